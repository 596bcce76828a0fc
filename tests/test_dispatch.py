"""Routes of the public calls, without a GPU: which kernels a call launches, and that no size which fits a
launch is refused."""
from tests.launch_recorder import routes


def test_very_many_rows_are_launched():
    """Up to 2^31 - 256 rows of few columns fit one launch; so do as many columns (70 GB and 140 GB of operands)."""
    most = 2 ** 31 - 256
    calls = [dict(op="nt", M=1_100_000_000, N=32, K=32), dict(op="nn", M=1_100_000_000, N=32, K=32), dict(op="nt", M=1, N=1_100_000_000, K=32),
             dict(op="nt", M=most, N=1, K=32), dict(op="nn", M=most, N=8, K=32), dict(op="splitk", M=most, N=1, K=64, splits=2)]
    got, _ = routes(calls)
    for c, (status, launches) in zip(calls, got):
        assert status == 0 and len(launches) == 1, (c, status, launches)
        name, grid, threads = launches[0]
        assert grid * threads < 2 ** 32 and grid >= max(c["M"], c["N"]) // 256, (c, launches)
