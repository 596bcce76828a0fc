// Work decomposition of the bf16 GEMM: one workgroup owns one BM x BN tile of C.
//
// The hardware hands consecutive workgroup ids to the 8 XCDs round-robin and each XCD has a
// private L2, so the tile list is cut into 8 contiguous pieces, one per XCD, and the list
// itself walks C in bands of GEMM_GROUP tile rows, column by column inside a band: the
// workgroups that are resident on one XCD at a time then cover a few tile rows x a few tile
// columns and share their A and B panels through that XCD's L2.  (The paper's GEMM gets the
// same reuse from cluster multicast and cluster launch control, section 4.2.)
#pragma once

#ifndef GEMM_HD
#define GEMM_HD __host__ __device__
#endif

#define GEMM_GROUP 4

struct GemmTileCoord {
  int tm, tn;
};

// entry L of the tile list
GEMM_HD inline GemmTileCoord gemm_tile_of_entry(int L, int tiles_m, int tiles_n) {
  const int width = GEMM_GROUP * tiles_n;
  const int band = L / width, in = L % width;
  const int first = band * GEMM_GROUP;
  const int rows = tiles_m - first < GEMM_GROUP ? tiles_m - first : GEMM_GROUP;
  GemmTileCoord c;
  c.tm = first + in % rows;
  c.tn = in / rows;
  return c;
}

// entry of a list of T that workgroup wg takes: XCD x owns base + (x < rem) consecutive entries,
// which is also how many workgroup ids it is handed
GEMM_HD inline int gemm_entry_of(int wg, int T) {
  const int xcd = wg & 7, idx = wg >> 3;
  const int base = T >> 3, rem = T & 7;
  return xcd * base + (xcd < rem ? xcd : rem) + idx;
}

GEMM_HD inline GemmTileCoord gemm_tile_coord_impl(int wg, int tiles_m, int tiles_n) {
  return gemm_tile_of_entry(gemm_entry_of(wg, tiles_m * tiles_n), tiles_m, tiles_n);
}

// Split-K launches: the list holds every tile of slice 0, then every tile of slice 1, ..., and is
// cut into 8 consecutive pieces as a whole: an XCD then works on one or two slices of k, and the
// tiles of a slice share their operand panels in its L2.  (Cutting every slice's tiles over the 8
// XCDs has each of them stream panels of all slices at once.)
GEMM_HD inline GemmTileCoord gemm_tile_coord_split(int wg, int tiles_m, int tiles_n, int splits, int* split) {
  const int ntile = tiles_m * tiles_n;
  const int L = gemm_entry_of(wg, ntile * splits);
  *split = L / ntile;
  return gemm_tile_of_entry(L - *split * ntile, tiles_m, tiles_n);
}
