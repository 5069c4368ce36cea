// Tile table of the tunable products and the rule for small FP64 products (host code).
#pragma once
#include <cstdint>

namespace qsgw {

// Tile shapes of the tunable products (qsgw_set_tiles).  Symmetric (upper
// tile) products take square shapes only.  The small-product rule alone takes 32 x 32.
enum Shape { SH_64x64 = 0, SH_128x64 = 1, SH_128x128 = 2, SH_COUNT, SH_32x32 };
enum Tunable { TU_MO1 = 0, TU_MO2, TU_CASIDA, TU_RHO, TU_SIGMA, TU_EXCHANGE, TU_COUNT };
struct Tiles {
  int shape[TU_COUNT] = {SH_128x64, SH_64x64, SH_128x128, SH_128x128, SH_64x64, SH_64x64};
  // workgroups a K-split aims for when the output tiles alone are few
  int64_t sigma_target = 4096, rho_target = 2048, exchange_target = 2048;
  // the qsMP2 contraction (K = nbf * block transitions) wants more splits
  int64_t mp2_target = 32768;
  // batched grouped products: 0 = one workgroup per tile, n > 0 = a
  // persistent grid of n workgroups per compute unit walking tile ranges
  int64_t persistent = 0;
  // projected divide and conquer of the two-stage eigensolver: tridiagonal
  // blocks up to this order are solved with their eigenvectors formed
  int64_t dc_leaf = 6144;
  // two-stage eigensolver: 1 = panel QR in one cooperative launch per panel
  // (the per-column launches when the device refuses it), 0 = per-column launches
  int64_t panel_coop = 1;
};
inline int shape_m(int s) { return s == SH_64x64 ? 64 : 128; }
inline int shape_n(int s) { return s == SH_128x128 ? 128 : 64; }

// FP64 products whose tiles would leave compute units idle take smaller ones:
// below 256 workgroups (the chip's compute units) 64 x 64, below that again
// 32 x 32.  The terms of an element and their order stay the same.  24 basis
// functions, 95 transitions: rho 33 -> 8 us, Casida matrix 28 -> 8 us, residues
// (tiles of 128 pairs x 128 or 32) 55 -> 24 us.  Just below the line: Casida
// matrix of order 2,800 (253 tiles of 128) with 480 auxiliary functions 175 ->
// 156 us, MO transform of 64 functions (250 tiles) 49 -> 47 us, residues of 78
// (210 tiles) 148 -> 128 us.
constexpr int64_t kFewWgs = 256;
inline int64_t tile_wgs(int64_t bm, int64_t bn, bool tri, int64_t M, int64_t N, int64_t batch,
                        int64_t nz) {
  const int64_t tm = (M + bm - 1) / bm, tn = (N + bn - 1) / bn;
  return (tri ? tm * (tm + 1) / 2 : tm * tn) * batch * (nz > 1 ? nz : 1);
}
inline int fitting_shape(int shape, bool tri, int64_t M, int64_t N, int64_t batch, int64_t nz) {
  if (tile_wgs(shape_m(shape), shape_n(shape), tri, M, N, batch, nz) >= kFewWgs) return shape;
  return tile_wgs(64, 64, tri, M, N, batch, nz) < kFewWgs ? SH_32x32 : SH_64x64;
}
// Shape of an FP64 product of the table: one that the table changed is taken as it
// is, the default one by the rule above.  (By the shape alone, so that a table
// written out and set again chooses as before.)
inline int table_shape(const Tiles& t, Tunable k, bool tri, int64_t M, int64_t N, int64_t batch,
                       int64_t nz) {
  const int shape = t.shape[k];
  return shape != Tiles{}.shape[k] ? shape : fitting_shape(shape, tri, M, N, batch, nz);
}

}  // namespace qsgw
