// Triangular factors of blocks of Householder reflectors.
#pragma once
#include "gemm_f64.hpp"
#include "wave.hpp"

namespace qsgw {

// T of N reflectors, H_0 H_1 .. = I - V T V^T (T upper triangular, T[j][j] =
// tau_j, T[0:j, j] = -tau_j T[0:j, 0:j] G[0:j, j] with the Gram matrix G = V^T V),
// by one workgroup of 256 threads.  g(i, j): G[i][j], i < j, 0 past the last
// reflector; tau[] in LDS, 0 there.  T in LDS, [N][N + 1], whole on return
// (zeros below the diagonal).
// The blocks of 16 by columns, a wave each (lane 16 p + i: row i, every fourth
// term), then pairs of neighbours joined by T12 = -T11 (G12 T22) on the matrix
// cores, G12 T22 in the place of the zeros under the diagonal: about 2 N serial
// steps become 16 and a few products.
template <int N, class G>
__device__ __forceinline__ void wy_factor(G g, const double* tau, double (*T)[N + 1]) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  typedef Mfma<double> MM;
  for (int e = tid; e < N * N; e += 256) T[e / N][e % N] = 0.0;
  lds_barrier();
  for (int d = wave; d < N / 16; d += 4) {
    const int o = 16 * d, i = lane & 15, p = lane >> 4;
    // (column j of the block's G in lane j, p: terms l = 4 u + p)
    double gl[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) gl[u] = 4 * u + p < i ? g(o + 4 * u + p, o + i) : 0.0;
    const double t = tau[o + i];
    double row[4] = {0.0, 0.0, 0.0, 0.0};  // T[i][4 u + p]
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      double s = 0.0;
#pragma unroll
      for (int u = 0; u < 4; ++u) s = fma(row[u], __shfl(gl[u], 16 * p + j), s);
      // over the four p
      s += __shfl_xor(s, 16);
      s += __shfl_xor(s, 32);
      const double tj = read_lane(t, j);
      const double x = i == j ? tj : (i < j ? -tj * s : 0.0);
      if (p == (j & 3)) row[j >> 2] = x;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) T[o + i][o + 4 * u + p] = row[u];
  }
  lds_barrier();
#pragma unroll
  for (int h = 16; h < N; h *= 2) {
    const int tiles = h / 16, per = tiles * tiles, all = N / (2 * h) * per;
    // T21's place <- G12 T22
    for (int e = wave; e < all; e += 4) {
      const int o = 2 * h * (e / per), r = 16 * (e % per / tiles), c = 16 * (e % tiles);
      typename MM::acc_t acc = MM::zero();
#pragma unroll 4
      for (int k = 0; k <= c + 12; k += 4)  // (T22 is upper triangular)
        acc = MM::mma(g(o + r + (lane & 15), o + h + k + (lane >> 4)),
                      T[o + h + k + (lane >> 4)][o + h + c + (lane & 15)], acc);
#pragma unroll
      for (int q = 0; q < 4; ++q) T[o + h + r + MM::row(lane, q)][o + c + (lane & 15)] = acc[q];
    }
    lds_barrier();
    // T12 <- -T11 (G12 T22)
    for (int e = wave; e < all; e += 4) {
      const int o = 2 * h * (e / per), r = 16 * (e % per / tiles), c = 16 * (e % tiles);
      typename MM::acc_t acc = MM::zero();
#pragma unroll 4
      for (int k = r; k < h; k += 4)
        acc = MM::mma(T[o + r + (lane & 15)][o + k + (lane >> 4)],
                      T[o + h + k + (lane >> 4)][o + c + (lane & 15)], acc);
#pragma unroll
      for (int q = 0; q < 4; ++q) T[o + r + MM::row(lane, q)][o + h + c + (lane & 15)] = -acc[q];
    }
    lds_barrier();
    for (int e = tid; e < N / (2 * h) * h * h; e += 256) {
      const int o = 2 * h * (e / (h * h)), w = e % (h * h);
      T[o + h + w / h][o + w % h] = 0.0;
    }
    lds_barrier();
  }
}

}  // namespace qsgw
