// Dense symmetric eigensolver for the orders where a one-stage reduction
// holds its matrix on the chip (n <= kEigTeamMax), one problem or many of
// different orders in the same launches.  Everything in FP64.
//
//   1. Reduction A = Q T Q^T (Householder, column j annihilates A[j+2.., j]):
//      a team of workgroups keeps the rows of A in registers for the whole
//      reduction, so a column costs its 3 m^2 multiply-adds and one exchange
//      between the workgroups instead of a pass over the matrix in memory
//      (k_tri_team).
//   2. Eigenpairs of T by divide and conquer: blocks of up to 64 rows are
//      solved in one workgroup (implicit QL on leaves of up to 8, then
//      merges in LDS: k_dc_base), larger ones merged level by level with all
//      nodes of a level in the same launches (k_dc_*), the eigenvectors of a
//      merge as two grouped products (each half's rows use only the columns
//      that are non-zero there).
//   3. Z = Q E by blocks of 128 reflectors in compact WY form, as products.
//
// The merge theory (Cuppen's tearing, deflation of small weights and of close
// poles by a rotation, the secular equation solved relative to the nearer
// pole, Gu and Eisenstat's weights from the computed roots) is that of
// eigdc.hip, with the tear's sign kept: beta = e[n1 - 1] comes off both
// touching diagonal entries and T = diag(T1, T2) + beta v v^T, v = e_{n1-1} +
// e_{n1}.  A negative beta is solved as -T (poles and roots negated, so their
// order reversed).  A root's vector is zh / (d - lambda) there, a deflated one keeps
// its half's sign.
#include "internal.hpp"
#include "wave.hpp"
#include "wy.hpp"

#include <algorithm>

namespace {

constexpr int kTeamThreads = 512;
constexpr int kBase = 64;   // largest block of the tridiagonal solved in one workgroup
constexpr int kLeaf = 8;    // largest QL leaf
constexpr int kBaseThreads = 512;
constexpr int kBk = 128;    // reflectors per WY block

// One eigenproblem on the device.
struct EigDev {
  double *A, *ev;      // matrix [n][ld] in, eigenvectors out; eigenvalues out
  double *E, *B, *U;   // n x n work: eigenvectors; gathered columns and W = V^T X; merge
                       // vectors and Y = V T (E and B: the exchange of the reduction)
  double *d, *e, *tau; // tridiagonal (scaled after k_dc_scale), reflector factors
  double* vec;         // merge vectors, kVec x n
  int* idx;            // merge index maps, kIdx x n
  double *G, *T;       // Gram matrices and T factors [blocks][128][128]
  double* scale;       // kScale words of the plan's, see below
  int64_t ld;
  int n, team, cfg, pad;
};
// scale[S_T]: power of two that T was divided by, [S_RANGE]: exponent of the one that the
// matrix was multiplied by (range_exponent), [S_MAX]: its largest magnitude.
enum { S_T = 0, S_RANGE, S_MAX, kScale = 8 };
enum { V_DK = 0, V_ZK, V_LAM, V_MU, V_DOR, V_ZH, V_DFS, V_RC, V_RS, kVec };
enum { I_COL = 0, I_P1, I_P2, I_DFC, I_DFF, I_POS, I_RA, I_RB, I_FLAG, kIdx };

struct TeamWg {
  int prob, g;
};
struct BaseNode {
  int prob, off, m;
};
struct Node {
  int prob, off, n1, n2;
};
// What a merge's deflation leaves for its later kernels.
struct NodeRes {
  double rho;
  int K, ndf, K1, K2, neg, pad;
};

// ------------------------------------------------------------ wave tools --
__device__ __forceinline__ double wave_max(double x) {
  for (int o = 32; o > 0; o >>= 1) x = fmax(x, __shfl_xor(x, o));
  return x;
}
__device__ __forceinline__ double wave_prod(double x) {
  for (int o = 32; o > 0; o >>= 1) x *= __shfl_xor(x, o);
  return x;
}
// Sums of 4 values over the 64 lanes into out[0..4): the first two steps halve
// the values as they halve the lanes (a swap of lane halves between two
// values, one add), the last four run within 16-lane rows.
__device__ __forceinline__ void reduce_rows4(const double (&s)[4], double* out) {
  const int lane = threadIdx.x & 63;
  double z = swap_add16(swap_add32(s[0], s[1]), swap_add32(s[2], s[3]));
  z = dpp_add<0x128, 0xf>(z);
  z = dpp_add<0x124, 0xf>(z);
  z = dpp_add<0x122, 0xf>(z);
  z = dpp_add<0x121, 0xf>(z);
  const int q = lane >> 4;
  if ((lane & 15) == 0) out[2 * (q & 1) + (q >> 1)] = z;
}

// ------------------------------------------------------------- reduction --
// Shared memory of a team workgroup.
struct TriSmem {
  double v[2][kEigTeamMax], w[2][kEigTeamMax];
  double y[128], r[128];   // single-workgroup teams
  double part[8][64];
  double red[2][4][8], al[2][4];
};

// The 16-byte slots (y, r) of a thread's columns tc + TC u, u < CU, read past
// the L2 of this XCD (the writers are anywhere on the chip); columns outside
// (j, n) read the nearest one inside.  All loads are waited for here.
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
template <int CU, int TC>
__device__ __forceinline__ void load_slots(const double* at, int j, int n, int tc, u32x4 (&x)[CU]) {
  const double* p[6];
#pragma unroll
  for (int u = 0; u < CU; ++u) {
    const int c = tc + TC * u;
    const int cc = c <= j ? j + 1 : (c < n ? c : n - 1);
    p[u] = at + 2 * (int64_t)(cc - tc);
  }
  static_assert(CU >= 1 && CU <= 6, "columns per thread");
  if constexpr (CU == 1)
    asm volatile("global_load_dwordx4 %0, %1, off sc1\n\ts_waitcnt vmcnt(0)"
                 : "=&v"(x[0])
                 : "v"(p[0])
                 : "memory");
  else if constexpr (CU == 2)
    asm volatile(
        "global_load_dwordx4 %0, %2, off sc1\n\tglobal_load_dwordx4 %1, %3, off sc1\n\t"
        "s_waitcnt vmcnt(0)"
        : "=&v"(x[0]), "=&v"(x[1])
        : "v"(p[0]), "v"(p[1])
        : "memory");
  else if constexpr (CU == 3)
    asm volatile(
        "global_load_dwordx4 %0, %3, off sc1\n\tglobal_load_dwordx4 %1, %4, off sc1\n\t"
        "global_load_dwordx4 %2, %5, off sc1\n\ts_waitcnt vmcnt(0)"
        : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2])
        : "v"(p[0]), "v"(p[1]), "v"(p[2])
        : "memory");
  else if constexpr (CU == 4)
    asm volatile(
        "global_load_dwordx4 %0, %4, off sc1\n\tglobal_load_dwordx4 %1, %5, off sc1\n\t"
        "global_load_dwordx4 %2, %6, off sc1\n\tglobal_load_dwordx4 %3, %7, off sc1\n\t"
        "s_waitcnt vmcnt(0)"
        : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3])
        : "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3])
        : "memory");
  else if constexpr (CU == 5)
    asm volatile(
        "global_load_dwordx4 %0, %5, off sc1\n\tglobal_load_dwordx4 %1, %6, off sc1\n\t"
        "global_load_dwordx4 %2, %7, off sc1\n\tglobal_load_dwordx4 %3, %8, off sc1\n\t"
        "global_load_dwordx4 %4, %9, off sc1\n\ts_waitcnt vmcnt(0)"
        : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(x[4])
        : "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3]), "v"(p[4])
        : "memory");
  else
    asm volatile(
        "global_load_dwordx4 %0, %6, off sc1\n\tglobal_load_dwordx4 %1, %7, off sc1\n\t"
        "global_load_dwordx4 %2, %8, off sc1\n\tglobal_load_dwordx4 %3, %9, off sc1\n\t"
        "global_load_dwordx4 %4, %10, off sc1\n\tglobal_load_dwordx4 %5, %11, off sc1\n\t"
        "s_waitcnt vmcnt(0)"
        : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(x[4]), "=&v"(x[5])
        : "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3]), "v"(p[4]), "v"(p[5])
        : "memory");
}

// Polls before a wait gives up (seconds; a team is resident as a whole, so its
// waits end).
constexpr int kTeamSpinMax = 1 << 21;

// The reduction of one matrix by a team of P.team workgroups, this one g.
// Rows are dealt cyclically to the team's VG = team * RG row groups (RG of TC
// lanes a workgroup), RL per group; lane tc of a group holds the columns
// tc + TC u, so A[i][c] is a[l][u] with i = l VG + vg.
// Iteration j, from column j of the reduced matrix A_j (col, held by every row
// group): v (v[j+1] = 1, zero up to j), tau, beta as in dlarfg; one pass over
// the registers applies the previous iteration's update A -= v w^T + w v^T and
// forms y = A_j v of the group's rows (above order 128 the update rounds an entry
// once, not twice: the eigenvalue errors, which grow with the order by these
// roundings, halve to 1.4e-15 of the norm at order 700, for 2 % of the time; at 95
// they are dsyevd's either way); y and row j + 1 of A_j are published
// and every group picks both up whole, forms w = tau y - (tau^2 (y . v) / 2) v
// and the next column A_j[j+1] - v w[j+1] - w.
// The exchange has no flags: slot (j, i) = (y_i, A_j[j+1][i]) is written once,
// each half by its owner, starts as kEmpty, and a reader polls the slots it needs.  Every group
// computes the same scalars from the same values in the same order.
// Row j of A takes v_j, once a whole workgroup has picked up y_j of every row: a
// wave polls its own columns alone, and a workgroup that starts late (other work on
// the device) may not have loaded its rows when another wave's slots are full.
// Indices here run from the matrix's last row to its first (index i is row
// n - 1 - i); T, the eigenvectors and the stored v are in the matrix's order.
// That is the order in which dsyevd reduces an upper triangle, and with the
// merges below the eigenvectors come out with the signs dsyevd gives them (every
// one of 8,871 vectors of ten Casida matrices), so that a caller sees the same
// Z whichever of the two solvers a call goes to.
template <int TC, int CU, int RL>
__device__ void tri_team(const EigDev& P, int g, TriSmem& sm, int* err) {
  constexpr int RG = kTeamThreads / TC, NW = TC / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int rg = __builtin_amdgcn_readfirstlane(tid / TC), tc = tid % TC;
  const int wr = __builtin_amdgcn_readfirstlane(wave % NW);
  const int n = P.n, G = P.team, VG = G * RG, vg = g * RG + rg;
  const int64_t ld = P.ld;
  double* A = P.A;
  double* YR = P.E;  // [column j][entry c][y, row j + 1]
  double a[RL][CU], v[CU], vp[CU], wp[CU], col[CU];
#pragma unroll
  for (int u = 0; u < CU; ++u) {
    const int c = tc + TC * u;
#pragma unroll
    for (int l = 0; l < RL; ++l) {
      const int i = l * VG + vg;
      a[l][u] = (i < n && c < n) ? A[(n - 1 - i) * ld + (n - 1 - c)] : 0.0;
    }
    col[u] = c < n ? A[(n - 1) * ld + (n - 1 - c)] : 0.0;
    v[u] = vp[u] = wp[u] = 0.0;
    if (c < n && rg == 0) sm.v[1][c] = sm.w[1][c] = 0.0;
  }
  // ---- entries far from 1 ----
  double mx = 0.0;
  if (G > 1) {
    mx = P.scale[S_MAX];  // (k_tri_clear)
  } else {
#pragma unroll
    for (int u = 0; u < CU; ++u)
#pragma unroll
      for (int l = 0; l < RL; ++l) mx = fmax(mx, finite_magnitude(a[l][u]));
    mx = wave_max(mx);
    if (lane == 0) sm.part[wave][0] = mx;
    lds_barrier();
#pragma unroll
    for (int q = 0; q < kTeamThreads / 64; ++q) mx = fmax(mx, sm.part[q][0]);
  }
  const int ex = __builtin_amdgcn_readfirstlane(range_exponent(mx));
  if (ex != 0) {
#pragma unroll
    for (int u = 0; u < CU; ++u) {
      col[u] = ldexp(col[u], ex);
#pragma unroll
      for (int l = 0; l < RL; ++l) a[l][u] = ldexp(a[l][u], ex);
    }
  }
  if (g == 0 && tid == 0) P.scale[S_RANGE] = ex;
  if (g == 0 && tid == 0) P.d[n - 1] = col[0];
  bool dead = false;
  for (int j = 0; j + 1 < n; ++j) {
    const int par = j & 1;
    // ---- reflector of column j ----
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < CU; ++u) {
      const int c = tc + TC * u;
      if (c > j + 1) s += col[u] * col[u];
      if (c == j + 1) sm.al[0][rg] = col[u];
    }
    s = wave_total(s);
    if (lane == 0) sm.red[0][rg][wr] = s;
    lds_barrier();
    double sig = 0.0;
#pragma unroll
    for (int q = 0; q < NW; ++q) sig += sm.red[0][rg][q];
    const double alpha = sm.al[0][rg];
    const auto [tau, beta, scale] = reflector(alpha, sig);
#pragma unroll
    for (int u = 0; u < CU; ++u) {
      const int c = tc + TC * u;
      v[u] = c > j + 1 ? col[u] * scale : (c == j + 1 ? 1.0 : 0.0);
      if (rg == 0 && c < n) sm.v[par][c] = v[u];
    }
    if (g == 0 && tid == 0) {
      P.e[n - 2 - j] = beta;
      P.tau[j] = tau;
    }
    // ---- previous update and y = A v on this group's rows ----
    double rv = 0.0, rw = 0.0;  // lane l: the previous v and w at row l
    {
      const int i = lane * VG + vg;
      if (lane < RL && i < n) {
        rv = sm.v[par ^ 1][i];
        rw = sm.w[par ^ 1][i];
      }
    }
    const int lr = (j + 1) % VG == vg ? (j + 1) / VG : -1;  // this group holds row j + 1
#pragma unroll
    for (int k = 0; k < RL / 4; ++k) {
      if ((4 * k + 3) * VG + vg <= j) continue;  // (a group of rows all reduced already)
      double s4[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int l = 4 * k + q;
        const double bv = read_lane(rv, l), bw = read_lane(rw, l);
        double t = 0.0;
#pragma unroll
        for (int u = 0; u < CU; ++u) {
          if constexpr (TC == 128)
            a[l][u] = fma(-bw, vp[u], fma(-bv, wp[u], a[l][u]));
          else
            a[l][u] -= fma(bv, wp[u], bw * vp[u]);
          t = fma(a[l][u], v[u], t);
        }
        s4[q] = t;
      }
      reduce_rows4(s4, sm.part[wave] + 4 * k);
      if (lr >> 2 == k) {
#pragma unroll
        for (int u = 0; u < CU; ++u) {
          const int c = tc + TC * u;
          const int q = lr & 3;
          const double x = q == 0 ? a[4 * k][u] : (q == 1 ? a[4 * k + 1][u]
                                                           : (q == 2 ? a[4 * k + 2][u] : a[4 * k + 3][u]));
          if (c > j && c < n) {
            if (G > 1)
              publish(YR + 2 * ((int64_t)j * n + c) + 1, x);
            else
              sm.r[c & 127] = x;
          }
        }
      }
    }
    lds_barrier();
    if (tc < RL) {
      const int i = tc * VG + vg;
      if (i > j && i < n) {
        double y = 0.0;
#pragma unroll
        for (int q = 0; q < NW; ++q) y += sm.part[rg * NW + q][tc];
        if (G > 1)
          publish(YR + 2 * ((int64_t)j * n + i), y);
        else
          sm.y[i & 127] = y;
      }
    }
    // ---- y and row j + 1, whole ----
    double y[CU], r[CU];
    if (G == 1) {
      lds_barrier();
#pragma unroll
      for (int u = 0; u < CU; ++u) {
        const int c = tc + TC * u;
        y[u] = c > j && c < n ? sm.y[c & 127] : 0.0;
        r[u] = c > j && c < n ? sm.r[c & 127] : 0.0;
      }
    } else {
      // (a first poll sent at once would arrive before the slowest workgroup's
      // stores and cost a second round trip: n = 1940, 14.1 -> 12.3 ms)
      if (CU < 6) __builtin_amdgcn_s_sleep(6);
      u32x4 x[CU];
      const double* at = YR + 2 * ((int64_t)j * n + tc);
      for (int spins = 0;; ++spins) {
        load_slots<CU, TC>(at, j, n, tc, x);
        bool all = true;
#pragma unroll
        for (int u = 0; u < CU; ++u) {
          const int c = tc + TC * u;
          if (c > j && c < n) all = all && (x[u][0] & x[u][1]) != ~0u && (x[u][2] & x[u][3]) != ~0u;
        }
        if (all || dead) break;
        if (spins > kTeamSpinMax) {
          dead = true;
          atomicOr(err, 1);
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
#pragma unroll
      for (int u = 0; u < CU; ++u) {
        const int c = tc + TC * u;
        const bool in = c > j && c < n;
        y[u] = in ? __builtin_bit_cast(double, u32x2{x[u][0], x[u][1]}) : 0.0;
        r[u] = in ? __builtin_bit_cast(double, u32x2{x[u][2], x[u][3]}) : 0.0;
      }
    }
    // ---- w and the next column ----
    double yv = 0.0;
#pragma unroll
    for (int u = 0; u < CU; ++u) {
      const int c = tc + TC * u;
      yv += y[u] * v[u];
      if (c == j + 1) sm.al[1][rg] = y[u];
    }
    yv = wave_total(yv);
    if (lane == 0) sm.red[1][rg][wr] = yv;
    lds_barrier();
    yv = 0.0;
#pragma unroll
    for (int q = 0; q < NW; ++q) yv += sm.red[1][rg][q];
    // (only now, after the barrier, have this workgroup's waves together seen y_j
    // of every row, and so each row's group has loaded it)
    if (j % G == g && rg == 0) {
#pragma unroll
      for (int u = 0; u < CU; ++u) {
        const int c = tc + TC * u;
        if (c < n) A[j * ld + (n - 1 - c)] = v[u];
      }
    }
    const double kap = 0.5 * tau * tau * yv;
    const double w1 = tau * sm.al[1][rg] - kap;
#pragma unroll
    for (int u = 0; u < CU; ++u) {
      const int c = tc + TC * u;
      const double w = c > j && c < n ? tau * y[u] - kap * v[u] : 0.0;
      if (rg == 0 && c < n) sm.w[par][c] = w;
      col[u] = c > j && c < n ? r[u] - v[u] * w1 - w : 0.0;
      if (c == j + 1 && g == 0 && rg == 0) P.d[n - 2 - j] = col[u];
      vp[u] = v[u];
      wp[u] = w;
    }
  }
}

// Row capacity of a workgroup and column capacity of each shape (RG RL rows,
// TC CU columns).
struct TeamShape {
  int rows, cols;
};
constexpr TeamShape kTeamShapes[] = {
    {128, 128}, {64, 256}, {16, 512}, {64, 512}, {16, 1024}, {40, 1024}, {12, 1536},
    {28, 1536}, {8, 2048}, {20, 2048}, {12, 2560}, {12, 3072},
};
__global__ __launch_bounds__(kTeamThreads, 2) void k_tri_team(const EigDev* __restrict__ P,
                                                              const TeamWg* __restrict__ wg,
                                                              int* __restrict__ err) {
  __shared__ TriSmem sm;
  const TeamWg t = wg[blockIdx.x];
  const EigDev p = P[t.prob];
  err += t.prob;
  switch (p.cfg) {
    case 0: tri_team<128, 1, 32>(p, t.g, sm, err); break;
    case 1: tri_team<256, 1, 32>(p, t.g, sm, err); break;
    case 2: tri_team<512, 1, 16>(p, t.g, sm, err); break;
    case 3: tri_team<512, 1, 64>(p, t.g, sm, err); break;
    case 4: tri_team<512, 2, 16>(p, t.g, sm, err); break;
    case 5: tri_team<512, 2, 40>(p, t.g, sm, err); break;
    case 6: tri_team<512, 3, 12>(p, t.g, sm, err); break;
    case 7: tri_team<512, 3, 28>(p, t.g, sm, err); break;
    case 8: tri_team<512, 4, 8>(p, t.g, sm, err); break;
    case 9: tri_team<512, 4, 20>(p, t.g, sm, err); break;
    case 10: tri_team<512, 5, 12>(p, t.g, sm, err); break;
    default: tri_team<512, 6, 12>(p, t.g, sm, err); break;
  }
}

__global__ void k_eig_init(double* scale, int* err, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n * kScale) scale[i] = 0.0;
  if (i < n) err[i] = 0;
}

// kEmpty into the exchange slots of every problem (blockIdx.y) solved by more
// than one workgroup, and its matrix's largest magnitude (bit patterns of
// numbers from 0 to infinity are in their order).
__global__ __launch_bounds__(256) void k_tri_clear(const EigDev* __restrict__ P) {
  __shared__ double red[4];
  const EigDev& p = P[blockIdx.y];
  if (p.team <= 1) return;
  const int64_t nn = (int64_t)p.n * p.n, step = (int64_t)gridDim.x * blockDim.x;
  ulonglong2* x = reinterpret_cast<ulonglong2*>(p.E);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nn; i += step)
    x[i] = ulonglong2{kEmpty, kEmpty};
  double m = 0.0;
  for (int64_t r = blockIdx.x; r < p.n; r += gridDim.x)
    for (int c = threadIdx.x; c < p.n; c += 256) m = fmax(m, finite_magnitude(p.A[r * p.ld + c]));
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  m = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
  if (threadIdx.x == 0 && m > __builtin_bit_cast(double, peek(p.scale + S_MAX)))
    atomicMax(reinterpret_cast<unsigned long long*>(p.scale + S_MAX),
              __builtin_bit_cast(unsigned long long, m));
}

// ------------------------------------------------------ divide and conquer --
// T divided by the power of two of its largest entry (one workgroup a problem).
// The merges' index maps take their places from comparisons of poles and are
// whole only for finite ones: a T with an entry that is not finite (a product
// that overflowed, a wait of the reduction that was given up) is replaced by
// zeros and flagged.
__global__ __launch_bounds__(256) void k_dc_scale(const EigDev* __restrict__ P,
                                                  int* __restrict__ err) {
  __shared__ double red[4];
  const EigDev& p = P[blockIdx.x];
  double m = 0.0;
  for (int i = threadIdx.x; i < p.n; i += 256) {
    m = fmax(m, finite_magnitude(p.d[i]));
    if (i + 1 < p.n) m = fmax(m, finite_magnitude(p.e[i]));
  }
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  m = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
  const bool ok = isfinite(m);
  int ex = 0;
  if (m > 0.0 && ok) (void)frexp(m, &ex);
  for (int i = threadIdx.x; i < p.n; i += 256) {
    p.d[i] = ok ? ldexp(p.d[i], -ex) : 0.0;
    if (i + 1 < p.n) p.e[i] = ok ? ldexp(p.e[i], -ex) : 0.0;
  }
  if (threadIdx.x == 0) {
    p.scale[S_T] = ldexp(1.0, ex);
    if (!ok) atomicOr(err + blockIdx.x, 4);
  }
}

// Root of the secular equation j of K (poles d ascending, weights z), by W
// lanes (4 or 64) that each sum every W-th term: the origin pole's index, mu
// (the root less that pole).  `total` sums a value over the W lanes.
// Each step replaces the poles up to j and those above it by one at d_j and
// one at d_{j+1} with the sums' values and slopes (the "middle way" of R.-C.
// Li, LAPACK Working Note 89) and takes that model's root, kept inside the
// bracket; it ends when f is as small as its own rounding.  3 to 4 steps on
// average, 11 at most in some 10,000 roots
// (Newton on mu f(mu) with a step test alone bisected on noise for most of
// its 40 or so: K = 24 by 4 lanes, 100,000 cycles).
template <int W, class F>
__device__ __forceinline__ void secular_root(const double* d, const double* z, int K, double rho,
                                             int j, int lane, F total, int& org, double& mu) {
  double a, b, m;
  int o;
  const int jl = j < K - 1 ? j : (K > 1 ? K - 2 : 0), jr = jl + 1 < K ? jl + 1 : jl;
  if (j < K - 1) {
    const double dj = d[j], gap = d[j + 1] - dj, half = 0.5 * gap;
    double s = 0.0;
#pragma unroll 4
    for (int i = lane; i < K; i += W) s += z[i] * z[i] * fast_rcp((d[i] - dj) - half);
    const double fm = 1.0 + rho * total(s);
    // first guess: the other poles as a constant
    const double u = rho * z[j] * z[j], v = rho * z[j + 1] * z[j + 1];
    const double c = fm + (u - v) * fast_rcp(half);
    if (fm >= 0.0) {
      o = j;
      a = 0.0;
      b = half;
      const double p = c * gap + u + v, q = sqrt(fabs(p * p - 4.0 * u * gap * c));
      m = p > 0.0 ? 2.0 * u * gap * fast_rcp(p + q) : (p - q) * 0.5 * fast_rcp(c);
    } else {
      o = j + 1;
      a = -half;
      b = 0.0;
      const double p = c * gap - u - v, q = sqrt(fabs(p * p + 4.0 * v * gap * c));
      m = p < 0.0 ? 2.0 * v * gap * fast_rcp(p - q) : -(p + q) * 0.5 * fast_rcp(c);
    }
    if (!(m > a && m < b)) m = 0.5 * (a + b);
  } else {
    o = j;
    a = 0.0;
    b = rho;
    m = 0.5 * rho;
  }
  const double d_o = d[o], dl_l = d[jl] - d_o, dl_r = d[jr] - d_o;
  for (int it = 0; it < 100; ++it) {
    double S = 0.0, Sa = 0.0, Pl = 0.0, Pr = 0.0;
#pragma unroll 4
    for (int i = lane; i < K; i += W) {
      const double r = fast_rcp((d[i] - d_o) - m);
      const double q = z[i] * z[i] * r, qr = q * r;
      S += q;
      Sa += fabs(q);
      Pl += i <= jl ? qr : 0.0;
      Pr += i <= jl ? 0.0 : qr;
    }
    S = total(S);
    Sa = total(Sa);
    Pl = rho * total(Pl);
    Pr = rho * total(Pr);
    const double f = 1.0 + rho * S;
    // (f increases over the bracket)
    if (f < 0.0) a = m; else b = m;
    if (fabs(f) <= __DBL_EPSILON__ * (8.0 * (1.0 + rho * Sa) + fabs(m) * (Pl + Pr))) break;
    const double Dl = dl_l - m, Dr = dl_r - m;
    const double c = f - Dl * Pl - Dr * Pr;
    const double p = (Dl + Dr) * f - Dl * Dr * (Pl + Pr), w = Dl * Dr * f;
    const double q = sqrt(fabs(p * p - 4.0 * w * c));
    double eta;
    if (j < K - 1)
      eta = p <= 0.0 ? (p - q) * 0.5 * fast_rcp(c) : 2.0 * w * fast_rcp(p + q);
    else
      eta = p >= 0.0 ? (p + q) * 0.5 * fast_rcp(c) : 2.0 * w * fast_rcp(p - q);
    if (!(f * eta < 0.0)) eta = -f * fast_rcp(Pl + Pr);
    double mn = m + eta;
    if (!(mn > a && mn < b)) mn = 0.5 * (a + b);
    const bool done = fabs(mn - m) <= __DBL_EPSILON__ * fabs(mn) ||
                      !(b - a > 2.0 * __DBL_EPSILON__ * fmax(fabs(a), fabs(b)));
    m = mn;
    if (done) break;
  }
  org = o;
  mu = m;
}

// Factor j of zh_i^2 (see eigdc.hip): lambda_j - d_i over the pole difference
// that interlaces with it.
__device__ __forceinline__ double zhat_factor(const double* d, int K, double rho, int i, int j,
                                              double dor_j, double mu_j) {
  const double di = d[i];
  const double lj = (dor_j - di) + mu_j;
  const double den = j < i ? d[j] - di : (j < K - 1 ? d[j + 1] - di : rho);
  return lj * fast_rcp(den);
}

// Serial deflation of n sorted poles ds with unit weights zs (one thread): the
// non-deflated positions nd[0..K) with values dk, zk, the deflated positions
// df with values dfv, the rotations (ra, rb, rc, rs) in order.  Returns K.
__device__ int dc_deflate_serial(const double* ds, const double* zs, int n, double rho, double tol,
                                 int* nd, double* dk, double* zk, int* df, double* dfv, int* ra,
                                 int* rb, double* rc, double* rs, int* nrot) {
  int K = 0, ndf = 0, nr = 0, prev = -1;
  double dp = 0.0, zp = 0.0;
  for (int j = 0; j < n; ++j) {
    const double dj = ds[j], zj = zs[j];
    if (rho * fabs(zj) <= tol) {
      df[ndf] = j;
      dfv[ndf++] = dj;
      continue;
    }
    if (prev >= 0) {
      // |(dj - dp) c s| <= tol with c = zj / t, s = zp / t; the square root and
      // the divisions only where it deflates
      const double t2 = zp * zp + zj * zj;
      if (fabs((dj - dp) * zj * zp) <= tol * t2) {
        const double t = sqrt(t2), cc = zj / t, ss = zp / t;
        ra[nr] = prev;
        rb[nr] = j;
        rc[nr] = cc;
        rs[nr++] = ss;
        df[ndf] = prev;
        dfv[ndf++] = dp * cc * cc + dj * ss * ss;
        prev = j;
        dp = dp * ss * ss + dj * cc * cc;
        zp = t;
        continue;
      }
      nd[K] = prev;
      dk[K] = dp;
      zk[K++] = zp;
    }
    prev = j;
    dp = dj;
    zp = zj;
  }
  if (prev >= 0) {
    nd[K] = prev;
    dk[K] = dp;
    zk[K++] = zp;
  }
  *nrot = nr;
  return K;
}

// ---- blocks of up to 64 rows in one workgroup ----
struct BaseSmem {
  double E[kBase][kBase + 1], E2[kBase][kBase + 1], U[kBase][kBase + 1];  // [column][row]
  double D[kBase], ds[kBase], zs[kBase], dk[kBase], zk[kBase], mu[kBase], dor[kBase], zh[kBase],
      dfv[kBase], rc[kBase], rs[kBase], lam[kBase];
  int src[kBase], nd[kBase], df[kBase], ra[kBase], rb[kBase], pos[kBase], col[kBase], K[4], nrot[4];
  double rho[4];
};

// Implicit QL with eigenvectors of a tridiagonal leaf of m <= 8 rows (lane i:
// d_i, and e_i between i and i + 1) by one wave, lane r row r of the
// eigenvectors in registers; eigenvalues ascending into D[b..b+m), vectors into
// the leaf's block of E.  If an eigenvalue does not converge it returns false
// and leaves the diagonal with unit vectors, which the merges can work on.
typedef double d8 __attribute__((ext_vector_type(8)));
__device__ bool ql_leaf(BaseSmem& sm, int b, int m, double d, double e) {
  const int lane = threadIdx.x & 63;
  const double d0 = d;
  bool ok = true;
  d8 Z;
#pragma unroll
  for (int c = 0; c < kLeaf; ++c) Z[c] = lane == c ? 1.0 : 0.0;
  for (int l = 0; l < m; ++l) {
    for (int it = 0;; ++it) {
      // first negligible e at or after l (the last row counts as one)
      const double dn = __shfl_down(d, 1);
      const unsigned long long small =
          __ballot(lane + 1 >= m || fabs(e) <= fmax(__DBL_EPSILON__ * (fabs(d) + fabs(dn)), kTinyEntry));
      const int q = l + __builtin_ctzll(small >> l);
      if (q == l) break;
      if (it >= 60) {
        ok = false;
        break;
      }
      const double dl = read_lane(d, l), el = read_lane(e, l);
      double gg = (read_lane(d, l + 1) - dl) / (2.0 * el);
      const double r = sqrt(gg * gg + 1.0);
      gg = read_lane(d, q) - dl + el / (gg + copysign(r, gg));
      double s = 1.0, c = 1.0, p = 0.0;
      int i = q - 1;
      for (; i >= l; --i) {
        const double ei = read_lane(e, i);
        const double f = s * ei, bb = c * ei;
        const double r2 = fma(f, f, gg * gg);
        if (r2 <= kTinySquare) {
          if (lane == i + 1) {
            e = 0.0;
            d -= p;
          }
          if (lane == q) e = 0.0;
          break;
        }
        const double ri = fast_rsqrt(r2);
        if (lane == i + 1) e = r2 * ri;
        s = f * ri;
        c = gg * ri;
        gg = read_lane(d, i + 1) - p;
        const double t = (read_lane(d, i) - gg) * s + 2.0 * c * bb;
        p = s * t;
        if (lane == i + 1) d = gg + p;
        gg = c * t - bb;
        const double z1 = Z[i + 1], z0 = Z[i];
        Z[i + 1] = s * z0 + c * z1;
        Z[i] = c * z0 - s * z1;
      }
      if (i >= l) continue;
      if (lane == l) {
        d -= p;
        e = gg;
      }
      if (lane == q) e = 0.0;
    }
  }
  if (!ok) {
    d = d0;
#pragma unroll
    for (int c = 0; c < kLeaf; ++c) Z[c] = lane == c ? 1.0 : 0.0;
  }
  int rank = 0;
  for (int k = 0; k < m; ++k) {
    const double dk = read_lane(d, k);
    rank += (dk < d || (dk == d && k < lane)) ? 1 : 0;
  }
  if (lane < m) sm.D[b + rank] = d;
#pragma unroll
  for (int k = 0; k < kLeaf; ++k) {
    const int rk = __builtin_amdgcn_readlane(rank, k);
    if (k < m && lane < m) sm.E[b + rk][b + lane] = Z[k];
  }
  return ok;
}

// Merge of D[o..o+m1) and D[o+m1..o+m1+m2) (each ascending, eigenvectors in
// the columns of E) by the TS threads of a team, rank tr; `team` numbers the
// teams of the workgroup, all of which call together.
template <int TS>
__device__ void base_merge(BaseSmem& sm, int team, int tr, int o, int m1, int m2, double beta) {
  const int m = m1 + m2;
  const bool neg = beta < 0.0;
  if (tr < m) {
    const double val = sm.D[o + tr];
    int pos = merged_place(sm.D + o, m1, m, tr);
    const double z = sm.E[o + tr][tr < m1 ? o + m1 - 1 : o + m1];
    if (neg) pos = m - 1 - pos;
    sm.ds[o + pos] = neg ? -val : val;
    sm.zs[o + pos] = z;
    sm.src[o + pos] = o + tr;
  }
  __syncthreads();
  if (tr < 64) {  // (the team's first wave)
    const double z = tr < m ? sm.zs[o + tr] : 0.0;
    const double s2 = wave_total(z * z), dm = wave_max(tr < m ? fabs(sm.ds[o + tr]) : 0.0);
    const double rho = fabs(beta) * s2, zi = z * fast_rsqrt(s2), di = tr < m ? sm.ds[o + tr] : 0.0;
    const double tol = fmax(8.0 * __DBL_EPSILON__ * fmax(dm, rho), kTinyEntry);
    // the poles that stay, and whether two neighbours among them are close
    const bool stays = tr < m && rho * fabs(zi) > tol;
    const unsigned long long mask = __ballot(stays);
    const int at = __popcll(mask & ((1ull << tr) - 1));
    const unsigned long long later = tr < 63 ? mask >> (tr + 1) : 0;
    const int nx = later ? tr + 1 + __builtin_ctzll(later) : tr;
    const double dn = __shfl(di, nx), zn = __shfl(zi, nx);
    const bool close =
        stays && later && fabs((dn - di) * zi * zn) <= tol * (zi * zi + zn * zn);
    if (__ballot(close) == 0) {
      if (stays) {
        sm.nd[o + at] = tr;
        sm.dk[o + at] = di;
        sm.zk[o + at] = zi;
      } else if (tr < m) {
        sm.df[o + tr - at] = tr;
        sm.dfv[o + tr - at] = di;
      }
      if (tr == 0) {
        sm.rho[team] = rho;
        sm.K[team] = __popcll(mask);
        sm.nrot[team] = 0;
      }
    } else {
      if (tr < m) sm.zs[o + tr] = zi;
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (tr == 0) {
        sm.rho[team] = rho;
        sm.K[team] = dc_deflate_serial(sm.ds + o, sm.zs + o, m, rho, tol, sm.nd + o, sm.dk + o,
                                       sm.zk + o, sm.df + o, sm.dfv + o, sm.ra + o, sm.rb + o,
                                       sm.rc + o, sm.rs + o, &sm.nrot[team]);
      }
    }
  }
  __syncthreads();
  const int K = sm.K[team], ndf = m - K, nrot = sm.nrot[team];
  const double rho = sm.rho[team];
  if (tr < K) sm.col[o + tr] = sm.src[o + sm.nd[o + tr]];
  if (tr < m)
    for (int q = 0; q < nrot; ++q) {
      double* xa = &sm.E[sm.src[o + sm.ra[o + q]]][o + tr];
      double* xb = &sm.E[sm.src[o + sm.rb[o + q]]][o + tr];
      const double a = *xa, b = *xb, c = sm.rc[o + q], s = sm.rs[o + q];
      *xa = c * a - s * b;
      *xb = s * a + c * b;
    }
  // roots, four lanes each (TS >= 4 m)
  const int j = tr >> 2, ql = tr & 3;
  if (j < K) {
    int org;
    double mu;
    secular_root<4>(sm.dk + o, sm.zk + o, K, rho, j, ql, [](double x) { return quad_total(x); },
                    org, mu);
    if (ql == 0) {
      sm.mu[o + j] = mu;
      sm.dor[o + j] = sm.dk[o + org];
      sm.lam[o + j] = sm.dk[o + org] + mu;
    }
  }
  __syncthreads();
  if (j < K) {
    double p = 1.0;
    for (int q = ql; q < K; q += 4)
      p *= zhat_factor(sm.dk + o, K, rho, j, q, sm.dor[o + q], sm.mu[o + q]);
    p *= __shfl_xor(p, 1);
    p *= __shfl_xor(p, 2);
    if (ql == 0) sm.zh[o + j] = copysign(sqrt(p), sm.zk[o + j]);
  }
  __syncthreads();
  if (j < K) {
    const double dj = sm.dor[o + j], mu = sm.mu[o + j];
    double s2 = 0.0;
    for (int i = ql; i < K; i += 4) {
      const double u = sm.zh[o + i] * fast_rcp((sm.dk[o + i] - dj) - mu);
      sm.U[o + j][o + i] = u;
      s2 += u * u;
    }
    s2 = quad_total(s2);
    const double inv = fast_rsqrt(s2);
    for (int i = ql; i < K; i += 4) sm.U[o + j][o + i] *= inv;
  }
  // final positions: roots j < K, then deflated values (rank by counting)
  if (tr < m) {
    double val;
    int pos;
    if (tr < K) {
      val = sm.lam[o + tr];
      pos = tr;
      for (int q = 0; q < ndf; ++q) pos += sm.dfv[o + q] < val ? 1 : 0;
    } else {
      const int q0 = tr - K;
      val = sm.dfv[o + q0];
      pos = dc_count(sm.lam + o, K, val, true);
      for (int q = 0; q < ndf; ++q)
        pos += (sm.dfv[o + q] < val || (sm.dfv[o + q] == val && q < q0)) ? 1 : 0;
    }
    if (neg) {
      pos = m - 1 - pos;
      val = -val;
    }
    sm.pos[o + tr] = o + pos;
    sm.D[o + pos] = val;  // (the old values were last read before the secular step)
  }
  __syncthreads();
  // E2[pos] = sum_i E[col_i] U[root][i] on the matrix cores (16 rows x 16 roots
  // a wave), the deflated columns as they are
  {
    typedef Mfma<double> MM;
    const int lane = tr & 63, l = lane & 15, nr = (m + 15) >> 4, nj = (K + 15) >> 4;
    for (int t = tr >> 6; t < nr * nj; t += TS / 64) {
      const int r = 16 * (t / nj) + l, j = 16 * (t % nj) + l;
      typename MM::acc_t acc = MM::zero();
#pragma unroll 4
      for (int k = lane >> 4; k < ((K + 3) & ~3); k += 4) {
        const int kk = k < K ? k : 0;
        const double x = sm.E[sm.col[o + kk]][o + (r < m ? r : 0)];
        const double y = sm.U[o + (j < K ? j : 0)][o + kk];
        acc = MM::mma(k < K ? x : 0.0, k < K ? y : 0.0, acc);
      }
      if (j < K) {
        const int at = sm.pos[o + j];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = 16 * (t / nj) + MM::row(lane, q);
          if (row < m) sm.E2[at][o + row] = acc[q];
        }
      }
    }
    for (int e = tr; e < ndf * m; e += TS) {
      const int q = e / m, row = e - q * m;
      sm.E2[sm.pos[o + K + q]][o + row] = sm.E[sm.src[o + sm.df[o + q]]][o + row];
    }
  }
  __syncthreads();
  for (int e = tr; e < m * m; e += TS) {
    const int c = e / m, r = e - c * m;
    sm.E[o + c][o + r] = sm.E2[o + c][o + r];
  }
  __syncthreads();
}

// One workgroup per block of up to 64 rows: eigenvalues (ascending) over the
// block of d, eigenvectors into the block of E.  Latency: the chain of a leaf's
// rotations (about 1.5 m^2 of some 600 cycles), then up to three merges of
// some 20,000 cycles each; leaves of 8 rows, a wave each.  Leaves of 16 with
// the vectors in LDS and square roots and divisions in the chain, merges with a
// serial deflation walk and scalar products took 160 us at n = 24, 289 at 95 and
// 440 at 1940; this 42, 76 and 104.
__global__ __launch_bounds__(kBaseThreads) void k_dc_base(const EigDev* __restrict__ P,
                                                          const BaseNode* __restrict__ nodes,
                                                          int* __restrict__ err) {
  __shared__ BaseSmem sm;
  const BaseNode nd = nodes[blockIdx.x];
  const EigDev& p = P[nd.prob];
  const int n = p.n, off = nd.off, m = nd.m, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // 2^depth leaves: halves of halves; boundary t of 2^level
  const int depth = m > 4 * kLeaf ? 3 : (m > 2 * kLeaf ? 2 : (m > kLeaf ? 1 : 0));
  auto bound = [&](int t, int level) {
    int lo = 0, len = m;
    if (t >> level) return m;
    for (int q = level - 1; q >= 0; --q) {
      const int h = len / 2;
      if ((t >> q) & 1) {
        lo += h;
        len -= h;
      } else {
        len = h;
      }
    }
    return lo;
  };
  for (int e = tid; e < kBase * kBase; e += kBaseThreads) sm.E[e / kBase][e % kBase] = 0.0;
  __syncthreads();
  auto edge = [&](int r) -> double {  // off-diagonal between rows r - 1 and r of T
    return r > 0 && r < n ? p.e[r - 1] : 0.0;
  };
  if (wave < 1 << depth) {
    const int b0 = bound(wave, depth), lm = bound(wave + 1, depth) - b0;
    double d = 0.0, e = 0.0;
    if (lane < lm) {
      d = p.d[off + b0 + lane];
      if (lane == 0) d -= edge(off + b0);
      if (lane == lm - 1) d -= edge(off + b0 + lm);
      if (lane + 1 < lm) e = p.e[off + b0 + lane];
    }
    if (!ql_leaf(sm, b0, lm, d, e) && lane == 0) atomicOr(err + nd.prob, 2);
  }
  __syncthreads();
  for (int level = depth; level > 0; --level) {
    const int teams = 1 << (level - 1), team = tid / (kBaseThreads / teams);
    const int o = bound(2 * team, level), mid = bound(2 * team + 1, level);
    const int end = bound(2 * team + 2, level), tr = tid % (kBaseThreads / teams);
    const double beta = p.e[off + mid - 1];
    if (level == 3)
      base_merge<kBaseThreads / 4>(sm, team, tr, o, mid - o, end - mid, beta);
    else if (level == 2)
      base_merge<kBaseThreads / 2>(sm, team, tr, o, mid - o, end - mid, beta);
    else
      base_merge<kBaseThreads>(sm, team, tr, o, mid - o, end - mid, beta);
  }
  for (int e = tid; e < m * m; e += kBaseThreads) {
    const int c = e / m, r = e - c * m;
    p.E[(int64_t)(off + c) * n + off + r] = sm.E[c][r];
  }
  if (tid < m) p.d[off + tid] = sm.D[tid];
}

// ---- merges of larger blocks, every node of a level in the same launches ----
// Node of global index q of the level (pre: first index of each node).
__device__ __forceinline__ int node_of(const int* pre, int nn, int q) {
  int lo = 0, hi = nn - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (pre[mid] <= q) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// E[off + pos[m]][off + n] (column-major columns): the new eigenvectors.
struct EpiEigCols {
  double* E;
  int64_t ld;
  const int* pos;
  __device__ __forceinline__ void operator()(int64_t, int64_t, int64_t m, int64_t n, double v,
                                             bool) const {
    E[pos[m] * ld + n] = v;
  }
};
typedef GemmJob<Strided<true>, Strided<false>, EpiEigCols> JobMerge;

constexpr int kPrepThreads = 1024;
struct PrepSmem {
  double ds[kEigTridiagMax], zs[kEigTridiagMax];
  int src[kEigTridiagMax], S[kEigTridiagMax];
  double red[2][16];
  int wsum[16], any, K, nrot;
};
// Exclusive sum of v over the workgroup's threads; *total the whole sum.
__device__ int block_scan(int v, int* wsum, int* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  int x = v;
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(x, o);
    if (lane >= o) x += t;
  }
  __syncthreads();
  if (lane == 63) wsum[w] = x;
  __syncthreads();
  int base = 0, all = 0;
  for (int q = 0; q < nw; ++q) {
    if (q < w) base += wsum[q];
    all += wsum[q];
  }
  *total = all;
  return base + x - v;
}

// Sorting and deflation of one node (one workgroup): the poles of both halves
// merged, small weights and, where two neighbouring poles are close, rotated
// ones deflated (the serial walk runs only then), the index maps of the later
// kernels, and the sizes of the node's two products.
__global__ __launch_bounds__(kPrepThreads) void k_dc_prep(const EigDev* __restrict__ P,
                                                          const Node* __restrict__ nodes,
                                                          NodeRes* __restrict__ res,
                                                          JobMerge* __restrict__ jobs) {
  __shared__ PrepSmem sm;
  const Node nd = nodes[blockIdx.x];
  const EigDev& p = P[nd.prob];
  const int N = p.n, off = nd.off, n1 = nd.n1, n = nd.n1 + nd.n2;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const double* d = p.d + off;
  double* vec = p.vec + off;
  int* idx = p.idx + off;
  const double beta = p.e[off + n1 - 1];
  const bool neg = beta < 0.0;
  double s2 = 0.0, dm = 0.0;
  for (int t = tid; t < n; t += kPrepThreads) {
    const double val = d[t];
    const double* Ec = p.E + (int64_t)(off + t) * N + off;
    int pos = merged_place(d, n1, n, t);
    const double z = Ec[t < n1 ? n1 - 1 : n1];
    if (neg) pos = n - 1 - pos;
    sm.ds[pos] = neg ? -val : val;
    sm.zs[pos] = z;
    sm.src[pos] = t;
    s2 += z * z;
    dm = fmax(dm, fabs(val));
  }
  s2 = wave_total(s2);
  dm = wave_max(dm);
  if (lane == 0) {
    sm.red[0][w] = s2;
    sm.red[1][w] = dm;
  }
  if (tid == 0) sm.any = 0;
  __syncthreads();
  s2 = 0.0;
  for (int q = 0; q < kPrepThreads / 64; ++q) {
    s2 += sm.red[0][q];
    dm = fmax(dm, sm.red[1][q]);
  }
  const double zi = 1.0 / sqrt(s2);
  const double rho = fabs(beta) * s2;
  const double tol = fmax(8.0 * __DBL_EPSILON__ * fmax(dm, rho), kTinyEntry);
  // survivors of the weight test, in order
  const int per = (n + kPrepThreads - 1) / kPrepThreads;
  const int t0 = tid * per, t1 = min(t0 + per, n);
  int cnt = 0;
  for (int t = t0; t < t1; ++t) {
    sm.zs[t] *= zi;
    cnt += rho * fabs(sm.zs[t]) > tol ? 1 : 0;
  }
  int ns = 0;
  int at = block_scan(cnt, sm.wsum, &ns);
  for (int t = t0; t < t1; ++t) {
    if (rho * fabs(sm.zs[t]) > tol)
      sm.S[at++] = t;
    else {
      vec[V_DFS * N + t - at] = sm.ds[t];
      idx[I_DFC * N + t - at] = sm.src[t];
      idx[I_DFF * N + t - at] = sm.src[t] < n1 ? 1 : 2;
    }
    idx[I_FLAG * N + t] = t < n1 ? 1 : 2;
  }
  __syncthreads();
  bool close = false;
  for (int k = tid; k + 1 < ns; k += kPrepThreads) {
    const int a = sm.S[k], b = sm.S[k + 1];
    const double zp = sm.zs[a], zj = sm.zs[b];
    const double t = sqrt(zp * zp + zj * zj);
    if (fabs((sm.ds[b] - sm.ds[a]) * (zj / t) * (zp / t)) <= tol) close = true;
  }
  if (close) sm.any = 1;
  __syncthreads();
  int K = ns;
  if (!sm.any) {
    for (int k = tid; k < K; k += kPrepThreads) {
      vec[V_DK * N + k] = sm.ds[sm.S[k]];
      vec[V_ZK * N + k] = sm.zs[sm.S[k]];
    }
  } else {
    // close poles: the serial walk, then its rotations on the columns of E
    // (a column that meets one of the other half gets its missing half as zeros)
    double *dfv = vec + V_LAM * N, *rc = vec + V_RC * N, *rs = vec + V_RS * N;
    int *df = idx + I_POS * N, *ra = idx + I_RA * N, *rb = idx + I_RB * N;
    if (tid == 0) {
      int nrot = 0;
      sm.K = dc_deflate_serial(sm.ds, sm.zs, n, rho, tol, sm.S, vec + V_DK * N, vec + V_ZK * N, df,
                               dfv, ra, rb, rc, rs, &nrot);
      sm.nrot = nrot;
    }
    __threadfence_block();
    __syncthreads();
    K = sm.K;
    int* flag = idx + I_FLAG * N;
    for (int q = 0; q < sm.nrot; ++q) {
      const int ca = sm.src[ra[q]], cb = sm.src[rb[q]];
      const int fa = flag[ca], fb = flag[cb];
      double* xa = p.E + (int64_t)(off + ca) * N + off;
      double* xb = p.E + (int64_t)(off + cb) * N + off;
      const double c = rc[q], s = rs[q];
      __syncthreads();
      for (int r = tid; r < n; r += kPrepThreads) {
        const int bit = r < n1 ? 1 : 2;
        if (!((fa | fb) & bit)) continue;
        const double a = fa & bit ? xa[r] : 0.0, b = fb & bit ? xb[r] : 0.0;
        xa[r] = c * a - s * b;
        xb[r] = s * a + c * b;
      }
      if (tid == 0) flag[ca] = flag[cb] = fa | fb;
      __threadfence_block();
      __syncthreads();
    }
    const int ndf = n - K;
    for (int q = tid; q < ndf; q += kPrepThreads) {
      const double val = dfv[q];
      int r = 0;
      for (int k = 0; k < ndf; ++k) r += (dfv[k] < val || (dfv[k] == val && k < q)) ? 1 : 0;
      const int col = sm.src[df[q]];
      vec[V_DFS * N + r] = val;
      idx[I_DFC * N + r] = col;
      idx[I_DFF * N + r] = flag[col];
    }
    __syncthreads();
  }
  // columns of the non-deflated poles, and their places among those with an
  // upper and with a lower part
  const int perk = (K + kPrepThreads - 1) / kPrepThreads;
  const int k0 = tid * perk, k1 = min(k0 + perk, K);
  int K1 = 0, K2 = 0;
  for (int half = 1; half <= 2; ++half) {
    int c2 = 0;
    for (int k = k0; k < k1; ++k) c2 += idx[I_FLAG * N + sm.src[sm.S[k]]] & half ? 1 : 0;
    int tot = 0;
    int pos = block_scan(c2, sm.wsum, &tot);
    for (int k = k0; k < k1; ++k) {
      const int col = sm.src[sm.S[k]];
      if (half == 1) idx[I_COL * N + k] = col;
      idx[(half == 1 ? I_P1 : I_P2) * N + k] = idx[I_FLAG * N + col] & half ? pos++ : -1;
    }
    if (half == 1) K1 = tot; else K2 = tot;
  }
  if (tid == 0) {
    res[blockIdx.x] = NodeRes{rho, K, n - K, K1, K2, neg ? 1 : 0, 0};
    JobMerge& u = jobs[2 * blockIdx.x];
    JobMerge& l = jobs[2 * blockIdx.x + 1];
    u.M = u.a.rows = l.M = l.a.rows = K;
    u.K = u.kchunk = K1;
    l.K = l.kchunk = K2;
    l.a.p = u.a.p + K1;
  }
}

// Gathered columns (workgroups [0, cols), one per column of a node) and secular
// roots (the others, four waves each one root).
__global__ __launch_bounds__(256) void k_dc_roots(const EigDev* __restrict__ P,
                                                  const Node* __restrict__ nodes, int nn,
                                                  const int* __restrict__ pre,
                                                  const int* __restrict__ preq, int cols,
                                                  const NodeRes* __restrict__ res) {
  const int tid = threadIdx.x;
  if ((int)blockIdx.x < cols) {
    const int ni = node_of(pre, nn, blockIdx.x);
    const Node nd = nodes[ni];
    const EigDev& p = P[nd.prob];
    const int N = p.n, off = nd.off, n1 = nd.n1, n = nd.n1 + nd.n2, t = blockIdx.x - pre[ni];
    const int K = res[ni].K;
    const int* idx = p.idx + off;
    double* Bc = p.B + (int64_t)off * N + off;
    if (t < K) {
      const double* Ec = p.E + (int64_t)(off + idx[I_COL * N + t]) * N + off;
      const int a = idx[I_P1 * N + t], b = idx[I_P2 * N + t];
      if (a >= 0)
        for (int r = tid; r < n1; r += 256) Bc[(int64_t)a * N + r] = Ec[r];
      if (b >= 0)
        for (int r = n1 + tid; r < n; r += 256) Bc[(int64_t)b * N + r] = Ec[r];
    } else {
      const double* Ec = p.E + (int64_t)(off + idx[I_DFC * N + t - K]) * N + off;
      const int f = idx[I_DFF * N + t - K];
      for (int r = tid; r < n; r += 256) Bc[(int64_t)t * N + r] = f & (r < n1 ? 1 : 2) ? Ec[r] : 0.0;
    }
    return;
  }
  const int q = blockIdx.x - cols;
  const int ni = node_of(preq, nn, q);
  const Node nd = nodes[ni];
  const EigDev& p = P[nd.prob];
  const int j = 4 * (q - preq[ni]) + (tid >> 6), K = res[ni].K, N = p.n;
  if (j >= K) return;
  double* vec = p.vec + nd.off;
  int org;
  double mu;
  secular_root<64>(vec + V_DK * N, vec + V_ZK * N, K, res[ni].rho, j, tid & 63,
                   [](double x) { return wave_total(x); }, org, mu);
  if ((tid & 63) == 0) {
    const double dor = vec[V_DK * N + org];
    vec[V_MU * N + j] = mu;
    vec[V_DOR * N + j] = dor;
    vec[V_LAM * N + j] = dor + mu;
  }
}

// Recomputed weights, one wave each.
__global__ __launch_bounds__(256) void k_dc_weights(const EigDev* __restrict__ P,
                                                    const Node* __restrict__ nodes, int nn,
                                                    const int* __restrict__ preq,
                                                    const NodeRes* __restrict__ res) {
  const int ni = node_of(preq, nn, blockIdx.x);
  const Node nd = nodes[ni];
  const EigDev& p = P[nd.prob];
  const int i = 4 * ((int)blockIdx.x - preq[ni]) + (threadIdx.x >> 6), K = res[ni].K, N = p.n;
  if (i >= K) return;
  double* vec = p.vec + nd.off;
  double q = 1.0;
  for (int j = threadIdx.x & 63; j < K; j += 64)
    q *= zhat_factor(vec + V_DK * N, K, res[ni].rho, i, j, vec[V_DOR * N + j], vec[V_MU * N + j]);
  q = wave_prod(q);
  if ((threadIdx.x & 63) == 0) vec[V_ZH * N + i] = copysign(sqrt(q), vec[V_ZK * N + i]);
}

// Eigenvectors of the merged matrix, one workgroup per column of a node: the
// unit vector of root t split into its parts on the upper and the lower
// columns (rows of U), or the deflated column copied to its place; the
// eigenvalue into the node's d.
__global__ __launch_bounds__(256) void k_dc_vecs(const EigDev* __restrict__ P,
                                                 const Node* __restrict__ nodes, int nn,
                                                 const int* __restrict__ pre,
                                                 const NodeRes* __restrict__ res) {
  __shared__ double red[4];
  const int ni = node_of(pre, nn, blockIdx.x);
  const Node nd = nodes[ni];
  const EigDev& p = P[nd.prob];
  const int N = p.n, off = nd.off, n = nd.n1 + nd.n2, t = blockIdx.x - pre[ni], tid = threadIdx.x;
  const int K = res[ni].K, ndf = res[ni].ndf, K1 = res[ni].K1;
  const bool neg = res[ni].neg != 0;
  double* vec = p.vec + off;
  int* idx = p.idx + off;
  if (t < K) {
    const double dor = vec[V_DOR * N + t], mu = vec[V_MU * N + t];
    const double *dk = vec + V_DK * N, *zh = vec + V_ZH * N;
    double s2 = 0.0;
    for (int i = tid; i < K; i += 256) {
      const double u = zh[i] / ((dk[i] - dor) - mu);
      s2 += u * u;
    }
    s2 = wave_total(s2);
    if ((tid & 63) == 0) red[tid >> 6] = s2;
    __syncthreads();
    const double inv = 1.0 / sqrt(red[0] + red[1] + red[2] + red[3]);
    double* Ur = p.U + (int64_t)off * N + (int64_t)t * n;
    for (int i = tid; i < K; i += 256) {
      const double u = zh[i] / ((dk[i] - dor) - mu) * inv;
      const int a = idx[I_P1 * N + i], b = idx[I_P2 * N + i];
      if (a >= 0) Ur[a] = u;
      if (b >= 0) Ur[K1 + b] = u;
    }
    if (tid == 0) {
      const double lam = vec[V_LAM * N + t];
      int pos = t + dc_count(vec + V_DFS * N, ndf, lam, false);
      if (neg) pos = n - 1 - pos;
      idx[I_POS * N + t] = pos;
      p.d[off + pos] = neg ? -lam : lam;
    }
  } else {
    const int r0 = t - K;
    const double val = vec[V_DFS * N + r0];
    int pos = r0 + dc_count(vec + V_LAM * N, K, val, true);
    if (neg) pos = n - 1 - pos;
    const double* Bc = p.B + (int64_t)(off + t) * N + off;
    double* Ec = p.E + (int64_t)(off + pos) * N + off;
    for (int r = tid; r < n; r += 256) Ec[r] = Bc[r];
    if (tid == 0) p.d[off + pos] = neg ? -val : val;
  }
}

// Eigenvalues; NaN if the problem's error flags are set.
__global__ void k_dc_finish(const EigDev* __restrict__ P, const int* __restrict__ err) {
  const EigDev& p = P[blockIdx.x];
  const double s = p.scale[S_T];
  const int ex = (int)p.scale[S_RANGE];
  const bool ok = err[blockIdx.x] == 0;
  for (int i = threadIdx.x; i < p.n; i += blockDim.x)
    p.ev[i] = !ok ? NAN : (ex == 0 ? p.d[i] * s : ldexp(p.d[i] * s, -ex));
  if (threadIdx.x == 0) p.scale[S_MAX] = 0.0;  // (for the plan's next run)
}

// ---------------------------------------------------- back-transformation --
// T of each block of kBk reflectors from their Gram matrix V^T V and tau, one
// workgroup a block (108 us by columns and halves, 36 us here).
struct TBlock {
  const double* G;
  const double* tau;
  double* T;
  int kb;
};
__global__ __launch_bounds__(256) void k_wy_t(const TBlock* __restrict__ blocks) {
  __shared__ double T[kBk][kBk + 1];
  __shared__ double tau[kBk];
  const TBlock b = blocks[blockIdx.x];
  const int tid = threadIdx.x;
  if (tid < kBk) tau[tid] = tid < b.kb ? b.tau[tid] : 0.0;
  wy_factor<kBk>([&](int i, int j) { return i < b.kb && j < b.kb ? b.G[i * kBk + j] : 0.0; }, tau, T);
  for (int e = tid; e < kBk * kBk; e += 256) b.T[e] = T[e / kBk][e % kBk];
}

// X[m][n] -= v
struct EpiMinus {
  double* X;
  int64_t ld;
  __device__ __forceinline__ void operator()(int64_t, int64_t, int64_t m, int64_t n, double v,
                                             bool) const {
    X[m * ld + n] -= v;
  }
};
typedef GemmJob<Strided<true>, Strided<true>, EpiStore> JobGW;    // Gram matrices, W = V^T X
typedef GemmJob<Strided<false>, Strided<false>, EpiStore> JobY;   // Y = V T
typedef GemmJob<Strided<false>, Strided<false>, EpiMinus> JobX;   // X -= Y W

__global__ void k_eig_out(const EigDev* __restrict__ P) {
  const EigDev& p = P[blockIdx.y];
  const int64_t nn = (int64_t)p.n * p.n, step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nn; i += step) {
    const int64_t s = i / p.n;
    p.A[s * p.ld + (i - s * p.n)] = p.E[i];
  }
}

// ------------------------------------------------------------- host side --
template <class J, class OA, class OB, class EPI>
void add_job(std::vector<J>& v, int64_t& wg, OA a, OB b, EPI e, int64_t M, int64_t N, int64_t K) {
  v.push_back(J{a, b, e, M, N, K, K > 0 ? K : 1, (M + 63) / 64, (N + 63) / 64, 1, wg});
  wg += ((M + 63) / 64) * ((N + 63) / 64);
}

// A grouped launch with fewer 64 x 64 tiles than the chip has compute units is
// bound by the matrix cores of those it reaches: it takes 32 x 32 tiles (k tiles
// of 32, half the barriers), as long as the launch stays this small.  Order 1940,
// V^T X of a block (62 tiles of 64): 59 -> 27 us.
constexpr int64_t kFewTiles = 256;
template <class J>
bool fine_tiles(std::vector<J>& v, int64_t& wg) {
  if (wg >= kFewTiles) return false;
  wg = 0;
  for (J& j : v) {
    j.tiles_m = (j.M + 31) / 32;
    j.tiles_n = (j.N + 31) / 32;
    j.wg_begin = wg;
    wg += j.tiles_m * j.tiles_n;
  }
  return true;
}

// Appends a table to the upload image; returns its offset.
template <class T>
size_t put(std::vector<char>& img, const std::vector<T>& v) {
  const size_t at = (img.size() + 255) / 256 * 256;
  img.resize(at + v.size() * sizeof(T));
  if (!v.empty()) memcpy(img.data() + at, v.data(), v.size() * sizeof(T));
  return at;
}

// Team of a problem: the smallest workgroup count whose rows hold it, in the
// shape with few rows per workgroup (`wide`: the columns of a single problem
// cost least) or with many (several problems share the chip).
void pick_team(int n, bool wide, int* cfg, int* team) {
  int c;
  if (n <= 128) c = 0;
  else if (n <= 256) c = 1;
  else if (n <= 512) c = wide ? 2 : 3;
  else if (n <= 1024) c = wide ? 4 : 5;
  else if (n <= 1536) c = wide ? 6 : 7;
  else if (n <= 2048) c = wide ? 8 : 9;
  else if (n <= 2560) c = 10;
  else c = 11;
  *cfg = c;
  *team = (n + kTeamShapes[c].rows - 1) / kTeamShapes[c].rows;
}

}  // namespace

struct EigPlan {
  struct Round {
    size_t at;
    unsigned wgs;
    bool coop;
  };
  struct Level {
    size_t nodes, pre, preq, res, jobs;
    int nn, cols, qblk;
    int64_t njobs, nwg;
    bool fine;
  };
  struct Products {
    size_t at;
    int64_t n, nwg;
    bool fine;  // 32 x 32 tiles
  };
  struct Step {
    Products w, x;
  };
  std::vector<EigProblem> prob;
  std::vector<char> img;  // host image of the device tables (alive until the run's last wait)
  char* dev = nullptr;
  int* err = nullptr;
  double* scale = nullptr;
  size_t probs = 0, base = 0, tblocks = 0;
  unsigned count = 0, nbase = 0, ntb = 0;
  bool clear = false;
  std::vector<Round> rounds;
  std::vector<Level> levels;
  Products gram{}, y{};
  std::vector<Step> steps;
};

EigPlan* eig_plan_new() { return new (std::nothrow) EigPlan(); }
void eig_plan_free(EigPlan* p) { delete p; }

// Workgroups of k_tri_team the device holds at once (0: cooperative launches are not available).
static int team_budget(qsgw_ctx* c) {
  if (c->team_wgs < 0) {
    int coop = 0, cus = 0, per = 0;
    c->team_wgs = 0;
    if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, c->device) == hipSuccess &&
        coop &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c->device) == hipSuccess &&
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, reinterpret_cast<const void*>(&k_tri_team),
                                                     kTeamThreads, 0) == hipSuccess)
      c->team_wgs = cus * per;
    (void)hipGetLastError();
  }
  return c->team_wgs;
}

bool eig_team_fits(qsgw_ctx* c, int64_t n) {
  if (n < 1 || n > kEigTeamMax) return false;
  int cfg, team;
  pick_team((int)n, false, &cfg, &team);
  return team <= 1 || team <= team_budget(c);
}

// Tables of the divide and conquer: base blocks, then the merges level by level.
static void plan_merges(EigPlan* pl, const std::vector<EigDev>& P) {
  std::vector<BaseNode> base;
  std::vector<std::vector<Node>> lev;
  struct Rec {
    int prob, off, n, depth;
  };
  std::vector<Rec> stack;
  for (size_t i = 0; i < P.size(); ++i) stack.push_back({(int)i, 0, P[i].n, 0});
  while (!stack.empty()) {
    const Rec r = stack.back();
    stack.pop_back();
    if (r.n <= kBase) {
      base.push_back({r.prob, r.off, r.n});
      continue;
    }
    if ((int)lev.size() <= r.depth) lev.resize((size_t)r.depth + 1);
    const int n1 = r.n / 2;
    lev[(size_t)r.depth].push_back({r.prob, r.off, n1, r.n - n1});
    stack.push_back({r.prob, r.off, n1, r.depth + 1});
    stack.push_back({r.prob, r.off + n1, r.n - n1, r.depth + 1});
  }
  pl->base = put(pl->img, base);
  pl->nbase = (unsigned)base.size();
  for (size_t dep = lev.size(); dep-- > 0;) {
    std::vector<int> pre, preq;
    std::vector<JobMerge> jobs;
    std::vector<NodeRes> res(lev[dep].size());
    int cols = 0, qb = 0;
    int64_t wg = 0;
    for (const Node& nd2 : lev[dep]) {
      const EigDev& p = P[(size_t)nd2.prob];
      const int64_t N = p.n, n = nd2.n1 + nd2.n2, off = nd2.off;
      pre.push_back(cols);
      preq.push_back(qb);
      cols += (int)n;
      qb += (int)((n + 3) / 4);
      const double* Ub = p.U + off * N;
      const double* Bb = p.B + off * N + off;
      const int* pos = p.idx + I_POS * N + off;
      double* Eb = p.E + off * N + off;
      add_job(jobs, wg, Strided<true>{Ub, n, 1, 0, n}, Strided<false>{Bb, 1, N, 0, nd2.n1},
              EpiEigCols{Eb, N, pos}, n, nd2.n1, n);
      add_job(jobs, wg, Strided<true>{Ub, n, 1, 0, n}, Strided<false>{Bb + nd2.n1, 1, N, 0, nd2.n2},
              EpiEigCols{Eb + nd2.n1, N, pos}, n, nd2.n2, n);
    }
    EigPlan::Level L;
    L.fine = fine_tiles(jobs, wg);
    L.nodes = put(pl->img, lev[dep]);
    L.pre = put(pl->img, pre);
    L.preq = put(pl->img, preq);
    L.res = put(pl->img, res);
    L.jobs = put(pl->img, jobs);
    L.nn = (int)lev[dep].size();
    L.cols = cols;
    L.qblk = qb;
    L.njobs = (int64_t)jobs.size();
    L.nwg = wg;
    pl->levels.push_back(L);
  }
}

// Error flags and range words cleared.
static int init_plan(qsgw_ctx* c, const EigPlan* pl) {
  hipLaunchKernelGGL(k_eig_init, dim3(blocks_for((int64_t)pl->count * kScale)), dim3(256), 0,
                     c->stream, pl->scale, pl->err, (int64_t)pl->count);
  return launch_check(c, "k_eig_init");
}

int eig_plan(qsgw_ctx* c, EigPlan* pl, const EigProblem* prob, int64_t count, int set) {
  pl->count = (unsigned)count;
  pl->prob.assign(prob, prob + count);
  std::vector<EigDev> P((size_t)count);
  // ---- sizes and teams ----
  int64_t wide_wgs = 0;
  for (int64_t i = 0; i < count; ++i) {
    int cfg, team;
    pick_team((int)prob[i].n, true, &cfg, &team);
    wide_wgs += team;
  }
  const int budget = team_budget(c);
  const bool wide = wide_wgs <= budget;
  size_t nd = 8, ni = (size_t)count;
  for (int64_t i = 0; i < count; ++i) {
    const int64_t n = prob[i].n, nb = (n - 1 + kBk - 1) / kBk;
    nd += (size_t)(3 * n * n + (3 + kVec) * n + 2 + 2 * nb * kBk * kBk + kScale);
    ni += (size_t)(kIdx * n);
  }
  double* D = nullptr;
  int* I = nullptr;
  CHECK(ws_get(c, W_EIGD_F + 3 * set, nd, &D));
  CHECK(ws_get(c, W_EIGD_I + 3 * set, ni, &I));
  pl->err = I;
  I += count;
  pl->scale = D;
  D += kScale * count;
  CHECK(init_plan(c, pl));
  for (int64_t i = 0; i < count; ++i) {
    const int64_t n = prob[i].n, nb = (n - 1 + kBk - 1) / kBk;
    EigDev& p = P[(size_t)i];
    p.A = prob[i].A;
    p.ev = prob[i].evals;
    p.ld = prob[i].ld;
    p.n = (int)n;
    p.pad = 0;
    pick_team((int)n, wide, &p.cfg, &p.team);
    p.E = D;
    p.B = D + n * n;
    p.U = D + 2 * n * n;
    D += (3 * n * n + 1) / 2 * 2;  // (16-byte slots of the exchange)
    p.d = D;
    p.e = D + n;
    p.tau = D + 2 * n;
    p.vec = D + 3 * n;
    D += ((3 + kVec) * n + 1) / 2 * 2;
    p.G = D;
    p.T = D + nb * kBk * kBk;
    D += 2 * nb * kBk * kBk;
    p.scale = pl->scale + kScale * i;
    p.idx = I;
    I += kIdx * n;
    pl->clear = pl->clear || p.team > 1;
  }
  pl->probs = put(pl->img, P);
  // ---- reduction rounds: largest first, each round filled up with what still fits ----
  std::vector<int> order((size_t)count);
  for (int64_t i = 0; i < count; ++i) order[(size_t)i] = (int)i;
  std::sort(order.begin(), order.end(), [&](int a, int b) {
    return P[(size_t)a].n != P[(size_t)b].n ? P[(size_t)a].n > P[(size_t)b].n : a < b;
  });
  // (a problem in one workgroup needs no other one resident: it fills a round up,
  // and what is left of them goes out in a launch of its own)
  std::vector<char> done((size_t)count, 0);
  std::vector<std::vector<TeamWg>> coop;
  auto add = [&](std::vector<TeamWg>& wg, int i) {
    for (int g = 0; g < P[(size_t)i].team; ++g) wg.push_back({i, g});
    done[(size_t)i] = 1;
  };
  for (int first : order) {
    if (done[(size_t)first] || P[(size_t)first].team <= 1) continue;
    if (P[(size_t)first].team > budget)
      return fail(c, QSGW_ERR_UNSUPPORTED, "eigensolver: a team exceeds the device");
    std::vector<TeamWg> wg;
    for (int i : order)
      if (!done[(size_t)i] && (int64_t)wg.size() + P[(size_t)i].team <= budget) add(wg, i);
    coop.push_back(std::move(wg));
  }
  // (the largest launch first: see eig_run)
  std::stable_sort(coop.begin(), coop.end(), [](const auto& a, const auto& b) { return a.size() > b.size(); });
  for (const auto& wg : coop) pl->rounds.push_back({put(pl->img, wg), (unsigned)wg.size(), true});
  std::vector<TeamWg> rest;
  for (int i : order)
    if (!done[(size_t)i]) add(rest, i);
  if (!rest.empty()) pl->rounds.push_back({put(pl->img, rest), (unsigned)rest.size(), false});
  plan_merges(pl, P);
  // ---- back-transformation ----
  std::vector<JobGW> gram;
  std::vector<JobY> yj;
  std::vector<TBlock> tb;
  int64_t gwg = 0, ywg = 0, maxb = 0;
  auto blocks = [](int64_t n) { return (n - 1 + kBk - 1) / kBk; };
  for (const EigDev& p : P) {
    const int64_t n = p.n, nb = blocks(n);
    maxb = std::max(maxb, nb);
    for (int64_t b = 0; b < nb; ++b) {
      const int64_t j0 = b * kBk, kb = std::min<int64_t>(kBk, n - 1 - j0), len = n - 1 - j0;
      const double* V = p.A + j0 * p.ld;  // (v_j is zero from column n - 1 - j on)
      double *G = p.G + b * kBk * kBk, *T = p.T + b * kBk * kBk;
      add_job(gram, gwg, Strided<true>{V, p.ld, 1, 0, kb}, Strided<true>{V, p.ld, 1, 0, kb},
              EpiStore{G, kBk, 0, 0, 1.0}, kb, kb, len);
      tb.push_back({G, p.tau + j0, T, (int)kb});
      add_job(yj, ywg, Strided<false>{T, 1, kBk, 0, kb}, Strided<false>{V, 1, p.ld, 0, len},
              EpiStore{p.U + j0 * n, n, 0, 0, 1.0}, kb, len, kb);
    }
  }
  const bool gf = fine_tiles(gram, gwg), yf = fine_tiles(yj, ywg);
  pl->gram = {put(pl->img, gram), (int64_t)gram.size(), gwg, gf};
  pl->y = {put(pl->img, yj), (int64_t)yj.size(), ywg, yf};
  pl->tblocks = put(pl->img, tb);
  pl->ntb = (unsigned)tb.size();
  for (int64_t s = 0; s < maxb; ++s) {
    std::vector<JobGW> wj;
    std::vector<JobX> xj;
    int64_t wwg = 0, xwg = 0;
    for (const EigDev& p : P) {
      const int64_t n = p.n, b = blocks(n) - 1 - s;
      if (b < 0) continue;
      const int64_t j0 = b * kBk, kb = std::min<int64_t>(kBk, n - 1 - j0), len = n - 1 - j0;
      const double* V = p.A + j0 * p.ld;
      add_job(wj, wwg, Strided<true>{V, p.ld, 1, 0, kb}, Strided<true>{p.E, n, 1, 0, n},
              EpiStore{p.B, n, 0, 0, 1.0}, kb, n, len);
      add_job(xj, xwg, Strided<false>{p.B, 1, n, 0, n},
              Strided<false>{p.U + j0 * n, 1, n, 0, len}, EpiMinus{p.E, n}, n, len, kb);
    }
    EigPlan::Step st;
    const bool wf = fine_tiles(wj, wwg), xf = fine_tiles(xj, xwg);
    st.w = {put(pl->img, wj), (int64_t)wj.size(), wwg, wf};
    st.x = {put(pl->img, xj), (int64_t)xj.size(), xwg, xf};
    pl->steps.push_back(st);
  }
  CHECK(ws_get(c, W_EIGD_T + 3 * set, pl->img.size() + 256, &pl->dev));
  HIP_TRY(c, hipMemcpyAsync(pl->dev, pl->img.data(), pl->img.size(), hipMemcpyHostToDevice,
                            c->stream));
  return QSGW_OK;
}

template <class J>
static int run_products(qsgw_ctx* c, const EigPlan* pl, const EigPlan::Products& g, const J*,
                        const char* what) {
  if (g.nwg <= 0) return QSGW_OK;
  if (g.nwg > 0x7fffffffLL) return fail(c, QSGW_ERR_INVALID_ARG, "%s: launch too large", what);
  const J* jobs = reinterpret_cast<const J*>(pl->dev + g.at);
  typedef decltype(jobs->a) OA;
  typedef decltype(jobs->b) OB;
  typedef decltype(jobs->e) EP;
  if (g.fine)
    hipLaunchKernelGGL((gemm_grouped_kernel<32, 32, OA, OB, EP, false, 32>),
                       dim3((unsigned)g.nwg), dim3(256), 0, c->stream, jobs, g.n, g.nwg);
  else
    hipLaunchKernelGGL((gemm_grouped_kernel<64, 64, OA, OB, EP, false>), dim3((unsigned)g.nwg),
                       dim3(256), 0, c->stream, jobs, g.n, g.nwg);
  return launch_check(c, what);
}

// Eigenpairs of every problem's d, e: E, and ev ascending.
static int run_merges(qsgw_ctx* c, const EigPlan* pl, const EigDev* P) {
  hipLaunchKernelGGL(k_dc_scale, dim3(pl->count), dim3(256), 0, c->stream, P, pl->err);
  hipLaunchKernelGGL(k_dc_base, dim3(pl->nbase), dim3(kBaseThreads), 0, c->stream, P,
                     reinterpret_cast<const BaseNode*>(pl->dev + pl->base), pl->err);
  CHECK(launch_check(c, "k_dc_base"));
  for (const auto& L : pl->levels) {
    const Node* nodes = reinterpret_cast<const Node*>(pl->dev + L.nodes);
    const int* pre = reinterpret_cast<const int*>(pl->dev + L.pre);
    const int* preq = reinterpret_cast<const int*>(pl->dev + L.preq);
    NodeRes* res = reinterpret_cast<NodeRes*>(pl->dev + L.res);
    JobMerge* jobs = reinterpret_cast<JobMerge*>(pl->dev + L.jobs);
    hipLaunchKernelGGL(k_dc_prep, dim3((unsigned)L.nn), dim3(kPrepThreads), 0, c->stream, P, nodes,
                       res, jobs);
    hipLaunchKernelGGL(k_dc_roots, dim3((unsigned)(L.cols + L.qblk)), dim3(256), 0, c->stream, P,
                       nodes, L.nn, pre, preq, L.cols, res);
    hipLaunchKernelGGL(k_dc_weights, dim3((unsigned)L.qblk), dim3(256), 0, c->stream, P, nodes, L.nn,
                       preq, res);
    hipLaunchKernelGGL(k_dc_vecs, dim3((unsigned)L.cols), dim3(256), 0, c->stream, P, nodes, L.nn,
                       pre, res);
    CHECK(launch_check(c, "k_dc_vecs"));
    CHECK(run_products(c, pl, EigPlan::Products{L.jobs, L.njobs, L.nwg, L.fine}, (const JobMerge*)nullptr,
                       "eig merge"));
  }
  hipLaunchKernelGGL(k_dc_finish, dim3(pl->count), dim3(256), 0, c->stream, P, pl->err);
  return launch_check(c, "k_dc_finish");
}

// Every problem of the plan by rocSOLVER dsyevd, one after another.
static int run_library(qsgw_ctx* c, const EigPlan* pl) {
  CHECK(init_plan(c, pl));  // (the range words of the round that did not run)
  for (const EigProblem& p : pl->prob) {
    if (p.ld != p.n) return fail(c, QSGW_ERR_UNSUPPORTED, "eigensolver: ld %lld", (long long)p.ld);
    CHECK(syevd(c, p.n, p.A, p.evals, "eigensolver"));
  }
  return QSGW_OK;
}

int eig_run(qsgw_ctx* c, const EigPlan* pl) {
  const EigDev* P = reinterpret_cast<const EigDev*>(pl->dev + pl->probs);
  const dim3 per_prob(pl->count > 8 ? 64 : 512, pl->count);
  if (pl->clear) hipLaunchKernelGGL(k_tri_clear, per_prob, dim3(256), 0, c->stream, P);
  CHECK(launch_check(c, "k_tri_clear"));
  for (const auto& r : pl->rounds) {
    const TeamWg* wg = reinterpret_cast<const TeamWg*>(pl->dev + r.at);
    int* err = pl->err;
    if (r.coop) {
      CHECK(aux_queues(c));
      void* args[] = {&P, &wg, &err};
      const hipError_t e =
          hipLaunchCooperativeKernel(reinterpret_cast<const void*>(&k_tri_team), dim3(r.wgs),
                                     dim3(kTeamThreads), args, 0, c->stream);
      if (e != hipSuccess) {
        // The device does not take the launch now, whatever its properties say
        // (another process may hold its queue for them).  A refusal of the first and
        // largest round leaves the matrices as they were; one after that means that
        // something else is wrong.
        (void)hipGetLastError();
        if (&r != &pl->rounds.front())
          return fail(c, QSGW_ERR_HIP, "cooperative launch: %s", hipGetErrorString(e));
        return run_library(c, pl);
      }
    } else {
      hipLaunchKernelGGL(k_tri_team, dim3(r.wgs), dim3(kTeamThreads), 0, c->stream, P, wg, err);
    }
    CHECK(launch_check(c, "k_tri_team"));
  }
  CHECK(run_merges(c, pl, P));
  CHECK(run_products(c, pl, pl->gram, (const JobGW*)nullptr, "eig Gram"));
  if (pl->ntb > 0)
    hipLaunchKernelGGL(k_wy_t, dim3(pl->ntb), dim3(256), 0, c->stream,
                       reinterpret_cast<const TBlock*>(pl->dev + pl->tblocks));
  CHECK(launch_check(c, "k_wy_t"));
  CHECK(run_products(c, pl, pl->y, (const JobY*)nullptr, "eig V T"));
  for (const auto& s : pl->steps) {
    CHECK(run_products(c, pl, s.w, (const JobGW*)nullptr, "eig V^T X"));
    CHECK(run_products(c, pl, s.x, (const JobX*)nullptr, "eig X update"));
  }
  hipLaunchKernelGGL(k_eig_out, per_prob, dim3(256), 0, c->stream, P);
  return launch_check(c, "k_eig_out");
}

// Error flags of the plan's runs so far (synchronizes); *at the first failing problem.
int eig_check(qsgw_ctx* c, const EigPlan* pl, const char* what, int64_t* at) {
  std::vector<int> e(pl->count, 0);
  HIP_TRY(c, hipMemcpyAsync(e.data(), pl->err, e.size() * sizeof(int), hipMemcpyDeviceToHost,
                            c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  for (size_t i = 0; i < e.size(); ++i) {
    if (!e[i]) continue;
    if (at) *at = (int64_t)i;
    if (e[i] & 1) return fail(c, QSGW_ERR_SOLVER, "%s: reduction wait exceeded its bound", what);
    if (e[i] & 4) return fail(c, QSGW_ERR_NONFINITE, "%s: a value is not finite", what);
    return fail(c, QSGW_ERR_SOLVER, "%s: a tridiagonal block did not converge", what);
  }
  return QSGW_OK;
}

int eig_team(qsgw_ctx* c, int64_t n, double* A, double* evals, const char* what) {
  EigPlan pl;
  const EigProblem p{n, n, A, evals};
  CHECK(eig_plan(c, &pl, &p, 1, 0));
  CHECK(eig_run(c, &pl));
  return eig_check(c, &pl, what, nullptr);
}

// Eigenpairs of the tridiagonal d, e of order n <= kEigTridiagMax: d ascending
// eigenvalues, E [n][n] the eigenvectors (column-major); e is destroyed.
int eig_tridiag(qsgw_ctx* c, int64_t n, double* d, double* e, double* E, const char* what) {
  if (n < 1 || n > kEigTridiagMax)
    return fail(c, QSGW_ERR_UNSUPPORTED, "%s: tridiagonal order %lld", what, (long long)n);
  EigPlan pl;
  pl.count = 1;
  double* D = nullptr;
  int* I = nullptr;
  CHECK(ws_get(c, W_EIGD_F, (size_t)(2 * n * n + kVec * n + kScale), &D));
  CHECK(ws_get(c, W_EIGD_I, (size_t)(1 + kIdx * n), &I));
  pl.err = I;
  pl.scale = D + 2 * n * n + kVec * n;
  CHECK(init_plan(c, &pl));
  EigDev p{};
  p.n = (int)n;
  p.ev = p.d = d;
  p.e = e;
  p.E = E;
  p.B = D;
  p.U = D + n * n;
  p.vec = D + 2 * n * n;
  p.scale = pl.scale;
  p.idx = I + 1;
  const std::vector<EigDev> P(1, p);
  pl.probs = put(pl.img, P);
  plan_merges(&pl, P);
  CHECK(ws_get(c, W_EIGD_T, pl.img.size() + 256, &pl.dev));
  HIP_TRY(c, hipMemcpyAsync(pl.dev, pl.img.data(), pl.img.size(), hipMemcpyHostToDevice,
                            c->stream));
  CHECK(run_merges(c, &pl, reinterpret_cast<const EigDev*>(pl.dev + pl.probs)));
  int64_t at = 0;
  return eig_check(c, &pl, what, &at);
}
