// Dense form of an orbital rotation (Sec. 2.3): Gamma' = C_{n_a}(U_a) Gamma C_{n_b}(U_b)^T with the
// compound matrices C_n(U)[J, I] = det U[J, I] (rows J and columns I the occupied orbitals of two
// configurations, ascending).  It is the plain definition of script-U(U) on the sector, evaluated as
// two complex matrix products on the FP64 matrix cores; the Givens sweeps reach the same result with
// 20 n (N - n) d^2 flops against this form's 16 d^3, so it is taken
// for small sectors only, where both are bound by latency.
//   * k_compound<n>: one thread per entry, the n x n minor gathered into registers and reduced by
//     Gaussian elimination with partial pivoting in complex FP64; both spins in one launch where that
//     costs nothing.
//   * Y = A B (complex128, row-major A and Y, B addressed through two strides so that C^T needs no
//     copy) by v_mfma_f64_16x16x4, the real and imaginary accumulators of a 16 x 16 tile taking four
//     products per k step: k_zgemm_tile for small products, k_zgemm_mfma for large ones.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <cstring>

#include "dev_common.h"
#include "device.h"

namespace ffx {
namespace dev {

// U (row-major complex norb x norb) from a buffer or, for up to kArgOrb
// orbitals, out of the kernel's own arguments: no upload before the launch.
constexpr int kArgOrb = 11;
struct CompoundSpin {
  const uint32_t* masks;
  const double* U;  // null: the arguments hold it
  zc128* C;
  int d, n;
};
struct CompoundArgs {
  CompoundSpin sp[2];
  int norb;
  int per;       // entries of a thread
  int which[2];  // the matrix in u that spin blockIdx.y takes
  double u[2][2 * kArgOrb * kArgOrb];
};

template <int NE>
__device__ __forceinline__ zc128 minor_det(uint32_t mj, uint32_t mi, int norb, const double* U) {
  if constexpr (NE == 0) {
    return zc128{1.0, 0.0};
  } else {
    int r[NE], c[NE];
#pragma unroll
    for (int k = 0; k < NE; ++k) {
      r[k] = __builtin_ctz(mj);
      mj &= mj - 1;
      c[k] = __builtin_ctz(mi);
      mi &= mi - 1;
    }
    double ar[NE][NE], ai[NE][NE];
#pragma unroll
    for (int p = 0; p < NE; ++p)
#pragma unroll
      for (int q = 0; q < NE; ++q) {
        ar[p][q] = U[2 * (r[p] * norb + c[q])];
        ai[p][q] = U[2 * (r[p] * norb + c[q]) + 1];
      }
    double dr = 1.0, di = 0.0;
#pragma unroll
    for (int k = 0; k < NE; ++k) {
      // pivot: the largest |a[p][k]| for p >= k; rows swapped by selects (fixed register indices)
      int piv = k;
      double best = ar[k][k] * ar[k][k] + ai[k][k] * ai[k][k];
#pragma unroll
      for (int p = k + 1; p < NE; ++p) {
        const double m = ar[p][k] * ar[p][k] + ai[p][k] * ai[p][k];
        if (m > best) {
          best = m;
          piv = p;
        }
      }
#pragma unroll
      for (int p = k + 1; p < NE; ++p) {
        const bool sw = p == piv;
#pragma unroll
        for (int q = k; q < NE; ++q) {
          const double tr = ar[k][q], ti = ai[k][q];
          ar[k][q] = sw ? ar[p][q] : tr;
          ai[k][q] = sw ? ai[p][q] : ti;
          ar[p][q] = sw ? tr : ar[p][q];
          ai[p][q] = sw ? ti : ai[p][q];
        }
      }
      if (piv != k) {
        dr = -dr;
        di = -di;
      }
      const double pr = ar[k][k], pi = ai[k][k];
      const double nr = dr * pr - di * pi, ni = dr * pi + di * pr;
      dr = nr;
      di = ni;
      if (best == 0.0) break;
      const double inv = 1.0 / best;  // 1 / pivot = conj(pivot) / |pivot|^2
      const double vr = pr * inv, vi = -pi * inv;
#pragma unroll
      for (int p = k + 1; p < NE; ++p) {
        const double fr = ar[p][k] * vr - ai[p][k] * vi, fi = ar[p][k] * vi + ai[p][k] * vr;
#pragma unroll
        for (int q = k + 1; q < NE; ++q) {
          ar[p][q] -= fr * ar[k][q] - fi * ai[k][q];
          ai[p][q] -= fr * ai[k][q] + fi * ar[k][q];
        }
      }
    }
    return zc128{dr, di};
  }
}

// Minors of LO or (HI = LO + 1) of either size.  The kernel of two sizes has the
// registers of the larger one (152 for 7 and 8, 120 for 7 alone): 860 us per
// matrix of 7 electrons at d = 3432, 630 us with 7 alone.
template <int LO, int HI>
__global__ __launch_bounds__(256) void k_compound(CompoundArgs) {
  extern __shared__ double su[];
  // (through the argument segment's address: indexed by lane, the struct itself would be copied to scratch)
  const CompoundArgs* P = (const CompoundArgs*)(uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
  const CompoundSpin sp = uniform_load(P->sp + blockIdx.y);
  const int norb = P->norb;
  const double* U = sp.U ? sp.U : P->u[P->which[blockIdx.y]];
  for (int i = threadIdx.x; i < 2 * norb * norb; i += 256) su[i] = U[i];
  __syncthreads();
  const int64_t d = sp.d;
  int64_t idx = (int64_t)blockIdx.x * P->per * 256 + threadIdx.x;
  for (int k = P->per; k > 0 && idx < d * d; --k, idx += 256) {
    const int64_t J = idx / d, I = idx - J * d;
    const uint32_t mj = sp.masks[J], mi = sp.masks[I];
    if (LO == HI || sp.n == LO)
      sp.C[idx] = minor_det<LO>(mj, mi, norb, su);
    else
      sp.C[idx] = minor_det<HI>(mj, mi, norb, su);
  }
}

int compound_arg_orbitals() { return kArgOrb; }

// Spins of different electron numbers share a launch while all its blocks fit
// the chip at once (two of 256 threads to a compute unit for each spin), where
// the launch is what counts.
constexpr int64_t kSharedEntries = 2 * 256 * 256;

void compound_matrices(const uint32_t* const masks[2], const int64_t d[2], const int n[2], int norb,
                       const double* const hU[2], const double* const dU[2], void* const C[2], hipStream_t s) {
  CompoundArgs a;
  a.norb = norb;
  for (int k = 0; k < 2; ++k) {
    a.sp[k] = CompoundSpin{masks[k], dU[k], (zc128*)C[k], (int)d[k], n[k]};
    a.which[k] = k;
    if (!dU[k]) std::memcpy(a.u[k], hU[k], sizeof(double) * 2 * norb * norb);
  }
  const size_t lds = sizeof(double) * 2 * norb * norb;
  auto grid = [&](int64_t dm, int spins) {
    // several entries to a thread where blocks abound: each stages all of U
    const int64_t groups = (dm * dm + 255) / 256;
    a.per = groups >= 4 * 4096 ? 4 : 1;
    return dim3((unsigned)((groups + a.per - 1) / a.per), (unsigned)spins);
  };
  auto one = [&](int size, int64_t dm, int spins) {
    const dim3 g = grid(dm, spins), b(256);
    switch (size) {
      case 0: hipLaunchKernelGGL((k_compound<0, 0>), g, b, lds, s, a); break;
      case 1: hipLaunchKernelGGL((k_compound<1, 1>), g, b, lds, s, a); break;
      case 2: hipLaunchKernelGGL((k_compound<2, 2>), g, b, lds, s, a); break;
      case 3: hipLaunchKernelGGL((k_compound<3, 3>), g, b, lds, s, a); break;
      case 4: hipLaunchKernelGGL((k_compound<4, 4>), g, b, lds, s, a); break;
      case 5: hipLaunchKernelGGL((k_compound<5, 5>), g, b, lds, s, a); break;
      case 6: hipLaunchKernelGGL((k_compound<6, 6>), g, b, lds, s, a); break;
      case 7: hipLaunchKernelGGL((k_compound<7, 7>), g, b, lds, s, a); break;
      default: hipLaunchKernelGGL((k_compound<8, 8>), g, b, lds, s, a); break;
    }
  };
  auto two = [&](int lo, int64_t dm) {
    const dim3 g = grid(dm, 2), b(256);
    switch (lo) {
      case 0: hipLaunchKernelGGL((k_compound<0, 1>), g, b, lds, s, a); break;
      case 1: hipLaunchKernelGGL((k_compound<1, 2>), g, b, lds, s, a); break;
      case 2: hipLaunchKernelGGL((k_compound<2, 3>), g, b, lds, s, a); break;
      case 3: hipLaunchKernelGGL((k_compound<3, 4>), g, b, lds, s, a); break;
      case 4: hipLaunchKernelGGL((k_compound<4, 5>), g, b, lds, s, a); break;
      case 5: hipLaunchKernelGGL((k_compound<5, 6>), g, b, lds, s, a); break;
      case 6: hipLaunchKernelGGL((k_compound<6, 7>), g, b, lds, s, a); break;
      default: hipLaunchKernelGGL((k_compound<7, 8>), g, b, lds, s, a); break;
    }
  };
  const int64_t dmax = std::max(d[0], d[1]);
  if (C[0] == C[1]) {
    one(n[0], d[0], 1);
  } else if (n[0] == n[1]) {
    one(n[0], dmax, 2);
  } else if (std::abs(n[0] - n[1]) == 1 && dmax * dmax <= kSharedEntries) {
    two(std::min(n[0], n[1]), dmax);
  } else {
    one(n[0], d[0], 1);
    a.sp[0] = a.sp[1];
    a.which[0] = 1;
    one(n[1], d[1], 1);
  }
}

// ---------------------------------------------------------------------------
// complex128 GEMM on the FP64 matrix cores.  v_mfma_f64_16x16x4: lane l holds
// A[l % 16][l / 16] and B[l / 16][l % 16] and receives D[l / 16 + 4 t][l % 16],
// t = 0..3.  Re Y += Ar Br - Ai Bi and Im Y += Ar Bi + Ai Br: four products
// into two accumulators per 16 x 16 tile.
// ---------------------------------------------------------------------------
typedef double zg_d4 __attribute__((ext_vector_type(4)));

// One 16 x 16 output tile per block, the k steps dealt to its four waves and
// their sums added in wave order.  Operands come straight from memory: a step's
// 2 KB cost 256 cycles of matrix work, which the L2 keeps up with.  For
// products with few tiles of 64 x 64, which leave most compute units idle.  70^3:
// 4.4 us (k_zgemm_mfma: 15.3 us in 4 blocks); 330^3 12 us (59 us).
constexpr int kZU = 4;  // k steps whose operands are requested together
__global__ __launch_bounds__(256) void k_zgemm_tile(const zc128* __restrict__ A, int64_t lda,
                                                    const zc128* __restrict__ B, int64_t sbk, int64_t sbn,
                                                    zc128* __restrict__ Y, int64_t ldy, int M, int N, int K) {
  __shared__ zc128 part[4][256];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m0 = blockIdx.y * 16, n0 = blockIdx.x * 16;
  const int r = lane & 15, q = lane >> 4;
  // rows and columns past the edge repeat the last one and are not stored
  const zc128* a = A + (int64_t)min(m0 + r, M - 1) * lda;
  const zc128* b = B + (int64_t)min(n0 + r, N - 1) * sbn;
  zg_d4 re{0.0, 0.0, 0.0, 0.0}, im = re;
  for (int k0 = 4 * wave; k0 < K; k0 += 16 * kZU) {
    zc128 av[kZU], bv[kZU];
#pragma unroll
    for (int u = 0; u < kZU; ++u) {
      const int k = k0 + 16 * u + q, kc = min(k, K - 1);
      av[u] = a[kc];
      bv[u] = b[(int64_t)kc * sbk];
      if (k >= K) av[u] = bv[u] = zc128{0.0, 0.0};
    }
#pragma unroll
    for (int u = 0; u < kZU; ++u) {
      re = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u].x, bv[u].x, re, 0, 0, 0);
      im = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u].x, bv[u].y, im, 0, 0, 0);
      re = __builtin_amdgcn_mfma_f64_16x16x4f64(-av[u].y, bv[u].y, re, 0, 0, 0);
      im = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u].y, bv[u].x, im, 0, 0, 0);
    }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) part[wave][16 * (q + 4 * t) + r] = zc128{re[t], im[t]};
  __syncthreads();
  const int gm = m0 + (tid >> 4), gn = n0 + (tid & 15);
  if (gm >= M || gn >= N) return;
  zc128 y = part[0][tid];
#pragma unroll
  for (int w = 1; w < 4; ++w) {
    y.x += part[w][tid].x;
    y.y += part[w][tid].y;
  }
  Y[(int64_t)gm * ldy + gn] = y;
}

constexpr int kGT = 64;  // output tile edge
constexpr int kGK = 16;  // k slice

__global__ __launch_bounds__(256) void k_zgemm_mfma(const zc128* __restrict__ A, int64_t lda,
                                                    const zc128* __restrict__ B, int64_t sbk, int64_t sbn,
                                                    zc128* __restrict__ Y, int64_t ldy, int M, int N, int K) {
  __shared__ double sar[kGK][kGT + 1], sai[kGK][kGT + 1];  // A slice, [k][m]
  __shared__ double sbr[kGK][kGT + 1], sbi[kGK][kGT + 1];  // B slice, [k][n]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m0 = blockIdx.y * kGT, n0 = blockIdx.x * kGT;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  const bool bk_fast = sbk == 1;
  zg_d4 re[2][2], im[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      re[i][j] = zg_d4{0.0, 0.0, 0.0, 0.0};
      im[i][j] = re[i][j];
    }
  for (int k0 = 0; k0 < K; k0 += kGK) {
    zc128 av[4], bv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = tid + 256 * u;
      const int am = e >> 4, ak = e & 15;  // k fastest: 16 consecutive elements of a row of A
      const int gm = m0 + am, gk = k0 + ak;
      av[u] = (gm < M && gk < K) ? A[(int64_t)gm * lda + gk] : zc128{0.0, 0.0};
      const int bk = bk_fast ? (e & 15) : (e >> 6), bn = bk_fast ? (e >> 4) : (e & 63);
      const int hk = k0 + bk, hn = n0 + bn;
      bv[u] = (hk < K && hn < N) ? B[(int64_t)hk * sbk + (int64_t)hn * sbn] : zc128{0.0, 0.0};
    }
    __syncthreads();  // the previous slice's readers are done
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = tid + 256 * u;
      sar[e & 15][e >> 4] = av[u].x;
      sai[e & 15][e >> 4] = av[u].y;
      const int bk = bk_fast ? (e & 15) : (e >> 6), bn = bk_fast ? (e >> 4) : (e & 63);
      sbr[bk][bn] = bv[u].x;
      sbi[bk][bn] = bv[u].y;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < kGK; kk += 4) {
      const int k = kk + (lane >> 4);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const double ar = sar[k][wm + 16 * i + (lane & 15)], ai = sai[k][wm + 16 * i + (lane & 15)];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const double br = sbr[k][wn + 16 * j + (lane & 15)], bi = sbi[k][wn + 16 * j + (lane & 15)];
          re[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, br, re[i][j], 0, 0, 0);
          re[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(-ai, bi, re[i][j], 0, 0, 0);
          im[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, bi, im[i][j], 0, 0, 0);
          im[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ai, br, im[i][j], 0, 0, 0);
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int gm = m0 + wm + 16 * i + (lane >> 4) + 4 * t, gn = n0 + wn + 16 * j + (lane & 15);
        if (gm < M && gn < N) Y[(int64_t)gm * ldy + gn] = zc128{re[i][j][t], im[i][j][t]};
      }
}

// 64 x 64 tiles once they fill the compute units, nine in ten of them: above, the
// smaller tiles read operands too often.  A rotation's two products, 16 x 16
// against 64 x 64 tiles: 225 tiles (924 x 924) 307 and 336 us, 195 tiles (924 x
// 792) 274 and 306, 192 tiles (364 x 2002) 412 and 416; 246 tiles (325 x 2600) 608
// and 524, 252 tiles (715 x 1287) 428 and 370, 256 tiles (1001 x 1001) 451 and 361.
constexpr unsigned kTileBlocks = 230;

void zgemm_mfma(const void* A, int64_t lda, const void* B, int64_t sbk, int64_t sbn, void* Y, int64_t ldy, int M,
                int N, int K, hipStream_t s) {
  const dim3 g((unsigned)((N + kGT - 1) / kGT), (unsigned)((M + kGT - 1) / kGT)), b(256);
  if (g.x * g.y < kTileBlocks) {
    const dim3 gt((unsigned)((N + 15) / 16), (unsigned)((M + 15) / 16));
    hipLaunchKernelGGL(k_zgemm_tile, gt, b, 0, s, (const zc128*)A, lda, (const zc128*)B, sbk, sbn, (zc128*)Y, ldy, M,
                       N, K);
    return;
  }
  hipLaunchKernelGGL(k_zgemm_mfma, g, b, 0, s, (const zc128*)A, lda, (const zc128*)B, sbk, sbn, (zc128*)Y, ldy, M, N,
                     K);
}

}  // namespace dev
}  // namespace ffx
