// Segment passes (gfx950): every Givens rotation and diagonal gate that acts
// on the column strings of one row of the state, applied with one HBM round
// trip of that row.
//
// The state is read row-wise (for the alpha-major matrix Gamma the column
// strings are the beta configurations; for its transpose they are the alpha
// configurations).  Rotations of the column spin never mix rows (Sec. 3.2.3:
// a Givens rotation of spin sigma pairs configurations that differ only in
// spin sigma), so a block can load a whole row -- or a contiguous segment of
// it whose configurations share the occupation of the orbitals above the
// segment window -- into LDS and run a list of stages on it:
//   * Givens stages: rotations confined to a register window [a, a+W); each
//     lane loads one class of configurations that agree outside the window
//     from LDS into registers, applies the stage's rotations there, and writes
//     the class back (one LDS round trip per stage, never per rotation);
//   * diagonal stages: per-configuration phases (number-operator sums,
//     diagonal Coulomb, deferred orbital phase layers), weights or weighted
//     norms, evaluated in FP64 from the row string, the column string and
//     byte-indexed partial-sum tables kept in LDS.
// The row segment is then stored once (or accumulated, or dropped after a
// reduction).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <utility>

#include "dev_common.h"
#include "device.h"

namespace ffx {
namespace dev {

// 12 waves per block (3 per SIMD): the widest complex128 window (W = 6) fits in
// the 168 registers this leaves a lane; complex64, narrower windows, and lanes
// that hold one part of each member fit in 128 registers and run 16 waves
template <int W, class R, bool SPLIT = false>
constexpr int seg_threads() {
  return SPLIT || sizeof(R) == 4 || W < kShapeW ? 1024 : 768;
}

// The rotation on the orbital pair that straddles the segment window, for
// the cnt strings own[0 .. cnt) of this segment and their partners peer[0 ..
// cnt) in another segment of the same row (read from the pass's source, which
// the pass does not write): role 0: own = x, x' = c x + s y; role 1: own = y,
// y' = c y - conj(s) x.  The first kCrossU partners of each thread are loaded
// together with the segment itself (cross_fetch, before the barrier that
// completes the segment); cross_apply then rotates, loading any further
// partners directly.
constexpr int kCrossU = 8;

__device__ const int4 kZeroWords = {0, 0, 0, 0};

// The block's row segment, the member-offset tables (int4 words) and the
// first kCrossU crossing partners per thread, requested in one straight-line
// batch before any is used: every thread issues all its loads (clamped to the
// last valid element, pointers chosen without branches), then stores the
// segment and the tables to LDS; the partners stay in registers (xt).  Further
// batches run only for segments longer than UR * nthr or tables longer than
// UM * nthr words.
// stride: distance between consecutive elements of the row in src and peer
// (1, or the row count of a gathering pass, whose src is the other layout).
template <int UR, int UM, class V>
__device__ __forceinline__ void stage_segment(V* __restrict__ row, const V* __restrict__ src, int len,
                                              int4* __restrict__ mt, const int4* mtg, int n4, const V* peer,
                                              int pcnt, V* xt, int tid, int nthr, int64_t stride) {
  const int4* pm = n4 > 0 ? mtg : &kZeroWords;
  const int pn4 = max(n4, 1);
  const V* pp = pcnt > 0 ? peer : src;
  const int pc = max(pcnt, 1);
  V t[UR];
  int4 q[UM];
#pragma unroll
  for (int u = 0; u < UR; ++u) t[u] = src[(int64_t)min(tid + u * nthr, len - 1) * stride];
#pragma unroll
  for (int u = 0; u < UM; ++u) q[u] = pm[min(tid + u * nthr, pn4 - 1)];
#pragma unroll
  for (int u = 0; u < kCrossU; ++u) xt[u] = pp[(int64_t)min(tid + u * nthr, pc - 1) * stride];
#pragma unroll
  for (int u = 0; u < UR; ++u) keep(t[u]);
#pragma unroll
  for (int u = 0; u < UM; ++u) keep(q[u]);
#pragma unroll
  for (int u = 0; u < UR; ++u)
    if (tid + u * nthr < len) row[tid + u * nthr] = t[u];
#pragma unroll
  for (int u = 0; u < UM; ++u)
    if (tid + u * nthr < n4) mt[tid + u * nthr] = q[u];
  for (int e = tid + UR * nthr; e < len; e += nthr) row[e] = src[(int64_t)e * stride];
  for (int e = tid + UM * nthr; e < n4; e += nthr) mt[e] = mtg[e];
}

template <class R>
__device__ __forceinline__ typename V2T<R>::type cross_rot(typename V2T<R>::type a, typename V2T<R>::type b, R c,
                                                           R sgn, R sr, R si) {
  // own' = c own + sgn * s' peer, s' = s (role 0) or conj(s) (role 1)
  typename V2T<R>::type o;
  o.x = c * a.x + sgn * (sr * b.x - si * b.y);
  o.y = c * a.y + sgn * (sr * b.y + si * b.x);
  return o;
}

template <class R>
__device__ __forceinline__ void cross_apply(typename V2T<R>::type* own, const typename V2T<R>::type* t,
                                            const typename V2T<R>::type* peer, int cnt, int role, double cd,
                                            double srd, double sid, int tid, int nthr, int64_t stride) {
  const R c = (R)cd, sr = (R)srd, si = role == 0 ? (R)sid : -(R)sid;
  const R sgn = role == 0 ? R(1) : R(-1);
#pragma unroll
  for (int u = 0; u < kCrossU; ++u) {
    const int e = tid + u * nthr;
    if (e < cnt) own[e] = cross_rot<R>(own[e], t[u], c, sgn, sr, si);
  }
  for (int e = tid + kCrossU * nthr; e < cnt; e += nthr)
    own[e] = cross_rot<R>(own[e], peer[(int64_t)e * stride], c, sgn, sr, si);
}

// Row-dependent part of a diagonal stage, computed by the whole block before
// the stage touches any element: the cross weights w[q] = sum_{p in row} C[p][q]
// (a column of C per thread, all its loads in flight at once, summed over p in
// a fixed order), the row value A[r], the row's phase factor (phase stages;
// with a cross term and byte tables it is folded into the first table), and
// the byte tables of the cross term: complex factors for phase stages, real
// sums otherwise.  With `direct` (segments shorter than the tables) the stage
// takes the sum of the weights, and a phase's sine and cosine, per element:
// a table of 256 entries per byte costs as many of them as 256 elements.
// Ends with a block barrier.
struct DiagRow {
  double arow;
  zc128 rowf;
  bool cross;
};

__device__ __forceinline__ DiagRow diag_stage_tables(const StageDev& st, const SegPassDev& P, int64_t r,
                                                     uint32_t rmask, zc128* ez, double* wq, int tid, int nthr,
                                                     int nbytes, bool direct) {
  double* tab = (double*)ez;
  DiagRow dr;
  dr.cross = st.C != nullptr;
  if (tid < P.norb) {
    double w = 0.0;
    if (dr.cross)
      for (int p0 = 0; p0 < P.norb; p0 += 16) {
        double c[16];
#pragma unroll
        for (int p = 0; p < 16; ++p) c[p] = st.C[min(p0 + p, P.norb - 1) * P.norb + tid];
#pragma unroll
        for (int p = 0; p < 16; ++p)
          if (p0 + p < P.norb && ((rmask >> (p0 + p)) & 1)) w += c[p];
      }
    wq[tid] = w;
  }
  dr.arow = st.A ? st.A[r] : 0.0;
  dr.rowf = zc128{1.0, 0.0};
  if (st.type == ST_PHASE) {
    double grow = 0.0;
    if (st.drow)
      for (int p = 0; p < P.norb; ++p)
        if ((rmask >> p) & 1) grow += st.drow[p];
    dr.rowf = phase_factor<double>(st.scale * dr.arow + grow);
    if (parity(rmask & st.sign_row)) {
      dr.rowf.x = -dr.rowf.x;
      dr.rowf.y = -dr.rowf.y;
    }
  }
  __syncthreads();
  if (dr.cross && !direct) {
    for (int i = tid; i < nbytes * 256; i += nthr) {
      const int k = i >> 8, b = i & 255;
      double v = 0.0;
      for (int q = 0; q < 8; ++q)
        if (((b >> q) & 1) && 8 * k + q < P.norb) v += wq[8 * k + q];
      if (st.type == ST_PHASE) {
        const zc128 e = phase_factor<double>(st.scale * v);
        ez[i] = k == 0 ? zmul(dr.rowf, e) : e;
      } else {
        tab[i] = v;
      }
    }
    __syncthreads();
  }
  return dr;
}

// The launch parameters, read again from the kernel's argument segment: kept
// across the stages they, and values computed from them, would hold (or spill)
// scalar registers that the rotation parameters need.
__device__ __forceinline__ SegPassDev reload_params() {
  using carg = const __attribute__((address_space(4))) char;
  carg* kp = (carg*)__builtin_amdgcn_kernarg_segment_ptr();
  uint64_t a = (uint64_t)kp;
  asm volatile("" : "+s"(a));
  return uniform_load((const SegPassDev*)a);
}

// LDS after the row: the byte tables (none for direct evaluation), the member
// offsets of every window, the cross weights and the reduction scratch
struct SegLds {
  zc128* ez;   // nbytes x 256 complex byte factors (or real byte sums)
  int4* mt;
  double* wq;  // 32 cross weights
  double* red;
};
__device__ __forceinline__ SegLds seg_lds_map(char* smem, const SegPassDev& P, int nbytes) {
  SegLds L;
  L.ez = (zc128*)(smem + P.lds_row_bytes);
  L.mt = (int4*)(L.ez + (P.direct ? 0 : nbytes * 256));
  L.wq = (double*)(L.mt + P.max_mt);
  L.red = L.wq + 32;
  return L;
}

// SPLIT (real rotations at W = 6): neighbouring lanes take the two parts of the
// members of one class (split_seg_window).  A lane then holds C(W, m) parts
// instead of twice as many, so a compute unit runs 16 waves of 20-member windows
// instead of 12, a stage's longest chain is half as long, and a row's few
// classes fill twice the lanes.  A 14-orbital DF step took 13.2 ms without it
// and 8.4 ms with it, a 10-orbital one 1.50 and 1.37 ms, a 16-orbital complex64
// one (whose rows fill a block either way) 52.8 and 52.4 ms.
template <int W, bool REAL, class R, bool SPLIT>
__global__ __launch_bounds__((seg_threads<W, R, SPLIT>())) void k_seg_pass(SegPassDev P) {
  using V = typename V2T<R>::type;
  extern __shared__ __align__(16) char smem[];
  V* row = (V*)smem;
  const SegLds L = seg_lds_map(smem, P, (P.norb + 7) >> 3);

  int si;
  int64_t r;
  if (P.xcd_rows > 0) {
    const int64_t k = blockIdx.x >> 3;
    r = (int64_t)(blockIdx.x & 7) * P.xcd_rows + k / P.n_seg;
    si = (int)(k % P.n_seg);
    if (r >= P.n_rows) return;  // the whole block: the grid rounds rows up to 8 XCDs
  } else {
    si = (int)(blockIdx.x % P.n_seg);
    r = blockIdx.x / P.n_seg;
  }
  const SegDev sg = uniform_load(P.segs + si);
  const int nthr = blockDim.x;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform in the wave: loops over chunks stay scalar
  const int nwaves = nthr >> 6;

  // row r of this layout: contiguous, or column r of the other layout
  const int64_t stride = P.gather ? P.n_rows : 1;
  const V* src = P.gather ? (const V*)P.src + r + (int64_t)sg.off * P.n_rows
                          : (const V*)P.src + r * P.row_len + sg.off;
  const bool xrot = P.cross && sg.cross_cnt > 0;
  const V* peer = P.gather ? (const V*)P.src + r + (int64_t)sg.cross_peer * P.n_rows
                           : (const V*)P.src + r * P.row_len + sg.cross_peer;
  V xt[kCrossU];
  // (the member-offset table of every window is a whole number of int4 words)
  stage_segment<sizeof(V) == 8 ? 13 : 9, 2>(row, src, sg.len, L.mt, sg.mt_all, sg.n_mt_all, peer,
                                            xrot ? sg.cross_cnt : 0, xt, tid, nthr, stride);
  __syncthreads();
  if (xrot) {
    cross_apply<R>(row + sg.cross_lo, xt, peer, sg.cross_cnt, sg.cross_role, P.cross_c, P.cross_sr, P.cross_si,
                   tid, nthr, stride);
    __syncthreads();
  }

  double acc = 0.0;

  // the vector-memory data of a Givens stage (its rotations, the wave's first
  // class codes) is requested one stage ahead, so that its latency overlaps the
  // stage before; descriptors come through the scalar cache
  RotLane<R> rl_next{nullptr};
  ChunkAhead fc_next{1, 1, -1, -1};
  auto fetch = [&](int s) {
    const StageDev st = uniform_load(P.stages + s);
    if (st.type == ST_GIVENS) {
      rl_next = fetch_rot_lane<R>(st.rots);
      fc_next = fetch_first_chunk(uniform_load(sg.win + st.a), wave, lane, nwaves);
    }
  };
  if (P.n_stages > 0) fetch(0);
  for (int s = 0; s < P.n_stages; ++s) {
    const StageDev st = uniform_load(P.stages + s);
    const RotLane<R> rl = rl_next;
    const ChunkAhead fc = fc_next;
    if (s + 1 < P.n_stages) fetch(s + 1);
    if (st.type == ST_GIVENS) {
      const SegWinDev wt = uniform_load(sg.win + st.a);
      givens_stage<W, REAL, R, SPLIT>(st.shape, row, (const char*)L.mt, wt, rl, st.nrot, wave, nwaves, lane, fc);
    } else {
      const SegPassDev P = reload_params();
      const int nbytes = (P.norb + 7) >> 3;
      const SegLds L = seg_lds_map(smem, P, nbytes);
      zc128* ez = L.ez;
      double* tab = (double*)ez;
      double* wq = L.wq;
      const uint32_t rmask = P.row_masks[r];
      const uint32_t* cmask = P.col_masks + sg.off;
      const DiagRow dr = diag_stage_tables(st, P, r, rmask, ez, wq, tid, nthr, nbytes, P.direct);
      const bool cross = dr.cross;
      const double arow = dr.arow;
      zc128 rowf = dr.rowf;
      // U elements per thread at a time (a whole segment per batch for the
      // usual block sizes): their column masks and tables are all requested
      // before the first is used
      constexpr int U = sizeof(V) == 8 ? 10 : 9;
      if (cross && P.direct) {
        // (a loop of its own, not unrolled: one copy of the sine and cosine)
        const zc128* colf = st.colf ? (const zc128*)st.colf + sg.off : nullptr;
        const double* Bs = st.B ? st.B + sg.off : nullptr;
#pragma unroll 1
        for (int e = tid; e < sg.len; e += nthr) {
          const uint32_t cm = cmask[e];
          double v = 0.0;
          for (uint32_t x = cm; x; x &= x - 1) v += wq[__builtin_ctz(x)];
          V y = row[e];
          if (st.type == ST_PHASE) {
            zc128 f = zmul(rowf, phase_factor<double>(st.scale * v));
            if (colf) f = zmul(f, colf[e]);
            if (parity(cm & st.sign_col)) {
              f.x = -f.x;
              f.y = -f.y;
            }
            V o;
            o.x = (R)((double)y.x * f.x - (double)y.y * f.y);
            o.y = (R)((double)y.x * f.y + (double)y.y * f.x);
            row[e] = o;
          } else {
            const double f = arow + (Bs ? Bs[e] : 0.0) + v;
            if (st.type == ST_SCALE) {
              y.x = (R)(f * (double)y.x);
              y.y = (R)(f * (double)y.y);
              row[e] = y;
            } else {
              acc += f * ((double)y.x * (double)y.x + (double)y.y * (double)y.y);
            }
          }
        }
      } else if (st.type == ST_PHASE) {
        if (cross) rowf = zc128{1.0, 0.0};
        const zc128* colf = st.colf ? (const zc128*)st.colf + sg.off : nullptr;
        const uint32_t sgn = st.sign_col;
        const bool use_cm = cross || sgn != 0;
        // signs only: negate where the row and column parities differ
        const bool signs_only = !cross && !colf && !st.A && !st.drow;
        const int rneg = rowf.x < 0.0;
        const zc128 one{1.0, 0.0};
        for (int e0 = tid; e0 < sg.len; e0 += U * nthr) {
          uint32_t cm[U];
          zc128 cf[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int e = min(e0 + u * nthr, sg.len - 1);
            cm[u] = use_cm ? cmask[e] : 0u;
            cf[u] = colf ? colf[e] : one;
          }
#pragma unroll
          for (int u = 0; u < U; ++u) asm volatile("" ::"v"(cm[u]), "v"(cf[u].x), "v"(cf[u].y));
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int e = e0 + u * nthr;
            if (e >= sg.len) continue;
            if (signs_only) {
              if (parity(cm[u] & sgn) != rneg) {
                V y = row[e];
                y.x = -y.x;
                y.y = -y.y;
                row[e] = y;
              }
              continue;
            }
            zc128 f = colf ? zmul(rowf, cf[u]) : rowf;
            if (cross)
              for (int k = 0; k < nbytes; ++k) f = zmul(f, ez[(k << 8) | ((cm[u] >> (8 * k)) & 255)]);
            if (parity(cm[u] & sgn)) {
              f.x = -f.x;
              f.y = -f.y;
            }
            V y = row[e];
            V o;
            o.x = (R)((double)y.x * f.x - (double)y.y * f.y);
            o.y = (R)((double)y.x * f.y + (double)y.y * f.x);
            row[e] = o;
          }
        }
      } else {
        const double* Bs = st.B ? st.B + sg.off : nullptr;
        for (int e0 = tid; e0 < sg.len; e0 += U * nthr) {
          uint32_t cm[U];
          double fb[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int e = min(e0 + u * nthr, sg.len - 1);
            cm[u] = cross ? cmask[e] : 0u;
            fb[u] = Bs ? Bs[e] : 0.0;
          }
#pragma unroll
          for (int u = 0; u < U; ++u) asm volatile("" ::"v"(cm[u]), "v"(fb[u]));
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int e = e0 + u * nthr;
            if (e < sg.len) {
              double f = arow + fb[u];
              if (cross)
                for (int k = 0; k < nbytes; ++k) f += tab[(k << 8) | ((cm[u] >> (8 * k)) & 255)];
              V y = row[e];
              if (st.type == ST_SCALE) {
                y.x = (R)(f * (double)y.x);
                y.y = (R)(f * (double)y.y);
                row[e] = y;
              } else {
                acc += f * ((double)y.x * (double)y.x + (double)y.y * (double)y.y);
              }
            }
          }
        }
      }
    }
    __syncthreads();
  }

  const SegPassDev Q = reload_params();
  if (Q.mode != SEG_NONE) {
    // row r of this layout, or (scatter) column r of the other one
    const int64_t ostride = Q.scatter ? Q.n_rows : 1;
    V* dst = Q.scatter ? (V*)Q.dst + r + (int64_t)sg.off * Q.n_rows : (V*)Q.dst + r * Q.row_len + sg.off;
    if (Q.mode == SEG_STORE) {
      if (Q.scatter)
        stage_out_strided<128 / sizeof(V)>(dst, row, sg.len, ostride, tid, nthr);
      else
        stage_in<128 / sizeof(V)>(dst, row, sg.len, tid, nthr);
    } else {
      for (int e = tid; e < sg.len; e += nthr) {
        V a = dst[e * ostride], b = row[e];
        a.x += b.x;
        a.y += b.y;
        dst[e * ostride] = a;
      }
    }
  }
  if (Q.partials) {
    // fixed-order block reduction: wave sums, then thread 0 adds them in order
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    double* red = seg_lds_map(smem, Q, (Q.norb + 7) >> 3).red;
    if (lane == 0) red[wave] = acc;
    __syncthreads();
    if (tid == 0) {
      double t = 0.0;
      for (int i = 0; i < nwaves; ++i) t += red[i];
      Q.partials[r * Q.n_seg + si] = t;
    }
  }
}

// ---------------------------------------------------------------------------
// Row planes.  A complex128 row that exceeds LDS, but whose real parts fit,
// is held as two planes when every Givens rotation of the pass is real: a real
// rotation matrix acts on the real and imaginary parts of the amplitudes alike
// and independently, so each run of consecutive Givens stages is applied to
// the plane in LDS, the planes are swapped, and the run is applied to the
// other.  The other plane stays in registers: thread t holds the parts of
// elements t, t + nthr, t + 2 nthr, ...  Diagonal stages combine the two parts
// of each element in the thread that holds its register part.  Where the real
// parts of a whole row fit, the row is one segment and no rotation crosses a
// segment: one pass per visit.  Longer rows are split, as in the segment pass,
// into segments of the strings that share their highest orbitals (the
// rotations on those orbitals run as whole-spin window passes between plane
// passes); each block holds one segment of one row.
// ---------------------------------------------------------------------------
// Block sizes: 768 threads hold 17 register parts each (rows of up to 13 056
// amplitudes, 168 registers a lane, 3 waves per SIMD; the default, 5 % faster
// on the DF step at 16 orbitals) or 512 threads 26 parts (13 312 amplitudes,
// 200 registers, 2 waves per SIMD).
template <int NT>
constexpr int plane_regs() {
  return NT == 512 ? 26 : 17;
}

int seg_pass_plane_max_len(int threads) { return threads * (threads == 512 ? plane_regs<512>() : plane_regs<768>()); }

// Givens stages [s0, s1) of a plane pass on the LDS plane; each stage's
// rotations and the wave's first class codes are requested one stage ahead.
template <int W>
__device__ __forceinline__ void plane_givens_run(const SegPassDev& P, const SegDev& sg, re128* pl, const char* mtl,
                                                 int s0, int s1, int wave, int nwaves, int lane) {
  StageDev st = uniform_load(P.stages + s0);
  RotLane<double> rl_next = fetch_rot_lane<double>(st.rots);
  ChunkAhead fc_next = fetch_first_chunk<false>(uniform_load(sg.win + st.a), wave, lane, nwaves);
  for (int s = s0; s < s1; ++s) {
    st = uniform_load(P.stages + s);
    const RotLane<double> rl = rl_next;
    const ChunkAhead fc = fc_next;
    if (s + 1 < s1) {
      const StageDev nx = uniform_load(P.stages + s + 1);
      rl_next = fetch_rot_lane<double>(nx.rots);
      fc_next = fetch_first_chunk<false>(uniform_load(sg.win + nx.a), wave, lane, nwaves);
    }
    const SegWinDev wt = uniform_load(sg.win + st.a);
    givens_stage_v<W, true, re128, 8, false>(st.shape, (char*)pl, mtl, wt, rl, st.nrot, wave, nwaves, lane, fc);
    __syncthreads();
  }
}

// Waves of a block that share a SIMD (wave w runs on SIMD w % 4) take
// different priorities, so that in a stage the first of them reads its class
// from LDS and starts on the rotations while the others still read (a
// 16-orbital step 142.8 -> 141.0 ms; segment passes, with shorter rows or 16
// waves, gained nothing and keep equal priorities).
__device__ __forceinline__ void stagger_waves(int wave) {
  switch ((wave >> 2) & 3) {
    case 0: __builtin_amdgcn_s_setprio(3); break;
    case 1: __builtin_amdgcn_s_setprio(2); break;
    case 2: __builtin_amdgcn_s_setprio(1); break;
    default: __builtin_amdgcn_s_setprio(0); break;
  }
}

// SEGS: rows split into segments (else one segment, the whole row, at offset 0)
template <int W, int NT, bool SEGS>
__global__ __launch_bounds__(NT) void k_seg_pass_planes(SegPassDev P) {
  constexpr int kPlaneRegs = plane_regs<NT>();
  extern __shared__ __align__(16) char smem[];
  re128* pl = (re128*)smem;  // the LDS plane
  const SegLds L = seg_lds_map(smem, P, (P.norb + 7) >> 3);
  const char* mtl = (const char*)L.mt;

  // block -> (row, segment) as in the segment pass
  int si = 0;
  int64_t r;
  if constexpr (SEGS) {
    if (P.xcd_rows > 0) {
      const int64_t k = blockIdx.x >> 3;
      r = (int64_t)(blockIdx.x & 7) * P.xcd_rows + k / P.n_seg;
      si = (int)(k % P.n_seg);
      if (r >= P.n_rows) return;  // the whole block: the grid rounds rows up to 8 XCDs
    } else {
      si = (int)(blockIdx.x % P.n_seg);
      r = blockIdx.x / P.n_seg;
    }
  } else {
    if (P.xcd_rows > 0) {
      r = (int64_t)(blockIdx.x & 7) * P.xcd_rows + (blockIdx.x >> 3);
      if (r >= P.n_rows) return;
    } else {
      r = blockIdx.x;
    }
  }
  const SegDev sg = uniform_load(P.segs + si);
  const int off = SEGS ? sg.off : 0;  // the segment's first column
  const int len = sg.len;
  const int nthr = blockDim.x;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform in the wave: loops over chunks stay scalar
  const int nwaves = nthr >> 6;
  stagger_waves(wave);
  const int64_t stride = P.gather ? P.n_rows : 1;
  const zc128* src = P.gather ? (const zc128*)P.src + r + (int64_t)off * P.n_rows
                              : (const zc128*)P.src + r * P.row_len + off;

  // the row: every load in flight before the first is used; real parts to the
  // LDS plane, imaginary parts to registers; then the member-offset tables
  double rp[kPlaneRegs];
  {
    zc128 t[kPlaneRegs];
#pragma unroll
    for (int k = 0; k < kPlaneRegs; ++k) t[k] = src[(int64_t)min(tid + k * nthr, len - 1) * stride];
#pragma unroll
    for (int k = 0; k < kPlaneRegs; ++k) keep(t[k]);
#pragma unroll
    for (int k = 0; k < kPlaneRegs; ++k) {
      const int e = tid + k * nthr;
      if (e < len) pl[e].x = t[k].x;
      rp[k] = t[k].y;
    }
  }
  for (int e = tid; e < sg.n_mt_all; e += nthr) L.mt[e] = sg.mt_all[e];
  __syncthreads();
  bool lds_re = true;  // the LDS plane holds the real parts (the same in every thread)

  double acc = 0.0;
  int s = 0;
  while (s < P.n_stages) {
    const StageDev st = uniform_load(P.stages + s);
    if (st.type == ST_GIVENS) {
      int s1 = s + 1;
      while (s1 < P.n_stages && uniform_load(P.stages + s1).type == ST_GIVENS) ++s1;
      // the run on one plane, a swap of the planes (the register plane into LDS
      // and back), the run on the other; a loop, so that the stages' code is
      // there once
#pragma unroll 1
      for (int half = 0;; ++half) {
        plane_givens_run<W>(P, sg, pl, mtl, s, s1, wave, nwaves, lane);
        if (half) break;
#pragma unroll
        for (int k = 0; k < kPlaneRegs; ++k) {
          int e = tid + k * nthr;
          asm volatile("" : "+v"(e));  // recomputed here: hoisted, 26 such offsets would stay live across stages
          if (e < len) {
            const double x = pl[e].x;
            pl[e].x = rp[k];
            rp[k] = x;
          }
        }
        __syncthreads();
      }
      lds_re = !lds_re;
      s = s1;
      continue;
    }
    const SegPassDev P = reload_params();
    const int nbytes = (P.norb + 7) >> 3;
    const SegLds L = seg_lds_map(smem, P, nbytes);
    zc128* ez = L.ez;
    double* tab = (double*)ez;
    double* wq = L.wq;
    const uint32_t rmask = P.row_masks[r];
    const uint32_t* cmask = P.col_masks + off;
    const DiagRow dr = diag_stage_tables(st, P, r, rmask, ez, wq, tid, nthr, nbytes, false);
    const bool cross = dr.cross;
    if (st.type == ST_PHASE) {
      const zc128 rowf = cross ? zc128{1.0, 0.0} : dr.rowf;
      const zc128* colf = st.colf ? (const zc128*)st.colf + off : nullptr;
      const uint32_t sgn = st.sign_col;
      const bool use_cm = cross || sgn != 0;
#pragma unroll
      for (int k = 0; k < kPlaneRegs; ++k) {
        int e = tid + k * nthr;
        asm volatile("" : "+v"(e));  // recomputed per element (see the swap)
        if (e >= len) continue;
        const uint32_t cm = use_cm ? cmask[e] : 0u;
        zc128 f = colf ? zmul(rowf, colf[e]) : rowf;
        if (cross)
          for (int b = 0; b < nbytes; ++b) f = zmul(f, ez[(b << 8) | ((cm >> (8 * b)) & 255)]);
        if (parity(cm & sgn)) {
          f.x = -f.x;
          f.y = -f.y;
        }
        const double a = pl[e].x, q = rp[k];
        const double re = lds_re ? a : q, im = lds_re ? q : a;
        const double nre = re * f.x - im * f.y, nim = re * f.y + im * f.x;
        pl[e].x = lds_re ? nre : nim;
        rp[k] = lds_re ? nim : nre;
      }
    } else {
      const double* Bs = st.B ? st.B + off : nullptr;
#pragma unroll
      for (int k = 0; k < kPlaneRegs; ++k) {
        int e = tid + k * nthr;
        asm volatile("" : "+v"(e));  // recomputed per element (see the swap)
        if (e >= len) continue;
        double f = dr.arow + (Bs ? Bs[e] : 0.0);
        if (cross) {
          const uint32_t cm = cmask[e];
          for (int b = 0; b < nbytes; ++b) f += tab[(b << 8) | ((cm >> (8 * b)) & 255)];
        }
        if (st.type == ST_SCALE) {
          pl[e].x *= f;
          rp[k] *= f;
        } else {
          const double a = pl[e].x, q = rp[k];
          acc += f * (a * a + q * q);
        }
      }
    }
    __syncthreads();
    ++s;
  }

  const SegPassDev Q = reload_params();
  if (Q.mode != SEG_NONE) {
    // row r of this layout, or (scatter) column r of the other one
    const int64_t ostride = Q.scatter ? Q.n_rows : 1;
    zc128* dst = Q.scatter ? (zc128*)Q.dst + r + (int64_t)off * Q.n_rows : (zc128*)Q.dst + r * Q.row_len + off;
#pragma unroll
    for (int k = 0; k < kPlaneRegs; ++k) {
      const int e = tid + k * nthr;
      if (e < len) {
        const double a = pl[e].x, q = rp[k];
        zc128 v = lds_re ? zc128{a, q} : zc128{q, a};
        if (Q.mode == SEG_ACCUM) {
          const zc128 o = dst[e * ostride];
          v.x += o.x;
          v.y += o.y;
        }
        dst[e * ostride] = v;
      }
    }
  }
  if (Q.partials) {
    // fixed-order block reduction: wave sums, then thread 0 adds them in order
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    double* red = seg_lds_map(smem, Q, (Q.norb + 7) >> 3).red;
    if (lane == 0) red[wave] = acc;
    __syncthreads();
    if (tid == 0) {
      double t = 0.0;
      for (int i = 0; i < nwaves; ++i) t += red[i];
      Q.partials[SEGS ? r * Q.n_seg + si : r] = t;
    }
  }
}

template <int W, int NT, bool SEGS>
static void launch_planes(const SegPassDev& p, size_t lds, hipStream_t s) {
  auto k = k_seg_pass_planes<W, NT, SEGS>;
  static bool attr_set = false;
  if (!attr_set) {
    (void)hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    attr_set = true;
  }
  const int64_t blocks = p.xcd_rows > 0 ? 8 * p.xcd_rows * p.n_seg : p.n_rows * p.n_seg;
  hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(NT), lds, s, p);
}

// rows split into segments only at window width 6 (the plan builds no
// narrower segmented plane set)
template <int NT>
static void planes_w(int W, const SegPassDev& p, size_t lds, hipStream_t s) {
  if (p.n_seg > 1) {
    if (W == 6) launch_planes<6, NT, true>(p, lds, s);
    return;
  }
  switch (W) {
    case 4: launch_planes<4, NT, false>(p, lds, s); break;
    case 5: launch_planes<5, NT, false>(p, lds, s); break;
    case 6: launch_planes<6, NT, false>(p, lds, s); break;
    default: break;
  }
}

void seg_pass_planes(int W, int threads, const SegPassDev& p, size_t lds, hipStream_t s) {
  if (threads == 768)
    planes_w<768>(W, p, lds, s);
  else
    planes_w<512>(W, p, lds, s);
}

size_t seg_pass_lds(bool c64, int norb, int max_len, int max_mt, bool direct) {
  size_t row = (size_t)max_len * (c64 ? 8 : 16);
  row = (row + 15) & ~(size_t)15;
  const size_t tabs = direct ? 0 : (size_t)((norb + 7) / 8) * 256 * sizeof(zc128);
  return row + tabs + (size_t)max_mt * 16 + (32 + 16) * sizeof(double);
}

int seg_pass_max_threads(bool c64, int W, bool split) {
  if (split) return seg_threads<kShapeW, double, true>();
  return c64 ? seg_threads<kShapeW, float>() : (W < kShapeW ? seg_threads<kShapeW - 1, double>() : seg_threads<kShapeW, double>());
}

template <int W, bool REAL, class R, bool SPLIT = false>
static void launch_seg(const SegPassDev& p, int threads, size_t lds, hipStream_t s) {
  auto k = k_seg_pass<W, REAL, R, SPLIT>;
  static bool attr_set = false;
  if (!attr_set) {
    (void)hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    attr_set = true;
  }
  const int64_t blocks = p.xcd_rows > 0 ? 8 * p.xcd_rows * p.n_seg : p.n_rows * p.n_seg;
  hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(std::min(threads, seg_threads<W, R, SPLIT>())), lds, s, p);
}

template <bool REAL, class R>
static void launch_seg_w(int W, const SegPassDev& p, int threads, size_t lds, hipStream_t s) {
  switch (W) {
    case 1: launch_seg<1, REAL, R>(p, threads, lds, s); break;
    case 2: launch_seg<2, REAL, R>(p, threads, lds, s); break;
    case 3: launch_seg<3, REAL, R>(p, threads, lds, s); break;
    case 4: launch_seg<4, REAL, R>(p, threads, lds, s); break;
    case 5: launch_seg<5, REAL, R>(p, threads, lds, s); break;
    case kShapeW: launch_seg<kShapeW, REAL, R, REAL>(p, threads, lds, s); break;
    default: break;
  }
}

void seg_pass(bool c64, bool real, int W, const SegPassDev& p, int threads, size_t lds, hipStream_t s) {
  if (c64) {
    if (real)
      launch_seg_w<true, float>(W, p, threads, lds, s);
    else
      launch_seg_w<false, float>(W, p, threads, lds, s);
  } else {
    if (real)
      launch_seg_w<true, double>(W, p, threads, lds, s);
    else
      launch_seg_w<false, double>(W, p, threads, lds, s);
  }
}

// ---------------------------------------------------------------------------
// in-place transpose of a square matrix: block (bx, by) with bx <= by swaps
// tile (by, bx) with tile (bx, by) through LDS (a diagonal tile is transposed
// in place).
// ---------------------------------------------------------------------------
template <class R>
__global__ __launch_bounds__(256) void k_transpose_square(typename V2T<R>::type* __restrict__ a, int64_t n,
                                                          int64_t ntiles) {
  using V = typename V2T<R>::type;
  __shared__ V t0[32][33];
  __shared__ V t1[32][33];
  // map the linear block index onto the lower triangle (bx <= by) of tile pairs
  int64_t k = blockIdx.x;
  int64_t by = (int64_t)((sqrt(8.0 * (double)k + 1.0) - 1.0) * 0.5);
  while ((by + 1) * (by + 2) / 2 <= k) ++by;
  while (by * (by + 1) / 2 > k) --by;
  const int64_t bx = k - by * (by + 1) / 2;
  if (by >= ntiles) return;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int64_t r0 = by * 32, c0 = bx * 32;  // tile (by, bx)
  for (int j = ty; j < 32; j += 8) {
    int64_t r = r0 + j, c = c0 + tx;
    if (r < n && c < n) t0[j][tx] = a[r * n + c];
    int64_t r2 = c0 + j, c2 = r0 + tx;  // tile (bx, by)
    if (r2 < n && c2 < n) t1[j][tx] = a[r2 * n + c2];
  }
  __syncthreads();
  for (int j = ty; j < 32; j += 8) {
    // tile (bx, by) <- transpose of tile (by, bx), and vice versa
    int64_t r2 = c0 + j, c2 = r0 + tx;
    if (r2 < n && c2 < n) a[r2 * n + c2] = t0[tx][j];
    int64_t r = r0 + j, c = c0 + tx;
    if (r < n && c < n) a[r * n + c] = t1[tx][j];
  }
}

void transpose_square(bool c64, void* vec, int64_t n, hipStream_t s) {
  const int64_t nt = (n + 31) / 32;
  const int64_t blocks = nt * (nt + 1) / 2;
  if (c64)
    hipLaunchKernelGGL(k_transpose_square<float>, dim3((unsigned)blocks), dim3(256), 0, s, (zc64*)vec, n, nt);
  else
    hipLaunchKernelGGL(k_transpose_square<double>, dim3((unsigned)blocks), dim3(256), 0, s, (zc128*)vec, n, nt);
}

}  // namespace dev
}  // namespace ffx
