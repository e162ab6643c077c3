// Host-side (CPU, FP64) building blocks of libffx: configuration tables,
// Givens decompositions, window scheduling and small dense linear algebra.
// Nothing here touches the GPU.
#pragma once

#include <complex>
#include <cstdint>
#include <stdexcept>
#include <string>
#include <utility>
#include <functional>
#include <vector>

namespace ffx {

using cd = std::complex<double>;

struct Error : std::runtime_error {
  int code;
  Error(int c, const std::string& m) : std::runtime_error(m), code(c) {}
};

int64_t binom(int n, int k);

// Error-path hook for tests: with FFX_FAULT="<site>:<k>" in the environment,
// the k-th call (k >= 1) at that site, counted from when the variable took its
// current value, reports failure, as if the runtime had refused the request.
// Site "alloc": the library's device and pinned host allocations (each then
// fails with FFX_ENOMEM).  Unset, empty or malformed: no effect.
bool fault_hit(const char* site);

// All n-subsets of {0..norb-1} as bit masks in ascending integer order
// (address = position).  Generated by Gosper's next-combination step, which
// visits equal-popcount integers in increasing order.
std::vector<uint64_t> make_strings(int norb, int n);

// One adjacent Givens rotation as seen by the state: on orbitals (p, p+1),
// for each configuration pair (I0: p occupied, p+1 empty; I1 = I0 with p -> p+1)
//   x' = c x + s y,   y' = -conj(s) x + c y,   x = gamma(I0), y = gamma(I1).
struct Givens {
  int p;
  double c;
  cd s;
};

// U = diag(exp(i phase)) G_K ... G_1 (G_1 applied first).
struct Decomposition {
  std::vector<Givens> rots;
  std::vector<double> phase;
  bool real = false;  // every s real and every phase in {0, pi}
};

// Checks unitarity (max |U^dag U - I| <= 1e-10, else Error(FFX_ENOTUNITARY)).
Decomposition givens_decompose(int norb, const cd* U);
double unitarity_defect(int norb, const cd* U);

// A pass applies, in order, a subset of the rotations whose orbitals all lie in
// the window [a, a + w).  Passes are listed in application order.
struct Pass {
  int a;
  std::vector<int> idx;  // indices into the rotation list, in application order
};
std::vector<Pass> schedule_windows(const std::vector<Givens>& rots, int norb, int w);
// The same with as few passes as a beam search of the given width finds: the
// partial schedules with the most rotations applied after each pass are kept
// (ties in a fixed order), and the first complete one is returned; the greedy
// schedule if the search fails.
std::vector<Pass> schedule_windows_beam(const std::vector<Givens>& rots, int norb, int w, int beam);

// Rotations some of which cross a segment window [0, wt): register-window
// stages [a, a + w) inside it (cost 1 each) and whole-spin window passes
// [a, a + W) anywhere that take at least one crossing rotation (cost
// win_cost each), in application order, with the least total cost a beam
// search over partial schedules of equal cost finds (beam states per cost,
// most rotations first, ties in a fixed order).  Empty if it finds none (or
// win_cost < 1).  When `shaped` is given, a stage whose rotation positions
// (relative to a) it rejects costs 2: the kernels run such a stage through
// run-time rotation dispatch instead of straight-line code.
struct SchedPass {
  bool win;  // whole-spin window pass (else a stage inside the segment window)
  int a;
  std::vector<int> idx;
};
std::vector<SchedPass> schedule_windows_cross(const std::vector<Givens>& rots, int norb, int wt, int w, int W,
                                              int beam, int win_cost,
                                              const std::function<bool(const std::vector<int>&)>* shaped = nullptr);

// Window class table of one spin for the window [a, a + w).
// A class is the set of configurations that agree outside the window; its
// members are listed by their in-window pattern in ascending order, so member k
// carries the k-th w-bit pattern with m bits set.  Every class is listed,
// including m = 0 and m = w (single members no rotation touches), so a pass
// can also apply a per-configuration phase to the whole state.  Classes are
// sorted by m and packed into chunks of 64 that share m;
// within a chunk, tab[chunk_off + k * 64 + lane] is the address of member k of
// the lane's class (-1 for padding lanes).
struct WindowTable {
  int a = 0, w = 0;
  std::vector<int> chunk_m, chunk_off, chunk_n;  // per chunk: m, table offset, live lanes
  std::vector<int> tab;
  std::vector<int> cls;  // live classes as (chunk << 6) | lane
};
WindowTable build_window_table(const std::vector<uint64_t>& strs, int norb, int n, int a, int w);

// Class tables of the register window [a, a + w) inside one segment of
// configurations (positions are indices into `seg`).  A segment is a run of
// configurations sharing the occupation of the orbitals >= wt, or several such
// runs back to back (a packed segment); within a run the configurations are in
// colex order of their part below wt.  For a configuration L | M | H (below,
// inside, above the window; l = |L|, m = |M|) the address splits as
// cbase(L, H) + mt(m, l, k), k = rank of M, so a class is described by
// (cbase, l) and the member offsets mt are shared.
struct SegWindowTable {
  int nl1 = 0;                     // number of l values (0 .. nl1-1)
  std::vector<int> code;           // per chunk lane: (cbase << 5) | l, or -1
  std::vector<int> chunk_m;        // per chunk, in order of decreasing work
  std::vector<int> mt;             // [(w+1) * nl1 offsets][tables]
};
// group: lanes that share one LDS access cycle (0: keep classes in address
// order).
SegWindowTable build_seg_window(const std::vector<uint64_t>& seg, int wt, int a, int w, int group = 0);

// The window table of one row replicated over R consecutive rows of length
// row_len held back to back in LDS (class bases shifted by r * row_len), with
// the classes of all rows re-packed into chunks of 64 sharing m.
SegWindowTable replicate_seg_window(const SegWindowTable& t, int w, int R, int row_len);

// The class codes as the device reads them: for a lane's class (cbase, l) in a
// chunk of m electrons in the window, (cbase << kCodeMoffBits) | moff with moff
// = mt_off + mt[m * nl1 + l], the index of the class's member-offset table in
// the segment's LDS table block (mt_off: where this window's tables start in
// it; 0 for compacted tables, whose mt holds that index already), so a lane
// finds its offsets without first looking up that index; -1 stays -1.  Error if cbase or moff does not fit its field.
constexpr int kCodeMoffBits = 14;
std::vector<int> pack_class_codes(const SegWindowTable& t, int mt_off);

// The member-offset tables of a window as the device keeps them: for every
// (m, l) that a class of the table uses (0 < m < w), the C(w, m) offsets as
// 16-bit values, padded to whole 16-byte words and appended to out.  Returns
// the table with mt[m * nl1 + l] = the index, in 16-byte words of out, of that
// (m, l)'s offsets (pack_class_codes then takes mt_off = 0).
SegWindowTable compact_members(const SegWindowTable& t, int w, std::vector<uint16_t>& out);

// The class table for real rotations with the real and imaginary parts of an
// amplitude in neighbouring lanes: lanes 2 j and 2 j + 1 of a chunk hold the
// two parts of one class, with bases counted in parts (2 cbase and 2 cbase +
// 1), so a chunk holds 32 classes.
SegWindowTable split_seg_window(const SegWindowTable& t, int w);

// Reorders the chunks of a segment-pass window table for a block of nwaves
// waves, which take chunks wave, wave + nwaves, ...: the chunks are spread over
// the four SIMDs (wave w runs on SIMD w % 4) so that their estimated work per
// SIMD is balanced (largest chunk first onto the least loaded SIMD); slots
// left over are filled with empty chunks.
void balance_seg_window(SegWindowTable& t, int w, int nwaves);

// Segments of one spin's configurations for the segment passes: runs of
// consecutive configurations (ascending order) that share their orbitals >= wt,
// as (first index, length).
std::vector<std::pair<int, int>> segment_runs(const std::vector<uint64_t>& strs, int wt);
// Consecutive runs packed back to back while their total length stays <= cap.
std::vector<std::pair<int, int>> pack_runs(const std::vector<std::pair<int, int>>& runs, int64_t cap);
// Partner ranges of the rotation on the pair (wt - 1, wt) that straddles the
// segment window, for unpacked runs of n-electron configurations: a run whose
// high part H lacks wt pairs its configurations holding wt - 1 (the last
// C(wt-1, k-1) of its C(wt, k), k = n - |H|) with the first C(wt-1, k-1)
// configurations of the run H + {wt}, which lack wt - 1 (role 0); that run's
// own range is [0, C(wt-1, k)) against the partner range starting at
// C(wt-1, k+1) in the first run (role 1).  Both ranges run in the same colex
// order of the other low orbitals.  has = false: no partner run.
struct CrossRange {
  bool has = false;
  int role = 0, lo = 0, cnt = 0, peer = 0;  // peer: first index of the partner range in strs
};
std::vector<CrossRange> crossing_ranges(const std::vector<uint64_t>& strs, const std::vector<std::pair<int, int>>& runs,
                                        int wt, int n);

// Small dense helpers (row-major, FP64).
std::vector<cd> matmul(int n, const std::vector<cd>& A, const std::vector<cd>& B);
std::vector<cd> dagger(int n, const std::vector<cd>& A);
// Hermitian eigendecomposition A = W diag(w) W^dag by cyclic complex Jacobi.
void eigh(int n, const std::vector<cd>& A, std::vector<double>& w, std::vector<cd>& W);
// expm of an anti-Hermitian K via K = W diag(i w) W^dag.
std::vector<cd> expm_antihermitian(int n, const std::vector<cd>& K);

// The one-body operator sum_pq h_pq a^dag_p a_q of one spin as a sparse matrix
// over its configurations, by target: row j of the result takes
// sum_{e in [off[j], off[j+1])} coef[e] * (row src[e] of the input).  An entry
// for every (p, q) with h_pq != 0, q in I, p not in I (or p == q), J = I - q + p,
// sign (-1)^(occupied orbitals of I strictly between p and q); the diagonal
// terms of a configuration are merged into one entry with src = J.
struct OneBodyTable {
  std::vector<int64_t> off;
  std::vector<int32_t> src;
  std::vector<double> coef;
};
OneBodyTable build_one_body_table(int norb, const std::vector<uint64_t>& strs, const std::vector<double>& h);

// Threads of a segment pass's block, one block for each of n_seg segments of
// each row: the waves that the registers leave a compute unit (max_threads /
// 64), shared by the blocks that its LDS holds (or by the fewer that the launch
// has for it), and no more than the widest window's chunks or four elements a
// thread can use.  At 14 orbitals a row of complex128 leaves room for two
// blocks: 256-thread blocks, one to a unit with 32-bit member tables beside the
// row, ran 963 us per pass.  Fewer where the launch (its rows rounded up to the
// 8 XCDs) would reach 2^32 work-items.
int seg_block_threads(int64_t chunks, size_t lds, int64_t rows, int64_t n_seg, int cus, int max_threads, int max_len);

// The blocks of the one-body row kernel over a rows x cols state: each takes 4
// rows and a tile of 64 columns.  A launch of blocks of 256 threads must stay
// below 2^32 work-items (HIP's limit on a grid dimension), which is 2^32
// amplitudes here, so larger states go out as several launches of at most
// kOneBodyLaunch blocks; it is a multiple of 8, so that a block's place in the
// whole grid still names its XCD.
constexpr int64_t kOneBodyLaunch = (int64_t)1 << 23;
struct OneBodyGrid {
  int64_t row_blocks, tiles;
  bool per_xcd;    // each XCD takes column tiles of its own
  int64_t blocks;  // of all launches; fewer than 2^32 for any state of up to 32 orbitals
};
OneBodyGrid onebody_grid(int64_t rows, int64_t cols, int elem_bytes);
// what block b of the whole grid takes
struct OneBodyBlock {
  uint32_t tile, row_block;
};
constexpr OneBodyBlock onebody_block(uint32_t b, uint32_t row_blocks, bool per_xcd) {
  const uint32_t k = per_xcd ? b >> 3 : b;
  return OneBodyBlock{per_xcd ? (b & 7) + 8 * (k / row_blocks) : k / row_blocks, k % row_blocks};
}

// Bessel functions of the first kind J_0(z) .. J_kmax(z), z >= 0, by Miller's
// backward recurrence J_{k-1} = (2k / z) J_k - J_{k+1} from a start index well
// above kmax, normalised by J_0 + 2 (J_2 + J_4 + ...) = 1.
std::vector<double> bessel_j_series(double z, int kmax);

// Per-string values for the Slater determinant script-U(U)|HF>: for each
// configuration J of n electrons, det U[J, 0:n] (Sec. 2.4), by Laplace
// expansion along the last column over subsets of growing size.
std::vector<cd> slater_column_minors(int norb, int n, const std::vector<cd>& U,
                                     const std::vector<uint64_t>& strs);

}  // namespace ffx
