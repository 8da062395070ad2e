// eps_solve.hip -- the epsilon form of Sec. 4 (Proposition 1, Theorem 1):
// X = (I - eps A)^-1 eps A in fp64, then R = [X > 0].
//
// Method: block Gauss-Jordan elimination without pivoting, in pivot panels p
// of rows and columns: with Q = W[p, p]^-1 (the same elimination in blocks of
// 128, those inverted by Gauss-Jordan in one workgroup)
//   Y = Q W[p, .];  W[q, .] -= W[q, p] Y for every row q outside p;
//   W[p, .] = Y                    (fp64 MFMA products)
// Closure form: in place on W = I - eps A, which becomes the inverse (its
// pivot columns take -W[q, p] Q and Q): 2 Np^3 flops.  X is the inverse off
// the diagonal; its diagonal comes from the equation (k_eps_diag).
// Measured at N = 8192 (degree 4): 21.9 ms against 29.4 ms for the augmented
// system [I - eps A | eps A], whose elimination takes 3 Np^3.
// General right-hand sides (tail-recursive layers): on [I - eps B | eps C],
// the columns right of the panel only, so the right part ends up as X.
//
// Why no pivoting: M = I - eps A has unit diagonal and off-diagonal entries
// <= 0 with eps * (row sum of A) < 1 (Lemma 1's eps bound), so M is a
// strictly diagonally dominant M-matrix; its Schur complements stay
// M-matrices, their inverses are entrywise >= 0, and every update above adds
// terms of one sign to the off-diagonal and right-hand-side entries (rows
// above the diagonal block hold entries <= 0 in the columns being
// eliminated, just like the rows below).  Exact
// zeros therefore stay exactly zero and positive entries never cancel:
// thresholding at > 0 is exact except where a true value underflows fp64
// (it is at least eps^L for a shortest path of length L, by the footnote to
// Lemma 2).  Denormals are kept.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <string>
#include <utility>
#include <vector>

#include "common.h"
#include "device.h"
#include "eps_solve.h"

namespace dl {

constexpr int NB = 128;  // block size of the elimination

// ----------------------------------------------------------------- fp64 MFMA GEMM
// D = A * B (cmode 0) or D = C - A * B (cmode 1);
// A: M x K, B: K x N, C/D: M x N, row-major.  BM x BN output tiles, 2 x 2
// waves (v_mfma_f64_16x16x4f64), K slices of 16 fetched straight into an LDS
// ring of STAGES slices (global_load_lds).  The accumulators start from zero
// and C is read at the end of the tile, so that the K terms round at the size
// of their own sum and C at its own once, not K times: with accumulators that
// start from C the closure form's error (relative, 2-norm, against the series)
// was 1.3e-15 at n = 1000 and 5.9e-15 at N = 8192 (augmented matrix; 1.4e-15 and
// 6.5e-15 in place), and is 5.0e-16 and 7.5e-16 (the block inverse sums the same
// way).  The time: n = 1000 487 -> 496 us, N = 8192 19.6 -> 19.7 ms; C's loads
// mostly hide behind the other workgroup of the compute unit.  D may alias C
// (every element is read and written by the same lane).  A and B must not
// overlap D.
//
// The elimination steps below change single tile rows and columns of a
// product (prow, pcol and np multiples of the launched tile's BM and BN; -1 =
// none):
//  - pivot rows prow .. prow + np - 1: D takes rows of B (row prow + i = B's
//    row i) instead of a product;
//  - pivot columns pcol .. pcol + np - 1: with pmode 1 C counts as zero there,
//    with pmode 2 D takes the columns of A (column
//    pcol + j = A's column j).
// A launch may also copy a matrix (copy_rows x copy_cols from cs to cd) in
// workgroups of its own after the product's.
//
// The doubling of the Stein equations uses the other forms: a second product
// of the same shape in one launch (D2 = A2 B2), B given transposed (template
// BT: B is N x K), a step that returns at once when the doubling before it
// was the last (stop), and the accumulating epilogue (template ACC).
// Counts after each doubling: [2 j] the positive entries of X_j, [2 j + 1] the
// entries that doubling j changed.  Doubling j (1-based) has nothing to do
// when the one before it added no positive entry and, if values are wanted,
// changed none; it then hands its predecessor's counts on, so that every
// later one stops too.
struct SteinStop {
  unsigned long long* cnt = nullptr;  // null: never stops
  int j = 0;
  int values = 0;
  __device__ bool done() const {
    return cnt && j >= 2 && cnt[2 * (j - 1)] == cnt[2 * (j - 2)] && (!values || cnt[2 * (j - 1) + 1] == 0ull);
  }
};

typedef double v2d __attribute__((ext_vector_type(2)));

struct GemmArgs {
  const double* A; int64_t lda;
  const double* B; int64_t ldb;
  const double* C; int64_t ldc;
  double* D; int64_t ldd;
  int M, N, K;
  int cmode;
  int np = 0;
  int prow = -1;
  int pcol = -1, pmode = 0;
  const double* cs = nullptr; int64_t csld = 0;
  double* cd = nullptr; int64_t cdld = 0;
  int copy_rows = 0, copy_cols = 0;
  const double* A2 = nullptr;  // second product, same leading dimensions
  const double* B2 = nullptr;
  double* D2 = nullptr;
  SteinStop stop;
  // K split between the owner of a tile and a helper (template SPLIT)
  double* part = nullptr;     // one partial tile per tile
  unsigned* state = nullptr;  // per tile: arrivals, kPartReady; zero between launches
  int full = 0;               // tiles before the split ones, each a workgroup's own
  int helpers = 0;
};

// Copies rows x cols doubles (cols even, rows 16-byte aligned) with the 256
// threads of a workgroup.
__device__ inline void copy_block(const double* src, int64_t lds_, double* dst, int64_t ldd, int rows, int cols) {
  const int half = cols / 2;
  for (int q = threadIdx.x; q < rows * half; q += 256) {
    const int r = q / half, c = 2 * (q - r * half);
    *(double2*)(dst + (int64_t)r * ldd + c) = *(const double2*)(src + (int64_t)r * lds_ + c);
  }
}
constexpr int kCopyRows = 32;  // rows of one copying workgroup

// Output coordinate of accumulator element `item` of lane `lane` for
// v_mfma_f64_16x16x4f64 (gfx950), as measured on the device.
__device__ inline void f64_acc_coord(int lane, int item, int& r, int& c) {
  r = (lane >> 4) + 4 * item;
  c = lane & 15;
}

// LDS of one slice: the A slice (BM rows x 16 doubles, 128-byte rows; the
// 16-byte chunk c of row r at position c ^ ((r >> 1) & 7)) then the B slice
// (16 k-rows x BN doubles; chunk c of k-row k at c ^ 8 (k & 1); a transposed
// B is laid out like A).  Either way
// the 32 lanes that one ds_read_b64 pass serves (two k values x 16 rows or
// columns) hit 64 distinct banks.
template <int BM, int BN, int STAGES>
struct Dgemm {
  static constexpr int WM = BM / 2, WN = BN / 2;  // four waves, 2 x 2
  static constexpr int FM = WM / 16, FN = WN / 16;
  static constexpr int kSlice = (BM + BN) * 128;
  static constexpr unsigned kLds = STAGES * kSlice;
  static constexpr int kA = BM / 32, kB = BN / 32;  // one-KB instructions per wave and slice
  static_assert(kLds <= 160 * 1024 && BM % 32 == 0 && (BN == 64 || BN == 128), "tile");
};

// What a product's epilogue does: store D, or ACC_ADD: X += product in place
// (X = D), counting the positive entries of the new X and the entries that
// changed, or ACC_SYM: the same for a symmetric result and a symmetric X, of
// which only the tiles on and above the diagonal (in blocks of BN) are
// computed, each off-diagonal one also written mirrored and counted twice.
enum Acc { ACC_NONE = 0, ACC_ADD = 1, ACC_SYM = 2 };

// s_waitcnt with vmcnt = N and no wait on the other counters
template <int N>
__device__ inline void dgemm_wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// Waits until slice kt of nk has landed: at most the later slices' PS
// instructions each (S - 2 slices at most, fewer at the end) are outstanding.
template <int PS, int S>
__device__ inline void dgemm_wait_slice(int later) {
  if constexpr (S <= 2) {
    dgemm_wait_vmcnt<0>();
  } else {
    if (later >= S - 2) dgemm_wait_vmcnt<PS*(S - 2)>();
    else dgemm_wait_slice<PS, S - 1>(later);
  }
}

// SPLIT: the tiles of a product's last pass, t of them, leave slots of the chip
// (two workgroups to a compute unit) without a tile.  Those get helpers:
// helper h takes the last K slices of the c tiles q with q helpers / t = h,
// K / (c + 1) of each, and the owner of a tile the others, so that all
// workgroups have about the same number of slices.  Whichever of the two
// finishes second adds the other's partial tile to its own: the first arrival
// stores its partial with write-through stores and then marks it ready, and
// the second waits for that mark -- of a workgroup that is running and waits
// for nobody -- so no workgroup ever waits for one that may not have started.
// A sum of two is the same in either order, so results do not depend on who
// was first.
constexpr unsigned kPartReady = 1u << 16;
struct SplitPlan {
  int first, count;  // tiles of a helper
  __host__ __device__ SplitPlan(int t, int helpers, int h) {
    first = (int)(((int64_t)h * t + helpers - 1) / helpers);
    count = (int)(((int64_t)(h + 1) * t + helpers - 1) / helpers) - first;
  }
  // K slices of nk that the owners of its tiles keep
  __host__ __device__ int owner_slices(int nk) const { return nk - (nk + count / 2) / (count + 1); }
};

template <int BM, int BN, int STAGES, bool BT = false, int ACC = ACC_NONE, bool SPLIT = false>
__global__ void __launch_bounds__(256, BM == 32 && STAGES == 2 ? 6 : BN == 128 && (SPLIT || ACC == ACC_SYM) ? 2 : 1) k_dgemm(GemmArgs g) {
  typedef Dgemm<BM, BN, STAGES> T;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  // the variant that runs beside a trailing update (see gj_blocks) issues first
  if constexpr (BM == 32 && STAGES == 2) __builtin_amdgcn_s_setprio(3);
  if (g.stop.done()) {
    if (ACC != ACC_NONE && blockIdx.x == 0 && tid == 0) g.stop.cnt[2 * g.stop.j] = g.stop.cnt[2 * (g.stop.j - 1)];
    return;
  }
  const int tiles_m = g.M / BM;
  // this workgroup's pieces: tiles first .. first + pieces - 1, slices kb .. ke - 1 of each
  const int nk = g.K / 16;
  int first = (int)blockIdx.x, pieces = 1, kb = 0, ke = nk;
  if constexpr (SPLIT) {
    const int t = (int)gridDim.x - g.full - g.helpers, q = first - g.full;
    if (q >= 0) {
      const SplitPlan plan(t, g.helpers, q < t ? (int)((int64_t)q * g.helpers / t) : q - t);
      if (q < t) {
        ke = plan.owner_slices(nk);
      } else {
        kb = plan.owner_slices(nk);
        first = g.full + plan.first;
        pieces = plan.count;
      }
    }
  }
  for (int piece = 0; piece < (SPLIT ? pieces : 1); ++piece) {
  const int tile = first + piece;
  // split: nothing derived from the lane stays in registers from piece to piece
  if constexpr (SPLIT) asm volatile("v_mov_b32 %0, %1" : "=v"(tid) : "v"((int)threadIdx.x));
  int lane = tid & 63;
  if (SPLIT && piece > 0) __syncthreads();  // every wave is done with the ring
  int m0, n0;
  if constexpr (ACC == ACC_SYM) {
    // block q of the upper triangle in column order, sub-tile tile % (BN / BM)
    const int q = tile / (BN / BM);
    int tn = (int)((sqrtf(8.0f * (float)q + 1.0f) - 1.0f) * 0.5f);
    while (tn * (tn + 1) / 2 > q) --tn;
    while ((tn + 1) * (tn + 2) / 2 <= q) ++tn;
    m0 = (q - tn * (tn + 1) / 2) * BN + (tile % (BN / BM)) * BM;
    n0 = tn * BN;
  } else {
    // column-major walk over tiles keeps one B column panel hot across rows
    int b = tile;
    if (!SPLIT && g.A2) {
      const int tiles = tiles_m * (g.N / BN);
      if (b >= tiles) {
        b -= tiles;
        g.A = g.A2;
        g.B = g.B2;
        g.D = g.D2;
      }
    }
    m0 = b % tiles_m * BM;
    n0 = b / tiles_m * BN;
  }
  if (!SPLIT && n0 >= g.N) {  // past the product: a copying workgroup
    const int r0 = ((int)blockIdx.x - tiles_m * (g.N / BN)) * kCopyRows;
    copy_block(g.cs + (int64_t)r0 * g.csld, g.csld, g.cd + (int64_t)r0 * g.cdld, g.cdld,
               min(kCopyRows, g.copy_rows - r0), g.copy_cols);
    return;
  }
  if (!SPLIT && g.prow >= 0 && m0 >= g.prow && m0 < g.prow + g.np) {
    copy_block(g.B + (int64_t)(m0 - g.prow) * g.ldb + n0, g.ldb, g.D + (int64_t)m0 * g.ldd + n0, g.ldd, BM, BN);
    return;
  }
  const bool in_pcol = !SPLIT && g.pcol >= 0 && n0 >= g.pcol && n0 < g.pcol + g.np;
  if (in_pcol && g.pmode == 2) {
    copy_block(g.A + (int64_t)m0 * g.lda + (n0 - g.pcol), g.lda, g.D + (int64_t)m0 * g.ldd + n0, g.ldd, BM, BN);
    return;
  }

  // Each wave issues its share of a slice's one-KB direct-to-LDS
  // instructions: A instruction a = wave + 4 jj covers rows 8a .. 8a + 7
  // (lane l: row 8a + l / 8, LDS chunk l % 8), B instruction b = wave + 4 jj
  // covers 128 / BN k-rows (lane l: LDS chunk l of that run).
  const double* asrc[T::kA];
  const double* bsrc[T::kB];
#pragma unroll
  for (int jj = 0; jj < T::kA; ++jj) {
    const int row = 8 * (wave + 4 * jj) + (lane >> 3);
    asrc[jj] = g.A + (int64_t)(m0 + row) * g.lda + 2 * ((lane & 7) ^ ((row >> 1) & 7));
  }
#pragma unroll
  for (int jj = 0; jj < T::kB; ++jj) {
    if constexpr (BT) {
      const int row = 8 * (wave + 4 * jj) + (lane >> 3);
      bsrc[jj] = g.B + (int64_t)(n0 + row) * g.ldb + 2 * ((lane & 7) ^ ((row >> 1) & 7));
    } else {
      const int q = (wave + 4 * jj) * 64 + lane, k = q / (BN / 2), ch = q % (BN / 2);
      bsrc[jj] = g.B + (int64_t)k * g.ldb + n0 + 2 * (ch ^ (8 * (k & 1)));
    }
  }
  auto issue = [&](int kt, int slot) {
    uint8_t* stage = lds + slot * T::kSlice;
    const int k0 = (kb + kt) * 16;
#pragma unroll
    for (int jj = 0; jj < T::kA; ++jj)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(asrc[jj] + k0),
                                       (__attribute__((address_space(3))) void*)(stage + (wave + 4 * jj) * 1024),
                                       16, 0, 0);
#pragma unroll
    for (int jj = 0; jj < T::kB; ++jj)
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)(bsrc[jj] + (BT ? k0 : (int64_t)k0 * g.ldb)),
          (__attribute__((address_space(3))) void*)(stage + BM * 128 + (wave + 4 * jj) * 1024), 16, 0, 0);
  };

  // fragment reads: lane (g4, r16) = (lane / 16, lane % 16) supplies
  // A[row r16][k g4] and B[k g4][column r16] of each 16 x 16 x 4 product
  const int g4 = lane >> 4, r16 = lane & 15;
  auto frags = [&](const uint8_t* st, int kk, double* af, double* bf) {
    const int k = kk + g4;
#pragma unroll
    for (int i = 0; i < T::FM; ++i) {
      const int r = wm * T::WM + i * 16 + r16;
      af[i] = *(const double*)(st + r * 128 + (((k >> 1) ^ ((r >> 1) & 7)) << 4) + ((k & 1) << 3));
    }
#pragma unroll
    for (int j = 0; j < T::FN; ++j) {
      const int n = wn * T::WN + j * 16 + r16;
      bf[j] = BT ? *(const double*)(st + BM * 128 + n * 128 + (((k >> 1) ^ ((n >> 1) & 7)) << 4) + ((k & 1) << 3))
                 : *(const double*)(st + BM * 128 + k * (BN * 8) + (((n >> 1) ^ (8 * (k & 1))) << 4) + ((n & 1) << 3));
    }
  };

  const int nks = ke - kb;
#pragma unroll
  for (int s0 = 0; s0 < STAGES - 1; ++s0)
    if (s0 < nks) issue(s0, s0);

  v4d acc[T::FM][T::FN];
#pragma unroll
  for (int i = 0; i < T::FM; ++i)
#pragma unroll
    for (int j = 0; j < T::FN; ++j) acc[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
  // C's and D's elements under this wave's fragments: one lane offset, and a
  // uniform one for each element (addresses of their own would take the
  // registers of a panel inverse beside this product)
  const int64_t row0 = m0 + wm * T::WM, col0 = n0 + wn * T::WN;
  const bool minus = ACC == ACC_NONE && !SPLIT && g.cmode == 1;
  auto tile_buffer = [&](const double* base, int64_t ld) {
    return buffer_of((void*)(base + row0 * ld + col0), (unsigned)(((T::WM - 1) * ld + T::WN) * sizeof(double)));
  };
  auto lane_offset = [&](int64_t ld) { return (int)(((lane >> 4) * ld + (lane & 15)) * sizeof(double)); };
  auto element_offset = [](int i, int j, int v, int64_t ld) {  // f64_acc_coord of the fragment
    return (int)(((i * 16 + 4 * v) * ld + j * 16) * sizeof(double));
  };
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  v4d cc[T::FN];
  auto load_c = [&](int i) {
    const __amdgpu_buffer_rsrc_t buf = tile_buffer(g.C, g.ldc);
    const int off = lane_offset(g.ldc);
#pragma unroll
    for (int j = 0; j < T::FN; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        cc[j][v] = __builtin_bit_cast(
            double, __builtin_amdgcn_raw_buffer_load_b64(buf, off, element_offset(i, j, v, g.ldc), 0));
  };

  int slot = 0;
  for (int kt = 0; kt < nks; ++kt) {
    // slice kt has landed once at most the later slices' instructions are
    // outstanding; the barrier extends that to every wave and retires every
    // read of the slot before it in the ring, refilled below
    dgemm_wait_slice<T::kA + T::kB, STAGES>(nks - 1 - kt);
    __builtin_amdgcn_s_barrier();
    if (kt + STAGES - 1 < nks) issue(kt + STAGES - 1, slot == 0 ? STAGES - 1 : slot - 1);
    const uint8_t* st = lds + slot * T::kSlice;
    slot = slot + 1 == STAGES ? 0 : slot + 1;
    double af[2][T::FM], bf[2][T::FN];
    frags(st, 0, af[0], bf[0]);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (q < 3) frags(st, 4 * (q + 1), af[(q + 1) & 1], bf[(q + 1) & 1]);
#pragma unroll
      for (int i = 0; i < T::FM; ++i)
#pragma unroll
        for (int j = 0; j < T::FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(af[q & 1][i], bf[q & 1][j], acc[i][j], 0, 0, 0);
    }
  }

  if constexpr (SPLIT || BM * BN == 128 * 128) {
    // re-derived: addresses computed from it are not kept live across the products
    asm volatile("v_mov_b32 %0, %1" : "=v"(tid) : "v"((int)threadIdx.x));
    lane = tid & 63;
  }
  if (SPLIT && tile >= g.full) {
    // element pair e of thread tid at 16 (256 e + tid): the same in either piece
    constexpr int kPairs = T::FM * T::FN * 2;
    constexpr unsigned kTile = BM * BN * 8;
    static_assert(kPairs * 256 * 16 == (int)kTile, "the partial tile");
    __shared__ unsigned s_before;
    const __amdgpu_buffer_rsrc_t part = buffer_of((uint8_t*)g.part + (size_t)(tile - g.full) * kTile, kTile);
    unsigned* state = g.state + (tile - g.full);
    __syncthreads();
    if (tid == 0) s_before = __hip_atomic_fetch_add(state, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if ((s_before & (kPartReady - 1)) == 0u) {  // first: leave the partial tile to the other
#pragma unroll
      for (int e = 0; e < kPairs; ++e) {
        const v4d& x = acc[e / 2 / T::FN][e / 2 % T::FN];
        st_agent_x4(part, (256 * e + tid) * 16, __builtin_bit_cast(u32x4, v2d{x[2 * (e & 1)], x[2 * (e & 1) + 1]}));
      }
      wait_stores();
      __syncthreads();
      if (tid == 0) __hip_atomic_fetch_add(state, kPartReady, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      continue;
    }
    if (tid == 0) {
      while (ld_agent(state) < kPartReady) __builtin_amdgcn_s_sleep(2);
      st_agent(state, 0u);
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kPairs; e += 4) {
      v2d w[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        w[u] = __builtin_bit_cast(
            v2d, __builtin_amdgcn_raw_buffer_load_b128(part, (256 * (e + u) + tid) * 16, 0, kCpolSc1));
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        v4d& x = acc[(e + u) / 2 / T::FN][(e + u) / 2 % T::FN];
        x[2 * (u & 1)] += w[u][0];
        x[2 * (u & 1) + 1] += w[u][1];
      }
      __builtin_amdgcn_sched_barrier(0);  // four loads in flight: more would spill accumulators
    }
  }
  int pos = 0, chg = 0;
  const bool mirror = ACC == ACC_SYM && m0 / BN < n0 / BN;
  if constexpr (ACC == ACC_NONE) {
    const __amdgpu_buffer_rsrc_t out = tile_buffer(g.D, g.ldd);
    const int out_off = lane_offset(g.ldd);
    auto store = [&](int i, int j, const v4d& x) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double d = x[v];
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, d), out, out_off,
                                              element_offset(i, j, v, g.ldd), 0);
      }
    };
    if (minus && !in_pcol) {
#pragma unroll
      for (int i = 0; i < T::FM; ++i) {
        load_c(i);
#pragma unroll
        for (int j = 0; j < T::FN; ++j) acc[i][j] = cc[j] - acc[i][j];
#pragma unroll
        for (int j = 0; j < T::FN; ++j) store(i, j, acc[i][j]);
        if constexpr (BM * BN == 128 * 128) __builtin_amdgcn_sched_barrier(0);  // more loads in flight would spill accumulators
      }
    } else {
      const double sign = minus ? -1.0 : 1.0;
#pragma unroll
      for (int i = 0; i < T::FM; ++i)
#pragma unroll
        for (int j = 0; j < T::FN; ++j) store(i, j, sign * acc[i][j]);
    }
  } else {
#pragma unroll
    for (int i = 0; i < T::FM; ++i)
#pragma unroll
      for (int j = 0; j < T::FN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          int r, c;
          f64_acc_coord(lane, v, r, c);
          const int64_t row = row0 + i * 16 + r, col = col0 + j * 16 + c;
          double* d = g.D + row * g.ldd + col;
          const double x = *d, y = x + acc[i][j][v];
          pos += y > 0.0;
          chg += y != x;
          *d = y;
          if (mirror) g.D[col * g.ldd + row] = y;
          if constexpr (BM * BN == 128 * 128)
            if (v == 3) __builtin_amdgcn_sched_barrier(0);  // more loads in flight would spill accumulators
        }
  }
  if constexpr (ACC != ACC_NONE) {
    __shared__ int red[2][4];
    for (int off = 32; off > 0; off >>= 1) {
      pos += __shfl_xor(pos, off, 64);
      chg += __shfl_xor(chg, off, 64);
    }
    if (lane == 0) {
      red[0][wave] = pos;
      red[1][wave] = chg;
    }
    __syncthreads();
    if (tid < 2) {
      const int t = red[tid][0] + red[tid][1] + red[tid][2] + red[tid][3];
      if (t) atomicAdd(g.stop.cnt + 2 * g.stop.j + tid, (unsigned long long)(mirror ? 2 * t : t));
    }
  }
  }
}

template <int BM, int BN, int STAGES, bool BT, int ACC>
static hipError_t dgemm_launch(const GemmArgs& g, hipStream_t s) {
  int64_t tiles = (int64_t)(g.M / BM) * (g.N / BN);
  if (ACC == ACC_SYM) {
    const int64_t side = g.N / BN;
    tiles = side * (side + 1) / 2 * (BN / BM);
  }
  const int64_t grid = (g.A2 ? 2 : 1) * tiles + (g.copy_rows + kCopyRows - 1) / kCopyRows;
  hipLaunchKernelGGL((k_dgemm<BM, BN, STAGES, BT, ACC>), dim3((unsigned)grid), dim3(256),
                     (Dgemm<BM, BN, STAGES>::kLds), s, g);
  return hipGetLastError();
}

template <int BM, int BN, bool BT, int ACC>
static hipError_t dgemm_launch_split(const GemmArgs& g, int tiles, hipStream_t s) {
  hipLaunchKernelGGL((k_dgemm<BM, BN, 2, BT, ACC, true>), dim3((unsigned)(tiles + g.helpers)), dim3(256),
                     (Dgemm<BM, BN, 2>::kLds), s, g);
  return hipGetLastError();
}

template <int BM, int BN, int STAGES, bool BT, int ACC>
static hipError_t dgemm_attr() {
  return hipFuncSetAttribute((const void*)k_dgemm<BM, BN, STAGES, BT, ACC>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)Dgemm<BM, BN, STAGES>::kLds);
}

template <bool BT, int ACC>
static hipError_t dgemm_attrs() {
  hipError_t e = dgemm_attr<ACC == ACC_SYM ? 64 : 128, 128, 2, BT, ACC>();
  if (e == hipSuccess) e = dgemm_attr<64, 64, 3, BT, ACC>();
  if (e == hipSuccess) e = dgemm_attr<32, 64, 4, BT, ACC>();
  return e;
}

// Tile rule, from the number t of 128 x 128 tiles (MI355X, 256 compute units;
// two-slice rings of 64 KB, so that two workgroups share a compute unit and
// one's barriers and tile ends are covered by the other's products):
//  - t fills whole passes over the 256 compute units to 85%: 128 x 128.
//    M = N = 8192, K = 512: 64.7 TFLOP/s (four-slice ring, one workgroup per
//    compute unit: 51.9; 64 x 64 tiles: 60.7); M = N = K = 4096: 69.1 (64.2).
//  - otherwise smaller tiles, whose last pass is shorter: 64 x 64 while they
//    number more than 256 (M = N = K = 2560: 55.9 against 53.4 TFLOP/s),
//    else 32 x 64 (1024: 46.1 against 16.0; M = N = 512, K = 128: 7.6 against
//    22.5 us).  A 64 x 64 tile moves 16 KB into LDS for 1024 clocks of
//    products, so small tiles stay bound by the products.
//  - with room for partial tiles (g.part), a last pass of 257 to 460 of the 512
//    slots is split (SPLIT).  M = N = K = 2304, 2560, 2688: 402, 540, 612 us;
//    whole 128 x 128 tiles 573, 633, 668, 64 x 64 tiles 463, 594, 633.  From
//    there on the slots left are too few (2816, 484 tiles: 753 against 695).
// A symmetric product takes halves of the 128 x 128 tiles, since the whole
// tile's epilogue does not fit in the registers of two workgroups to a compute
// unit (2816: 382 against 406 us), and splits them where 64 x 64 tiles fill
// their passes to less than 85% (2048, 2560: 199, 317 us against 210, 352;
// 2432, filled to 96%: 261 against 252).
constexpr int kSplitSlots = 512;
template <bool BT = false, int ACC = ACC_NONE>
static hipError_t dgemm(const GemmArgs& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (g.M % 128 || g.N % 128 || g.K % 16) return hipErrorInvalidValue;
  constexpr int BM = ACC == ACC_SYM ? 64 : 128;
  const int64_t side = g.N / 128;
  const int64_t t = ACC == ACC_SYM ? side * (side + 1) / 2 : (g.A2 ? 2 : 1) * (int64_t)(g.M / 128) * side;
  auto fills = [](int64_t tiles) { return tiles * 100 >= (tiles + 255) / 256 * 256 * 85; };
  if (g.part && !g.A2 && !(ACC == ACC_SYM && fills(side * (2 * side + 1)))) {
    const int64_t tiles = t * (128 / BM), last = tiles % kSplitSlots;
    if (last > kSplitSlots / 2 && last <= 460) {
      GemmArgs h = g;
      h.full = (int)(tiles - last);
      h.helpers = kSplitSlots - (int)last;
      return dgemm_launch_split<BM, 128, BT, ACC>(h, (int)tiles, s);
    }
  }
  if (fills(t)) return dgemm_launch<BM, 128, 2, BT, ACC>(g, s);
  return 4 * t > 256 ? dgemm_launch<64, 64, 3, BT, ACC>(g, s) : dgemm_launch<32, 64, 4, BT, ACC>(g, s);
}

// ----------------------------------------------------------------- diagonal block inverse
// In-place Gauss-Jordan inversion of the NB x NB block at W (ld), written to
// Dinv (ldd; may be W itself), in NB / 16 steps of 16 x 16 pivot blocks on the matrix cores.
// Eight waves own a column of eight 16 x 16 tiles each, kept in MFMA
// accumulators for the whole kernel; a ninth wave inverts the pivot blocks.
// Step k, with Q = a[k][k]^-1 and C = a[.][k] in LDS (C negated):
//   Y = Q a[k][j]                       (the wave's own tile: the accumulator
//                                        layout is the layout of operand B)
//   a[i][j] += (-C[i]) Y  (i != k),  a[k][j] = Y
// and in the pivot column j = k the same with a[i][k] = 0 and Y = Q, which
// leaves -C[i] Q and Q.  Every wave updates its tile of row k + 1 first; the
// owner of the next pivot block hands it to the ninth wave, which inverts it
// while the others finish step k, so the serial chain (16 pivots in a block)
// runs beside the products.
// Bound by one compute unit's fp64 matrix cores: 2 NB^3 operations at 128 per
// clock are 13.7 us.  Measured per 128 x 128 block (MI355X): 31 us, against
// 175 us of the version before it, which took 64 steps of 2 x 2 pivots, each a
// barrier, two dependent divisions and a rank-2 update on the vector units.
// Signs: the block is a strictly diagonally dominant M-matrix, so every
// inverse is >= 0 entrywise and, as for single pivots, every update adds
// terms of one sign to each off-diagonal entry (columns already pivoted hold
// entries >= 0, the others <= 0), so zeros stay exact and nothing cancels.
constexpr int kInvPitch = 17;  // doubles per 16-wide LDS row: operand reads and tile writes hit distinct banks

// Lane n of each row of 16 lanes, to all lanes of that row.
template <int N>
__device__ inline double row_lane(double v) {
  const int2 x = __builtin_bit_cast(int2, v);
  int2 r;
  r.x = __builtin_amdgcn_update_dpp(0, x.x, 0x150 + N, 0xf, 0xf, true);  // row_newbcast:N
  r.y = __builtin_amdgcn_update_dpp(0, x.y, 0x150 + N, 0xf, 0xf, true);
  return __builtin_bit_cast(double, r);
}

// Row G (lanes 16 G .. 16 G + 15) of v, to all four rows of lanes.
template <int G>
__device__ inline int lane_row(int v) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 h = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
  const unsigned w = G < 2 ? h[0] : h[1];  // the half that holds row G, twice
  const u32x2 q = __builtin_amdgcn_permlane16_swap(w, w, false, false);
  return (int)((G & 1) ? q[1] : q[0]);
}

// 1 / x for the pivots, which lie in (1 / 65537, 1]: the hardware estimate and
// two Newton steps (each squares the relative error, and the second one's
// rounding is that of its last multiply-add).
__device__ inline double pivot_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
  return __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
}

// Gauss-Jordan step P of the 16 x 16 inverse held by one wave: lane (r, g) =
// (lane % 16, lane / 16) has columns 4 g .. 4 g + 3 of row r.
template <int P>
__device__ inline void inv16_step(double (&a)[4], int r, int g) {
  constexpr int G = P >> 2, J = P & 3;
  const int2 x = __builtin_bit_cast(int2, a[J]);
  int2 cx;
  cx.x = lane_row<G>(x.x);
  cx.y = lane_row<G>(x.y);
  const double col = __builtin_bit_cast(double, cx);  // a[r][P]
  const double inv = pivot_rcp(row_lane<P>(col));
  const double f = -col * inv;
  // row P becomes a inv = a + (inv - 1) a: the other rows' multiply-add (the
  // difference is rounded once, and not at all for pivots in [1/2, 1])
  const double m = r == P ? inv - 1.0 : f;
#pragma unroll
  for (int j = 0; j < 4; ++j) a[j] = __builtin_fma(m, row_lane<P>(a[j]), a[j]);  // a[P][4 g + j]
  if (g == G) a[J] = r == P ? inv : f;
}

template <int P>
__device__ inline void inv16_steps(double (&a)[4], int r, int g) {
  inv16_step<P>(a, r, g);
  if constexpr (P < 15) inv16_steps<P + 1>(a, r, g);
}

// NT = 8: blocks of 128, eight column waves and the inverting wave.  NT = 4:
// blocks of 64 for a panel inverse that runs beside the trailing update: four
// waves of 72 registers and 24 KB of LDS, which fit on a compute unit beside two
// update workgroups (2 x 184 registers a SIMD lane, 2 x 64 KB); the wave that
// owns the next pivot block inverts it itself.
template <int NT>
__global__ void __launch_bounds__(NT == 8 ? 576 : 256, NT == 8 ? 1 : 6)
k_block_inverse(const double* W, int64_t ld, double* Dinv, int64_t ldd) {
  // beside a trailing update its waves issue first: it is the longer chain
  __builtin_amdgcn_s_setprio(3);
  constexpr bool kOwn = NT == 4;
  __shared__ double cbuf[2][16 * NT * kInvPitch];  // -C of steps k and k + 1
  __shared__ double dbuf[16 * kInvPitch];          // pivot block to invert
  __shared__ double qbuf[2][16 * kInvPitch];       // its inverse, steps k and k + 1
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, c = lane & 15;
  // Q of step k from the pivot block in dbuf, by one wave
  auto invert = [&](int k) {
    double a[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) a[j] = dbuf[c * kInvPitch + 4 * g + j];
    inv16_steps<0>(a, c, g);
#pragma unroll
    for (int j = 0; j < 4; ++j) qbuf[k & 1][c * kInvPitch + 4 * g + j] = a[j];
  };
  if (wave == NT) {  // the inverting wave
    for (int k = 0; k < NT; ++k) {
      __syncthreads();  // pivot block k is in dbuf
      invert(k);
      __syncthreads();  // Q and C of step k are in LDS
    }
    return;
  }
  // tile i of this wave: element v of a lane is row 16 i + g + 4 v, column 16 wave + c
  v4d acc[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[i][v] = W[(int64_t)(16 * i + g + 4 * v) * ld + 16 * wave + c];
  // this wave's column as the panel -C of step k (k = wave)
  auto publish_c = [&]() {
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) cbuf[wave & 1][(16 * i + g + 4 * v) * kInvPitch + c] = -acc[i][v];
  };
  // hands the pivot block of step k over (and inverts it, without a wave for that)
  auto pivot = [&](const v4d& t, int k) {
#pragma unroll
    for (int v = 0; v < 4; ++v) dbuf[(g + 4 * v) * kInvPitch + c] = t[v];
    if constexpr (kOwn) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      invert(k);
    }
  };
  // the first pivot block (kOwn: as step -1, so that the inverse's code is there once)
  if constexpr (!kOwn) {
    if (wave == 0) pivot(acc[0], 0);
    __syncthreads();
    if (wave == 0) publish_c();
    __syncthreads();
  }
  for (int k = kOwn ? -1 : 0; k < NT; ++k) {
    const double* q = qbuf[k & 1];
    const double* cb = cbuf[k & 1];
    v4d y = {0.0, 0.0, 0.0, 0.0};
    if (kOwn && k < 0) {
    } else if (wave == k) {
#pragma unroll
      for (int v = 0; v < 4; ++v) y[v] = q[(g + 4 * v) * kInvPitch + c];
#pragma unroll
      for (int i = 0; i < NT; ++i) acc[i] = v4d{0.0, 0.0, 0.0, 0.0};
    } else {
      v4d t = acc[0];
#pragma unroll
      for (int i = 1; i < NT; ++i)
        if (i == k) t = acc[i];
#pragma unroll
      for (int v = 0; v < 4; ++v)
        y = __builtin_amdgcn_mfma_f64_16x16x4f64(q[c * kInvPitch + 4 * v + g], t[v], y, 0, 0, 0);
    }
    auto update = [&](int i) {
      if (i == k) {
        acc[i] = y;
        return;
      }
      v4d z = {0.0, 0.0, 0.0, 0.0};  // from zero: see k_dgemm
#pragma unroll
      for (int v = 0; v < 4; ++v)
        z = __builtin_amdgcn_mfma_f64_16x16x4f64(cb[(16 * i + c) * kInvPitch + 4 * v + g], y[v], z, 0, 0, 0);
      acc[i] += z;
      if constexpr (kOwn) __builtin_amdgcn_sched_barrier(0);  // operand reads of later tiles would cost registers
    };
    if (k + 1 < NT) {
      v4d t = acc[0];
#pragma unroll
      for (int i = 0; i < NT; ++i)
        if (i == k + 1) {
          if (!kOwn || k >= 0) update(i);
          if (!kOwn && wave == i) pivot(acc[i], i);
          t = acc[i];
        }
      if (kOwn && wave == k + 1) pivot(t, k + 1);
      if constexpr (!kOwn) __syncthreads();  // the next pivot block is ready
    }
    if (!kOwn || k >= 0) {
#pragma unroll
      for (int i = 0; i < NT; ++i)
        if (i != k + 1) update(i);
    }
    if (k + 1 < NT) {
      if (wave == k + 1) publish_c();
      __syncthreads();
    }
  }
  int lane2;  // re-derived: addresses computed from it are not kept live across the steps
  asm volatile("v_mov_b32 %0, %1" : "=v"(lane2) : "v"(lane));
  double* dst = Dinv + (lane2 >> 4) * ldd + 16 * wave + (lane2 & 15);
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) dst[(int64_t)(16 * i + 4 * v) * ldd] = acc[i][v];
}

// ----------------------------------------------------------------- setup / copy / emit
// Four consecutive doubles, two 16-byte accesses; 8-byte alignment for the
// caller's matrices (their stride may be odd).
typedef v2d v2d_8 __attribute__((aligned(8)));
typedef unsigned u32_any __attribute__((aligned(1)));

// The bytes j .. j + 3 of a row of n as flags, 0 past its end.
__device__ inline unsigned bytes4(const uint8_t* row, int j, int n) {
  if (j + 4 <= n) {
    unsigned x = *(const u32_any*)(row + j);
    x |= x >> 4;
    x |= x >> 2;
    x |= x >> 1;
    return x & 0x01010101u;
  }
  unsigned x = 0u;
  for (int e = 0; e < 4; ++e)
    if (j + e < n && row[j + e] != 0) x |= 1u << (8 * e);
  return x;
}

// W[i][j] = [i == j] - eps b_ij  and, with C, W[i][Np + j] = eps c_ij; padded
// rows and columns carry the identity and zeros.  Four columns a thread.
__global__ void __launch_bounds__(256) k_eps_init(const uint8_t* B, int64_t ldb, const uint8_t* C, int64_t ldc,
                                                  int n, int Np, double eps, double* W) {
  const int i = blockIdx.y;
  const int64_t ld = C ? 2 * (int64_t)Np : Np;
  for (int j = 4 * (blockIdx.x * 256 + threadIdx.x); j < Np; j += 1024 * gridDim.x) {
    const unsigned b = i < n ? bytes4(B + (int64_t)i * ldb, j, n) : 0u;
    v2d w[2];
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e >> 1][e & 1] = (i == j + e ? 1.0 : 0.0) - (((b >> (8 * e)) & 1u) ? eps : 0.0);
    *(v2d*)(W + i * ld + j) = w[0];
    *(v2d*)(W + i * ld + j + 2) = w[1];
    if (C) {
      const unsigned c = i < n ? bytes4(C + (int64_t)i * ldc, j, n) : 0u;
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e >> 1][e & 1] = ((c >> (8 * e)) & 1u) ? eps : 0.0;
      *(v2d*)(W + i * ld + Np + j) = w[0];
      *(v2d*)(W + i * ld + Np + j + 2) = w[1];
    }
  }
}

// The diagonal of X in the closure form.  There X = (I - eps A)^-1 - I: off
// the diagonal the inverse itself, on it a difference that would cancel; the
// equation X = eps A + eps A X gives it from terms of one sign instead:
//   X_ii = eps (a_ii + sum_{k != i} a_ik X_ki) / (1 - eps a_ii).
// part[chunk][i] receives the sum over the chunk's k (added up by k_eps_emit
// in chunk order).  A workgroup takes 64 columns i and the rows k of one
// chunk; A is read 16 bytes at a time.
// Chunks of 128: n = 1000 13 us (512, one load at a time: 30 us).
constexpr int kDiagChunk = 128;
__global__ void __launch_bounds__(256)
k_eps_diag(const uint8_t* A, int64_t lda, const double* W, int n, int Np, double* part) {
  __shared__ double red[4][64];
  const int c = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + c;
  const int k1 = min(n, ((int)blockIdx.y + 1) * kDiagChunk);
  double sum = 0.0;
  if (i < n) {
    for (int k0 = blockIdx.y * kDiagChunk + 16 * q; k0 < k1; k0 += 64) {
      const uint8_t* src = A + (int64_t)i * lda + k0;
      uint8_t b[16] = {};
      if (k0 + 16 <= k1) __builtin_memcpy(b, src, 16);
      else
        for (int e = 0; e < k1 - k0; ++e) b[e] = src[e];
      // every lane loads (those without the edge W[0], unused), so that the
      // sixteen loads are in flight together
      double v[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) v[e] = W[b[e] != 0 ? (int64_t)(k0 + e) * Np + i : 0];
#pragma unroll
      for (int e = 0; e < 16; ++e) sum += b[e] != 0 && k0 + e != i ? v[e] : 0.0;
    }
  }
  red[q][c] = sum;
  __syncthreads();
  if (q == 0 && i < n) part[(int64_t)blockIdx.y * Np + i] = (red[0][c] + red[1][c]) + (red[2][c] + red[3][c]);
}

// R = [X > 0] (and X itself when asked for), plus the smallest positive
// entry of X: its bits go into *minpos by an unsigned atomic minimum (positive
// doubles order like their bit patterns), one per workgroup.  A fixed grid of
// 16-wave workgroups walks the rows, four columns a thread, so the atomics
// stay few (1024 of them took most of 17 us at n = 1000, now 10; n = 8192,
// X written: 292 us with one column a thread, now 254).  X is n x n with row
// stride ldw (even); with part set its diagonal comes from the sums of
// k_eps_diag.
constexpr int kEmitBlocks = 512;
__global__ void __launch_bounds__(1024)
k_eps_emit(const double* Xw, int64_t ldw, int n, uint8_t* R, int64_t ldr, double* X, int64_t ldx,
           unsigned long long* minpos, const double* part, int Np, int nchunk, const uint8_t* A, int64_t lda,
           double eps) {
  __shared__ unsigned long long red[16];
  unsigned long long m = ~0ull;
  const int tpr = (n + 3) / 4 < 1024 ? ((n + 3) / 4 + 63) / 64 * 64 : 1024;  // threads per row
  const int rpb = 1024 / tpr;                                               // rows at once
  const int sub = (int)threadIdx.x / tpr, tj = (int)threadIdx.x % tpr;
  for (int i = blockIdx.x * rpb + sub; i < n && sub < rpb; i += gridDim.x * rpb) {
    for (int j = 4 * tj; j < n; j += 4 * tpr) {
      // whole groups of four lie inside the padded row
      const v2d a = *(const v2d*)(Xw + i * ldw + j), b = *(const v2d*)(Xw + i * ldw + j + 2);
      double x[4] = {a.x, a.y, b.x, b.y};
      if (part && i >= j && i < j + 4) {
        const double aii = A[(int64_t)i * lda + i] != 0 ? 1.0 : 0.0;
        double d = aii;
        for (int ch = 0; ch < nchunk; ++ch) d += part[(int64_t)ch * Np + i];
        d = eps * d / (1.0 - eps * aii);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (i == j + e) x[e] = d;
      }
      unsigned r = 0u;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (x[e] > 0.0 && j + e < n) {
          r |= 1u << (8 * e);
          const unsigned long long v = (unsigned long long)__double_as_longlong(x[e]);
          m = v < m ? v : m;
        }
      if (j + 4 <= n) {
        *(u32_any*)(R + (int64_t)i * ldr + j) = r;
        if (X) {
          *(v2d_8*)(X + (int64_t)i * ldx + j) = v2d{x[0], x[1]};
          *(v2d_8*)(X + (int64_t)i * ldx + j + 2) = v2d{x[2], x[3]};
        }
      } else {
        for (int e = 0; e < 4 && j + e < n; ++e) {
          R[(int64_t)i * ldr + j + e] = (uint8_t)((r >> (8 * e)) & 1u);
          if (X) X[(int64_t)i * ldx + j + e] = x[e];
        }
      }
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long v = __shfl_xor(m, o);
    m = v < m ? v : m;
  }
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 16; ++w) m = red[w] < m ? red[w] : m;
    if (m != ~0ull) atomicMin(minpos, m);
  }
}

__global__ void k_set_word(unsigned long long* p, unsigned long long v) { *p = v; }

// ----------------------------------------------------------------- driver
hipError_t eps_kernels_init() {
  hipError_t e = dgemm_attrs<false, ACC_NONE>();
  if (e == hipSuccess) e = dgemm_attrs<false, ACC_ADD>();
  if (e == hipSuccess) e = dgemm_attrs<true, ACC_SYM>();
  // the split products' rings are 64 KB or less: no attribute
  return e;
}

int64_t eps_padded_size(int64_t n) { return n <= 0 ? 0 : ((n + NB - 1) / NB) * NB; }

void eps_free(EpsWorkspace* ws) {
  if (ws->buf) (void)hipFree(ws->buf);
  ws->buf = nullptr;
  ws->size = 0;
}

void eps_release(EpsWorkspace* ws) {
  eps_free(ws);
  for (auto& e : ws->ev) {
    if (e) (void)hipEventDestroy(e);
    e = nullptr;
  }
  if (ws->side) (void)hipStreamDestroy(ws->side);
  if (ws->work) (void)hipStreamDestroy(ws->work);
  ws->side = ws->work = nullptr;
}

static hipError_t ensure(EpsWorkspace* ws, size_t budget_left, size_t need, const char* what, std::string* err) {
  if (need <= ws->size) return hipSuccess;
  if (budget_left && need > budget_left) {
    *err = std::string(what) + " workspace of " + std::to_string(need) + " bytes exceeds the budget";
    return hipErrorOutOfMemory;
  }
  eps_free(ws);
  hipError_t e = hipMalloc(&ws->buf, need);
  if (e != hipSuccess && ws->spare) {
    (void)hipGetLastError();
    ws->spare();
    e = hipMalloc(&ws->buf, need);
  }
  if (e != hipSuccess) {
    (void)hipGetLastError();
    ws->buf = nullptr;
    *err = "hipMalloc of " + std::to_string(need) + " bytes for the " + what + " failed";
    return hipErrorOutOfMemory;
  }
  ws->size = need;
  return hipSuccess;
}

#define EPS_CK(x, what)            \
  do {                             \
    hipError_t e_ = (x);           \
    if (e_ != hipSuccess) {        \
      *err = what;                 \
      return e_;                   \
    }                              \
  } while (0)

// One elimination step on pivot rows and columns p = K0 .. K0 + P - 1 of W
// (Ns rows, row stride ldw), given Q = W[p, p]^-1 (row stride ldq): two
// launches, Y (P rows, row stride ldw) and then the update.
//  - inplace: the system becomes its inverse (columns 0 .. Ns - 1):
//      Y = Q W[p, .] with Y[., p] = Q;  W[q, .] -= W[q, p] Y for q outside p,
//      with W[q, p] taken as 0 in the difference;  W[p, .] = Y.
//    Cb (Ns x P) holds W[., p] meanwhile, which other workgroups overwrite.
//  - otherwise only the columns T right of the panel change (right-hand
//    sides stand there; the columns left of T would hold the identity).
static GemmArgs gj_panel(double* W, int64_t Ns, int64_t ldw, int64_t K0, int P, const double* Q, int64_t ldq,
                           bool inplace, double* Y, double* Cb) {
  const int64_t c0 = inplace ? 0 : K0 + P;
  const int64_t cols = inplace ? Ns : ldw - c0;
  GemmArgs y{Q, ldq, W + K0 * ldw + c0, ldw, nullptr, 0, Y + c0, ldw, P, (int)cols, P, 0};
  if (inplace) {
    y.np = P;
    y.pcol = (int)K0;
    y.pmode = 2;
    y.cs = W + K0;
    y.csld = ldw;
    y.cd = Cb;
    y.cdld = P;
    y.copy_rows = (int)Ns;
    y.copy_cols = P;
  }
  return y;
}

static GemmArgs gj_update(double* W, int64_t Ns, int64_t ldw, int64_t K0, int P, bool inplace, const double* Y,
                          const double* Cb) {
  const int64_t c0 = inplace ? 0 : K0 + P;
  GemmArgs u{inplace ? Cb : W + K0, inplace ? (int64_t)P : ldw, Y + c0, ldw, W + c0, ldw, W + c0, ldw,
             (int)Ns, (int)(inplace ? Ns : ldw - c0), P, 1};
  u.np = P;
  u.prow = (int)K0;
  if (inplace) {
    u.pcol = (int)K0;
    u.pmode = 1;
  }
  return u;
}

// In-place inverse of the n x n matrix V (row stride ldv, n a multiple of
// NB), pivot blocks of NB: three launches a block.  scratch: NB x NB, then
// Y (NB x ldv) and the saved column block (n x NB).
// beside: the inverse runs on another stream beside a trailing update, whose
// workgroups fill the chip and take every slot that comes free (a 128-block
// inverse waited up to 1.1 ms for a compute unit, 240 us on average): all its
// launches then are of a size that fits beside two update workgroups, pivot
// blocks of 64 and products of 32 x 64 tiles with a 24 KB ring.
// N = 8192 21.7 -> 19.5 ms.
static size_t gj_blocks_scratch(int64_t n, int64_t ldv) { return (size_t)NB * NB + (size_t)NB * ldv + (size_t)n * NB; }
static hipError_t gj_blocks(double* V, int64_t n, int64_t ldv, double* scratch, bool beside, hipStream_t s,
                            std::string* err) {
  const int nb = beside ? 64 : NB;
  double* Dinv = scratch;
  double* Y = Dinv + (size_t)NB * NB;
  double* Cb = Y + (size_t)NB * ldv;
  for (int64_t K0 = 0; K0 < n; K0 += nb) {
    const double* blk = V + K0 * ldv + K0;
    const bool whole = n == nb;
    if (beside)
      hipLaunchKernelGGL(k_block_inverse<4>, dim3(1), dim3(256), 0, s, blk, ldv, Dinv, (int64_t)nb);
    else
      hipLaunchKernelGGL(k_block_inverse<8>, dim3(1), dim3(576), 0, s, blk, ldv, whole ? V : Dinv,
                         whole ? ldv : (int64_t)nb);
    EPS_CK(hipGetLastError(), "block inverse");
    if (whole) break;
    const GemmArgs y = gj_panel(V, n, ldv, K0, nb, Dinv, nb, true, Y, Cb), u = gj_update(V, n, ldv, K0, nb, true, Y, Cb);
    EPS_CK((beside ? dgemm_launch<32, 64, 2, false, ACC_NONE>(y, s) : dgemm(y, s)), "row panel product");
    EPS_CK((beside ? dgemm_launch<32, 64, 2, false, ACC_NONE>(u, s) : dgemm(u, s)), "elimination update");
  }
  return hipSuccess;
}

// V = W[r0 : r0 + P, r0 : r0 + P]  (P x P)
__global__ void __launch_bounds__(256)
k_panel_copy(const double* W, int64_t ldw, int64_t r0, int P, double* V) {
  const int i = blockIdx.y;
  for (int j = blockIdx.x * 256 + threadIdx.x; j < P; j += gridDim.x * 256)
    V[(int64_t)i * P + j] = W[(r0 + i) * ldw + r0 + j];
}

// Block Gauss-Jordan elimination of the Ns x Ns system held in the left part
// of W (Ns rows, row stride ldw; Ns a multiple of NB), in pivot panels of
// kPanel rows and columns.  inplace: W becomes the inverse, 2 Ns^3
// operations; otherwise columns Ns .. ldw of W (right-hand sides) end up
// holding the solution.  Each panel's trailing update reads and writes the
// matrix once with K = kPanel.  Look-ahead: once Y is known, the next pivot
// block alone is updated into a buffer of its own and inverted there
// (gj_blocks) on the side stream while the full update runs.
// Systems of at most kDirectMax rows are inverted in pivot blocks of NB
// directly: their updates are too short to hide a panel's inverse behind.
constexpr int kPanel = 4 * NB;
constexpr int64_t kDirectMax = 2048;

// The elimination's two streams (default priority): the work stream takes
// the updates, the side stream the look-ahead panel inverse.
static hipError_t ensure_streams(EpsWorkspace* ws, std::string* err) {
  if (ws->side) return hipSuccess;
  EPS_CK(hipStreamCreateWithFlags(&ws->side, hipStreamNonBlocking), "side stream");
  EPS_CK(hipStreamCreateWithFlags(&ws->work, hipStreamNonBlocking), "work stream");
  for (auto& e : ws->ev) EPS_CK(hipEventCreateWithFlags(&e, hipEventDisableTiming), "event");
  return hipSuccess;
}

// Scratch doubles gj_eliminate needs beyond W.
static size_t gj_scratch_doubles(int64_t ldw) {
  return (size_t)4 * kPanel * kPanel + (size_t)NB * NB + (size_t)kPanel * ldw;
}
static size_t gj_inplace_scratch_doubles(int64_t Ns) {
  return Ns <= kDirectMax ? gj_blocks_scratch(Ns, Ns)
                          : (size_t)2 * kPanel * kPanel + gj_blocks_scratch(kPanel, kPanel) + (size_t)2 * kPanel * Ns;
}

static hipError_t gj_eliminate(EpsWorkspace* ws, double* W, int64_t Ns, int64_t ldw, bool inplace, double* scratch,
                               hipStream_t s, bool timing, std::vector<std::pair<hipEvent_t, hipEvent_t>>* evs,
                               std::string* err) {
  if (inplace && Ns <= kDirectMax) return gj_blocks(W, Ns, ldw, scratch, false, s, err);
  // the caller's stream s hands over to the work stream and takes it back
  EPS_CK(ensure_streams(ws, err), *err);
  EPS_CK(hipEventRecord(ws->ev[2], s), "event");
  EPS_CK(hipStreamWaitEvent(ws->work, ws->ev[2], 0), "wait");
  const hipStream_t caller = s;
  s = ws->work;
  auto timed = [&](const GemmArgs& g) -> hipError_t {
    hipEvent_t ea = nullptr, eb = nullptr;
    if (timing && hipEventCreate(&ea) == hipSuccess && hipEventCreate(&eb) == hipSuccess) (void)hipEventRecord(ea, s);
    hipError_t e = dgemm(g, s);
    if (ea && eb) {
      (void)hipEventRecord(eb, s);
      evs->push_back({ea, eb});
    }
    return e;
  };
  // scratch: V[2] (kPanel x kPanel each), the panel inverse's, Y (kPanel x ldw), Cb (Ns x kPanel, in place only)
  double* V[2] = {scratch, scratch + (size_t)kPanel * kPanel};
  double* inner = V[1] + (size_t)kPanel * kPanel;
  double* Y = inner + gj_blocks_scratch(kPanel, kPanel);
  double* Cb = Y + (size_t)kPanel * ldw;
  int P = (int)std::min<int64_t>(kPanel, Ns);
  hipLaunchKernelGGL(k_panel_copy, dim3((unsigned)((P + 255) / 256), (unsigned)P), dim3(256), 0, s, (const double*)W,
                     ldw, (int64_t)0, P, V[0]);
  EPS_CK(hipGetLastError(), "panel copy");
  EPS_CK(gj_blocks(V[0], P, P, inner, false, s, err), *err);
  int t = 0;
  for (int64_t K0 = 0; K0 < Ns; K0 += P, ++t) {
    P = (int)std::min<int64_t>(kPanel, Ns - K0);
    const int64_t T0 = K0 + P;
    EPS_CK(dgemm(gj_panel(W, Ns, ldw, K0, P, V[t & 1], P, inplace, Y, Cb), s), "panel row product");
    const bool ahead = T0 < Ns;
    if (ahead) {
      // the next pivot block, W[p', p'] - W[p', p] Y[., p'], and its inverse
      const int Pn = (int)std::min<int64_t>(kPanel, Ns - T0);
      double* Vn = V[(t + 1) & 1];
      GemmArgs nd{W + T0 * ldw + K0, ldw, Y + T0, ldw, W + T0 * ldw + T0, ldw, Vn, Pn, Pn, Pn, P, 1};
      EPS_CK(dgemm(nd, s), "next pivot block");
      EPS_CK(hipEventRecord(ws->ev[0], s), "event");
      EPS_CK(hipStreamWaitEvent(ws->side, ws->ev[0], 0), "wait");
      EPS_CK(gj_blocks(Vn, Pn, Pn, inner, true, ws->side, err), *err);
      EPS_CK(hipEventRecord(ws->ev[1], ws->side), "event");
    }
    EPS_CK(timed(gj_update(W, Ns, ldw, K0, P, inplace, Y, Cb)), "elimination update");
    if (ahead) EPS_CK(hipStreamWaitEvent(s, ws->ev[1], 0), "wait");
  }
  EPS_CK(hipEventRecord(ws->ev[3], s), "event");
  EPS_CK(hipStreamWaitEvent(caller, ws->ev[3], 0), "wait");
  return hipSuccess;
}

hipError_t eps_solve(EpsWorkspace* ws, size_t budget_left, int64_t n, const uint8_t* B, int64_t ldb,
                     const uint8_t* C, int64_t ldc, double eps, uint8_t* R, int64_t ldr, double* X_out,
                     int64_t ldx, hipStream_t s, bool timing, double* trailing_ms, int64_t* trailing_launches,
                     double* min_positive, std::string* err) {
  *trailing_ms = 0.0;
  *trailing_launches = 0;
  const int64_t Np = eps_padded_size(n);
  // the closure form (C = B) needs the inverse alone, in place in W: X is
  // (I - eps B)^-1 - I.  The workspace is the general form's either way.
  const bool closure = C == B && ldc == ldb;
  const int64_t ldw = closure ? Np : 2 * Np;
  const size_t wbytes = (size_t)Np * 2 * Np * sizeof(double);
  const size_t dbytes = gj_scratch_doubles(2 * Np) * sizeof(double);
  EPS_CK(ensure(ws, budget_left, wbytes + dbytes + 256, "epsilon-solve", err), *err);
  double* W = (double*)ws->buf;
  double* scratch = W + (size_t)Np * ldw;
  const int nchunk = (int)((n + kDiagChunk - 1) / kDiagChunk);
  double* part = scratch + gj_inplace_scratch_doubles(Np);  // closure: nchunk x Np diagonal sums
  unsigned long long* minpos = (unsigned long long*)((char*)ws->buf + wbytes + dbytes);
  hipLaunchKernelGGL(k_set_word, dim3(1), dim3(1), 0, s, minpos, ~0ull);
  EPS_CK(hipGetLastError(), "epsilon init");

  hipLaunchKernelGGL(k_eps_init, dim3((unsigned)((Np + 1023) / 1024), (unsigned)Np), dim3(256), 0, s, B, ldb,
                     closure ? (const uint8_t*)nullptr : C, ldc, (int)n, (int)Np, eps, W);
  EPS_CK(hipGetLastError(), "epsilon init");
  std::vector<std::pair<hipEvent_t, hipEvent_t>> evs;
  hipError_t e = gj_eliminate(ws, W, Np, ldw, closure, scratch, s, timing, &evs, err);
  if (e == hipSuccess && closure) {
    hipLaunchKernelGGL(k_eps_diag, dim3((unsigned)((n + 63) / 64), (unsigned)nchunk), dim3(256), 0, s, B, ldb,
                       (const double*)W, (int)n, (int)Np, part);
    e = hipGetLastError();
    if (e != hipSuccess) *err = "diagonal";
  }
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_eps_emit, dim3((unsigned)std::min<int64_t>((n + 3) / 4, kEmitBlocks)), dim3(1024), 0, s,
                       (const double*)(closure ? W : W + Np), ldw, (int)n, R, ldr, X_out, ldx, minpos,
                       (const double*)(closure ? part : nullptr), (int)Np, nchunk, B, ldb, eps);
    e = hipGetLastError();
    if (e != hipSuccess) *err = "threshold";
  }
  unsigned long long mp = ~0ull;
  if (e == hipSuccess) {
    e = hipMemcpyAsync(&mp, minpos, sizeof mp, hipMemcpyDeviceToHost, s);
    if (e != hipSuccess) *err = "smallest positive entry read-back";
  }
  if (e == hipSuccess) {
    e = hipStreamSynchronize(s);
    if (e != hipSuccess) *err = "epsilon solve sync";
  }
  if (min_positive) {
    double v = INFINITY;
    if (mp != ~0ull) memcpy(&v, &mp, sizeof v);
    *min_positive = v;
  }
  for (auto& p : evs) {
    float t = 0.f;
    if (e == hipSuccess && hipEventElapsedTime(&t, p.first, p.second) == hipSuccess) {
      *trailing_ms += t;
      *trailing_launches += 1;
    }
    (void)hipEventDestroy(p.first);
    (void)hipEventDestroy(p.second);
  }
  return e;
}

// ----------------------------------------------------------------- stacked tail-recursive system
// W = [ I - E BB | E AA ] for the heads h = 0 .. M-1 of one layer (Ns = M Np
// rows, ldw = Ns + Np): block (h, j) of BB is the int8 0/1 matrix B[h][j]
// (null = zero), block h of AA is A[h], E = diag(eps_h) row-block-wise.
__global__ void __launch_bounds__(256) k_stack_init(StackDesc d, int64_t Ns, int64_t ldw, double* W) {
  const int64_t i = blockIdx.y;
  const int h = (int)(i / d.Np), ii = (int)(i % d.Np);
  const double eps = d.eps[h];
  for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < ldw; j += (int64_t)gridDim.x * 256) {
    double v;
    if (j < Ns) {
      const int jb = (int)(j / d.Np), jj = (int)(j % d.Np);
      const int8_t* b = d.B[h][jb];
      const double bij = (b && b[(int64_t)ii * d.Np + jj] != 0) ? 1.0 : 0.0;
      v = (i == j ? 1.0 : 0.0) - eps * bij;
    } else {
      const int8_t* a = d.A[h];
      const int jj = (int)(j - Ns);
      v = (a && a[(int64_t)ii * d.Np + jj] != 0) ? eps : 0.0;
    }
    W[i * ldw + j] = v;
  }
}

// R[h] = [X_h > 0] as int8 0/1 (Np x Np), counting the ones of each head.
__global__ void __launch_bounds__(256) k_stack_emit(StackDesc d, int64_t Ns, int64_t ldw, const double* W) {
  const int64_t i = blockIdx.y;
  const int h = (int)(i / d.Np), ii = (int)(i % d.Np);
  int c = 0;
  for (int j = blockIdx.x * 256 + threadIdx.x; j < d.Np; j += gridDim.x * 256) {
    const int8_t v = W[i * ldw + Ns + j] > 0.0 ? 1 : 0;
    d.R[h][(int64_t)ii * (d.ldr ? d.ldr : d.Np) + j] = v;
    c += v;
  }
  if (!d.cnt) return;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
  __shared__ int red[4];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    const int t = red[0] + red[1] + red[2] + red[3];
    if (t) atomicAdd(d.cnt + h, (unsigned long long)t);
  }
}

hipError_t stacked_solve(EpsWorkspace* ws, size_t budget_left, const StackDesc& d, hipStream_t s, std::string* err) {
  if (d.M < 1 || d.M > kMaxStack || d.Np % NB) {
    *err = "bad stacked system";
    return hipErrorInvalidValue;
  }
  const int64_t Ns = (int64_t)d.M * d.Np;
  const int64_t ldw = Ns + d.Np;
  const size_t wbytes = (size_t)Ns * ldw * sizeof(double);
  const size_t dbytes = gj_scratch_doubles(ldw) * sizeof(double);
  EPS_CK(ensure(ws, budget_left, wbytes + dbytes, "stacked linear solve", err), *err);
  double* W = (double*)ws->buf;
  double* scratch = W + (size_t)Ns * ldw;
  hipLaunchKernelGGL(k_stack_init, dim3((unsigned)((ldw + 255) / 256), (unsigned)Ns), dim3(256), 0, s, d, Ns, ldw, W);
  EPS_CK(hipGetLastError(), "stacked init");
  std::vector<std::pair<hipEvent_t, hipEvent_t>> evs;
  EPS_CK(gj_eliminate(ws, W, Ns, ldw, false, scratch, s, false, &evs, err), *err);
  hipLaunchKernelGGL(k_stack_emit, dim3((unsigned)((d.Np + 255) / 256), (unsigned)Ns), dim3(256), 0, s, d, Ns, ldw,
                     (const double*)W);
  EPS_CK(hipGetLastError(), "stacked threshold");
  return hipSuccess;
}

// ----------------------------------------------------------------- two-sided (Stein) equations
// X = Q + B X C with B, C, Q >= 0 and a convergent series, solved by Smith's
// doubling in fp64:
//   X_0 = Q,  B_0 = B,  C_0 = C,
//   X_{j+1} = X_j + B_j X_j C_j,  B_{j+1} = B_j B_j,  C_{j+1} = C_j C_j,
// so X_j = sum_{m < 2^j} B^m Q C^m.  Every term is >= 0, so the zero pattern
// of X_j is exact: it is the 2^j-th iterate of the Boolean series
// Y' = [Q + B Y C] from Y = 0.  When a doubling leaves the number of positive
// entries unchanged, that series has repeated (it is monotone), so the
// pattern is the least model.  When the real solution is wanted as well,
// doublings go on until one also leaves every fp64 value unchanged (the
// increments shrink doubly exponentially, so the truncated series is then
// within rounding of the limit).  A Schur-based Sylvester solver would
// cancel terms and lose the exact zero pattern.  For the same-generation
// form C = B^T, which is kept as the transpose of B instead of a product.
__global__ void __launch_bounds__(256)
k_f64_from_bytes(const uint8_t* src, int64_t ld, int n, int Np, double scale, int identity, double* dst) {
  const int i = blockIdx.y;
  for (int j = 4 * (blockIdx.x * 256 + threadIdx.x); j < Np; j += 1024 * gridDim.x) {
    unsigned b = 0u;
    if (i < n) b = identity ? (i >= j && i < j + 4 ? 1u << (8 * (i - j)) : 0u) : bytes4(src + (int64_t)i * ld, j, n);
    v2d w[2];
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e >> 1][e & 1] = ((b >> (8 * e)) & 1u) ? scale : 0.0;
    *(v2d*)(dst + (int64_t)i * Np + j) = w[0];
    *(v2d*)(dst + (int64_t)i * Np + j + 2) = w[1];
  }
}

// Adds the positive entries of X (count entries, an even number) to *out: a
// fixed grid, one atomic per workgroup (2048 workgroups spent 18 us on them
// at Np = 1024).
constexpr int kElemGrid = 256;
__global__ void __launch_bounds__(256) k_count_positive(const double* X, int64_t count, unsigned long long* out) {
  __shared__ int red[4];
  int c = 0;
  const double2* X2 = (const double2*)X;
  for (int64_t q = blockIdx.x * 256 + threadIdx.x; q < count / 2; q += (int64_t)gridDim.x * 256) {
    const double2 x = X2[q];
    c += (x.x > 0.0) + (x.y > 0.0);
  }
  for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    const int t = red[0] + red[1] + red[2] + red[3];
    if (t) atomicAdd(out, (unsigned long long)t);
  }
}

// The words of a doubling loop: its counts, counts[0] starting at `first`, and
// behind those of kSteinDoublings doublings the states of the split products'
// tiles; all zeroed.
constexpr int kSteinDoublings = 127;
constexpr int kSteinState = 2 * (kSteinDoublings + 1);
constexpr int kSteinWords = kSteinState + kSplitSlots / 2;
static_assert(kSteinWords <= kRing, "the ring of a slot");
__global__ void __launch_bounds__(256) k_stein_clear(unsigned long long* cnt, int words, unsigned long long first) {
  for (int i = threadIdx.x; i < words; i += 256) cnt[i] = i == 0 ? first : 0ull;
}

__global__ void __launch_bounds__(256)
k_f64_emit(const double* X, int Np, int n, uint8_t* S, int64_t lds, double* Xo, int64_t ldx) {
  const int i = blockIdx.y;
  for (int j = 4 * (blockIdx.x * 256 + threadIdx.x); j < n; j += 1024 * gridDim.x) {
    const v2d a = *(const v2d*)(X + (int64_t)i * Np + j), b = *(const v2d*)(X + (int64_t)i * Np + j + 2);
    const double x[4] = {a.x, a.y, b.x, b.y};
    if (j + 4 <= n) {
      unsigned r = 0u;
#pragma unroll
      for (int e = 0; e < 4; ++e) r |= (x[e] > 0.0 ? 1u : 0u) << (8 * e);
      *(u32_any*)(S + (int64_t)i * lds + j) = r;
      if (Xo) {
        *(v2d_8*)(Xo + (int64_t)i * ldx + j) = a;
        *(v2d_8*)(Xo + (int64_t)i * ldx + j + 2) = b;
      }
    } else {
      for (int e = 0; e < 4 && j + e < n; ++e) {
        S[(int64_t)i * lds + j + e] = x[e] > 0.0 ? 1 : 0;
        if (Xo) Xo[(int64_t)i * ldx + j + e] = x[e];
      }
    }
  }
}

// Doubling loop on buffers already initialised: X = X_0 and the factors B and
// C (C = null: C = B^T, and X symmetric); with t_ready T = B X_0 as well.  T,
// Bn and Cn (unless C is null) are scratch.  counts: 2 (max_doublings + 1)
// device words, [0] = the positive entries of X_0, the others zero.
// Per doubling: the factors' squares (the first doubling needs none), T = B X
// and X += T C with its counts in the product's epilogue.  For C = B^T the
// increment is symmetric: its upper triangle is computed and B is its own
// right operand, read transposed.  Doublings are enqueued in groups, each
// launch checking the counts before it, and the host reads the counts once
// per group: a doubling after the last one costs its empty launches only.
// Against each product its own full launch, the squares before the check, a
// read-back per doubling and separate passes for the transpose and the sum:
// same generation, n = 2500, five doublings 9.4 -> 6.7 ms (5.9 with split products); two-sided, n =
// 1024, six doublings 1.65 -> 1.07 ms.
static hipError_t stein_doubling(int64_t Np, double* X, double* B, double* C, double* T, double* Bn, double* Cn,
                                 bool t_ready, bool want_values, int max_doublings, hipStream_t s,
                                 unsigned long long* counts, unsigned long long* h_counts,
                                 unsigned long long* h_counts_dev, int64_t* positives, int32_t* doublings,
                                 bool* done_out, std::string* err) {
  const int N = (int)Np;
  int issued = 0, last = 0;
  bool done = false;
  while (!done && issued < max_doublings) {
    const int group = std::min(issued == 0 ? 4 : 2, max_doublings - issued);
    for (int q = 0; q < group; ++q) {
      const int j = ++issued;
      // partial tiles of the split products: the square's fit in T, which holds
      // nothing then, the others' in Bn
      unsigned* state = max_doublings <= kSteinDoublings ? (unsigned*)(counts + kSteinState) : nullptr;
      SteinStop stop;
      stop.cnt = counts;
      stop.j = j;
      stop.values = want_values ? 1 : 0;
      if (j > 1) {
        GemmArgs sq{B, Np, B, Np, nullptr, 0, Bn, Np, N, N, N, 0};
        sq.stop = stop;
        sq.part = state ? T : nullptr;
        sq.state = state;
        if (C) {
          sq.A2 = C;
          sq.B2 = C;
          sq.D2 = Cn;
        }
        EPS_CK(dgemm(sq, s), "factor squares");
        std::swap(B, Bn);
        if (C) std::swap(C, Cn);
      }
      if (j > 1 || !t_ready) {
        GemmArgs tx{B, Np, X, Np, nullptr, 0, T, Np, N, N, N, 0};
        tx.stop = stop;
        tx.part = state ? Bn : nullptr;
        tx.state = state;
        EPS_CK(dgemm(tx, s), "B X");
      }
      GemmArgs ac{T, Np, C ? C : B, Np, nullptr, 0, X, Np, N, N, N, 0};
      ac.stop = stop;
      ac.part = state ? Bn : nullptr;
      ac.state = state;
      EPS_CK((C ? dgemm<false, ACC_ADD>(ac, s) : dgemm<true, ACC_SYM>(ac, s)), "T C");
    }
    EPS_CK(launch_publish(counts, h_counts_dev, 2 * (issued + 1), s), "readback");
    EPS_CK(hipStreamSynchronize(s), "sync");
    while (!done && last < issued) {
      ++last;
      done = h_counts[2 * last] == h_counts[2 * (last - 1)] && (!want_values || h_counts[2 * last + 1] == 0ull);
    }
  }
  *positives = (int64_t)h_counts[2 * last];
  *doublings = last;
  *done_out = done;
  return hipSuccess;
}

hipError_t sg_eps_solve(EpsWorkspace* ws, size_t budget_left, int64_t n, const uint8_t* P, int64_t ldp, double eps,
                        uint8_t* S, int64_t lds, double* X_out, int64_t ldx, int max_doublings, hipStream_t s,
                        int32_t* doublings, int64_t* positives, unsigned long long* counts,
                        unsigned long long* h_counts, unsigned long long* h_counts_dev, std::string* err) {
  const int64_t Np = eps_padded_size(n);
  const size_t mat = (size_t)Np * Np;
  EPS_CK(ensure(ws, budget_left, 5 * mat * sizeof(double), "same-generation epsilon solve", err), *err);
  double* X = (double*)ws->buf;
  double* A = X + mat;
  double* T = A + mat;
  double* An = T + mat;
  const dim3 rows((unsigned)((Np + 1023) / 1024), (unsigned)Np);
  // X_0 = eps I, A_0 = sqrt(eps) P, T = A_0 X_0 (one product per entry)
  const double se = sqrt(eps);
  hipLaunchKernelGGL(k_f64_from_bytes, rows, dim3(256), 0, s, (const uint8_t*)nullptr, (int64_t)0, (int)n, (int)Np,
                     eps, 1, X);
  hipLaunchKernelGGL(k_f64_from_bytes, rows, dim3(256), 0, s, P, ldp, (int)n, (int)Np, se, 0, A);
  hipLaunchKernelGGL(k_f64_from_bytes, rows, dim3(256), 0, s, P, ldp, (int)n, (int)Np, se * eps, 0, T);
  hipLaunchKernelGGL(k_stein_clear, dim3(1), dim3(256), 0, s, counts, std::max(2 * (max_doublings + 1), kSteinWords),
                     (unsigned long long)n);
  EPS_CK(hipGetLastError(), "init");
  bool done = false;
  EPS_CK(stein_doubling(Np, X, A, nullptr, T, An, nullptr, true, X_out != nullptr, max_doublings, s, counts, h_counts,
                        h_counts_dev, positives, doublings, &done, err),
         *err);
  hipLaunchKernelGGL(k_f64_emit, dim3((unsigned)((n + 1023) / 1024), (unsigned)n), dim3(256), 0, s, (const double*)X,
                     (int)Np, (int)n, S, lds, X_out, ldx);
  EPS_CK(hipGetLastError(), "threshold");
  EPS_CK(hipStreamSynchronize(s), "sync");
  return done ? hipSuccess : hipErrorNotReady;
}

hipError_t two_sided_solve(EpsWorkspace* ws, size_t budget_left, int64_t n, const uint8_t* Q, int64_t ldq,
                           const uint8_t* B, int64_t ldb, const uint8_t* C, int64_t ldc, double eps, uint8_t* R,
                           int64_t ldr, double* X_out, int64_t ldx, int8_t* R8, int64_t ld8,
                           unsigned long long* r8_count, int max_doublings, hipStream_t s, int32_t* doublings, unsigned long long* counts,
                           unsigned long long* h_counts, unsigned long long* h_counts_dev, std::string* err) {
  const int64_t Np = eps_padded_size(n);
  const size_t mat = (size_t)Np * Np;
  EPS_CK(ensure(ws, budget_left, 6 * mat * sizeof(double), "two-sided solve", err), *err);
  double* X = (double*)ws->buf;
  double* Bd = X + mat;
  double* Cd = Bd + mat;
  double* T = Cd + mat;
  double* Bn = T + mat;
  double* Cn = Bn + mat;
  const dim3 rows((unsigned)((Np + 1023) / 1024), (unsigned)Np);
  // X = eps (Q + B X C): X_0 = eps Q, B_0 = sqrt(eps) B, C_0 = sqrt(eps) C
  const double se = sqrt(eps);
  hipLaunchKernelGGL(k_f64_from_bytes, rows, dim3(256), 0, s, Q, ldq, (int)n, (int)Np, eps, 0, X);
  hipLaunchKernelGGL(k_f64_from_bytes, rows, dim3(256), 0, s, B, ldb, (int)n, (int)Np, se, 0, Bd);
  hipLaunchKernelGGL(k_f64_from_bytes, rows, dim3(256), 0, s, C, ldc, (int)n, (int)Np, se, 0, Cd);
  hipLaunchKernelGGL(k_stein_clear, dim3(1), dim3(256), 0, s, counts, std::max(2 * (max_doublings + 1), kSteinWords), 0ull);
  hipLaunchKernelGGL(k_count_positive, dim3(kElemGrid), dim3(256), 0, s, (const double*)X, (int64_t)mat, counts);
  EPS_CK(hipGetLastError(), "init");
  bool done = false;
  int64_t pos = 0;
  EPS_CK(stein_doubling(Np, X, Bd, Cd, T, Bn, Cn, false, X_out != nullptr, max_doublings, s, counts, h_counts,
                        h_counts_dev, &pos, doublings, &done, err),
         *err);
  if (R) {
    hipLaunchKernelGGL(k_f64_emit, dim3((unsigned)((n + 1023) / 1024), (unsigned)n), dim3(256), 0, s, (const double*)X,
                       (int)Np, (int)n, R, ldr, X_out, ldx);
    EPS_CK(hipGetLastError(), "threshold");
  }
  if (R8) {
    StackDesc d{};
    d.M = 1;
    d.Np = (int)Np;
    d.R[0] = R8;
    d.ldr = ld8;
    d.cnt = r8_count;
    hipLaunchKernelGGL(k_stack_emit, dim3((unsigned)((Np + 255) / 256), (unsigned)Np), dim3(256), 0, s, d,
                       (int64_t)0, (int64_t)Np, (const double*)X);
    EPS_CK(hipGetLastError(), "threshold");
  }
  EPS_CK(hipStreamSynchronize(s), "sync");
  return done ? hipSuccess : hipErrorNotReady;
}

#undef EPS_CK

}  // namespace dl
