// list_kernels.hip -- the same-generation series for a relation with few
// entries a row: products with P as gathers over lists, on bits, the whole
// series in one launch.
//
// S' = [I + P S P^T] (Sec. 7.2) multiplies by P twice a step, and P -- parents,
// typically one or two of them -- never changes.  As dense products a step at
// n = 4096 takes 90 us of matrix-core work whatever P holds.  With the columns
// of the nonzero entries of each row of P as a list, (M P^T)[i][j] is the OR
// of M[i][q] over the list of j, and with 32 rows of M in the bits of a word,
// one word per column, a list of c entries costs c LDS reads for 32 entries
// of the result, and a step moves n^2 / 8 bytes instead of reading and writing
// n^2 four times.
//
// Layout ("slices"): word j of slice b of a matrix holds rows 32 b ..
// 32 b + 31 of column j, bit r = row 32 b + r; pitch = 32 nb words, nb =
// ceil(n / 32).  Rows and columns from n on are zero.
//
// k_sg_lists: workgroup b keeps slice b of S in LDS for the whole series.  A
// step gathers V = S P^T and stores it transposed, in 32 x 32 blocks, to the
// slices of V^T = P S (S is symmetric) that other workgroups
// read; when all have arrived it fetches its slice, gathers V^T P^T = P S P^T
// -- symmetric again -- and adds I.  An arrival carries the ones of the slice
// of S^(t-1), so every workgroup learns the model size of step t - 1 while it
// waits for step t's exchange, and all stop together at the first repeat; the
// exchange of step t is then left unused.  V^T is double buffered: a slice of
// step t + 2 is stored by workgroups that have seen all the others arrive at
// t + 1, and so done with step t's.
//
// All workgroups have to run together: see kResidentTicks.  Coherence across
// XCDs as in k_fix_bits: device-scope stores, loads and atomics.
//
// A step takes 5 us at n = 4096, bound by the round trips of the exchange (10
// us with the blocks transposed by a ballot a row).  Measured, same generation
// of random forests, by products and now: n = 1024 277, 68 us a call; n = 4096
// 1212, 105; n = 8192 10560, 220.
#include "common.h"
#include "device.h"

namespace dl {

typedef unsigned long long u64;

// Lists of the rows of P: entry k of row j at idx[k n + j], len[j] entries,
// kListMax + 1 for a row with more.  A wave a row.  Where one of the first
// rows is too long the host hears of it at once, and queues the products while
// their first operands are written; of any other row it hears from the next
// launch.  (One word that all rows report to took 140 us of stores to one address.)  With ring, the
// words of the product series start over as well (see DenseStart).
__global__ void __launch_bounds__(256) k_row_lists(const uint8_t* P, int64_t ldp, int n, unsigned short* idx,
                                                   unsigned short* len, unsigned* status_out,
                                                   unsigned long long* ring, int* conv) {
  if (ring) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    for (int q = t; q < kRing; q += gridDim.x * 256) ring[q] = 0ull;
    if (t == 0) *conv = kNotConverged;
  }
  const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n) return;
  const uint8_t* src = P + (int64_t)row * ldp;
  int base = 0;
  for (int c0 = 0; c0 < n; c0 += 4096) {
    unsigned m[4];  // four 1024-column pieces of the row, all loads in flight together
    int own = 0;
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      const int j0 = c0 + 1024 * h + 16 * lane;
      m[h] = 0u;
      if (j0 + 16 <= n) {
        m[h] = bit16_of_bytes(bytes01(load16_any(src + j0)));
      } else {
        for (int e = 0; j0 + e < n; ++e) m[h] |= (src[j0 + e] != 0 ? 1u : 0u) << e;
      }
      own += __popc(m[h]);
    }
    if (__ballot((int)(own != 0)) == 0ull) continue;
    int upto = own;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int v = __shfl_up(upto, off, 64);
      if (lane >= off) upto += v;
    }
    const int total = __shfl(upto, 63, 64);
    if (base + total > kListMax) {
      base = kListMax + 1;
      if (row < 8 && lane == 0) st_system(status_out, 0u);
      break;
    }
    int k = base + upto - own;  // any order within the list
#pragma unroll
    for (int h = 0; h < 4; ++h)
      for (unsigned rest = m[h]; rest != 0u; rest &= rest - 1, ++k)
        idx[(int64_t)k * n + row] = (unsigned short)(c0 + 1024 * h + 16 * lane + __ffs((int)rest) - 1);
    base += total;
  }
  if (lane == 0) len[row] = (unsigned short)base;
}

// The 32 x 32 bit matrix of lanes 0 .. 31 (row = lane, column = bit), and that
// of lanes 32 .. 63, transposed: five exchanges with lane ^ s, each moving the
// quarter whose row and column differ in bit s (a rotation, then a select by
// mask; what the rotation carries round is outside the mask).
template <int S>
__device__ inline unsigned swap_quarters(unsigned v, int lane) {
  constexpr unsigned M = S == 16 ? 0x0000ffffu : S == 8 ? 0x00ff00ffu : S == 4 ? 0x0f0f0f0fu : S == 2 ? 0x33333333u : 0x55555555u;
  unsigned y;
  if constexpr (S == 8) y = (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, true);  // row_ror:8
  else if constexpr (S == 2) y = (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x4e, 0xf, 0xf, true);  // quad_perm 2 3 0 1
  else if constexpr (S == 1) y = (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0xb1, 0xf, 0xf, true);  // quad_perm 1 0 3 2
  else y = (unsigned)__builtin_amdgcn_ds_swizzle((int)v, 0x1f | (S << 10));
  const bool upper = (lane & S) != 0;
  const unsigned x = __builtin_amdgcn_alignbit(y, y, upper ? S : 32 - S), k = upper ? M : ~M;
  return (x & k) | (v & ~k);
}
__device__ inline unsigned transpose32(unsigned v, int lane) {
  v = swap_quarters<16>(v, lane);
  v = swap_quarters<8>(v, lane);
  v = swap_quarters<4>(v, lane);
  v = swap_quarters<2>(v, lane);
  return swap_quarters<1>(v, lane);
}

constexpr u64 kArrived = 1ull << 40;  // above any sum of ones
constexpr int kListThreads = 1024;

// Bytes c .. c + 15 of a caller's row of n as 0/1 bytes, 0 from n on.
__device__ inline u32x4 row16(const uint8_t* row, int c, int n) {
  if (c + 16 <= n) return bytes01(load16_any(row + c));
  u32x4 v = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int e = 0; e < 16; ++e)
    if (c + e < n && row[c + e] != 0) v[e >> 2] |= 1u << (8 * (e & 3));
  return v;
}

// Bit r of words c .. c + 15 as bytes: 16 elements of row r of a slice.
__device__ inline u32x4 strip_row16(const unsigned* bits, int c, int r) {
  u32x4 v;
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    const u32x4 w = *(const u32x4*)(bits + c + 4 * x);
    v[x] = ((w[0] >> r) & 1u) | ((w[1] >> r) & 1u) << 8 | ((w[2] >> r) & 1u) << 16 | ((w[3] >> r) & 1u) << 24;
  }
  return v;
}

// DenseStart of the same generation, by all workgroups of k_sg_lists: a wave a row.
__device__ inline void sg_dense_start(const ListParams& p) {
  const DenseStart& d = p.dense;
  const int wave = blockIdx.x * (kListThreads / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  for (int row = wave; row < d.Np; row += gridDim.x * (kListThreads / 64))
    for (int c = 16 * lane; c < d.Np; c += 1024) {
      u32x4 v = {0u, 0u, 0u, 0u}, e = v;
      if (row < p.n) {
        v = row16(p.P + (int64_t)row * p.ldp, c, p.n);
        if (row >= c && row < c + 16) e[(row - c) >> 2] = 1u << (8 * ((row - c) & 3));
      }
      *(u32x4*)(d.Y + (int64_t)row * d.Np + c) = v;
      *(u32x4*)(d.S1 + (int64_t)row * d.Np + c) = e;
    }
  if (blockIdx.x == 0) {
    for (int i = threadIdx.x; i < d.words; i += kListThreads) d.zero[i] = 0u;
    if (threadIdx.x == 0) d.ring[1] = (u64)p.n;
  }
}

__device__ inline u64* arrival(const ListParams& p, int t, int k) { return p.cnt + ((t & 3) * kListArrivals + k) * 16; }

__global__ void __launch_bounds__(kListThreads) k_sg_lists(ListParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned lds[];
  __shared__ int red[kListThreads / 64];
  __shared__ u64 s_total;
  __shared__ int s_go;
  unsigned* S = lds;            // slice b of S
  unsigned* VT = lds + p.pitch;  // slice b of P S
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const unsigned bytes = (unsigned)((size_t)p.nb * p.pitch * 4);
  // length and first entry of every column's list
  unsigned* head = lds + 2 * p.pitch;
  if (tid == 0) s_go = 1;
  __syncthreads();
  for (int j = tid; j < p.pitch; j += kListThreads) {
    unsigned h = 0u;
    if (j < p.n) {
      const unsigned c = p.len[j];
      if (c > (unsigned)kListMax) s_go = 0;
      h = c << 16 | (c ? p.idx[j] : 0u);
    }
    head[j] = h;
  }
  auto gather = [&](const unsigned* m, int j) {
    const unsigned h = head[j], c = h >> 16;
    unsigned v = c ? m[h & 0xffffu] : 0u;
    for (unsigned k = 1; k < c; ++k) v |= m[p.idx[(int64_t)k * p.n + j]];
    return v;
  };
  __syncthreads();
  if (s_go == 0) {  // some row is too long for a list: every workgroup sees that
    if (b == 0 && tid == 0) st_system(p.status_out, 0u);
    sg_dense_start(p);
    return;
  }
  // S^(1) = I
  int ones = 0;
  for (int j = tid; j < p.pitch; j += kListThreads) {
    const unsigned v = j >> 5 == b && j < p.n ? 1u << (j & 31) : 0u;
    S[j] = v;
    ones += v != 0u;
  }
  u64 prev = 0ull;  // size of S^(t-2)
  int t = 2, converged = 0;
  for (;; ++t) {
    ones = wave_sum(ones);
    if (lane == 0) red[wave] = ones;
    __syncthreads();  // S^(t-1) is complete
    const __amdgpu_buffer_rsrc_t X = buffer_of(p.VT[t & 1], bytes);
    for (int j0 = 64 * wave; j0 < p.pitch; j0 += kListThreads) {
      const unsigned v = j0 + lane < p.pitch ? gather(S, j0 + lane) : 0u;
      const unsigned w = transpose32(v, lane);  // row lane % 32 of the lane's 32 x 32 block
      const int tile = (j0 >> 5) + (lane >> 5);
      if (tile < p.nb)
        __builtin_amdgcn_raw_buffer_store_b32(w, X, (tile * p.pitch + 32 * b + (lane & 31)) * 4, 0, kCpolSc1);
    }
    wait_stores();
    __syncthreads();
    if (wave == 0) {
      u64 sum = lane < kListThreads / 64 ? (u64)red[lane] : 0ull;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
      if (lane == 0) atomicAdd(arrival(p, t, b % kListArrivals), kArrived + sum);
      const long long t0 = (long long)__builtin_amdgcn_s_memrealtime();
      int go = 1;
      u64 v = 0ull;
      for (;;) {
        if (lane < kListArrivals) v = ld_agent64(arrival(p, t, lane));
        int arrived = lane < kListArrivals ? (int)(v >> 40) : 0;
        arrived = wave_sum(arrived);
        if (arrived == p.nb) break;
        if (ld_agent(p.finished + 1) != 0u) {
          go = -1;
          break;
        }
        if ((long long)__builtin_amdgcn_s_memrealtime() - t0 > (t == 2 ? kResidentTicks : p.wait_limit)) {
          if (lane == 0) {
            st_agent(p.finished + 1, 1u);
            st_system(p.status_out + 1, t == 2 ? kNotResident : 1u);
          }
          go = -1;
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
      u64 total = lane < kListArrivals ? v & (kArrived - 1) : 0ull;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) total += __shfl_xor(total, off, 64);
      if (b == 0) {
        // everybody has left the words of step t - 2: they are step t + 2's
        // (complete before this workgroup arrives at t + 1)
        if (lane < kListArrivals)
          __hip_atomic_store(arrival(p, t + 2, lane), 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (lane == 0) st_system64(p.ring_out + (t - 1), total);
        wait_stores();
      }
      if (lane == 0) {
        s_total = total;
        s_go = go;
      }
    }
    __syncthreads();
    if (s_go < 0) return;
    const u64 now = s_total;
    converged = now == prev ? 1 : 0;
    if (converged || t > p.max_steps) break;
    prev = now;
    for (int q = 4 * tid; q < p.pitch; q += 4 * kListThreads)
      *(u32x4*)(VT + q) = __builtin_amdgcn_raw_buffer_load_b128(X, (b * p.pitch + q) * 4, 0, kCpolSc1);
    __syncthreads();
    ones = 0;
    for (int j = tid; j < p.pitch; j += kListThreads) {
      unsigned v = gather(VT, j);
      if (j >> 5 == b && j < p.n) v |= 1u << (j & 31);
      S[j] = v;
      ones += __popc(v);
    }
  }

  // S^(t-1) as 0/1 bytes, a wave a row, 16 columns a lane; every store of the
  // slice completes before the workgroup counts itself finished
  for (int r = wave; r < 32; r += kListThreads / 64) {
    const int row = 32 * b + r;
    if (row >= p.n) break;
    uint8_t* dst = p.R + (int64_t)row * p.ldr;
    const __amdgpu_buffer_rsrc_t D = buffer_of(dst, (unsigned)p.n);
    const bool aligned = ((uintptr_t)dst & 15) == 0;
    for (int c = 16 * lane; c < p.n; c += 1024) {
      const u32x4 v = strip_row16(S, c, r);
      if (aligned && c + 16 <= p.n) st_agent_x4(D, c, v);
      else store16_agent_any(dst + c, v, p.n - c);
    }
  }
  wait_stores();
  __syncthreads();
  if (tid == 0) s_go = atomicAdd(p.finished, 1u) == (unsigned)p.nb - 1u ? 1 : 0;
  __syncthreads();
  if (!s_go) return;
  // the last workgroup: cleared words, then the status
  if (tid < 4 * kListArrivals)
    __hip_atomic_store(p.cnt + tid * 16, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (tid == 0) st_agent(p.finished, 0u);
  wait_stores();
  __syncthreads();
  if (tid == 0) {
    st_system(p.status_out + 1, 0u);
    st_system(p.status_out, (unsigned)(t - 1));  // >= 1: the last step computed
  }
}

// The Boolean series R^(t) = A + P R^(t-1) from R^(1) = A of a program's
// layer, by P's lists: (P R)[i] is the OR of rows R[q] over the list of i, so
// 32 columns of R depend on no others.  Workgroup b runs its own series of
// columns 32 b .. 32 b + 31 in LDS, one word a row, without a word to the
// others, until a step changes nothing (k_b); the whole series has repeated
// at K = max k_b.  For R S on the right, the transposed matrices: R^T = A^T +
// S^T R^T.  At n = 4000, P with three entries a row, 17 steps take 53 us with
// the reading of A and the writing of both orientations of R; as products,
// each 50 us, 850.  A program of three layers with two such series: 2130 -> 541
// us.
// E: entries of every row's list in LDS, the row itself in place of those that
// it does not have, so that a step reads them without a test; 8 where they fit
// (90 us for 17 steps at n = 4000 with 4, since the longer lists of a wave's 64
// rows then come from memory entry by entry).
// CALLER: A and R are a caller's matrices (n x n, any stride and alignment),
// and no transpose is written.
// DenseStart of the plain closure, by all workgroups of k_layer_lists, the b-th
// of them: units of 128 columns (whole lines of A and Y) by a quarter of the
// rows, as bits through LDS, word k of a row at k (Np / 4 + 16) + row (Np + 64
// words; the pitch keeps four words of a row in different banks).  n = 8192,
// 67 MB read and 134 MB written: 78 us in strips of 32 columns.
__device__ inline void plain_dense_start(const LayerLists& p, int b, unsigned* bits) {
  const DenseStart& d = p.dense;
  __shared__ int s_ones;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int rows = d.Np / 4, pitch = rows + 16;
  if (tid == 0) s_ones = 0;
  int ones = 0;
  for (int u = b; u < d.Np / 32; u += gridDim.x) {
    const int c0 = u / 4 * 128, r0 = u % 4 * rows;
    __syncthreads();
    auto put = [&](int k, int r, u32x4 lo, u32x4 hi) {
      const int i = r0 + r, c = c0 + 32 * k;
      unsigned w = bit16_of_bytes(lo) | bit16_of_bytes(hi) << 16;
      bits[k * pitch + r] = w;
      ones += __popc(w);
      if (i < p.n && i >= c && i < c + 32) w |= 1u << (i - c);
      u32x4* y = (u32x4*)(d.Y + (int64_t)i * d.Np + c);
      y[0] = bytes_of_bit16(w & 0xffffu);
      y[1] = bytes_of_bit16(w >> 16);
    };
    const int k = tid & 3, left = p.n - r0 < rows ? p.n - r0 : rows;  // rows of the relation in this unit
    const uint8_t* a = (const uint8_t*)p.A + (int64_t)(r0 + (tid >> 2)) * p.lda + c0 + 32 * k;
    int r = tid >> 2;
    if (c0 + 128 <= p.n)
      for (; r + 3 * (kListThreads / 4) < left; r += kListThreads) {  // eight loads in flight
        u32x4 x[4][2];
#pragma unroll
        for (int e = 0; e < 4; ++e, a += (int64_t)(kListThreads / 4) * p.lda) {
          x[e][0] = load16_any(a);
          x[e][1] = load16_any(a + 16);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) put(k, r + e * (kListThreads / 4), x[e][0], x[e][1]);
      }
    for (; r < rows; r += kListThreads / 4) {
      u32x4 x[2] = {};
      if (r < left) {
        const uint8_t* row = (const uint8_t*)p.A + (int64_t)(r0 + r) * p.lda;
        x[0] = row16(row, c0 + 32 * k, p.n);
        x[1] = row16(row, c0 + 32 * k + 16, p.n);
      }
      put(k, r, x[0], x[1]);
    }
    __syncthreads();
    for (int col = wave; col < 128; col += kListThreads / 64)
      for (int r = 16 * lane; r < rows; r += 1024)
        *(u32x4*)(d.S1 + (int64_t)(c0 + col) * d.Np + r0 + r) = strip_row16(bits + (col >> 5) * pitch, r, col & 31);
  }
  ones = wave_sum(ones);
  if (lane == 0 && ones) atomicAdd(&s_ones, ones);
  __syncthreads();
  if (tid == 0 && s_ones) atomicAdd(d.ring + 1, (u64)s_ones);
}

template <int E, bool CALLER>
__global__ void __launch_bounds__(kListThreads) k_layer_lists(LayerLists p) {
  typedef unsigned short Entries __attribute__((ext_vector_type(E)));
  constexpr unsigned short kMore = 0x8000u;  // in the last entry: the list goes on
  extern __shared__ __attribute__((aligned(16))) unsigned lds[];
  __shared__ int s_go, s_changed[3];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int b = xcd_logical(blockIdx.x, gridDim.x);  // neighbours share the lines of A and M
  if (tid == 0) s_go = 1;
  if (tid < 3) s_changed[tid] = 0;
  __syncthreads();
  unsigned* cur = lds;
  unsigned* nxt = lds + p.Np;
  Entries* first = (Entries*)(lds + 2 * p.Np);
  for (int i = tid; i < p.n; i += kListThreads)
    if (p.len[i] > kListMax) s_go = 0;
  __syncthreads();
  if (s_go == 0) {  // some row is too long for a list: every workgroup sees that
    if (blockIdx.x == 0 && tid == 0) st_system(p.status_out, 0u);
    if constexpr (CALLER) plain_dense_start(p, b, lds);
    return;
  }
  unsigned any = 0u;
  for (int i = tid; i < p.Np; i += kListThreads) {
    Entries e;
    const int c = i < p.n ? p.len[i] : 0;
#pragma unroll
    for (int k = 0; k < E; ++k) e[k] = k < c ? p.idx[(int64_t)k * p.n + i] : (unsigned short)i;
    if (c > E) e[E - 1] |= kMore;
    first[i] = e;
    unsigned v = 0u;
    const uint8_t* a = (const uint8_t*)p.A + (int64_t)i * p.lda + 32 * b;
    if (!CALLER) {
      v = bit16_of_bytes(((const u32x4*)a)[0]) | bit16_of_bytes(((const u32x4*)a)[1]) << 16;
    } else if (i < p.n) {
      if (32 * b + 32 <= p.n)
        v = bit16_of_bytes(bytes01(load16_any(a))) | bit16_of_bytes(bytes01(load16_any(a + 16))) << 16;
      else
        for (int x = 0; 32 * b + x < p.n; ++x) v |= (a[x] != 0 ? 1u : 0u) << x;
    }
    cur[i] = v;
    any |= v;
  }
  if (any != 0u) s_changed[1] = 1;
  __syncthreads();
  int t = 1;  // cur is R^(t); s_changed[t % 3]: it differs from R^(t-1)
  while (s_changed[t % 3]) {
    if (tid == 0) s_changed[(t + 2) % 3] = 0;  // read by all before the last barrier
    bool changed = false;
    for (int i = tid; i < p.Np; i += kListThreads) {
      const Entries e = first[i];
      const unsigned was = cur[i];  // R^(t-1) in place of A: the same iterates, since they grow
      unsigned v = was | cur[e[E - 1] & (kMore - 1)];
#pragma unroll
      for (int k = 0; k < E - 1; ++k) v |= cur[e[k]];
      if (e[E - 1] & kMore)
        for (int k = E, c = p.len[i]; k < c; ++k) v |= cur[p.idx[(int64_t)k * p.n + i]];
      nxt[i] = v;
      changed |= v != was;
    }
    ++t;
    if (changed) s_changed[t % 3] = 1;
    unsigned* x = cur;
    cur = nxt;
    nxt = x;
    __syncthreads();
  }
  for (int i = tid; i < (CALLER ? p.n : p.Np); i += kListThreads) {
    uint8_t* m = (uint8_t*)p.M + (int64_t)i * p.ldm + 32 * b;
    const unsigned w = cur[i];
    if (!CALLER) {
      ((u32x4*)m)[0] = bytes_of_bit16(w & 0xffffu);
      ((u32x4*)m)[1] = bytes_of_bit16(w >> 16);
    } else if (32 * b + 32 <= p.n) {
      store16_any(m, bytes_of_bit16(w & 0xffffu));
      store16_any(m + 16, bytes_of_bit16(w >> 16));
    } else {
      for (int x = 0; 32 * b + x < p.n; ++x) m[x] = (uint8_t)((w >> x) & 1u);
    }
  }
  for (int r = wave; !CALLER && r < 32; r += kListThreads / 64)
    for (int c = 16 * lane; c < p.Np; c += 1024)
      *(u32x4*)(p.T + (int64_t)(32 * b + r) * p.Np + c) = strip_row16(cur, c, r);
  // the last workgroup reports K
  if (tid == 0) {
    atomicMax(p.words + 1, (unsigned)t);
    wait_stores();
    if (atomicAdd(p.words, 1u) == gridDim.x - 1) {
      const unsigned K = ld_agent(p.words + 1);
      st_agent(p.words, 0u);
      st_agent(p.words + 1, 0u);
      wait_stores();
      st_system(p.status_out, K);
    }
  }
}

constexpr int kListsOf8 = kListMaxN * 5 / 8;  // up to here 8 entries a row fit: 24 bytes a row, 120 KB

template <bool CALLER>
static hipError_t launch_layer(const LayerLists& p, const uint8_t* P, int64_t ldp, hipStream_t s) {
  hipLaunchKernelGGL(k_row_lists, dim3((p.n + 3) / 4), dim3(256), 0, s, P, ldp, p.n, p.idx, p.len, p.status_out,
                     CALLER ? p.dense.ring : nullptr, p.dense.conv);
  const dim3 grid(p.Np / 32);
  if (p.Np <= kListsOf8)
    hipLaunchKernelGGL((k_layer_lists<8, CALLER>), grid, dim3(kListThreads), 24 * p.Np, s, p);
  else
    hipLaunchKernelGGL((k_layer_lists<4, CALLER>), grid, dim3(kListThreads), 16 * p.Np, s, p);
  return hipGetLastError();
}

hipError_t launch_layer_lists(const LayerLists& q, const int8_t* P, hipStream_t s) {
  if (q.n <= 0 || q.Np > kListMaxN || q.Np % 64 || q.Np < q.n) return hipErrorInvalidValue;
  LayerLists p = q;
  p.lda = p.ldm = p.Np;
  return launch_layer<false>(p, (const uint8_t*)P, p.Np, s);
}

hipError_t launch_closure_lists(const LayerLists& q, const uint8_t* A, int64_t lda, uint8_t* R, int64_t ldr,
                                hipStream_t s) {
  if (q.n <= 0 || q.n > kListMaxN || q.dense.Np < q.n || q.dense.Np % 128) return hipErrorInvalidValue;
  LayerLists p = q;
  p.Np = (p.n + 31) / 32 * 32;
  if (p.dense.Np + 64 > 4 * p.Np) return hipErrorInvalidValue;  // the LDS that the lists' launch has
  p.A = (const int8_t*)A;
  p.lda = lda;
  p.M = (int8_t*)R;
  p.ldm = ldr;
  return launch_layer<true>(p, A, lda, s);
}

__global__ void __launch_bounds__(256) k_lists_clear(ListParams p) {
  for (int i = threadIdx.x; i < kListWords; i += 256) ((unsigned*)p.cnt)[i] = 0u;
}

size_t sg_lists_bytes(int64_t n) {
  const size_t nb = (size_t)((n + 31) / 32);
  return 2 * nb * 32 * nb * 4 + (size_t)(kListMax + 1) * n * 2;
}

template <int E, bool CALLER>
static hipError_t layer_lists_attr(int bytes) {
  return hipFuncSetAttribute((const void*)k_layer_lists<E, CALLER>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

hipError_t sg_lists_init() {
  hipError_t e = layer_lists_attr<8, false>(24 * kListsOf8);
  if (e == hipSuccess) e = layer_lists_attr<8, true>(24 * kListsOf8);
  if (e == hipSuccess) e = layer_lists_attr<4, false>(16 * kListMaxN);
  if (e == hipSuccess) e = layer_lists_attr<4, true>(16 * kListMaxN);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute((const void*)k_sg_lists, hipFuncAttributeMaxDynamicSharedMemorySize, 3 * kListMaxN * 4);
}

hipError_t launch_sg_lists(ListParams p, uint8_t* ws, unsigned* words, bool clear_first, hipStream_t s) {
  if (p.dense.Np < p.n || p.dense.Np % 16) return hipErrorInvalidValue;
  if (p.n <= 0 || p.n > kListMaxN || p.max_steps < 2 || p.max_steps >= kRing) return hipErrorInvalidValue;
  p.nb = (p.n + 31) / 32;
  p.pitch = 32 * p.nb;
  const size_t slices = (size_t)p.nb * p.pitch;
  p.VT[0] = (unsigned*)ws;
  p.VT[1] = p.VT[0] + slices;
  p.idx = (unsigned short*)(p.VT[1] + slices);
  p.len = p.idx + (size_t)kListMax * p.n;
  p.cnt = (u64*)words;
  p.finished = words + 4 * kListArrivals * 32;
  if (clear_first) hipLaunchKernelGGL(k_lists_clear, dim3(1), dim3(256), 0, s, p);
  hipLaunchKernelGGL(k_row_lists, dim3((p.n + 3) / 4), dim3(256), 0, s, p.P, p.ldp, p.n, p.idx, p.len,
                     p.status_out, p.dense.ring, p.dense.conv);
  hipLaunchKernelGGL(k_sg_lists, dim3(p.nb), dim3(kListThreads), 3 * p.pitch * 4, s, p);
  return hipGetLastError();
}

}  // namespace dl
