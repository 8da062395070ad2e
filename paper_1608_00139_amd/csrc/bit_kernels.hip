// bit_kernels.hip -- the int8 squaring closure of a small relation in one
// launch, with bit-packed iterates.
//
// At n <= 1920 a fixpoint of product launches is bound by its launches, each
// product's wait for its first loads, and the host's read-back (n = 300: 65 us
// of kernels in a call of 107 us), not by arithmetic.  Here the whole series
// runs in one launch; workgroups hand their tiles to each other as bits (an
// eighth of the int8 bytes), so each fetches its two operand panels whole, and
// the bits become int8 operands in registers, in front of the MFMA.
//
// k_fix_bits: one workgroup per 64 x 64 tile (ti, tj) of R, all resident at
// once (see kResidentTicks), T = ceil(n / 64) <= 30 tiles a side.  Step 1
// packs the workgroup's tile of A; step t >= 2 computes its tile of
//   R^(t) = R^(t-1) | [R^(t-1) R^(t-1) != 0]
// (adding the previous iterate instead of A leaves the iterates unchanged)
// from row panel ti of R^(t-1) and row panel tj of its transpose.  A tile is
// published as 64 words of R and 64 of R^T, stored tile by tile, so a panel is
// contiguous.
//
// Arrivals: each step has one 64-bit word per tile row, to which a workgroup
// adds 2^40 + the ones of its tile once its stores have completed; a
// workgroup starts the next step when every row's word counts T arrivals
// (one load of T words by one wave), and the words' low parts sum to the model
// size, so all workgroups see the same repeat and stop together.  A tile of
// R^(t) overwrites the tile of R^(t-2), whose readers have all arrived at
// t - 1.  Coherence across XCDs and the bounded waits are those of
// k_fix_small: device-scope stores, loads and atomics.  On stopping each
// workgroup writes its tile as 0/1 bytes into the caller's R, and the last to
// finish writes the model sizes and the status and clears the words.
//
// Product: four waves of 32 x 32 (v_mfma_i32_16x16x64_i8, 2 x 2 fragments).
// Both operands use the same assignment of K to lanes, so the lanes of group g
// take word 4 q + g of their row and its 16-bit quarters in four K steps: one
// 8-byte LDS read feeds four MFMA operands.  Rows are padded to an odd number
// of words, so the 16 rows one read touches hit distinct banks.
//
// Measured (MI355X, a call as the caller sees it, degree 2, product launches
// and this one): n = 300 108, 50 us; n = 1000 116, 63 us; n = 1920 176, 174
// us.  Of the 50 us in the kernel at n = 1000 (seven steps) the waits for
// other workgroups take 24, the products 11 (AND and OR of the bits on the
// vector units instead: 17), publishing 6, fetching 4: bound by the chain of
// device-scope round trips.  At the top of the range the products are about 40% of it.
#include "common.h"
#include "device.h"

namespace dl {

typedef unsigned long long u64;

// Bits 16 q .. 16 q + 15 of w as 16 int8 operand elements, nonzero where the
// bit is set: 1, 2, 4 or 8, which v_perm and one mask give (the product's sums
// of at most 2048 terms <= 64 stay positive int32 numbers, and only their
// being nonzero is used).
__device__ inline v4i bytes_nz(u64 w, int q) {
  const unsigned x = q < 2 ? (unsigned)w : (unsigned)(w >> 32), y = x >> 4;
  const unsigned lo = (q & 1) ? 0x02020202u : 0x00000000u, hi = lo | 0x01010101u;  // byte selectors
  v4i v;
  v[0] = (int)(__builtin_amdgcn_perm(x, x, lo) & 0x08040201u);
  v[1] = (int)(__builtin_amdgcn_perm(y, y, lo) & 0x08040201u);
  v[2] = (int)(__builtin_amdgcn_perm(x, x, hi) & 0x08040201u);
  v[3] = (int)(__builtin_amdgcn_perm(y, y, hi) & 0x08040201u);
  return v;
}

constexpr u64 kArrive = 1ull << 40;  // above any sum of ones of a tile row

// Arrival word of a step and tile row, one per 128-byte line: arrivals of
// different rows and the polls of other workgroups do not queue on one line.
__device__ inline int bit_word(int step, int row) { return (step * kBitTiles + row) * kBitLine; }

__global__ void __launch_bounds__(256, 4) k_fix_bits(FixBitsParams p) {
  extern __shared__ __attribute__((aligned(16))) u64 lds64[];
  __shared__ u64 rows[64];  // the tile: word r = row 64 ti + r, columns 64 tj ..
  __shared__ u64 s_total;
  __shared__ int s_go;
  const int T = p.T, Tp = (T + 3) & ~3, pitch = Tp + 1;
  u64* xs = lds64;  // 64 rows of X, then of Y; words T .. Tp - 1 of a row stay zero
  u64* ys = lds64 + 64 * pitch;
  const int G = (int)gridDim.x;
  const int L = xcd_logical(blockIdx.x, G);
  const int ti = L / T, tj = L % T;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const unsigned mat = (unsigned)((size_t)T * T * 512);

  // step 1: the tile of A, 16 bytes a thread
  const int pr = tid >> 2, pc = (tid & 3) * 16;
  {
    const int gi = 64 * ti + pr, gj = 64 * tj + pc;
    unsigned m = 0u;
    if (gi < p.n) {
      const uint8_t* src = p.A + (int64_t)gi * p.lda + gj;
      if (gj + 16 <= p.n) {
        m = bit16_of_bytes(load16_any(src));
      } else {
        for (int e = 0; e < 16; ++e)
          if (gj + e < p.n && src[e] != 0) m |= 1u << e;
      }
    }
    ((unsigned short*)rows)[4 * pr + (tid & 3)] = (unsigned short)m;
  }
  for (int q = tid; q < 128 * (Tp - T); q += 256) lds64[(q / (Tp - T)) * pitch + T + q % (Tp - T)] = 0ull;
  __syncthreads();

  const u64 none = ~0ull;
  u64 sizes = 0ull;  // lane s of wave 0: the model size of step s
  u64 prev = none;   // size of the step before
  int t = 1;
  for (;;) {
    // publish: wave w has rows 16 w .. 16 w + 15 of the tile and of its transpose
    const u64 word = rows[lane];
    u64 col = 0ull;
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      const u64 b = __ballot((int)((word >> (16 * wave + c)) & 1ull));
      if (lane == c) col = b;
    }
    const __amdgpu_buffer_rsrc_t S = buffer_of(p.S[t & 1], mat), ST = buffer_of(p.ST[t & 1], mat);
    if ((lane >> 4) == wave) st_agent_x2(S, ((ti * T + tj) * 64 + lane) * 8, (unsigned)word, (unsigned)(word >> 32));
    if (lane < 16)
      st_agent_x2(ST, ((tj * T + ti) * 64 + 16 * wave + lane) * 8, (unsigned)col, (unsigned)(col >> 32));
    wait_stores();
    __syncthreads();
    if (wave == 0) {
      const int ones = wave_sum(__popcll(word));
      if (lane == 0) atomicAdd(p.cnt + bit_word(t, ti), kArrive + (u64)ones);
      // every tile row's arrivals at step t, and the model size
      const long long t0 = (long long)__builtin_amdgcn_s_memrealtime();
      int go = 1;
      u64 v = 0ull;
      for (;;) {
        if (lane < T) v = ld_agent64(p.cnt + bit_word(t, lane));
        if (__ballot(lane < T && (v >> 40) != (u64)T) == 0ull) break;
        if (ld_agent(p.finished + 1) != 0u) {
          go = -1;
          break;
        }
        if ((long long)__builtin_amdgcn_s_memrealtime() - t0 > (t == 1 ? kResidentTicks : p.wait_limit)) {
          if (lane == 0) {
            st_agent(p.finished + 1, 1u);
            st_system(p.status_out + 1, t == 1 ? kNotResident : 1u);
          }
          go = -1;
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
      u64 total = lane < T ? v & (kArrive - 1) : 0ull;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) total += __shfl_xor(total, off, 64);
      if (lane == t) sizes = total;
      if (lane == 0) {
        s_total = total;
        s_go = go;
      }
    }
    __syncthreads();
    if (s_go < 0) return;
    const u64 now = s_total;
    if (now == (t == 1 ? 0ull : prev) || t >= p.max_steps) break;
    prev = now;
    ++t;
    // the operands: T x 32 16-byte units (two rows' words of one tile) a panel
    const __amdgpu_buffer_rsrc_t X = buffer_of(p.S[(t - 1) & 1], mat), Y = buffer_of(p.ST[(t - 1) & 1], mat);
    for (int q = tid; q < 32 * T; q += 256) {
      const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(X, (ti * T * 64 + 2 * q) * 8, 0, kCpolSc1);
      const u32x4 y = __builtin_amdgcn_raw_buffer_load_b128(Y, (tj * T * 64 + 2 * q) * 8, 0, kCpolSc1);
      const int w = q >> 5, r = 2 * (q & 31);
      xs[r * pitch + w] = (u64)x[0] | (u64)x[1] << 32;
      xs[(r + 1) * pitch + w] = (u64)x[2] | (u64)x[3] << 32;
      ys[r * pitch + w] = (u64)y[0] | (u64)y[1] << 32;
      ys[(r + 1) * pitch + w] = (u64)y[2] | (u64)y[3] << 32;
    }
    __syncthreads();
    v4i acc[2][2] = {};
    const int g = lane >> 4, c = lane & 15;
    const int wm = wave >> 1, wn = wave & 1;
    const u64* xr = xs + (32 * wm + c) * pitch + g;
    const u64* yr = ys + (32 * wn + c) * pitch + g;
#pragma unroll 2
    for (int w = 0; w < Tp; w += 4) {
      const u64 x[2] = {xr[w], xr[16 * pitch + w]};
      const u64 y[2] = {yr[w], yr[16 * pitch + w]};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        v4i xf[2], yf[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          xf[i] = bytes_nz(x[i], q);
          yf[i] = bytes_nz(y[i], q);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xf[i], yf[j], acc[i][j], 0, 0, 0);
      }
    }
    // element v of fragment (i, j): row 32 wm + 16 i + 4 g + v, column
    // 32 wn + 16 j + c; lane c of group g takes fragment (c / 8, c / 4 % 2),
    // element c % 4 of the group's rows, 16 columns
    unsigned mine = 0u;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const u64 b = __ballot((int)(acc[i][j][v] != 0));
          if (c == 8 * i + 4 * j + v) mine = (unsigned)(b >> (16 * g)) & 0xffffu;
        }
    {
      const int r = 32 * wm + 16 * (c >> 3) + 4 * g + (c & 3), quarter = 2 * wn + ((c >> 2) & 1);
      ((unsigned short*)rows)[4 * r + quarter] =
          (unsigned short)(mine | ((const unsigned short*)(xs + r * pitch + tj))[quarter]);
    }
    __syncthreads();
  }

  // R^(t) as bytes, cropped; every store completes before the workgroup
  // counts itself finished
  {
    const int gi = 64 * ti + pr, gj = 64 * tj + pc;
    if (gi < p.n && gj < p.n) {
      const u32x4 v = bytes_of_bit16(((const unsigned short*)rows)[4 * pr + (tid & 3)]);
      store16_agent_any(p.R + (int64_t)gi * p.ldr + gj, v, p.n - gj);
    }
  }
  wait_stores();
  __syncthreads();
  if (tid == 0) s_go = atomicAdd(p.finished, 1u) == (unsigned)G - 1u ? 1 : 0;
  __syncthreads();
  if (!s_go) return;
  // the last workgroup: model sizes, cleared words, then the status
  if (wave == 0 && lane <= t) st_system64(p.ring_out + lane, sizes);
  for (int i = tid; i < (t + 1) * T; i += 256)
    __hip_atomic_store(p.cnt + bit_word(i / T, i % T), 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (tid == 0) st_agent(p.finished, 0u);
  wait_stores();
  __syncthreads();
  if (tid == 0) {
    st_system(p.status_out + 1, 0u);
    st_system(p.status_out, (unsigned)t);
  }
}

__global__ void __launch_bounds__(256) k_fix_bits_clear(FixBitsParams p) {
  for (int i = threadIdx.x; i < (kBitSteps + 1) * kBitTiles; i += 256) p.cnt[i * kBitLine] = 0ull;
  if (threadIdx.x < 2) p.finished[threadIdx.x] = 0u;
}

size_t fix_bits_bytes(int64_t n) {
  const size_t T = (size_t)((n + 63) / 64);
  return 4 * T * T * 512;
}

hipError_t launch_fix_bits(const FixBitsParams& q, bool clear_first, hipStream_t s) {
  const FixBitsParams& p = q;
  if (p.n <= 0 || p.T != (p.n + 63) / 64 || p.T > kBitTiles || p.max_steps < 1 || p.max_steps > kBitSteps)
    return hipErrorInvalidValue;
  if (clear_first) {
    hipLaunchKernelGGL(k_fix_bits_clear, dim3(1), dim3(256), 0, s, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_fix_bits, dim3(p.T * p.T), dim3(256),
                     (unsigned)(2 * 64 * (((p.T + 3) & ~3) + 1) * sizeof(u64)), s, p);
  return hipGetLastError();
}

}  // namespace dl
