// common.h -- types and helpers shared by the library's HIP sources (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dl {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef double v4d __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// Precision codes, identical to dl_prec in include/dl.h.
enum Prec { P_I8 = 0, P_F32 = 1, P_BF16 = 2, P_FP8 = 3, P_FP4 = 4 };

// Slots of the per-step model-size ring kept on the device.  Step s of a
// fixpoint accumulates the number of true entries of its iterate into
// ones[s % kRing]; kRing exceeds the largest chunk of steps launched between
// two host read-backs.
constexpr int kRing = 4096;
constexpr int kNotConverged = 0x7fffffff;

// 4-bit units (nibbles) per operand element: fp4 packs two elements per
// byte, element 2t in the low nibble of byte t.
__host__ __device__ constexpr int elem_nibbles(int prec) {
  return prec == P_F32 ? 8 : (prec == P_BF16 ? 4 : (prec == P_FP4 ? 1 : 2));
}
// Byte offset of element index e, and bytes of an Np x Np operand.
__host__ __device__ constexpr int64_t elem_offset(int prec, int64_t e) { return e * elem_nibbles(prec) / 2; }
__host__ __device__ constexpr int64_t mat_bytes(int prec, int64_t np) { return np * np * elem_nibbles(prec) / 2; }

// Parameters of one boolean product step  out = [add + X * Y^T != 0].
// Closure steps need no addend: with the identity stored in Y (Y = R^T + I
// for squaring, A + I for the plain series), X Y^T = R R + R already holds
// the previous iterate; outT_ident writes the next Y that way.
struct NTParams {
  const void* X;        // [Np x Np] operand, row-major, K contiguous
  const void* Y;        // [Np x Np] operand; row j of Y is column j of the right factor
  int64_t ld;           // leading dimension of X, Y, out, outT in elements (= Np)
  int Np;               // padded size: M = N = K = Np
  const int8_t* add;    // optional addend [Np x Np], row-major: int8 0/1 (pitch Np) or, with
                        // add_op, in operand precision (pitch ld; nonzero = true)
  int add_op;           // the addend is in operand precision
  int add_identity;     // if set, OR in (i, i) for i < n_valid
  int n_valid;          // number of real constants
  void* out;            // [Np x Np] next iterate in operand precision
  void* outT;           // optional transposed copy of out
  int outT_ident;       // outT gets (i, i) for i < n_valid as well: out^T + I
  unsigned long long* ones;  // model-size ring (read for the repeat test)
  int count;            // 1: add this iterate's number of ones to ones[step % kRing]
  int* conv;            // convergence step (null: no early exit)
  int step;             // index s of the iterate this launch produces
  int check;            // 1: detect a repeat from ones[s-1] == ones[s-2]
  int tiles_m, tiles_n; // grid in tiles
};

// Early exit of the element-wise kernels of a series: the test every product
// launch makes (step_is_done).  done() is true when the fixpoint was reached
// before step `step`; the first launch that sees the repeat records it.
// conv null: never.
struct StepGate {
  const unsigned long long* ones = nullptr;
  int* conv = nullptr;
  int step = 0;
  __device__ bool done() const {
    if (!conv) return false;
    if (*(volatile const int*)conv < step) return true;
    if (step < 2 || *(volatile const unsigned long long*)(ones + (step - 1) % kRing) !=
                        *(volatile const unsigned long long*)(ones + (step - 2) % kRing))
      return false;
    if (threadIdx.x == 0) atomicMin(conv, step - 1);
    return true;
  }
};

// One request's product in a grouped (serving) launch: T x T output tiles
// of an Np x Np int8 product, Np a multiple of T.
struct GroupDesc {
  const void* X;
  const void* Y;
  const int8_t* add;
  void* out;
  void* outT;
  unsigned long long* cnt;  // ones of this product's output (null: do not count)
  int Np;
  int n_valid;
  int add_identity;
  int outT_ident;  // outT = out^T + I (see NTParams)
  int tile_start;  // first work-list index of this request
  int sym;         // the result is symmetric (same generation's S'): only the
                   // tiles tm <= tn are listed, each off-diagonal one also
                   // written mirrored into out and counted twice
  // Skip test of a product issued before the previous round's model sizes
  // were read back: the request finished in that round exactly when its
  // cumulative counter *chk equals chk_val, and then this product gets no
  // tiles (see k_group_upload).  chk null: never skipped.
  const unsigned long long* chk;
  unsigned long long chk_val;
};

// The tile lists of one serving round, in descriptor order: segment k holds
// descriptors [begin[k], begin[k + 1]) of tile size tile[k] (begin[3] = all).
struct GroupLists {
  int begin[4];
  int tile[3];
};

// One request of a grouped admission (serving): clear its buffers, write the
// identity where same generation needs S^(1) = I, zero its admission counter,
// then scatter its edge list.  clear_start / edge_start are running totals
// (16-byte units, edges) over the requests before it.
struct AdmitDesc {
  int8_t* base;            // start of the region to clear
  long long clear_units;   // 16-byte units to clear from base
  long long clear_start;
  long long ident_off;     // byte offset from base of an Np x Np identity block, -1 if none
  int8_t* M;               // scatter targets (see k_scatter_edges); M2 / MT may be null
  int8_t* M2;
  int8_t* MT;
  unsigned long long* ones;  // distinct edges counter (may be null), zeroed by the clear
  const int32_t* edges;
  long long m;
  long long edge_start;
  int n;
  int Np;
};
hipError_t launch_admit(const AdmitDesc* d, int nreq, long long total_units, long long total_edges, hipStream_t s);

// The one-launch fixpoints need all their workgroups (k_fix_small: those of a
// tile row) on the chip together.  A cooperative launch does not see to that
// beside another one or beside other work (several threads' launches held
// parts of the chip and waited for the rest until their time limit), and costs
// 11.5 us more than an ordinary one (17.7 against 6.2 us from the call to a
// status word in host memory).  So they are launched the ordinary way, and
// each workgroup's first wait is for all the others' first tiles: once it is
// over they are all running, and nothing can keep them from finishing.  If it
// takes longer than kResidentTicks -- other work holds the chip -- the launch
// ends with kNotResident in status_out[1], and the series is run by product
// launches, which wait for nobody.
constexpr long long kResidentTicks = 20000;  // 200 us of s_memrealtime (100 MHz)
constexpr unsigned kNotResident = 2u;

// The whole plain closure fixpoint in one launch (k_fix_small in
// bool_kernels.hip): one workgroup per 32 x 32 tile of S = R^T, for
// operand rows of at most 2 KB and Np <= 512.
struct FixSmallParams {
  const uint8_t* A;
  int64_t lda;
  uint8_t* R;
  int64_t ldr;
  // counters: zero when the launch starts, and left zero by a launch that
  // ends normally (the last workgroup clears them); see fix_small_words
  unsigned long long* ones_row;  // [tiles][Np + 3] model size of each row block per step
  unsigned* krow;                // [tiles] last step of each row block
  unsigned* finished;            // [0] workgroups done, [1] abort (a wait ran past its limit)
  // tiles of the iterates as bits, S^(t) in half t & 1: [tile row][tile][row]
  // words of (tag + t) << 32 | 32 columns; no word holds one of this launch's
  // tags tag + 1 .. tag + max_steps when it starts
  unsigned long long* exchange;
  unsigned tag;
  // outputs (device or mapped host memory), written by the last workgroup
  unsigned long long* ring_out;  // ring_out[t] = size of S^(t), t = 0 .. K
  unsigned* status_out;          // [0] K, the last step of any row block; [1] 1 after an abort, or kNotResident
  int n, Np, tiles;              // tiles = Np / 32 per side
  int max_steps;                 // at most Np + 2
  long long wait_limit;          // ticks
};
bool fix_small_supported(int prec, int64_t np);
// Tile-configuration id that selects it for the plain series (the product
// kernels' configurations are 0 .. nt_config_count - 1; for every other use
// of the product step this id falls back to the size rule).
constexpr int kCfgWholeFixpoint = 5;
// The launch; with clear_first, a kernel that zeroes the counters of every size
// and the exchanged words runs before it (needed once for fresh memory, after
// an abort and when the tags start again).
// Words (32-bit) for padded size np: the counters of fix_small_counters(np),
// the first 2 tiles (np + 3) of them holding ones_row, then the exchanged
// words, as many for every size (8-byte aligned).
hipError_t launch_fix_small(int prec, const FixSmallParams& p, bool clear_first, hipStream_t s);
constexpr int64_t kFixSmallExchange = 2 * 16 * 16 * 32;  // words of 8 bytes: Np = 512
inline constexpr int64_t fix_small_counters(int64_t np) { return (2 * (np / 32) * (np + 3) + (np / 32) + 3) / 2 * 2; }
inline constexpr int64_t fix_small_words(int64_t np) { return fix_small_counters(np) + 2 * kFixSmallExchange; }
// Points the counters and exchanged words of p into `words` (fix_small_words(512)
// of them, 8-byte aligned): the exchanged words lie behind the largest size's
// counters, at one place for every size.
inline void fix_small_place(FixSmallParams& p, unsigned* words) {
  p.ones_row = (unsigned long long*)words;
  p.krow = words + 2 * (int64_t)p.tiles * (p.Np + 3);
  p.finished = p.krow + p.tiles;
  p.exchange = (unsigned long long*)(words + fix_small_counters(512));
}
// The tags of the next launch over one set of words, of which `last` is the
// last launch's: from it on, or from zero, in words cleared first, before they
// would run over.
constexpr unsigned kFixSmallTags = 1024;  // above Np + 2
inline unsigned fix_small_tag(unsigned* last, bool* clear) {
  if (*last > ~0u - 2 * kFixSmallTags) {
    *last = 0u;
    *clear = true;
  }
  return *last += kFixSmallTags;
}

// The squaring closure of n <= 64 kBitTiles constants in one launch, on bits (k_fix_bits in bit_kernels.hip).
constexpr int kBitTiles = 30;  // 64 x 64 tiles a side at most
constexpr int kBitLine = 16;   // 64-bit words per arrival word: a 128-byte line
constexpr int kBitSteps = 16;  // squaring repeats by step 2 + ceil(log2(1920))
struct FixBitsParams {
  const uint8_t* A;
  int64_t lda;
  uint8_t* R;
  int64_t ldr;
  void* S[2];               // iterates, tile by tile (T x T tiles of 64 words): S^(t) in S[t & 1]
  void* ST[2];              // their transposes
  unsigned long long* cnt;  // [kBitSteps + 1][kBitTiles][kBitLine] arrivals and ones per step and tile row (the
                            // first word of each line), zero between launches
  unsigned* finished;       // [0] workgroups done, [1] abort, zero between launches
  unsigned long long* ring_out;  // model sizes of steps 0 .. K
  unsigned* status_out;          // [0] K, [1] 1 after an abort
  int n, T;                      // T = ceil(n / 64)
  int max_steps;                 // 1 .. kBitSteps
  long long wait_limit;          // ticks
};
// Bytes of the four iterate buffers; counter words (32-bit, 8-byte aligned).
size_t fix_bits_bytes(int64_t n);
constexpr int64_t kFixBitsWords = 2 * (kBitSteps + 1) * kBitTiles * kBitLine + 2;
hipError_t launch_fix_bits(const FixBitsParams& p, bool clear_first, hipStream_t s);

// Where a row turns out too long for lists, the launch that would have run the
// series writes the first operands of its products instead (int8, Np x Np, as
// launch_ingest and launch_identity do): with the ring of model sizes reset by
// the pass that makes the lists, finding out costs a dense relation no launch.
// Calls in us, without lists and with: same generation, density 0.3, n = 64, 512,
// 2048, 4096: 96, 100, 164, 265 and 94, 91, 136, 250; plain closure, 300 entries a
// row, n = 600, 1000, 4096, 8192: 91, 98, 180, 1052 and 79, 83, 175, 1075 (with a
// launch that only says no, then those of the product series: 116, 114, 158, 281
// and 109, 114, 204, 1075).
//   same generation: Y = P, S1 = I, ring[1] = n, `words` zeros at `zero`
//   plain closure:   Y = A + I, S1 = A^T, ring[1] = the ones of A
struct DenseStart {
  int8_t* Y;
  int8_t* S1;
  int Np;
  unsigned long long* ring;
  int* conv;
  unsigned* zero;
  int words;
};

// The same-generation series by lists of P's entries, on bits, in one launch
// (list_kernels.hip), for n <= kListMaxN and at most kListMax entries a row.
//
// Series with a relation of few entries a row go by lists at every size up to
// kListMaxN (a slice of 32 rows a compute unit) and up to kListMax entries in
// every row: at 32 they still win everywhere.  Calls in us, lists / products,
// relations with exactly 4, 16 and 32 entries in every row (5 to 7, 4 or 5, 3 to
// 5 steps):
//   same generation  n = 64 54/102, 59/99, 64/94; 512 61/153, 64/100, 82/101;
//                    4096 96/547, 145/428, 189/347; 8192 168/3795, 261/2544, 358/1946
//   plain closure    n = 1024 45/168, 47/103, 55/98; 4096 73/624, 91/351, 126/270;
//                    8192 111/3855, 172/1699, 238/1356
//   program closure  n = 64 52/113, 51/77, 53/73; 512 50/123, 51/83, 59/78;
//                    4096 106/706, 122/368, 155/291; 8192 208/4750, 270/2050, 334/1648
constexpr int kListMax = 32;
constexpr int kListMaxN = 8192;
constexpr int kListArrivals = 8;  // words that a step's arrivals are spread over, a line each
struct ListParams {
  const uint8_t* P;
  int64_t ldp;
  uint8_t* R;
  int64_t ldr;
  unsigned* VT[2];      // slices of P S, step t in VT[t & 1] ...
  unsigned short* idx;  // [kListMax][n] list entries, [k n + j] = entry k of row j ...
  unsigned short* len;  // ... and [n] their numbers
  unsigned long long* cnt;  // [4][kListArrivals][16] arrivals and ones of steps t % 4, zero between launches
  unsigned* finished;       // [0] workgroups done, [1] abort, zero between launches
  unsigned long long* ring_out;  // model sizes of steps 1 .. K
  unsigned* status_out;          // [0] K, 0 if a row is too long; [1] 1 after an abort, or kNotResident
  int n, nb, pitch;              // nb = ceil(n / 32) slices of pitch = 32 nb words
  int max_steps;                 // 2 .. kRing - 1
  long long wait_limit;          // ticks
  DenseStart dense;
};
size_t sg_lists_bytes(int64_t n);
constexpr int kListWords = 4 * kListArrivals * 32 + 2;  // 32-bit, 8-byte aligned
hipError_t sg_lists_init();
// ws: sg_lists_bytes(n), 16-byte aligned; words: kListWords of them.
hipError_t launch_sg_lists(ListParams p, uint8_t* ws, unsigned* words, bool clear_first, hipStream_t s);

// The series of a program's layer with one recursive term, R = A + P R, by
// lists of P's entries (k_layer_lists), Np <= kListMaxN.
struct LayerLists {
  const int8_t* A;      // Np x Np, zero from row and column n on
  int8_t *M, *T;        // the model and its transpose
  int64_t lda, ldm;     // set by the launch
  unsigned short* idx;  // lists as in ListParams
  unsigned short* len;
  unsigned* words;       // [0] workgroups done, [1] their last steps; zero between launches
  unsigned* status_out;  // host memory: K, the first step that repeats, or 0 if a row is too long
  int n, Np;
  DenseStart dense;  // the plain closure's (otherwise nothing is written for a row too long)
};
constexpr int kLayerWords = 2;
hipError_t launch_layer_lists(const LayerLists& p, const int8_t* P, hipStream_t s);
// The plain closure R = A + A R of a caller's relation the same way (idx, len,
// words, status_out, n and dense of p are used).
hipError_t launch_closure_lists(const LayerLists& p, const uint8_t* A, int64_t lda, uint8_t* R, int64_t ldr,
                                hipStream_t s);

// Launch helpers implemented in bool_kernels.hip.
struct TileCfg {
  int bm, bn, kb, threads;
  size_t lds_bytes;
};

hipError_t launch_nt_step(int prec, int cfg_id, const NTParams& p, hipStream_t s);

// Stream-K split of a product whose result is symmetric (the same-generation
// S' = [I + T P^T]): only the tiles tm <= tn of the 256 x 256 int8 tiling are
// computed, their tiles x (Np / 128) K slices dealt to the workgroups in runs
// of `share` slices, so that every compute unit gets the same number of
// slices.  A tile split over several workgroups is finished by the last of
// them to arrive: each stores its partial Boolean tile as bits in scratch slot
// (t * maxc + contributor) with write-through stores and counts itself in
// tile_cnt[t]; the last ORs the partials (device-scope loads), adds
// the identity, counts, writes the tile and its mirror image and clears
// tile_cnt[t] for the next launch.  tile_cnt starts at zero.
constexpr unsigned kSkSlot = 256 * 256 / 8;
struct SkParams {
  uint8_t* scratch;    // tiles * maxc slots of kSkSlot bytes
  unsigned* tile_cnt;  // [tiles] arrivals, zero between launches
  int side;            // tiles per side, Np / 256
  int tiles;           // side (side + 1) / 2
  int share;           // K slices per workgroup
  int maxc;            // slots per tile (contributors at most)
};
// Whether the split applies (int8 operands, the direct-to-LDS configuration,
// Np a multiple of 256), the plan for Np, and the scratch it needs (slots,
// then the counters).
bool sk_supported(int prec, int cfg_id, int64_t Np);
void sk_plan(int64_t Np, SkParams& q);
size_t sk_scratch_bytes(const SkParams& q);
hipError_t launch_nt_sym_sk(const NTParams& p, const SkParams& q, hipStream_t s);
TileCfg nt_config(int prec, int cfg_id);
int choose_nt_config(int prec, int64_t n);
int nt_config_count(int prec);  // cfg ids are 0 .. count - 1
bool nt_config_valid(int prec, int cfg, int64_t np);  // cfg usable at padded size np
hipError_t launch_hash_bool(uint8_t* M, int64_t ld, int n, int Np, unsigned seed, hipStream_t s);
hipError_t launch_publish(const unsigned long long* src, unsigned long long* dst, int n, hipStream_t s);
int64_t padded_size_for(int prec, int64_t n);

// ident: bit 0 adds the identity (first n constants) to Aop, bit 1 to ATop;
// the ones counted are those of A alone.
hipError_t launch_ingest(int prec, const uint8_t* A, int64_t lda, int n, int Np, int8_t* A8,
                         int8_t* AT8, void* Aop, void* ATop, int ident, unsigned long long* ones_slot,
                         hipStream_t s);
hipError_t launch_identity(int prec, void* S, int Np, int n, hipStream_t s);
// An int8 matrix cropped to n x n into R, its true entries counted into
// *sum_out (mapped host memory).  words: two, zero between launches.
hipError_t launch_emit_sum(const void* S, int Np, int n, uint8_t* R, int64_t ldr, unsigned long long* words,
                           unsigned long long* sum_out, hipStream_t s);
// Models of several int8 iterates to callers' matrices in one launch.
struct EmitDesc {
  const uint8_t* S;  // Np x Np iterate
  uint8_t* R;        // n x ldr
  int64_t ldr;
  int Np, n;
  int tile_start;  // set by launch_emit_group
  int pad;
};
constexpr int kEmitGroup = 64;  // matrices per launch: their descriptors are its arguments
hipError_t launch_emit_group(const EmitDesc* d, int count, hipStream_t s);
hipError_t launch_emit(int prec, const void* S, int Np, int transpose, int n, uint8_t* R,
                       int64_t ldr, hipStream_t s);
hipError_t launch_ring_clear(unsigned long long* ones, int* conv, int s0, int count, int reset_conv,
                             hipStream_t s);
hipError_t launch_ring_set(unsigned long long* ones, int slot, unsigned long long value, hipStream_t s);
hipError_t launch_row_max(const uint8_t* A, int64_t lda, int n, int* out_max, hipStream_t s);
hipError_t launch_col_max(const uint8_t* A, int64_t lda, int n, int* out_max, hipStream_t s);
// out = (a | b | [ident] I), or its complement within the n x n constants when
// `complement` is set; int8 0/1 Np x Np operands (a, b, out, outT may be null;
// out may alias a or b).  Adds the ones of the result to *cnt if cnt is set.
hipError_t launch_bytes_op(const int8_t* a, const int8_t* b, int ident, int complement, int n, int Np, int8_t* out,
                           int8_t* outT, unsigned long long* cnt, hipStream_t s, const StepGate& gate = StepGate());
// Sets byte (i, j) of M (and of M2, and byte (j, i) of MT, when not null) for
// every edge (i, j) of the device list edges[2 m] with 0 <= i, j < n; adds
// the number of distinct edges to *ones.  The matrices must be zeroed.
hipError_t launch_scatter_edges(const int32_t* edges, int64_t m, int n, int Np, int8_t* M, int8_t* M2, int8_t* MT,
                                unsigned long long* ones, hipStream_t s);
hipError_t bool_kernels_init();
// Measured matrix-core throughput (operations per second) of MFMA kind 0 int8,
// 1 fp32, 2 bf16, 3 fp8, 4 fp4, 5 fp64 on the current device, or bytes per
// second of kind 6 (LDS reads, ds_read_b128) and 7 (global-to-LDS fill,
// global_load_lds_dwordx4 from 1 MB at src); kind 8 is kind 5 with AGPR
// accumulators.  `sink` must hold 256 ints (never written).
hipError_t measure_peak(int kind, int* sink, double* ops_per_s, hipStream_t s, const uint8_t* src);
// tile: 64, 128 or 256 (every request of the list has Np a multiple of it);
// at most kMaxGroupRequests requests per launch
constexpr int kMaxGroupRequests = kRing;
// dyn_total (device int, may be null): the live tile count written by
// k_group_upload; total_tiles is then the bound the grid was sized for.
hipError_t launch_group_step(int tile, const GroupDesc* desc, int nreq, int total_tiles, hipStream_t s,
                             const int* dyn_total = nullptr);
// Copy a round's descriptors from src (a device mapping of host memory) to
// dst and renumber the tiles of each segment over the products that are not
// skipped (GroupDesc::chk); totals[k] receives segment k's live tile count.
hipError_t launch_group_upload(const GroupDesc* src, GroupDesc* dst, const GroupLists& lists, int* totals,
                               hipStream_t s);

}  // namespace dl
