// Internal declarations shared by the translation units of libclover.so.
// Host-side launch wrappers only: every wrapper validates nothing (the C-ABI layer does) and
// enqueues on the given stream.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include <type_traits>

#include "../../include/clover.h"
#include "once_per_device.h"

namespace clv {

typedef unsigned short bf16_t;  // raw bfloat16 bit pattern

enum KernelClass {
  KC_EMBED = 0, KC_RMSNORM, KC_GEMM_QKV, KC_ROPE_KV, KC_ATTN, KC_GEMM_WO, KC_GEMM_GATEUP, KC_GEMM_DOWN,
  KC_GEMM_LMHEAD, KC_GEMM_DRAFT, KC_AD_GATE, KC_TOPK, KC_DRAFT_MISC, KC_ACCEPT, KC_COMPACT, KC_ELTWISE,
  KC_COUNT
};

// Rows are laid out [B, R]; row (b,i) exists for i < n and is valid iff i < (n_valid ? n_valid[b] : n).
struct RowMap {
  int B, R, n;
  const int* n_valid;  // dev [B] or null
};

constexpr int KV_PAGE = 32;   // cached positions per page (= the key tile of the MFMA attention)
struct KVLayout {
  // Paged caches, one pair per layer.  A page holds KV_PAGE consecutive positions of one sequence for all KV heads:
  // so K, and V^T, of one (page, head) -- one key tile of the attention -- are one contiguous block each.  Position `slot` of
  // sequence b lives in page pages[(b + b0) * T + slot / KV_PAGE] (identity when pages is null), at row r = slot % KV_PAGE.
  //   planes 1 (kvdtype 0): fp32 elements, K [n_kv][KV_PAGE][d], V transposed [n_kv][d][KV_PAGE].
  //   planes 2 (kvdtype 1): two bf16 planes (hi, then lo `plane` elements later) with hi + lo == value to 16 mantissa bits,
  // [n_kv][planes][KV_PAGE x d] in the order in which the MFMA attention stages a block: KBs of 64 lanes x 8 elements, lane
  // 16 g + l of KB (half, k) of K holding row 8 (l / 4) + 4 half + l % 4, columns 32 k + 8 g .., of KB k of V^T row (channel)
  // 16 k + l, positions 8 g ...  A staging load then takes its KB lane by lane; with rows in the cache its lanes jumped by 256
  // bytes in K and by 64 in V^T.  And a key tile is two streams of 16 KB instead of four of 8.  Attention, us per
  // launch: 96 nodes at 8192 keys 49 -> 45, a 1024-token prompt 53.7 -> 50.5, an 8192-token one 345 -> 342.
  int max_batch, max_seq, n_kv, d;
  int planes;
  size_t plane;
  int T;               // pages per sequence = max_seq / KV_PAGE
  int b0;              // added to every sequence index (a call that works on one sequence of the batch)
  const int* pages;    // dev [max_batch * T] page table, or null
};
#ifdef __HIPCC__
// element index of block (page, head) of the position
__device__ __forceinline__ size_t kv_block(const KVLayout& kv, int b, int slot, int head) {
  const int lp = (b + kv.b0) * kv.T + slot / KV_PAGE;
  return ((size_t)(kv.pages ? kv.pages[lp] : lp) * kv.n_kv + head) * kv.planes * (KV_PAGE * kv.d);
}
// element index of K[b][slot][head][c] = kv_k_at + kv_k_col(c); four columns c % 4 == 0 are contiguous
__device__ __forceinline__ size_t kv_k_at(const KVLayout& kv, int b, int slot, int head) {
  const int r = slot % KV_PAGE;
  return kv_block(kv, b, slot, head) + (kv.planes == 1 ? r * kv.d : ((r >> 2) & 1) * 16 * kv.d + ((r >> 3) * 4 + (r & 3)) * 8);
}
__device__ __forceinline__ int kv_k_col(const KVLayout& kv, int c) {
  return kv.planes == 1 ? c : (c >> 5) * 512 + ((c >> 3) & 3) * 128 + (c & 7);
}
// element index of V^T[b][head][dim][slot]; four positions slot % 4 == 0 are contiguous
__device__ __forceinline__ size_t kv_v_at(const KVLayout& kv, int b, int head, int dim, int slot) {
  const int r = slot % KV_PAGE;
  return kv_block(kv, b, slot, head) + (kv.planes == 1 ? dim * KV_PAGE + r : (dim >> 4) * 512 + ((r >> 3) * 16 + (dim & 15)) * 8 + (r & 7));
}
#endif

// ---- launch helper -----------------------------------------------------------------------------
// what a launcher of this thread could not launch, until the entry point that called it reports it (null: nothing)
inline thread_local const char* g_not_launched = nullptr;
// f(integral constant n) for n in LO .. HI: a kernel's loads of n partial results are counted at compile time.  Another count is
// not rounded to one of these -- the kernel would leave out ranges or add what nothing wrote: nothing is launched and the call fails.
template <int LO, int HI, class F>
inline void with_count(int n, F&& f) {
  if (n == LO) return f(std::integral_constant<int, LO>{});
  if constexpr (LO < HI)
    if (n > LO) return with_count<LO + 1, HI>(n, f);
  g_not_launched = "no kernel for this count of partial results";
}

// ---- rankings by (value, id) keys ----------------------------------------------------------------
#ifdef __HIPCC__
// largest of the wavefront's values, along the lanes of a row, then over the rows (a few clocks a step; an exchange through the
// LDS crossbar takes 50 to 100, and a ranking is a chain of them: the chunks of a top-8 of 8 rows x 128256 8.6 -> 6.8 us)
__device__ __forceinline__ unsigned wave_max_u32(unsigned v) {
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));   // row_shr:1, 2, 4, 8
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));   // row_bcast:15 into rows 1 and 3
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));   // row_bcast:31 into rows 2 and 3
  return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ unsigned long long wave_max_key(unsigned long long v) {
  const unsigned hi = (unsigned)(v >> 32), top = wave_max_u32(hi);
  return ((unsigned long long)top << 32) | wave_max_u32(hi == top ? (unsigned)v : 0u);
}
// the largest key of 256 threads, round r of a ranking: the rounds take turns in `red`, so one barrier each is enough
__device__ __forceinline__ unsigned long long block_max_key(unsigned long long v, unsigned long long (&red)[2][4], int r) {
  v = wave_max_key(v);
  unsigned long long* q = red[r & 1];
  if ((threadIdx.x & 63) == 0) q[threadIdx.x >> 6] = v;
  __syncthreads();
  const unsigned long long a = q[0] > q[1] ? q[0] : q[1], b = q[2] > q[3] ? q[2] : q[3];
  return a > b ? a : b;
}
#endif

// ---- staging loads: global -> LDS without a stop in registers -------------------------------------
#ifdef __HIPCC__
typedef const __attribute__((address_space(1))) char* gbyte_ptr;
// 64 lanes x 16 bytes from (uniform base) + (lane offset) to the KB at LDS byte address `dst` (the same for all lanes;
// the hardware adds lane * 16, lane l's piece lands at dst + 16 l).  The compiler is not told that this writes the LDS:
// it would wait for every load in flight before each LDS read that follows.  The waits before the barriers are written by
// hand, and there is no memory clobber (the staged data is read only behind a later barrier, which is a fence for the
// compiler; a clobber would turn scalar loads around it into vector loads that wait for the staging loads in flight).
// The no-op is the wait state gfx950 needs between a scalar write of M0 and a load to the LDS that reads it; the compiler
// places it for its own loads but does not look inside an asm string.  It is one issue slot beside a load of 64 clocks.
// NT: non-temporal.
template <bool NT>
__device__ __forceinline__ void lds_load16(gbyte_ptr base, unsigned lane_off, unsigned dst) {
  const unsigned m0 = __builtin_amdgcn_readfirstlane(dst);
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" : : "s"(m0), "v"(lane_off), "s"(base) : "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(m0), "v"(lane_off), "s"(base) : "m0");
}
#endif

// ---- GEMM activations in fragment order ---------------------------------------------------------
// An activation matrix that feeds the MFMA GEMM is kept as two bf16 planes (hi, lo) with hi + lo == x to 16 mantissa
// bits, stored as the GEMM stages them: [K/32][mb row blocks][hi, lo][16 rows][32 columns], every (row block, plane) of
// a 32-column step one contiguous KB.  A compute unit pulls contiguous KBs from the L2 at 124 GB/s and 16 rows of 64 or
// 128 bytes out of a row-major matrix at 62 (256 compute units at once, 8 KB row stride), and the activations are half
// of what a GEMM workgroup loads.  The four 16-byte pieces of a row's 64 bytes are permuted by the row, so that the
// 16-row fragment reads from the (identical) LDS image run without bank conflicts; a producer that owns a row still
// writes whole 64-byte segments.
struct FragPlanes {
  bf16_t* p;
  int mb;   // row blocks = ceil(rows / 16); rows past the matrix in the last block are never initialised
};
inline FragPlanes frag_planes(void* buf, int rows) { return FragPlanes{(bf16_t*)buf, (rows + 15) / 16}; }
#ifdef __HIPCC__
// element index of the hi value at (row, col); the lo value is 512 elements further.  The 8 columns of a piece
// (col % 8 == 0) are contiguous.
__device__ __forceinline__ size_t frag_at(const FragPlanes& f, int row, int col) {
  const int r = row & 15, pc = ((col >> 3) & 3) ^ ((0 - (r >> 2)) & 3);
  return ((size_t)(col >> 5) * f.mb + (row >> 4)) * 1024 + r * 32 + pc * 8 + (col & 7);
}
// four adjacent columns (col % 4 == 0) of one row
__device__ __forceinline__ void frag_store4(const FragPlanes& f, int row, int col, float o0, float o1, float o2, float o3) {
  const float o[4] = {o0, o1, o2, o3};
  unsigned h[4], l[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {   // round to nearest even through the hardware conversion (v_cvt_pk_bf16_f32)
    h[r] = (unsigned)__builtin_bit_cast(unsigned short, (__bf16)o[r]);
    l[r] = (unsigned)__builtin_bit_cast(unsigned short, (__bf16)(o[r] - __uint_as_float(h[r] << 16)));
  }
  bf16_t* dst = f.p + frag_at(f, row, col);
  *(uint2*)dst = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
  *(uint2*)(dst + 512) = make_uint2(l[0] | (l[1] << 16), l[2] | (l[3] << 16));
}
#endif

#ifdef __HIPCC__
// Four elements at once from wherever an element may lie: callers owe their tensors no more, and the load instruction takes it.
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef bf16_t bf16x4_any __attribute__((ext_vector_type(4), aligned(2)));
__device__ __forceinline__ float4 ld4_any(const float* p) {
  const f32x4_any u = *(const f32x4_any*)p;
  return make_float4(u[0], u[1], u[2], u[3]);
}
__device__ __forceinline__ float4 ld4_any(const bf16_t* p) {
  const bf16x4_any u = *(const bf16x4_any*)p;
  return make_float4(__uint_as_float((unsigned)u[0] << 16), __uint_as_float((unsigned)u[1] << 16), __uint_as_float((unsigned)u[2] << 16),
                     __uint_as_float((unsigned)u[3] << 16));
}
__device__ __forceinline__ int rows_valid(const RowMap& rm, int b) { return rm.n_valid ? min(rm.n_valid[b], rm.n) : rm.n; }

// raises the limit of a kernel's dynamic LDS, once per device
inline void allow_dynamic_lds(OncePerDevice& once, const void* kernel, int bytes) {
  int dev = -1;
  hipGetDevice(&dev);
  once(dev, [&] { hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes); });
}
#endif

// ---- generic (fp32 ALU) kernels; wdtype: 0 fp32, 1 bf16 ---------------------------------------
// rotary tables: row (b, i) of the pass sits at position base_len[b] + (depth ? depth[i] : i)
struct RopeRows {
  const int *base_len, *depth;   // dev [B]; dev [n] or null
  int depth_stride;              // nodes per sequence in a per-sequence depth table, 0: one table for all
  float base; int d;
  float *cos_t, *sin_t;          // [rows][d / 2]
};
#ifdef __HIPCC__
__device__ __forceinline__ void rope_row(const RopeRows& r, int b, int i, size_t row) {
  const int half = r.d / 2;
  if ((int)threadIdx.x >= half) return;
  const int pos = r.base_len[b] + (r.depth ? r.depth[(size_t)b * r.depth_stride + i] : i);
  for (int c = threadIdx.x; c < half; c += blockDim.x) {
    const double inv = pow((double)r.base, -2.0 * (double)c / (double)r.d);
    const double ang = (double)pos * inv;
    r.cos_t[row * half + c] = (float)cos(ang);
    r.sin_t[row * half + c] = (float)sin(ang);
  }
}
#endif
// start of a pass: out[row] = table[tok[row]], the rotary tables, and where gain is given (bf16 models) planes of RMSNorm(out) * gain
struct PassStart {
  const void* table; const int* tok; int vocab;
  float* out; int ldo, H;
  RowMap rm;
  RopeRows rope;
  const void* gain; float eps; FragPlanes planes;
};
void launch_pass_start(const PassStart& p, int wdtype, hipStream_t st);
void launch_rmsnorm(const float* x, int ldx, const void* gain, int wdtype, float eps, float* out, int ldo, int H,
                    int rows, hipStream_t st);
void launch_rope_kv_write(const float* qkv, int ldqkv, const float* cos_t, const float* sin_t, float* q_out, int ldq, float* k_cache,
                          float* v_cache, KVLayout kv, const int* base_len, int n_q, RowMap rm, int* err_flag, hipStream_t st);
// the same behind a QKV GEMM that left partial tiles, heads of q and k in rotary order; caches of two planes.  q in fp32, few rows:
void launch_rope_kv_parts(const float* qkv, int ldqkv, int splits, size_t split_stride, const float* cos_t, const float* sin_t, float* q_out,
                          int ldq, bf16_t* k_cache, bf16_t* v_cache, KVLayout kv, const int* base_len, int n_q, RowMap rm, int* err_flag,
                          hipStream_t st);
// q as planes:
void launch_rope_kv_planes(const float* qkv, int ldqkv, int splits, size_t split_stride, const float* cos_t, const float* sin_t, bf16_t* k_cache,
                           bf16_t* v_cache, KVLayout kv, const int* base_len, int n_q, RowMap rm, int* err_flag, bf16_t* q_hi, bf16_t* q_lo,
                           int ldq, float q_scale, hipStream_t st);
void launch_attn_generic(const float* q, int ldq, const void* k_cache, const void* v_cache, int kvdtype, KVLayout kv,
                         const int* base_len, const unsigned long long* anc /*[n][2]*/, int n_q, float* out /*of fp32 caches*/, int ldo,
                         FragPlanes planes /*the results over caches of bf16 planes*/, RowMap rm,
                         hipStream_t st, int anc_stride = 0 /*nodes per sequence in a per-sequence mask table, 0: shared*/,
                         const int* iv = nullptr /*[n][2] interval labels: decide visibility instead of anc when given*/);
// mode 0: Y = X W^T (+bias); mode 1: Y += X W^T (+bias)
void launch_gemm_generic(const float* X, int ldx, const void* W, const void* bias, int wdtype, float* Y, int ldy,
                         int M, int N, int K, int mode, hipStream_t st);
// Up to three such products over the same M rows and K in one launch.  gain non-null: of RMSNorm(X) * gain.  swiglu: Y of
// g[0] = silu(X g[0].W^T) * (X g[1].W^T) (no bias, mode 0).  Only where gemm_small_joins says so: the outputs are too few for
// larger tiles, and one launch is faster than the norm and the products by themselves.
struct SmallGemm {
  const float* X; int ldx;
  const void *W, *bias, *gain;
  float* Y; int ldy, N;
};
bool gemm_small_joins(const SmallGemm* g, int n, bool swiglu, int wdtype, int M, int K);
void launch_gemm_small(const SmallGemm* g, int n, bool swiglu, int wdtype, int M, int K, int mode, float eps, hipStream_t st);
void launch_swiglu(const float* g, const float* u, float* h, size_t n, hipStream_t st);
// nodes non-null: row b * n_lvl + r of the result goes to row b * R + nodes[b * stride + r] of out, and to cat[row][0 .. H-1]
struct AdNodes { const int* nodes; int n_lvl, R, stride; float* cat /*[rows, 2H]*/; };
void launch_ad_gate(const float* x, int ldx, const float* q, const float* k, const float* v, int H, int heads,
                    float* out, int rows, hipStream_t st, AdNodes to = AdNodes{});

// top-k of each row of z[rows, V] by (value desc, id asc); k <= CLOVER_MAX_RANK.
// cand: scratch [rows][chunks][16] of (float,int) pairs; out_ids [rows][16]; chunks = topk_chunks(V).
int topk_chunks(int V);
// tokens non-null: row b * n_lvl + r ranks node u = nodes[r] of sequence b, and tokens[b * R + c] = the row's id of rank[c] for each
// child c of u (rank[c] < k); sequences with m[b] < 1 are left alone
struct TopkChildren { const int *nodes, *first_child, *n_child, *rank, *m; int n_lvl, R; int* tokens; };
void launch_topk(const float* z, int ldz, int V, int rows, int k, void* cand, int* out_ids, hipStream_t st,
                 TopkChildren to = TopkChildren{});

// ---- draft-tree bookkeeping -------------------------------------------------------------------
// gather for level rows: row (b,r) <- node u = lvl_nodes[r]; xs = state[b][parent(u)], e = lm_head[token[b][u]]
// (nodes_stride / parent_stride: per-sequence strides of the index tables, 0 when all sequences share them)
void launch_draft_gather(const float* state, const int* tokens, const int* lvl_nodes, const int* parent, int n_lvl,
                         int B, int R, int H, const void* lm_head, int wdtype, int vocab, float* xs, float* e,
                         float* cat /*[rows,2H], second half <- e*/, hipStream_t st, int nodes_stride = 0,
                         int parent_stride = 0);
// root rows: xs_root[b] = a[b][m[b]-1]; state[b][0] = same; tokens[b][0] = next_tok[b][m[b]-1]; aug_len[b] += m[b]
// (Rs: row stride of state and tokens when it differs from R, the stride of a and next_tok)
void launch_draft_root(const float* a, const int* next_tok, const int* m, int B, int R, int H, float* root_x,
                       float* state, int* tokens, int* aug_len, hipStream_t st, int Rs = 0);
void launch_add_scalar(int* p, int v, hipStream_t st);   // *p += v

// ---- accept / compact -------------------------------------------------------------------------
void launch_accept_walk(const int* argmax, const int* tokens, const int* first_child, const int* n_child, int n_nodes,
                        int B, int R, const int* n_forced, const int* forced_next, int* m, int* acc_idx,
                        int* new_tokens, int* next_tok, int* seq_len /* += m */, hipStream_t st, int child_stride = 0);
// behind the walk (len includes m): K/V rows of the accepted nodes to their slots in every layer, hid_acc[b][i] = hidden[b][acc_idx[i]];
// m[b] <= max_rows
void launch_accept_move(void* k_cache, void* v_cache, int kvdtype, KVLayout kv, int n_layers, size_t layer_elems, const int* len,
                        const int* m, const int* acc_idx, int B, int R, int max_rows, const float* hidden, int H, float* hid_acc,
                        hipStream_t st);
void launch_read_kv(const void* k_cache, const void* v_cache, int kvdtype, KVLayout kv, int b, int slot0, int n_slots,
                    float* k_out, float* v_out, hipStream_t st);
void launch_write_kv(void* k_cache, void* v_cache, int kvdtype, KVLayout kv, int b, int slot0, int n_slots,
                     const float* k_in, const float* v_in, hipStream_t st);
void launch_fill_i32(int* p, int v, int n, hipStream_t st);

// ---- activation planes and partial-sum consumers ------------------------------------------------
void launch_split_planes(const float* x, int ldx, FragPlanes out, int rows, int K, hipStream_t st);
// Y[m,n] (=|+=) sum_s P[s*split_stride + m*ldp + n] (+ bias[n]);  mode 0 store, 1 add
void launch_reduce(const float* P, int splits, size_t split_stride, int ldp, const void* bias, int wdtype, float* Y,
                   int ldy, int M, int N, int mode, hipStream_t st);
// bf16 models: x[m,:] += sum_s P[s][m][:]  (splits may be 0); then, if gain: out[m,:] = planes of rmsnorm(x[m,:]) * gain
// bias non-null: x[m,:] = bias + sum_s P[s][m][:] (the old x is not read)
void launch_reduce_add_norm(float* x, int ldx, const float* P, int splits, size_t split_stride, int ldp,
                            const void* gain, float eps, FragPlanes out, int rows, int H,
                            hipStream_t st, const void* bias = nullptr);

// ---- MFMA tree attention (head_dim 128, caches as bf16 planes) ---------------------------------
// How the key tiles of a launch's sequences are dealt to workgroups.  Every sequence is cut into ranges of `tiles` key tiles, so a
// short one has fewer ranges than a long one; a unit is a (sequence, range).  With a table unit[u] = sequence | range << 8 | (the
// only range: 1) << 15, ranges[b] = ranges of sequence b; without (more sequences or units than it holds) all sequences have `most` ranges,
// those behind a sequence's last tile idle.
constexpr int ATTN_TAB = 256;
struct AttnUnits {
  int tiles, n_units, most, tab;
  unsigned short unit[ATTN_TAB];
};
struct AttnPlan : AttnUnits {
  unsigned char ranges[ATTN_TAB];        // (the merge's)
};
struct AttnParams {
  const bf16_t *q_hi, *q_lo; int ldq;    // [rows, n_q*128] planes: RoPE applied, scaled by 1/sqrt(128)
  const bf16_t *k, *v;                   // K and V^T planes of one layer (paged, see KVLayout)
  KVLayout kv;
  int max_seq, n_kv, n_q;
  const int* base_len;                   // dev [B]
  const unsigned long long* anc;         // dev [n][2]; null (and no interval labels): the nodes form a chain
  const int* iv;                         // dev [n][2] interval labels (enter, exit) of a depth-first numbering, or null:
                                         //   when given they decide visibility instead of the bit sets
  int anc_stride;                        // nodes per sequence in a per-sequence mask table, 0: one table for all
  RowMap rm;
  float* o_part;                         // [plan.most][rows_total][n_q][128]
  float* ml_part;                        // [plan.most][rows_total][n_q][2]
  int rows_total;
  FragPlanes out;                        // finished rows
  AttnUnits plan;
};
bool attn_mfma_supported(int head_dim, int n_q, int n_kv, int max_seq);
// keys[b]: host-side upper bound of base_len[b] + n for each of the B sequences of n rows; max_ranges: what the partial results
// have room for; chain: the rows form a chain
AttnPlan attn_plan(const int* keys, int B, int n, int n_kv, int n_q, bool chain, int max_ranges);
void launch_attn_mfma(AttnParams p, const AttnPlan& plan, hipStream_t st);

// ---- fragment-major weights and the GEMM that reads them ----------------------------------------
// [N,K] row-major bf16 -> rows row0 .. row0+N-1 of a packed matrix of n_rows rows, [K/32][n_rows/16][64 lanes][8]: lane
// l of block (kt, nb) holds row nb*16 + l%16, columns kt*32 + (l/16)*8 .. +7, so a matrix-instruction operand is one
// contiguous KB.  K steps outermost: the workgroups of a launch walk K side by side and so read one contiguous region
// at a time.  (Row blocks outermost, every workgroup reads at the same offset of its own power-of-two-sized blocks;
// gate+up at one row 43 -> 40 us, LM head 168 -> 164, 64 rows and more within noise.)
// rotary_d > 0: the rows of each head of that size in rotary order, so that a block of 16 holds 8 rows 8j .. of the head's first half and
// the 8 rows of the second half that are rotated with them.
void launch_pack_weight(const void* src, void* dst, int N, int K, int row0, int n_rows, hipStream_t st, int rotary_d = 0);
// gate and up, each [F,K], as one matrix of 2F rows: block b holds rows 8b .. 8b+7 of the gate, then those of the up
void launch_pack_gate_up(const void* gate, const void* up, void* dst, int F, int K, hipStream_t st);
// What the QKV projection's launch does with its sums: q and k rotated (half-split pairing), q out, k and v into the cache.  W holds the
// q and k rows of every head in rotary order (launch_pack_weight).
struct QkvOut {
  int n_q, d;                         // query heads; the caches' KV heads follow from kv
  bf16_t *q_hi, *q_lo; float q_scale; // planes of q * q_scale for the MFMA attention; q_hi null: fp32 q
  float* q; int ldq;
  bf16_t *kc, *vc; KVLayout kv;
  const float *cos_t, *sin_t;         // [rows][d / 2]
  const int* base_len; RowMap rm; int* err_flag;
};
struct TileGemm {
  FragPlanes X;                       // activations [M, K]
  const bf16_t* W;                    // packed [N, K]; epi 1: gate and up interleaved, [2N, K]
  float* Y; int ldy;                  // epi 0: fp32 [M, N]; range r of K writes Y + r * split_stride
  FragPlanes out;                     // epi 1: planes of silu(X Wg^T) * (X Wu^T), [M, N]
  int M, N, K;
  int epi;                            // 0 plain, 1 SwiGLU
  int k_parts; size_t split_stride;   // (split_stride: epi 0 only)
  int n_units;                        // filled in by launch_gemm_tile: column tiles x K ranges
};
// epi 3.  (Apart from the others, whose launches would otherwise carry the longer arguments: 0.2 us each.)
struct TileGemmQkv : TileGemm {
  QkvOut qkv;
  // over several ranges of K: their workgroups exchange partial tiles in `part` (tile_gemm_exchange_bytes) and finish the tile in
  // shares, and meet in `meet`, TILE_MEETINGS words MEET_STRIDE apart (zero before the first launch that uses them)
  float* part; unsigned* meet; int polls;
  // filled in by launch_gemm_qkv: row blocks of a row tile that has them all; 1: the ranges of a tile are on different XCDs
  int row_blocks, spread;
};
constexpr int TILE_MEETINGS = 256, MEET_STRIDE = 16;
constexpr int MEET_POLLS = 256;       // looks of a member at the word before it leaves its share to the last one (100 us or so)
void set_meet_polls(clover_ctx* x, int polls);   // of this context's launches
constexpr int TILE_MAX_K_PARTS = 8;
// K ranges of a narrow output; the same for all M that round up to the same multiple of 32
int tile_gemm_pick_k_parts(int M, int N, int K);
void launch_gemm_tile(const TileGemm& g, hipStream_t st);
// what launch_gemm_tile runs for M rows (N = F for epi 1; k_parts 0: its own choice)
struct TileForm { int rb, wb /* column blocks of 16 */, row_tiles, k_parts, stages; };
TileForm tile_gemm_form(int M, int N, int K, int epi, int k_parts);
// whether the QKV projection's launch rotates and stores by itself (epi 3; which form of it, if so) or leaves that to a second one
bool tile_gemm_qkv_joins(int M, int N, int K, int k_parts, bool mfma_attention, TileForm* form);
// bytes of `part` for M rows
size_t tile_gemm_exchange_bytes(const TileForm& t, int M, int N);
void launch_gemm_qkv(const TileGemmQkv& g, const TileForm& t, hipStream_t st);

// ---- fused bookkeeping kernels of the draft head (MFMA path, bf16 weights) ----------------------
// planes of RMSNorm(hid[row]) * gain -> a and of the embedding of tok[row] -> y, rows of `rm` in,
// row b * rm.n + i out, and its rotary table (for every i < rm.n)
void launch_draft_pre(const float* hid, const int* tok, const void* gain, float eps, const void* table, int vocab, int H,
                      RowMap rm, const RopeRows& rope, FragPlanes a, FragPlanes y, hipStream_t st);
// Attention-Decoder gate reading the q and (k|v) GEMMs' partial tiles and adding the biases itself
struct AdGateArgs {
  const float* x; int ldx;                    // residual input rows
  const float* Pq; int Sq; size_t sps_q;      // [Sq][M][H], Sq <= 8
  const float* Pkv; int Skv; size_t sps_kv;   // [Skv][M][2H]: k columns, then v columns, Skv <= 8
  const void *bq, *bk, *bv;                   // bf16 [H]
  int H, heads;
  const int *nodes, *parent; int n_lvl, R;    // nodes null: row g -> row g, read from row (g / n_lvl)*R + g % n_lvl if n_lvl > 0; else g = b*n_lvl + r, u = nodes[r]: row b*R+parent[u] -> row b*R+u
  int nodes_stride, parent_stride;            // per-sequence strides of nodes / parent (0: shared by all sequences)
  const int* m;                               // with nodes: sequences with m[b] < 1 are skipped (null: none)
  float* out; int ldo;
  const void* gain; float eps; FragPlanes norm;   // gain non-null: planes of RMSNorm(result)*gain, row g
  FragPlanes cat;                             // cat.p non-null: planes of the result, row g (columns 0 .. H-1)
};
bool ad_gate_fused_supported(int H, int heads);
void launch_ad_gate_fused(const AdGateArgs& a, int rows, hipStream_t st);
// root state/token from the last accepted row, its planes in row b of y, aug_len[b] += m[b]; R, Ra: rows per
// sequence of next_tok and of a
void launch_draft_root_fused(const float* a, const int* next_tok, const int* m, int B, int R, int Ra, int H, float* state,
                             int* tokens, FragPlanes y, int* aug_len, hipStream_t st, int Rs = 0);
// per internal node r of one depth (u = nodes[r]), row b*n_lvl + r: planes of RMSNorm(state[parent(u)]) * gain in a,
// planes of the embedding of tokens[u] in y and in columns H .. 2H-1 of cat
void launch_draft_level(const float* state, const int* tokens, const int* nodes, const int* parent, int n_lvl, int B,
                        int R, int H, const void* table, int vocab, const void* gain, float eps, FragPlanes a,
                        FragPlanes y, FragPlanes cat, hipStream_t st, int nodes_stride = 0, int parent_stride = 0);

// ---- dynamic (score-pruned) draft tree ----------------------------------------------------------
constexpr int DYN_MAX_CAND = 256;    // candidates per sequence, the root included
constexpr int DYN_MAX_FRONT = 64;    // candidates expanded per depth
struct DynTree {
  int C, D, topk, N;                       // candidates, depths, children per expansion, tree nodes
  int off[CLOVER_MAX_DEPTH + 2];           // candidates of depth j are [off[j], off[j + 1])
  int F[CLOVER_MAX_DEPTH + 1];             // candidates expanded at depth j (F[0] = 1: the root)
  int* cand_tok; float* cand_score; int* cand_par;   // dev [B][C]
  int* frontier;                           // dev [B][CLOVER_MAX_DEPTH][DYN_MAX_FRONT]: expanded candidates, best first
  int *t_parent, *t_rank, *t_depth, *t_first_child, *t_n_child, *t_keep;   // dev [B][R]: the tree as verified
  unsigned long long* t_anc;               // dev [B][R][2]
  int* t_iv;                               // dev [B][R][2]: interval labels (enter, exit) of the tree as verified
};
// log-sum-exp of each row of z[rows, V], every value multiplied by `scale` first (an inverse temperature).  cand:
// [rows][chunks][16] 64-bit keys, aux: [rows][chunks][2] floats, chunks = ceil(V / 2048)
// to non-null (k = to->topk): row b * F[j] + r ranks candidate frontier[b][j][r] by (value descending, id ascending); token, cumulative
// score and parent of its k children go to their candidates (sequences with m[b] < 1 are left alone)
void launch_topk_lse(const float* z, int ldz, int V, int rows, int k, void* cand, float* aux, float* out_lse, hipStream_t st,
                     float scale = 1.0f, const DynTree* to = nullptr, int j = 0, const int* m = nullptr);
// verification at a temperature > 0: lse[row] = log-sum-exp of logits[row] * inv_temp; uniforms [B][R][17]
int sample_chunks(int V);
void launch_accept_sample(const float* logits, int V, const float* lse, float inv_temp, const int* tokens,
                          const int* first_child, const int* n_child, int child_stride, int B, int R,
                          const float* uniforms, int* m, int* acc_idx, int* new_tokens, int* next_tok, int* seq_len /* += m */,
                          double* mass /* scratch, B * sample_chunks(V) */, hipStream_t st);
void launch_dyn_frontier(const DynTree& t, int j, int B, const int* m, hipStream_t st);
void launch_dyn_finalize(const DynTree& t, int B, int R, const int* m, int* tree_tokens, hipStream_t st);   // (also t.t_iv when set)

// ---- tuning knobs -------------------------------------------------------------------------------
// The shipped library reads no environment variable: every knob is its default.  A build with
// -DCLOVER_ABLATE (kernel-tuning experiments only) reads CLOVER_<NAME> at every use instead, so that one process can
// sweep them.
#ifdef CLOVER_ABLATE
int tune_int(const char* name, int dflt);
#else
inline int tune_int(const char*, int dflt) { return dflt; }
#endif

}  // namespace clv
