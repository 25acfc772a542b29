// C-ABI layer of libclover.so: context, validation, workspace carving and the kernel sequences of
// the three calls of a speculative step.  All arithmetic runs in the kernels this file launches.
#include "../../include/clover.h"
#include "clover_internal.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <string>
#include <utility>
#include <vector>

using namespace clv;

#ifdef CLOVER_ABLATE
#include <cstdlib>
namespace clv {
int tune_int(const char* name, int dflt) {
  const char* v = getenv(name);
  return v ? atoi(v) : dflt;
}
}  // namespace clv
#endif

namespace {

thread_local std::string g_err;

int op_gemm_impl(int32_t path, int32_t dtype, const float* X, const void* W, float* Y, int32_t ldy, int32_t M,
                 int32_t N, int32_t K, void* scratch, size_t scratch_bytes, void* hip_stream);

// Scratch of clover_op_gemm_static: one copy per GPU, held until the process ends.  In host code the name below is
// only a handle for hipGetSymbolAddress; every use goes through the per-device address looked up once.
// The limit that callers know counts M rows of activations; the array also holds the rows that pad them to a whole row
// block: at most 15 rows of 4 K bytes, K at most limit / 36 (one row and 16 columns).
constexpr size_t kStaticScratch = (size_t)CLOVER_STATIC_SCRATCH_BYTES + 15 * 4 * ((size_t)CLOVER_STATIC_SCRATCH_BYTES / 36);
__device__ __align__(256) unsigned char g_static_scratch[kStaticScratch];
constexpr int kMaxDevices = 64;
void* g_static_scratch_ptr[kMaxDevices] = {};
int static_scratch_ptr(void** out);

const char* kClassNames[KC_COUNT] = {"embed",     "rmsnorm",     "gemm_qkv",   "rope_kv_write", "tree_attention", "gemm_wo",
                                     "gemm_gate_up", "gemm_down", "gemm_lm_head", "gemm_draft",  "ad_gate",        "topk",
                                     "draft_misc", "accept_walk", "compact_kv", "eltwise"};

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct TreeHost {
  int n = 0, max_depth = 0;
  std::vector<int> parent, rank, depth, first_child, n_child;
  std::vector<int> lvl_nodes;           // internal nodes, grouped by depth
  std::vector<int> lvl_off;             // [max_depth+2]: internal nodes of depth j are lvl_nodes[lvl_off[j]..lvl_off[j+1])
  std::vector<int> kmax;                // per depth j: 1 + max rank among children of depth-j nodes
  std::vector<unsigned long long> anc;  // [n][2] (all zero for trees of more than 128 nodes: those use the labels)
  std::vector<int> iv;                  // [n][2] interval labels: enter, exit of a depth-first numbering
  bool is_chain = false;
};

struct ProfEvent {
  int cls;
  hipEvent_t a, b;
};

// The buffers over the rows of a pass.  Two sets share the same memory: one for the rows of a step, all of it side by side with
// what drafting and ranking need, and one for the longer passes of a prompt (carve).
struct RowBufs {
  int rows;                // their capacity
  float *xd, *a_norm, *qkv, *q_rot, *attn_out, *h_ffn, *tmp_ffn, *cos_t, *sin_t, *ad_q, *ad_k, *ad_v, *d_xs, *d_e;
  float* pl_y;             // planes of draft-side GEMM inputs
  float* partial;          // partial tiles of the MFMA GEMMs over K ranges
  float *o_part, *ml_part; // partial results of the MFMA attention
  size_t split_rows;       // rows times key splits that they hold
};

}  // namespace

struct clover_ctx : RowBufs {
  clover_config cfg;
  hipStream_t st;
  clover_weights w;
  std::vector<clover_layer_weights> layers, aug;
  std::vector<const void*> fc_w, fc_b;
  TreeHost tree;
  std::string err;
  // sizes
  int R, H, QKVN, NQD;
  RowBufs step, pass;      // clover_prefill works on `pass`, every other call on `step`
  KVLayout kv;
  size_t k_layer_elems, v_layer_elems, esz, kv_esz;
  int kvdtype;  // 0: fp32 cache elements; 1: (hi, lo) bf16 planes, same bytes (a random-init 32-layer stack amplifies
                // plain bf16 cache rounding ~20x, so 16 mantissa bits are kept either way)
  size_t kv_layer_stride;  // cache elements (of the kvdtype's element type) per layer
  bool attn_fast;
  // device regions
  int *d_seq_len, *d_aug_len, *d_err;
  int *d_depth, *d_parent, *d_rank, *d_first_child, *d_n_child, *d_lvl_nodes;
  unsigned* d_meet;        // meetings of the workgroups that share a GEMM tile
  int meet_polls;          // looks of one of them before it leaves its share to the last
  unsigned long long* d_anc;
  int* d_pages;            // page table [max_batch][max_seq / KV_PAGE] (used once clover_set_page_table was called)
  int* d_iv;               // interval labels of the static tree [R][2]
  bool interval;           // CLOVER_FLAG_INTERVAL_MASK: tree attention reads the labels instead of the bit sets
  char *kc, *vc, *aug_kc, *aug_vc;
  float *d_cat, *d_g, *d_state, *d_rootx, *z;
  void* cand;
  int* topk_ids;
  char* packed;            // fragment-major copies of every linear weight (MFMA path)
  size_t packed_bytes;
  const void* lm_head_pk;
  bool fast;               // bf16 model on the MFMA path
  // dynamic (score-pruned) tree: candidates, frontiers and the per-sequence topology tables
  bool dyn_on = false;
  DynTree dyn{};
  float *topk_lse, *topk_aux;
  float* dyn_state;        // [B][DYN_MAX_CAND][H] draft states of the expanded candidates
  float* draft_capture = nullptr;   // test hook: device buffer that receives every depth's draft logits
  size_t draft_capture_floats = 0;
  // host-side bounds
  std::vector<int> len_ub, aug_ub;
  int m_upper;
  bool only_prefills;   // no accept call since init / reset: every pending hand-off has m = 1
  // profiling
  bool prof = false;
  std::vector<ProfEvent> prof_events;
  std::vector<ProfEvent> prof_pool;
};

// (test hook: with 0 nearly every member leaves its share to the last arrival)
void clv::set_meet_polls(clover_ctx* x, int polls) { x->meet_polls = polls; }

namespace {

int fail(clover_ctx* ctx, int code, const std::string& msg) {
  if (ctx) ctx->err = msg; else g_err = msg;
  return code;
}

int check_config(const clover_config* c, std::string& why) {
  auto bad = [&](const char* m) { why = m; return CLOVER_E_CONFIG; };
  if (c->n_layers < 1 || c->hidden < 1 || c->n_q_heads < 1 || c->n_kv_heads < 1 || c->ffn < 1) return bad("non-positive model dimension");
  if (c->head_dim != 64 && c->head_dim != 128) return bad("head_dim must be 64 or 128");
  if (c->n_q_heads % c->n_kv_heads != 0) return bad("n_q_heads must be a multiple of n_kv_heads");
  if (c->ad_heads < 1 || c->hidden % c->ad_heads != 0) return bad("hidden must be a multiple of ad_heads");
  if (c->hidden % 4 != 0 || c->ffn % 4 != 0) return bad("hidden and ffn must be multiples of 4");
  if (c->vocab < 16 || c->vocab > 262144) return bad("vocab must be in [16, 262144]");
  if (c->dtype != CLOVER_DTYPE_F32 && c->dtype != CLOVER_DTYPE_BF16) return bad("unknown dtype");
  if (c->aug_layers < 1 || c->aug_layers > 8) return bad("aug_layers must be in [1, 8]");
  if (c->draft_depths < 1 || c->draft_depths > CLOVER_MAX_DEPTH) return bad("draft_depths out of range");
  if (c->max_batch < 1 || c->max_batch > 1024) return bad("max_batch out of range");
  if (c->max_seq % KV_PAGE != 0) return bad("max_seq must be a multiple of 32 (the page size of the caches)");
  if (c->max_nodes < 1 || c->max_nodes > ((c->flags & CLOVER_FLAG_INTERVAL_MASK) ? CLOVER_MAX_NODES_INTERVAL : CLOVER_MAX_NODES))
    return bad("max_nodes must be in [1, 128] (in [1, 256] with CLOVER_FLAG_INTERVAL_MASK)");
  if (c->prefill_rows < 0 || c->prefill_rows > CLOVER_MAX_PREFILL_ROWS) return bad("prefill_rows must be in [0, 256]");
  if (c->max_seq < c->max_nodes) return bad("max_seq smaller than max_nodes");
  if (!(c->rope_base > 1.f) || !(c->rms_eps > 0.f)) return bad("rope_base must be > 1 and rms_eps > 0");
  return CLOVER_OK;
}

int build_tree(const clover_config& cfg, const clover_tree* t, TreeHost& out, std::string& why) {
  auto bad = [&](const char* m) { why = m; return CLOVER_E_TREE; };
  if (!t->parent || !t->rank) { why = "tree arrays are null"; return CLOVER_E_NULL; }
  const int n = t->n_nodes;
  if (n < 1 || n > cfg.max_nodes) return bad("n_nodes outside [1, max_nodes]");
  if (t->parent[0] != -1) return bad("parent[0] must be -1");
  TreeHost h;
  h.n = n;
  h.parent.assign(t->parent, t->parent + n);
  h.rank.assign(t->rank, t->rank + n);
  h.depth.assign(n, 0);
  h.first_child.assign(n, 0);
  h.n_child.assign(n, 0);
  for (int u = 1; u < n; ++u) {
    const int p = h.parent[u];
    if (p < 0 || p >= u) return bad("parent index must satisfy 0 <= parent[u] < u");
    if (u >= 2 && p < h.parent[u - 1]) return bad("nodes must be in breadth-first order (parent non-decreasing)");
    if (h.rank[u] < 0 || h.rank[u] >= CLOVER_MAX_RANK) return bad("rank outside [0, 16)");
    h.depth[u] = h.depth[p] + 1;
    if (h.n_child[p] == 0) h.first_child[p] = u;
    h.n_child[p]++;
  }
  for (int u = 0; u < n; ++u) {
    unsigned seen = 0;
    for (int c = h.first_child[u]; c < h.first_child[u] + h.n_child[u]; ++c) {
      if (seen & (1u << h.rank[c])) return bad("siblings must have distinct ranks");
      seen |= 1u << h.rank[c];
    }
  }
  h.max_depth = h.depth[n - 1];
  h.is_chain = true;
  for (int u = 1; u < n; ++u) h.is_chain = h.is_chain && (h.parent[u] == u - 1);
  h.lvl_off.assign(h.max_depth + 2, 0);
  h.kmax.assign(h.max_depth + 1, 0);
  for (int j = 0; j <= h.max_depth; ++j) {
    h.lvl_off[j] = (int)h.lvl_nodes.size();
    for (int u = 0; u < n; ++u) {
      if (h.depth[u] != j) continue;
      if (h.n_child[u] > 0) {
        h.lvl_nodes.push_back(u);
        for (int c = h.first_child[u]; c < h.first_child[u] + h.n_child[u]; ++c) h.kmax[j] = std::max(h.kmax[j], h.rank[c] + 1);
      }
    }
  }
  h.lvl_off[h.max_depth + 1] = (int)h.lvl_nodes.size();
  for (int u = 1; u < n; ++u)
    if (h.depth[u] < h.depth[u - 1]) return bad("depth must be non-decreasing");
  h.anc.assign((size_t)2 * n, 0ull);
  for (int u = 0; u < n && n <= CLOVER_MAX_NODES; ++u) {
    if (u > 0) { h.anc[2 * u] = h.anc[2 * h.parent[u]]; h.anc[2 * u + 1] = h.anc[2 * h.parent[u] + 1]; }
    h.anc[2 * u + (u >> 6)] |= 1ull << (u & 63);
  }
  // interval labels (Appendix A.1, linear-size mask): subtree sizes bottom-up (children have larger indices), then
  // enter[child] = enter[parent] + 1 + sizes of the earlier siblings; exit = enter + size - 1
  {
    std::vector<int> size(n, 1);
    for (int u = n - 1; u >= 1; --u) size[h.parent[u]] += size[u];
    h.iv.assign((size_t)2 * n, 0);
    for (int u = 0; u < n; ++u) {
      int e = h.iv[2 * u] + 1;
      for (int c = h.first_child[u]; c < h.first_child[u] + h.n_child[u]; ++c) { h.iv[2 * c] = e; e += size[c]; }
      h.iv[2 * u + 1] = h.iv[2 * u] + size[u] - 1;
    }
  }
  out = std::move(h);
  return CLOVER_OK;
}

// ---- workspace carving ---------------------------------------------------------------------
struct Carver {
  char* base;
  size_t off = 0;
  template <typename T>
  T* take(size_t count) {
    T* p = base ? (T*)(base + off) : nullptr;
    off = align256(off + count * sizeof(T));
    return p;
  }
};

struct GemmShape { int N, K; };

// every GEMM of the MFMA path that writes partial tiles
void model_gemm_shapes(const clover_config& c, std::vector<GemmShape>& v) {
  const int H = c.hidden, nqd = c.n_q_heads * c.head_dim, qkvn = (c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim;
  v = {{qkvn, H}, {H, nqd}, {H, c.ffn}, {H, H}, {H, 2 * H}};
}
bool mfma_shape_ok(int N, int K) { return N % 16 == 0 && K % 128 == 0; }

// Bytes of the partial tiles of launches over up to a number of rows: QKV and Wo, down, the projections of an Attention Decoder
// (q and k|v lie side by side), the draft head's FC.
struct TileBytes {
  size_t attn = 0, down = 0, ad = 0, fc = 0;
  size_t most() const { return std::max(std::max(attn, down), std::max(ad, fc)); }
};
// for up to 32, 64 .. rows
std::vector<TileBytes> tile_bytes(const clover_config& c, int rows) {
  std::vector<GemmShape> s;
  model_gemm_shapes(c, s);   // QKV, Wo, down, an Attention Decoder's q, the FC
  std::vector<TileBytes> v;
  TileBytes t{256, 256, 256, 256};
  const bool mfma_attention = attn_mfma_supported(c.head_dim, c.n_q_heads, c.n_kv_heads, c.max_seq);
  for (int M = 32; M < rows + 32; M += 32) {   // one row count of each class of equal K ranges
    auto bytes = [&](int N, int K) {   // (a tuning build that changes the ranges afterwards makes room for them here)
      return (size_t)std::max(tile_gemm_pick_k_parts(M, N, K), tune_int("CLOVER_TILE_KP_ROOM", 1)) * std::min(M, rows) * N * sizeof(float);
    };
    auto exchanged = [&](int N, int K) {
      const int m = std::min(M, rows), room = tune_int("CLOVER_TILE_KP_ROOM", 1);
      if (room > 1) return tile_gemm_exchange_bytes(tile_gemm_form(m, N, K, 0, std::max(tile_gemm_pick_k_parts(m, N, K), room)), m, N);
      TileForm form;
      const bool joins = tile_gemm_qkv_joins(m, N, K, tile_gemm_pick_k_parts(m, N, K), mfma_attention, &form);
      return joins ? tile_gemm_exchange_bytes(form, m, N) : 0;
    };
    t.attn = std::max({t.attn, bytes(s[0].N, s[0].K), exchanged(s[0].N, s[0].K), bytes(s[1].N, s[1].K)});
    t.down = std::max(t.down, bytes(s[2].N, s[2].K));
    t.ad = std::max(t.ad, align256(bytes(s[3].N, s[3].K)) + bytes(2 * c.hidden, c.hidden));
    t.fc = std::max(t.fc, bytes(s[4].N, s[4].K));
    v.push_back(t);
  }
  return v;
}

// The layout of a prompt pass of `rows` rows: what is alive at the same time side by side, the rest on top of each other.
// Returns its bytes.
size_t carve_pass(const clover_ctx* x, char* base, int rows, const TileBytes& t, RowBufs& b) {
  const clover_config& c = x->cfg;
  Carver cv{base};
  const size_t H = c.hidden, rows16 = ((size_t)rows + 15) / 16 * 16;
  const bool fused = x->fast && ad_gate_fused_supported(c.hidden, c.ad_heads);
  b = RowBufs{};
  b.rows = rows;
  b.cos_t = cv.take<float>((size_t)rows * c.head_dim / 2);
  b.sin_t = cv.take<float>((size_t)rows * c.head_dim / 2);
  b.d_xs = cv.take<float>(rows * H);
  b.xd = fused ? b.d_xs : cv.take<float>(rows * H);   // (the fused gate kernel writes where it read)
  b.a_norm = cv.take<float>(rows16 * H);
  // attention | FFN | Attention Decoder 1, each behind its own partial tiles
  Carver at = cv, ff = cv, ad = cv;
  b.partial = (float*)at.take<char>(t.attn);
  ff.take<char>(t.down);
  ad.take<char>(t.ad);
  b.h_ffn = ff.take<float>(rows16 * c.ffn);
  if (!x->fast) b.tmp_ffn = ff.take<float>((size_t)rows * c.ffn);
  b.d_e = ad.take<float>(rows * H);
  if (x->fast) b.pl_y = ad.take<float>(rows16 * H);
  if (!fused)
    for (float** p : {&b.ad_q, &b.ad_k, &b.ad_v}) *p = ad.take<float>(rows * H);
  auto attention = [&](Carver& a) {
    if (!x->fast) b.qkv = a.take<float>((size_t)rows * x->QKVN);
    b.q_rot = a.take<float>((size_t)rows * x->NQD);
    b.attn_out = a.take<float>(rows16 * x->NQD);
  };
  const size_t tiles_end = at.off;
  attention(at);
  const size_t end = std::max(at.off, std::max(ff.off, ad.off));
  // The attention's partial results lie on the projection's partial tiles, which are summed by then, and on what is free
  // behind them: its own rows stand at the end.
  Carver rows_at{base, end - (at.off - tiles_end)};
  const size_t room = rows_at.off - cv.off;
  attention(rows_at);
  b.split_rows = x->attn_fast ? (room - 256) / (sizeof(float) * (x->NQD + 2 * c.n_q_heads)) : 0;
  b.o_part = b.partial;
  b.ml_part = base ? (float*)((char*)b.partial + align256(b.split_rows * x->NQD * sizeof(float))) : nullptr;
  return end;
}

// Rows of a prompt pass: as many as the memory of a step's buffers holds, up to 2048, where the narrow GEMMs (QKV, Wo, down) fill
// the chip without ranges of K and every weight byte staged serves 256 rows.  (8B shape, step buffers of 256 rows: 2048.)  Per
// 256 rows and layer there in passes of 256 / 2048 rows: gate+up 91 / 75 us, QKV, Wo and down with the kernels behind them
// 125 / 75.
void carve_passes(clover_ctx* x, char* base, size_t bytes) {
  const int most = std::min(2048, x->cfg.max_seq), own = std::min(x->step.rows, std::min(most, 256));
  const std::vector<TileBytes> tiles = x->fast ? tile_bytes(x->cfg, most) : std::vector<TileBytes>(most / 32);
  int rows = most;
  while (rows > own && carve_pass(x, nullptr, rows, tiles[rows / 32 - 1], x->pass) > bytes)
    rows = rows > 256 ? (rows - 1) / 256 * 256 : (rows - 1) / 32 * 32;
  if (rows > own) carve_pass(x, base, rows, tiles[rows / 32 - 1], x->pass);
  else carve_pass(x, base, own, x->fast ? tile_bytes(x->cfg, own).back() : TileBytes{}, x->pass);   // (a part of the step's: fits)
}

// Bytes that a step has no use for, so that prompt passes are longer: a row of the residual stream per row.  Without them 29 of
// 500 configurations have shorter passes (hidden 4096, 32 KV heads, 2 x 32 nodes: 256 rows instead of 512; hidden 5120, 128 nodes: 768
// instead of 1024).
size_t pass_room(const clover_config& c, int rows) { return (size_t)rows * c.hidden * sizeof(float); }

void carve(clover_ctx* x, char* base, size_t* total) {
  const clover_config& c = x->cfg;
  Carver cv{base};
  const int B = c.max_batch, R = c.max_nodes, H = c.hidden, d = c.head_dim;
  const int rows = std::max(B * R, c.prefill_rows);   // row capacity of every activation buffer
  const size_t rows16 = (size_t)(rows + 15) / 16 * 16;   // of those that hold planes in fragment order (whole row blocks)
  const size_t esz = c.dtype == CLOVER_DTYPE_F32 ? 4 : 2;
  x->R = R; x->H = H; x->esz = esz;
  x->kv_esz = 4;  // bytes per cached value in both formats
  x->NQD = c.n_q_heads * d;
  x->QKVN = (c.n_q_heads + 2 * c.n_kv_heads) * d;
  x->k_layer_elems = (size_t)B * c.max_seq * c.n_kv_heads * d;
  x->d_pages = cv.take<int>((size_t)B * (c.max_seq / KV_PAGE));
  x->kv = KVLayout{B, c.max_seq, c.n_kv_heads, d, 1, 0, c.max_seq / KV_PAGE, 0, nullptr};
  x->v_layer_elems = x->k_layer_elems;
  x->d_seq_len = cv.take<int>(B);
  x->d_aug_len = cv.take<int>(B);
  x->d_err = cv.take<int>(1);
  x->d_depth = cv.take<int>(R);
  x->d_parent = cv.take<int>(R);
  x->d_rank = cv.take<int>(R);
  x->d_first_child = cv.take<int>(R);
  x->d_n_child = cv.take<int>(R);
  x->d_lvl_nodes = cv.take<int>(R);
  x->d_anc = cv.take<unsigned long long>(2 * R);
  x->d_iv = cv.take<int>(2 * R);
  x->kc = cv.take<char>(x->k_layer_elems * x->kv_esz * c.n_layers);
  x->vc = cv.take<char>(x->v_layer_elems * x->kv_esz * c.n_layers);
  x->aug_kc = cv.take<char>(x->k_layer_elems * x->kv_esz * c.aug_layers);
  x->aug_vc = cv.take<char>(x->v_layer_elems * x->kv_esz * c.aug_layers);
  x->cand = cv.take<unsigned long long>((size_t)rows * topk_chunks(c.vocab) * 16);
  x->topk_ids = cv.take<int>((size_t)rows * 16);
  x->dyn.cand_tok = cv.take<int>((size_t)B * DYN_MAX_CAND);
  x->dyn.cand_score = cv.take<float>((size_t)B * DYN_MAX_CAND);
  x->dyn.cand_par = cv.take<int>((size_t)B * DYN_MAX_CAND);
  x->dyn.frontier = cv.take<int>((size_t)B * CLOVER_MAX_DEPTH * DYN_MAX_FRONT);
  x->dyn.t_parent = cv.take<int>((size_t)rows);
  x->dyn.t_rank = cv.take<int>((size_t)rows);
  x->dyn.t_depth = cv.take<int>((size_t)rows);
  x->dyn.t_first_child = cv.take<int>((size_t)rows);
  x->dyn.t_n_child = cv.take<int>((size_t)rows);
  x->dyn.t_keep = cv.take<int>((size_t)rows);
  x->dyn.t_anc = cv.take<unsigned long long>((size_t)rows * 2);
  x->dyn.t_iv = cv.take<int>((size_t)rows * 2);
  // MFMA path: is every GEMM shape of this model supported?
  bool fast = c.dtype == CLOVER_DTYPE_BF16 && !(c.flags & CLOVER_FLAG_GENERIC);
  if (fast) {
    std::vector<GemmShape> shapes;
    model_gemm_shapes(c, shapes);
    for (const GemmShape& s : shapes) fast = fast && mfma_shape_ok(s.N, s.K);
    fast = fast && mfma_shape_ok(c.ffn, H) && mfma_shape_ok(c.vocab, H);
    fast = fast && (c.n_kv_heads * d) % 16 == 0;
  }
  size_t packed_bytes = 0;
  if (fast) {
    const size_t layer_elems = (size_t)x->QKVN * H + (size_t)H * x->NQD + (size_t)3 * c.ffn * H;
    packed_bytes = 2 * ((size_t)(c.n_layers + c.aug_layers) * layer_elems + (size_t)c.vocab * H + (size_t)7 * H * H +
                        (size_t)(c.draft_depths - 1) * 2 * H * H);
  }
  x->packed_bytes = packed_bytes;
  x->packed = cv.take<char>(packed_bytes ? packed_bytes : 256);
  x->fast = fast;
  x->kvdtype = fast ? 1 : 0;
  x->kv.planes = fast ? 2 : 1;
  x->kv.plane = fast ? (size_t)KV_PAGE * d : 0;
  x->kv_layer_stride = fast ? 2 * x->k_layer_elems : x->k_layer_elems;
  x->attn_fast = fast && attn_mfma_supported(d, c.n_q_heads, c.n_kv_heads, c.max_seq);
  // From here on nothing outlives the call that wrote it, so a prompt pass may lay it out in its own way.
  const size_t own = cv.off;
  RowBufs& b = x->step;
  b.rows = rows;
  b.xd = cv.take<float>((size_t)rows * H);
  b.a_norm = cv.take<float>(rows16 * H);
  b.qkv = cv.take<float>((size_t)rows * x->QKVN);
  b.q_rot = cv.take<float>((size_t)rows * x->NQD);
  b.attn_out = cv.take<float>(rows16 * x->NQD);
  b.h_ffn = cv.take<float>(rows16 * c.ffn);
  b.tmp_ffn = cv.take<float>((size_t)rows * c.ffn);
  b.cos_t = cv.take<float>((size_t)rows * d / 2);
  b.sin_t = cv.take<float>((size_t)rows * d / 2);
  b.ad_q = cv.take<float>((size_t)rows * H);
  b.ad_k = cv.take<float>((size_t)rows * H);
  b.ad_v = cv.take<float>((size_t)rows * H);
  b.d_xs = cv.take<float>((size_t)rows * H);
  b.d_e = cv.take<float>((size_t)rows * H);
  x->d_cat = cv.take<float>(rows16 * 2 * H);
  x->d_g = cv.take<float>((size_t)rows * H);
  cv.take<char>(pass_room(c, rows));
  x->d_state = cv.take<float>((size_t)rows * H);
  x->d_rootx = cv.take<float>((size_t)B * H);
  x->z = cv.take<float>((size_t)rows * c.vocab);
  x->topk_lse = cv.take<float>((size_t)rows);
  x->topk_aux = cv.take<float>(std::max((size_t)rows * topk_chunks(c.vocab), (size_t)B * sample_chunks(c.vocab)) * 2);
  x->dyn_state = cv.take<float>((size_t)B * DYN_MAX_CAND * H);
  const size_t splits = 16;
  b.split_rows = splits * rows;
  b.o_part = cv.take<float>(x->attn_fast ? splits * rows * x->NQD : 64);
  b.ml_part = cv.take<float>(x->attn_fast ? splits * rows * c.n_q_heads * 2 : 64);
  b.partial = (float*)cv.take<char>(fast ? tile_bytes(c, rows).back().most() : 256);
  b.pl_y = cv.take<float>(rows16 * 2 * H);
  static_cast<RowBufs&>(*x) = b;
  if (base) carve_passes(x, base + own, cv.off - own);
  x->d_meet = cv.take<unsigned>(TILE_MEETINGS * MEET_STRIDE);   // (behind what passes lay out: it outlives them)
  *total = cv.off;
}

// the buffers of prompt passes, for as long as this lives
struct PassBufs {
  clover_ctx* x;
  explicit PassBufs(clover_ctx* ctx) : x(ctx) { static_cast<RowBufs&>(*x) = x->pass; }
  ~PassBufs() { static_cast<RowBufs&>(*x) = x->step; }
};

// ---- profiling ------------------------------------------------------------------------------
struct Scope {
  clover_ctx* x;
  ProfEvent ev;
  bool on;
  Scope(clover_ctx* ctx, int cls) : x(ctx), on(ctx->prof) {
    if (!on) return;
    if (!x->prof_pool.empty()) { ev = x->prof_pool.back(); x->prof_pool.pop_back(); }
    else { hipEventCreate(&ev.a); hipEventCreate(&ev.b); }
    ev.cls = cls;
    hipEventRecord(ev.a, x->st);
  }
  ~Scope() {
    if (!on) return;
    hipEventRecord(ev.b, x->st);
    x->prof_events.push_back(ev);
  }
};

// ---- GEMM dispatch ----------------------------------------------------------------------------
// MFMA path: part[r][M][N] = X W^T over K range r (default: x->partial).  Returns the number of ranges.
int gemm_fast(clover_ctx* x, int cls, FragPlanes X, const void* W, int M, int N, int K, float* part = nullptr) {
  Scope sc(x, cls);
  TileGemm g;
  memset(&g, 0, sizeof(g));
  g.X = X;
  g.W = (const bf16_t*)W;
  g.Y = part ? part : x->partial; g.ldy = N; g.split_stride = (size_t)M * N;
  g.M = M; g.N = N; g.K = K; g.epi = 0;
  g.k_parts = tile_gemm_pick_k_parts(M, N, K);
  launch_gemm_tile(g, x->st);
  return g.k_parts;
}
// Y = X W^T + bias through the MFMA path, for the small draft-side linears
void linear_fast(clover_ctx* x, FragPlanes X, const void* W, const void* bias, float* Y, int ldy, int M, int N, int K) {
  const int sp = gemm_fast(x, KC_GEMM_DRAFT, X, W, M, N, K);
  Scope sc(x, KC_ELTWISE);
  launch_reduce(x->partial, sp, (size_t)M * N, N, bias, x->cfg.dtype, Y, ldy, M, N, 0, x->st);
}
FragPlanes split_to(clover_ctx* x, const float* src, int ld, float* planes_buf, int rows, int K) {
  FragPlanes P = frag_planes(planes_buf, rows);
  Scope sc(x, KC_ELTWISE);
  launch_split_planes(src, ld, P, rows, K, x->st);
  return P;
}

// generic path: Y = X W^T (+bias), mode 1 adds into Y
void gemm_generic(clover_ctx* x, int cls, const float* X, int ldx, const void* W, const void* bias, float* Y, int ldy,
                  int M, int N, int K, int mode) {
  Scope sc(x, cls);
  launch_gemm_generic(X, ldx, W, bias, x->cfg.dtype, Y, ldy, M, N, K, mode, x->st);
}

// The split of the MFMA attention over the sequences of `rm` (M rows in all) behind at most cached[b] keys each.
AttnPlan plan_attention(clover_ctx* x, const int* cached, const RowMap& rm, int M, bool chain) {
  if (!x->attn_fast) return AttnPlan{};
  std::vector<int> keys(rm.B);
  for (int b = 0; b < rm.B; ++b) keys[b] = cached[b] + rm.n;
  return attn_plan(keys.data(), rm.B, rm.n, x->cfg.n_kv_heads, x->cfg.n_q_heads, chain, (int)(x->split_rows / M));
}

// One LLaMA decoder layer over the rows of `rm` (residual stream xres, leading dimension H).
// MFMA path: on entry the planes of a_norm hold RMSNorm(xres) * attn_norm of this layer; on exit they
// hold RMSNorm(xres) * next_gain (skipped when next_gain is null).  Generic path: norms are computed here.
void run_layer(clover_ctx* x, const clover_layer_weights& lw, float* xres, RowMap rm, int M, char* kc_layer,
               char* vc_layer, const int* base_len, const unsigned long long* anc, const void* next_gain,
               const AttnPlan& attn /* of the MFMA attention */, int anc_stride = 0 /* nodes per sequence in a per-sequence mask table */,
               const int* iv = nullptr /* interval labels: decide visibility instead of anc */,
               int seq0 = 0 /* the rows belong to sequence seq0 + (their index in rm) */) {
  const clover_config& c = x->cfg;
  KVLayout kvl = x->kv;
  kvl.b0 = seq0;
  const int H = x->H, d = c.head_dim, F = c.ffn;
  const int sn[3] = {c.n_q_heads * d, c.n_kv_heads * d, c.n_kv_heads * d};
  const void* ws[3] = {lw.wq, lw.wk, lw.wv};
  if (x->fast) {
    const FragPlanes A = frag_planes(x->a_norm, M), O = frag_planes(x->attn_out, M), Hf = frag_planes(x->h_ffn, M);
    bf16_t* const q_hi = (bf16_t*)x->q_rot;
    bf16_t* const q_lo = q_hi + (size_t)x->rows * x->NQD;
    const int sq = tile_gemm_pick_k_parts(M, x->QKVN, H);
    TileForm form;
    if (tile_gemm_qkv_joins(M, x->QKVN, H, sq, x->attn_fast, &form)) {
      Scope s(x, KC_GEMM_QKV);
      TileGemmQkv g;
      memset(&g, 0, sizeof(g));
      g.X = A;
      g.W = (const bf16_t*)lw.wq;   // q, k and v rows
      g.M = M; g.N = x->QKVN; g.K = H;
      g.part = x->partial; g.meet = x->d_meet; g.polls = x->meet_polls;
      g.qkv = QkvOut{c.n_q_heads, d, x->attn_fast ? q_hi : nullptr, q_lo, 1.0f / sqrtf((float)d), x->q_rot, x->NQD,
                     (bf16_t*)kc_layer, (bf16_t*)vc_layer, kvl, x->cos_t, x->sin_t, base_len, rm, x->d_err};
      launch_gemm_qkv(g, form, x->st);
    } else {
      gemm_fast(x, KC_GEMM_QKV, A, lw.wq, M, x->QKVN, H);
      Scope s(x, KC_ROPE_KV);
      const size_t stride = (size_t)M * x->QKVN;
      bf16_t *const kc = (bf16_t*)kc_layer, *const vc = (bf16_t*)vc_layer;
      if (x->attn_fast)
        launch_rope_kv_planes(x->partial, x->QKVN, sq, stride, x->cos_t, x->sin_t, kc, vc, kvl, base_len, c.n_q_heads, rm, x->d_err, q_hi, q_lo,
                              x->NQD, 1.0f / sqrtf((float)d), x->st);
      else
        launch_rope_kv_parts(x->partial, x->QKVN, sq, stride, x->cos_t, x->sin_t, x->q_rot, x->NQD, kc, vc, kvl, base_len, c.n_q_heads, rm,
                             x->d_err, x->st);
    }
    { Scope s(x, KC_ATTN);
      if (x->attn_fast) {
        AttnParams ap;
        memset(&ap, 0, sizeof(ap));
        ap.q_hi = q_hi; ap.q_lo = q_lo; ap.ldq = x->NQD;
        ap.k = (const bf16_t*)kc_layer; ap.v = (const bf16_t*)vc_layer;
        ap.kv = kvl; ap.max_seq = c.max_seq; ap.n_kv = c.n_kv_heads; ap.n_q = c.n_q_heads;
        ap.base_len = base_len; ap.anc = anc; ap.iv = iv; ap.anc_stride = anc_stride; ap.rm = rm;
        ap.o_part = x->o_part; ap.ml_part = x->ml_part; ap.rows_total = M; ap.out = O;
        launch_attn_mfma(ap, attn, x->st);
      } else {
        launch_attn_generic(x->q_rot, x->NQD, kc_layer, vc_layer, x->kvdtype, kvl, base_len, anc, c.n_q_heads, nullptr,
                            x->NQD, O, rm, x->st, anc_stride, iv);
      } }
    const int sw = gemm_fast(x, KC_GEMM_WO, O, lw.wo, M, H, x->NQD);
    { Scope s(x, KC_RMSNORM);
      launch_reduce_add_norm(xres, H, x->partial, sw, (size_t)M * H, H, lw.ffn_norm, c.rms_eps, A, M, H, x->st); }
    { Scope s(x, KC_GEMM_GATEUP);
      TileGemm g;
      memset(&g, 0, sizeof(g));
      g.X = A;
      g.W = (const bf16_t*)lw.w_gate;   // gate and up rows interleaved
      g.out = Hf;
      g.M = M; g.N = F; g.K = H; g.epi = 1; g.k_parts = 1;
      launch_gemm_tile(g, x->st); }
    const int sd = gemm_fast(x, KC_GEMM_DOWN, Hf, lw.w_down, M, H, F);
    { Scope s(x, KC_RMSNORM);
      launch_reduce_add_norm(xres, H, x->partial, sd, (size_t)M * H, H, next_gain, c.rms_eps, A, M, H, x->st); }
    return;
  }
  // (few rows: the norm and the three projections in one launch, below the norm, both projections and SwiGLU)
  SmallGemm g3[3];
  for (int sgm = 0, off = 0; sgm < 3; off += sn[sgm++]) g3[sgm] = SmallGemm{xres, H, ws[sgm], nullptr, lw.attn_norm, x->qkv + off, x->QKVN, sn[sgm]};
  if (gemm_small_joins(g3, 3, false, c.dtype, M, H)) {
    Scope s(x, KC_GEMM_QKV);
    launch_gemm_small(g3, 3, false, c.dtype, M, H, 0, c.rms_eps, x->st);
  } else {
    { Scope s(x, KC_RMSNORM); launch_rmsnorm(xres, H, lw.attn_norm, c.dtype, c.rms_eps, x->a_norm, H, H, M, x->st); }
    for (int sgm = 0, off = 0; sgm < 3; off += sn[sgm++])
      gemm_generic(x, KC_GEMM_QKV, x->a_norm, H, ws[sgm], nullptr, x->qkv + off, x->QKVN, M, sn[sgm], H, 0);
  }
  { Scope s(x, KC_ROPE_KV);
    launch_rope_kv_write(x->qkv, x->QKVN, x->cos_t, x->sin_t, x->q_rot, x->NQD, (float*)kc_layer, (float*)vc_layer, kvl, base_len,
                         c.n_q_heads, rm, x->d_err, x->st); }
  { Scope s(x, KC_ATTN);
    launch_attn_generic(x->q_rot, x->NQD, kc_layer, vc_layer, x->kvdtype, kvl, base_len, anc, c.n_q_heads, x->attn_out,
                        x->NQD, FragPlanes{}, rm, x->st, anc_stride, iv); }
  gemm_generic(x, KC_GEMM_WO, x->attn_out, x->NQD, lw.wo, nullptr, xres, H, M, H, x->NQD, 1);
  const SmallGemm gu[2] = {{xres, H, lw.w_gate, nullptr, lw.ffn_norm, x->h_ffn, F, F}, {xres, H, lw.w_up, nullptr, lw.ffn_norm, nullptr, F, F}};
  if (gemm_small_joins(gu, 2, true, c.dtype, M, H)) {
    Scope s(x, KC_GEMM_GATEUP);
    launch_gemm_small(gu, 2, true, c.dtype, M, H, 0, c.rms_eps, x->st);
  } else {
    { Scope s(x, KC_RMSNORM); launch_rmsnorm(xres, H, lw.ffn_norm, c.dtype, c.rms_eps, x->a_norm, H, H, M, x->st); }
    gemm_generic(x, KC_GEMM_GATEUP, x->a_norm, H, lw.w_gate, nullptr, x->tmp_ffn, F, M, F, H, 0);
    gemm_generic(x, KC_GEMM_GATEUP, x->a_norm, H, lw.w_up, nullptr, x->h_ffn, F, M, F, H, 0);
    Scope s(x, KC_ELTWISE);
    launch_swiglu(x->tmp_ffn, x->h_ffn, x->h_ffn, (size_t)M * F, x->st);
  }
  gemm_generic(x, KC_GEMM_DOWN, x->h_ffn, F, lw.w_down, nullptr, xres, H, M, H, F, 1);
}


// planes of RMSNorm(src) * gain in the a_norm buffer (MFMA path)
FragPlanes norm_planes(clover_ctx* x, const float* src, const void* gain, int rows) {
  const clover_config& c = x->cfg;
  const FragPlanes A = frag_planes(x->a_norm, rows);
  Scope s(x, KC_RMSNORM);
  launch_reduce_add_norm(const_cast<float*>(src), x->H, nullptr, 0, 0, 0, gain, c.rms_eps, A, rows, x->H, x->st);
  return A;
}

// rotary tables of a pass behind base_len cached positions
RopeRows rope_rows(const clover_ctx* x, const int* base_len, const int* depth = nullptr, int depth_stride = 0) {
  return RopeRows{base_len, depth, depth_stride, x->cfg.rope_base, x->cfg.head_dim, x->cos_t, x->sin_t};
}
// start of a pass over the target's layers: embeddings in `res`, rotary tables, on the MFMA path planes for the first layer
void start_pass(clover_ctx* x, const int* tok, float* res, const RowMap& rm, int M, const RopeRows& rope) {
  const clover_config& c = x->cfg;
  Scope s(x, KC_EMBED);
  launch_pass_start(PassStart{x->w.embed, tok, c.vocab, res, x->H, x->H, rm, rope, x->fast ? x->layers[0].attn_norm : nullptr,
                              c.rms_eps, frag_planes(x->a_norm, M)}, c.dtype, x->st);
}

// Can draft_tree take the fused route?  (The gate kernel deals whole heads to its lanes.)
bool draft_fused_ok(clover_ctx* x) { return x->fast && ad_gate_fused_supported(x->H, x->cfg.ad_heads); }

// Attention Decoder on the fused route: planes A = RMSNorm(x)*norm, Y = y are in place; q and k|v projections leave
// their partial tiles side by side, the gate kernel does the rest.
void run_ad_fused(clover_ctx* x, const clover_ad_weights& ad, FragPlanes A, FragPlanes Y, int rows, AdGateArgs g) {
  const int H = x->H;
  g.Pq = x->partial; g.sps_q = (size_t)rows * H;
  g.Sq = gemm_fast(x, KC_GEMM_DRAFT, A, ad.wq, rows, H, H);
  float* Pkv = x->partial + align256((size_t)g.Sq * rows * H * sizeof(float)) / sizeof(float);
  g.Pkv = Pkv; g.sps_kv = (size_t)rows * 2 * H;
  g.Skv = gemm_fast(x, KC_GEMM_DRAFT, Y, ad.wk /* k and v rows */, rows, 2 * H, H, Pkv);
  g.bq = ad.bq; g.bk = ad.bk; g.bv = ad.bv;
  g.H = H; g.heads = x->cfg.ad_heads; g.eps = x->cfg.rms_eps;
  Scope sc(x, KC_AD_GATE);
  launch_ad_gate_fused(g, rows, x->st);
}

// Attention Decoder on `rows` contiguous rows: out = x + gate(q(norm(x)), k(y)) * v(y)
void run_ad(clover_ctx* x, const clover_ad_weights& ad, const float* xin, const float* y, int rows, float* out,
            AdNodes to = AdNodes{} /* of the routes without draft_fused_ok */) {
  const clover_config& c = x->cfg;
  const int H = x->H;
  if (x->fast) {
    const FragPlanes A = norm_planes(x, xin, ad.norm, rows);
    const FragPlanes Y = split_to(x, y, H, x->pl_y, rows, H);
    if (draft_fused_ok(x)) {
      AdGateArgs g;
      memset(&g, 0, sizeof(g));
      g.x = xin; g.ldx = H; g.out = out; g.ldo = H;
      run_ad_fused(x, ad, A, Y, rows, g);
      return;
    }
    linear_fast(x, A, ad.wq, ad.bq, x->ad_q, H, rows, H, H);
    const int sp = gemm_fast(x, KC_GEMM_DRAFT, Y, ad.wk /* k and v rows */, rows, 2 * H, H);
    Scope sc(x, KC_ELTWISE);
    launch_reduce(x->partial, sp, (size_t)rows * 2 * H, 2 * H, ad.bk, c.dtype, x->ad_k, H, rows, H, 0, x->st);
    launch_reduce(x->partial + H, sp, (size_t)rows * 2 * H, 2 * H, ad.bv, c.dtype, x->ad_v, H, rows, H, 0, x->st);
  } else {
    const SmallGemm g[3] = {{xin, H, ad.wq, ad.bq, ad.norm, x->ad_q, H, H}, {y, H, ad.wk, ad.bk, nullptr, x->ad_k, H, H},
                            {y, H, ad.wv, ad.bv, nullptr, x->ad_v, H, H}};
    if (gemm_small_joins(g, 3, false, c.dtype, rows, H)) {
      Scope s(x, KC_GEMM_DRAFT);
      launch_gemm_small(g, 3, false, c.dtype, rows, H, 0, c.rms_eps, x->st);
    } else {
      { Scope s(x, KC_RMSNORM); launch_rmsnorm(xin, H, ad.norm, c.dtype, c.rms_eps, x->a_norm, H, H, rows, x->st); }
      gemm_generic(x, KC_GEMM_DRAFT, x->a_norm, H, ad.wq, ad.bq, x->ad_q, H, rows, H, H, 0);
      gemm_generic(x, KC_GEMM_DRAFT, y, H, ad.wk, ad.bk, x->ad_k, H, rows, H, H, 0);
      gemm_generic(x, KC_GEMM_DRAFT, y, H, ad.wv, ad.bv, x->ad_v, H, rows, H, H, 0);
    }
  }
  { Scope s(x, KC_AD_GATE);
    launch_ad_gate(xin, H, x->ad_q, x->ad_k, x->ad_v, H, c.ad_heads, out, rows, x->st, to); }
}

// Y = X W^T + bias for a draft-side FC with fp32 input X [rows, K]
void run_fc(clover_ctx* x, const float* X, int K, const void* W, const void* bias, float* Y, int rows) {
  const int H = x->H;
  if (x->fast) {
    const FragPlanes P = split_to(x, X, K, x->pl_y, rows, K);
    linear_fast(x, P, W, bias, Y, H, rows, H, K);
  } else {
    gemm_generic(x, KC_GEMM_DRAFT, X, K, W, bias, Y, H, rows, H, K, 0);
  }
}

// out[rows, vocab] = A * lm_head^T (MFMA path)
void lm_head_fast(clover_ctx* x, FragPlanes A, int rows, float* out) {
  const clover_config& c = x->cfg;
  Scope s(x, KC_GEMM_LMHEAD);
  TileGemm g;
  memset(&g, 0, sizeof(g));
  g.X = A;
  g.W = (const bf16_t*)x->lm_head_pk;
  g.Y = out; g.ldy = c.vocab; g.M = rows; g.N = c.vocab; g.K = x->H; g.epi = 0; g.k_parts = 1;
  launch_gemm_tile(g, x->st);
}

// out[rows, vocab] = RMSNorm(src) * gain through the LM head (generic path)
void lm_head_generic(clover_ctx* x, const float* src, const void* gain, int rows, float* out) {
  const clover_config& c = x->cfg;
  const int H = x->H;
  const SmallGemm g{src, H, x->w.lm_head, nullptr, gain, out, c.vocab, c.vocab};
  if (gemm_small_joins(&g, 1, false, c.dtype, rows, H)) {
    Scope s(x, KC_GEMM_LMHEAD);
    return launch_gemm_small(&g, 1, false, c.dtype, rows, H, 0, c.rms_eps, x->st);
  }
  { Scope s(x, KC_RMSNORM); launch_rmsnorm(src, H, gain, c.dtype, c.rms_eps, x->a_norm, H, H, rows, x->st); }
  gemm_generic(x, KC_GEMM_LMHEAD, x->a_norm, H, x->w.lm_head, nullptr, out, c.vocab, rows, c.vocab, H, 0);
}

// logits of `rows` contiguous rows of g through the head norm and the shared LM head, into x->z
void run_head(clover_ctx* x, const float* g, int rows) {
  const clover_config& c = x->cfg;
  const int H = x->H;
  if (x->fast) {
    const FragPlanes A = norm_planes(x, g, x->w.head_norm, rows);
    lm_head_fast(x, A, rows, x->z);
  } else {
    lm_head_generic(x, g, x->w.head_norm, rows, x->z);
  }
}

// test hook: copy the logits of the depth-j internal nodes (rows x vocab in x->z) behind those of the shallower depths
void capture_draft_logits(clover_ctx* x, int j, int rows) {
  if (!x->draft_capture) return;
  const size_t V = (size_t)x->cfg.vocab;
  size_t off;
  if (x->dyn_on) {   // rows of depth j start behind the rows of the shallower depths: batch * (F[0] + .. + F[j-1]) rows
    int before = 0;
    for (int i = 0; i < j; ++i) before += x->dyn.F[i];
    off = (size_t)(rows / std::max(1, x->dyn.F[j])) * before * V;
  } else {
    off = (size_t)(rows / std::max(1, x->tree.lvl_off[j + 1] - x->tree.lvl_off[j])) * x->tree.lvl_off[j] * V;
  }
  if (off + (size_t)rows * V > x->draft_capture_floats) return;
  hipMemcpyAsync(x->draft_capture + off, x->z, (size_t)rows * V * sizeof(float), hipMemcpyDeviceToDevice, x->st);
}

// Dynamic tree: expansion depth by depth (the root state and token are in candidate 0), then the selection.
// Depth j expands F[j] candidates per sequence; their logits go through a log-softmax so that scores add up
// along a path.
void draft_expand_dynamic(clover_ctx* x, int B, const int* m, int* tree_tokens, bool fused) {
  const clover_config& c = x->cfg;
  const DynTree& t = x->dyn;
  const int H = x->H, C = t.C, ns = CLOVER_MAX_DEPTH * DYN_MAX_FRONT;
  for (int j = 0; j < t.D; ++j) {
    const int n_lvl = t.F[j], rows = B * n_lvl;
    const int* nodes = t.frontier + (size_t)j * DYN_MAX_FRONT;
    if (fused) {
      const FragPlanes A = frag_planes(x->a_norm, rows), Y = frag_planes(x->pl_y, rows), Cc = frag_planes(x->d_cat, rows);
      int sp;
      if (j == 0) {
        sp = gemm_fast(x, KC_GEMM_DRAFT, Y, x->w.fc0_w, rows, H, H);
      } else {
        { Scope s(x, KC_DRAFT_MISC);
          launch_draft_level(x->dyn_state, t.cand_tok, nodes, t.cand_par, n_lvl, B, C, H, x->w.lm_head, c.vocab,
                             x->w.ad2.norm, c.rms_eps, A, Y, Cc, x->st, ns, C); }
        AdGateArgs g;
        memset(&g, 0, sizeof(g));
        g.x = x->dyn_state; g.ldx = H; g.out = x->dyn_state; g.ldo = H;
        g.nodes = nodes; g.parent = t.cand_par; g.n_lvl = n_lvl; g.R = C; g.m = m;
        g.nodes_stride = ns; g.parent_stride = C;
        g.cat = Cc;
        run_ad_fused(x, x->w.ad2, A, Y, rows, g);
        sp = gemm_fast(x, KC_GEMM_DRAFT, Cc, x->fc_w[j], rows, H, 2 * H);
      }
      { Scope s(x, KC_RMSNORM);
        launch_reduce_add_norm(x->d_g, H, x->partial, sp, (size_t)rows * H, H, x->w.head_norm, c.rms_eps, A,
                               rows, H, x->st, j == 0 ? x->w.fc0_b : x->fc_b[j]); }
      lm_head_fast(x, A, rows, x->z);
    } else {
      if (j == 0) {
        run_fc(x, x->d_rootx, H, x->w.fc0_w, x->w.fc0_b, x->d_g, rows);
      } else {
        { Scope s(x, KC_DRAFT_MISC);
          launch_draft_gather(x->dyn_state, t.cand_tok, nodes, t.cand_par, n_lvl, B, C, H, x->w.lm_head, c.dtype, c.vocab,
                              x->d_xs, x->d_e, x->d_cat, x->st, ns, C); }
        run_ad(x, x->w.ad2, x->d_xs, x->d_e, rows, x->dyn_state, AdNodes{nodes, n_lvl, C, ns, x->d_cat});
        run_fc(x, x->d_cat, 2 * H, x->fc_w[j], x->fc_b[j], x->d_g, rows);
      }
      run_head(x, x->d_g, rows);
    }
    capture_draft_logits(x, j, rows);
    { Scope s(x, KC_TOPK);
      launch_topk_lse(x->z, c.vocab, c.vocab, rows, t.topk, x->cand, x->topk_aux, x->topk_lse, x->st, 1.0f, &t, j, m); }
    if (j + 1 < t.D) { Scope s(x, KC_DRAFT_MISC); launch_dyn_frontier(t, j + 1, B, m, x->st); }
  }
  { Scope s(x, KC_DRAFT_MISC); launch_dyn_finalize(t, B, x->R, m, tree_tokens, x->st); }
}

int upload_tree(clover_ctx* x) {
  const TreeHost& t = x->tree;
  const int n = t.n;
  hipError_t e = hipSuccess;
  auto up = [&](void* dst, const void* src, size_t bytes) {
    if (bytes && e == hipSuccess) e = hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, x->st);
  };
  up(x->d_depth, t.depth.data(), n * sizeof(int));
  up(x->d_parent, t.parent.data(), n * sizeof(int));
  up(x->d_rank, t.rank.data(), n * sizeof(int));
  up(x->d_first_child, t.first_child.data(), n * sizeof(int));
  up(x->d_n_child, t.n_child.data(), n * sizeof(int));
  up(x->d_lvl_nodes, t.lvl_nodes.data(), t.lvl_nodes.size() * sizeof(int));
  up(x->d_anc, t.anc.data(), 2 * n * sizeof(unsigned long long));
  up(x->d_iv, t.iv.data(), 2 * n * sizeof(int));
  if (e == hipSuccess) e = hipStreamSynchronize(x->st);  // the host vectors may change after return
  if (e != hipSuccess) return fail(x, CLOVER_E_HIP, std::string("tree upload: ") + hipGetErrorString(e));
  return CLOVER_OK;
}

int finish(clover_ctx* x, const char* what) {
  if (const char* why = std::exchange(g_not_launched, nullptr)) return fail(x, CLOVER_E_STATE, std::string(what) + ": " + why);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(x, CLOVER_E_HIP, std::string(what) + ": " + hipGetErrorString(e));
  return CLOVER_OK;
}

int check_batch(clover_ctx* x, int batch) {
  if (batch < 1 || batch > x->cfg.max_batch) return fail(x, CLOVER_E_SHAPE, "batch outside [1, max_batch]");
  return CLOVER_OK;
}

int accept_common(clover_ctx* x, int batch, const int* tree_tokens, const float* logits, const float* hidden,
                  const int* n_forced, const int* forced_next, int* m, int* acc_idx, int* new_tokens, float* hid_acc,
                  int* next_tok, float temperature = 0.f, const float* uniforms = nullptr) {
  const clover_config& c = x->cfg;
  const TreeHost& t = x->tree;
  const int n_nodes = x->dyn_on ? x->dyn.N : t.n;
  const int R = x->R, M = (batch - 1) * R + n_nodes;
  x->only_prefills = false;
  const int* fc_tab = x->dyn_on ? x->dyn.t_first_child : x->d_first_child;
  const int* nc_tab = x->dyn_on ? x->dyn.t_n_child : x->d_n_child;
  if (uniforms) {
    // temperature > 0: per-row log-sum-exp of logits / T, then the sampled walk
    const float inv_t = 1.0f / temperature;
    { Scope s(x, KC_TOPK);
      launch_topk_lse(logits, c.vocab, c.vocab, M, 1, x->cand, x->topk_aux, x->topk_lse, x->st, inv_t); }
    { Scope s(x, KC_ACCEPT);
      launch_accept_sample(logits, c.vocab, x->topk_lse, inv_t, tree_tokens, fc_tab, nc_tab, x->dyn_on ? R : 0, batch, R,
                           uniforms, m, acc_idx, new_tokens, next_tok, x->d_seq_len,
                           (double*)x->topk_aux /* read by the launch above, free now */, x->st); }
  } else {
  { Scope s(x, KC_TOPK); launch_topk(logits, c.vocab, c.vocab, M, 1, x->cand, x->topk_ids, x->st); }
  { Scope s(x, KC_ACCEPT);
    launch_accept_walk(x->topk_ids, tree_tokens, x->dyn_on ? x->dyn.t_first_child : x->d_first_child,
                       x->dyn_on ? x->dyn.t_n_child : x->d_n_child, n_nodes, batch, R, n_forced, forced_next,
                       m, acc_idx, new_tokens, next_tok, x->d_seq_len, x->st, x->dyn_on ? R : 0); }
  }
  { Scope s(x, KC_COMPACT);
    const int most = n_forced ? n_nodes : std::min((x->dyn_on ? x->dyn.D : t.max_depth) + 1, R);
    launch_accept_move(x->kc, x->vc, x->kvdtype, x->kv, c.n_layers, x->kv_layer_stride, x->d_seq_len, m, acc_idx, batch, R, most,
                       hidden, x->H, hid_acc, x->st); }
  return finish(x, "accept");
}

int static_scratch_ptr(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) { g_err = std::string("hipGetDevice: ") + hipGetErrorString(e); return CLOVER_E_HIP; }
  if (dev < 0 || dev >= kMaxDevices) { g_err = "device index beyond the static scratch table"; return CLOVER_E_SHAPE; }
  if (!g_static_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(g_static_scratch));
    if (e != hipSuccess || !p) {
      g_err = std::string("hipGetSymbolAddress(static scratch): ") + hipGetErrorString(e);
      return CLOVER_E_HIP;
    }
    g_static_scratch_ptr[dev] = p;
  }
  *out = g_static_scratch_ptr[dev];
  return CLOVER_OK;
}

}  // namespace

// ================================================================================================
extern "C" {

int clover_workspace_bytes(const clover_config* cfg, size_t* bytes_out) {
  if (!cfg || !bytes_out) return fail(nullptr, CLOVER_E_NULL, "null argument");
  std::string why;
  const int rc = check_config(cfg, why);
  if (rc) return fail(nullptr, rc, why);
  clover_ctx tmp{};
  tmp.cfg = *cfg;
  size_t total = 0;
  carve(&tmp, nullptr, &total);
  *bytes_out = total;
  return CLOVER_OK;
}

int clover_init(const clover_config* cfg, const clover_weights* w, const clover_tree* tree, void* workspace,
                size_t workspace_bytes, void* hip_stream, clover_ctx** ctx_out) {
  if (!cfg || !w || !tree || !workspace || !ctx_out) return fail(nullptr, CLOVER_E_NULL, "null argument");
  std::string why;
  int rc = check_config(cfg, why);
  if (rc) return fail(nullptr, rc, why);
  if (((uintptr_t)workspace & 255) != 0) return fail(nullptr, CLOVER_E_CONFIG, "workspace must be 256-byte aligned");
  if (!w->embed || !w->layers || !w->final_norm || !w->lm_head || !w->aug || !w->fc0_w || !w->fc0_b || !w->fc_w ||
      !w->fc_b || !w->head_norm)
    return fail(nullptr, CLOVER_E_NULL, "null weight pointer");
  const clover_ad_weights* ads[2] = {&w->ad1, &w->ad2};
  for (const clover_ad_weights* a : ads)
    if (!a->norm || !a->wq || !a->bq || !a->wk || !a->bk || !a->wv || !a->bv) return fail(nullptr, CLOVER_E_NULL, "null Attention-Decoder weight");
  auto layer_ok = [](const clover_layer_weights& l) {
    return l.attn_norm && l.wq && l.wk && l.wv && l.wo && l.ffn_norm && l.w_gate && l.w_up && l.w_down;
  };
  for (int i = 0; i < cfg->n_layers; ++i) if (!layer_ok(w->layers[i])) return fail(nullptr, CLOVER_E_NULL, "null target layer weight");
  for (int i = 0; i < cfg->aug_layers; ++i) if (!layer_ok(w->aug[i])) return fail(nullptr, CLOVER_E_NULL, "null augmenting layer weight");
  for (int j = 1; j < cfg->draft_depths; ++j) if (!w->fc_w[j] || !w->fc_b[j]) return fail(nullptr, CLOVER_E_NULL, "null FC weight");
  TreeHost th;
  rc = build_tree(*cfg, tree, th, why);
  if (rc) return fail(nullptr, rc, why);

  clover_ctx* x = new clover_ctx{};
  x->cfg = *cfg;
  x->st = (hipStream_t)hip_stream;
  x->w = *w;
  x->layers.assign(w->layers, w->layers + cfg->n_layers);
  x->aug.assign(w->aug, w->aug + cfg->aug_layers);
  x->fc_w.assign(w->fc_w, w->fc_w + cfg->draft_depths);
  x->fc_b.assign(w->fc_b, w->fc_b + cfg->draft_depths);
  x->tree = std::move(th);
  size_t total = 0;
  carve(x, (char*)workspace, &total);
  if (total > workspace_bytes) { delete x; return fail(nullptr, CLOVER_E_CAPACITY, "workspace too small"); }
  x->len_ub.assign(cfg->max_batch, 0);
  x->aug_ub.assign(cfg->max_batch, 0);
  x->m_upper = cfg->max_nodes;
  x->only_prefills = true;
  x->interval = (cfg->flags & CLOVER_FLAG_INTERVAL_MASK) != 0;
  x->meet_polls = MEET_POLLS;
  launch_fill_i32(x->d_seq_len, 0, cfg->max_batch, x->st);
  launch_fill_i32(x->d_aug_len, 0, cfg->max_batch, x->st);
  launch_fill_i32(x->d_err, 0, 1, x->st);
  launch_fill_i32((int*)x->d_meet, 0, TILE_MEETINGS * MEET_STRIDE, x->st);
  // A draft call leaves a skipped sequence's dynamic tables alone, but its rows are computed along and index by them: candidate 0
  // and a root without children until a call fills them in.
  launch_fill_i32(x->dyn.cand_tok, 0, (int)(x->dyn.t_iv + 2 * x->step.rows - x->dyn.cand_tok), x->st);
  if (x->fast) {
    // the MFMA attention multiplies masked probabilities (exact zeros) with whatever the cache rows of a
    // tile hold, so the caches must never contain non-finite garbage
    hipMemsetAsync(x->kc, 0, x->k_layer_elems * x->kv_esz * cfg->n_layers, x->st);
    hipMemsetAsync(x->vc, 0, x->v_layer_elems * x->kv_esz * cfg->n_layers, x->st);
    hipMemsetAsync(x->aug_kc, 0, x->k_layer_elems * x->kv_esz * cfg->aug_layers, x->st);
    hipMemsetAsync(x->aug_vc, 0, x->v_layer_elems * x->kv_esz * cfg->aug_layers, x->st);
    // private fragment-major copies of every linear weight; the originals are only read here
    // (and, for the LM head, by the draft's embedding gathers)
    char* cur = x->packed;
    auto pack = [&](const void*& w, int N, int K) {
      launch_pack_weight(w, cur, N, K, 0, N, x->st);
      w = cur;
      cur += (size_t)N * K * 2;
    };
    // linears that share their input, as one matrix: every pointer names the whole
    struct Part { const void** w; int rows, rotary_d; };
    auto pack_joint = [&](std::initializer_list<Part> parts, int K) {
      int n_rows = 0, row0 = 0;
      for (const Part& p : parts) n_rows += p.rows;
      for (const Part& p : parts) {
        launch_pack_weight(*p.w, cur, p.rows, K, row0, n_rows, x->st, p.rotary_d);
        *p.w = cur;
        row0 += p.rows;
      }
      cur += (size_t)n_rows * K * 2;
    };
    const int H = x->H, d = cfg->head_dim, F = cfg->ffn;
    auto pack_layer = [&](clover_layer_weights& l) {
      pack_joint({{&l.wq, cfg->n_q_heads * d, d}, {&l.wk, cfg->n_kv_heads * d, d}, {&l.wv, cfg->n_kv_heads * d, 0}}, H);
      pack(l.wo, H, x->NQD);
      launch_pack_gate_up(l.w_gate, l.w_up, cur, F, H, x->st);
      l.w_gate = l.w_up = cur;
      cur += (size_t)2 * F * H * 2;
      pack(l.w_down, H, F);
    };
    for (auto& l : x->layers) pack_layer(l);
    for (auto& l : x->aug) pack_layer(l);
    x->lm_head_pk = x->w.lm_head;
    pack(x->lm_head_pk, cfg->vocab, H);
    for (clover_ad_weights* a : {&x->w.ad1, &x->w.ad2}) { pack(a->wq, H, H); pack_joint({{&a->wk, H, 0}, {&a->wv, H, 0}}, H); }
    pack(x->w.fc0_w, H, H);
    for (int j = 1; j < cfg->draft_depths; ++j) pack(x->fc_w[j], H, 2 * H);
    if ((size_t)(cur - x->packed) > x->packed_bytes) { delete x; return fail(nullptr, CLOVER_E_CAPACITY, "internal: packed weights overflow"); }
  }
  rc = upload_tree(x);
  if (rc == CLOVER_OK) rc = finish(x, "init");
  if (rc) { g_err = x->err; delete x; return rc; }
  *ctx_out = x;
  return CLOVER_OK;
}

int clover_destroy(clover_ctx* x) {
  if (!x) return CLOVER_E_NULL;
  hipStreamSynchronize(x->st);
  for (ProfEvent& ev : x->prof_events) { hipEventDestroy(ev.a); hipEventDestroy(ev.b); }
  for (ProfEvent& ev : x->prof_pool) { hipEventDestroy(ev.a); hipEventDestroy(ev.b); }
  delete x;
  return CLOVER_OK;
}

int clover_reset(clover_ctx* x) {
  if (!x) return CLOVER_E_NULL;
  launch_fill_i32(x->d_seq_len, 0, x->cfg.max_batch, x->st);
  launch_fill_i32(x->d_aug_len, 0, x->cfg.max_batch, x->st);
  launch_fill_i32(x->d_err, 0, 1, x->st);
  std::fill(x->len_ub.begin(), x->len_ub.end(), 0);
  std::fill(x->aug_ub.begin(), x->aug_ub.end(), 0);
  x->m_upper = x->cfg.max_nodes;
  x->only_prefills = true;
  return finish(x, "reset");
}

int clover_set_tree(clover_ctx* x, const clover_tree* tree) {
  if (!x || !tree) return fail(x, CLOVER_E_NULL, "null argument");
  TreeHost th;
  std::string why;
  const int rc = build_tree(x->cfg, tree, th, why);
  if (rc) return fail(x, rc, why);
  hipError_t e = hipStreamSynchronize(x->st);  // kernels in flight still read the old tables
  if (e != hipSuccess) return fail(x, CLOVER_E_HIP, hipGetErrorString(e));
  x->tree = std::move(th);
  x->dyn_on = false;
  return upload_tree(x);
}

int clover_set_dynamic_tree(clover_ctx* x, int32_t n_nodes, int32_t topk, int32_t frontier) {
  if (!x) return CLOVER_E_NULL;
  const clover_config& c = x->cfg;
  if (n_nodes < 1 || n_nodes > c.max_nodes) return fail(x, CLOVER_E_TREE, "n_nodes outside [1, max_nodes]");
  if (n_nodes > CLOVER_MAX_NODES) return fail(x, CLOVER_E_TREE, "a dynamic tree has at most 128 nodes");
  if (topk < 1 || topk > CLOVER_MAX_RANK) return fail(x, CLOVER_E_TREE, "topk outside [1, 16]");
  if (frontier < 1 || frontier > DYN_MAX_FRONT || frontier > c.max_nodes)
    return fail(x, CLOVER_E_TREE, "frontier outside [1, min(64, max_nodes)]");
  DynTree t = x->dyn;   // keeps the workspace pointers
  t.D = c.draft_depths; t.topk = topk; t.N = n_nodes;
  t.off[0] = 0; t.off[1] = 1; t.F[0] = 1;
  int n_cand = topk;                               // candidates of depth 1
  for (int j = 1; j <= t.D; ++j) {
    t.off[j + 1] = t.off[j] + n_cand;
    if (n_cand > DYN_MAX_CAND) return fail(x, CLOVER_E_TREE, "more than 256 candidates in one depth");
    t.F[j] = std::min(frontier, n_cand);
    n_cand = t.F[j] * topk;
  }
  t.C = t.off[t.D + 1];
  if (t.C > DYN_MAX_CAND) return fail(x, CLOVER_E_TREE, "more than 256 candidates: lower topk, frontier or draft_depths");
  if (t.C < n_nodes) return fail(x, CLOVER_E_TREE, "fewer candidates than tree nodes");
  hipError_t e = hipStreamSynchronize(x->st);  // kernels in flight still read the old tables
  if (e != hipSuccess) return fail(x, CLOVER_E_HIP, hipGetErrorString(e));
  x->dyn = t;
  x->dyn_on = true;
  return CLOVER_OK;
}

int clover_read_dynamic_tree(clover_ctx* x, int32_t b, int32_t* parent_out, int32_t* rank_out, int32_t* keep_out,
                             int32_t* cand_token_out, float* cand_score_out, int32_t* cand_parent_out,
                             int32_t* frontier_out) {
  if (!x || !parent_out || !rank_out || !keep_out || !cand_token_out || !cand_score_out || !cand_parent_out || !frontier_out)
    return fail(x, CLOVER_E_NULL, "null argument");
  if (!x->dyn_on) return fail(x, CLOVER_E_TREE, "no dynamic tree is set");
  if (b < 0 || b >= x->cfg.max_batch) return fail(x, CLOVER_E_SHAPE, "sequence index out of range");
  const DynTree& t = x->dyn;
  const size_t ro = (size_t)b * x->R, co = (size_t)b * t.C;
  hipError_t e = hipSuccess;
  auto down = [&](void* dst, const void* src, size_t bytes) {
    if (e == hipSuccess) e = hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, x->st);
  };
  down(parent_out, t.t_parent + ro, t.N * sizeof(int));
  down(rank_out, t.t_rank + ro, t.N * sizeof(int));
  down(keep_out, t.t_keep + ro, t.N * sizeof(int));
  down(cand_token_out, t.cand_tok + co, t.C * sizeof(int));
  down(cand_score_out, t.cand_score + co, t.C * sizeof(float));
  down(cand_parent_out, t.cand_par + co, t.C * sizeof(int));
  down(frontier_out, t.frontier + (size_t)b * CLOVER_MAX_DEPTH * DYN_MAX_FRONT, CLOVER_MAX_DEPTH * DYN_MAX_FRONT * sizeof(int));
  if (e == hipSuccess) e = hipStreamSynchronize(x->st);
  if (e != hipSuccess) return fail(x, CLOVER_E_HIP, std::string("clover_read_dynamic_tree: ") + hipGetErrorString(e));
  return CLOVER_OK;
}

int draft_tree(clover_ctx* x, int32_t batch, const float* hid_acc, const int32_t* next_tok, const int32_t* m,
               int32_t* tree_tokens) {
  if (!x || !hid_acc || !next_tok || !m || !tree_tokens) return fail(x, CLOVER_E_NULL, "null argument");
  int rc = check_batch(x, batch);
  if (rc) return rc;
  const clover_config& c = x->cfg;
  const TreeHost& t = x->tree;
  const int B = batch, R = x->R, H = x->H, n = std::min(x->m_upper, R);
  for (int b = 0; b < B; ++b)
    if (x->aug_ub[b] + n > c.max_seq) return fail(x, CLOVER_E_CAPACITY, "augmenting-block cache could exceed max_seq");
  const bool fused = draft_fused_ok(x);
  // rows of the accepted tokens: the caller's arrays hold R rows per sequence of which at most n are accepted; the fused
  // route packs them (16 sequences x 32 nodes: 80 rows instead of 485)
  const RowMap in{B, R, n, m}, rm{B, fused ? n : R, n, m};
  const int M = (B - 1) * rm.R + n;
  const AttnPlan plan = plan_attention(x, x->aug_ub.data(), rm, M, true);
  const RopeRows rope = rope_rows(x, x->d_aug_len);
  if (fused) {
    const FragPlanes A = frag_planes(x->a_norm, M), Y = frag_planes(x->pl_y, M);
    // embeddings of the follow-up tokens come from the LM-head rows; AD1 over (hidden state, embedding)
    { Scope s(x, KC_DRAFT_MISC);
      launch_draft_pre(hid_acc, next_tok, x->w.ad1.norm, c.rms_eps, x->w.lm_head, c.vocab, H, in,
                       rope, A, Y, x->st); }
    AdGateArgs g;
    memset(&g, 0, sizeof(g));
    g.x = hid_acc; g.ldx = H; g.out = x->xd; g.ldo = H; g.n_lvl = n; g.R = R;
    g.gain = x->aug[0].attn_norm; g.norm = A;   // planes for the Augmenting Block's first layer
    run_ad_fused(x, x->w.ad1, A, Y, M, g);
  } else {
  // embeddings of the follow-up tokens come from the LM-head rows
  { Scope s(x, KC_EMBED); launch_pass_start(PassStart{x->w.lm_head, next_tok, c.vocab, x->d_e, H, H, rm, rope, nullptr, 0.f, {}}, c.dtype, x->st); }
  run_ad(x, x->w.ad1, hid_acc, x->d_e, M, x->xd);
  if (x->fast) norm_planes(x, x->xd, x->aug[0].attn_norm, M);
  }
  for (int l = 0; l < c.aug_layers; ++l)
    run_layer(x, x->aug[l], x->xd, rm, M, x->aug_kc + (size_t)l * x->k_layer_elems * x->kv_esz,
              x->aug_vc + (size_t)l * x->v_layer_elems * x->kv_esz, x->d_aug_len, nullptr /* the new rows form a chain */,
              l + 1 < c.aug_layers ? x->aug[l + 1].attn_norm : nullptr, plan);
  {
    // root state and token: node 0 of the static tree, candidate 0 of the dynamic one
    float* root_state = x->dyn_on ? x->dyn_state : x->d_state;
    int* root_tok = x->dyn_on ? x->dyn.cand_tok : tree_tokens;
    const int Rs = x->dyn_on ? x->dyn.C : R;
    Scope s(x, KC_DRAFT_MISC);
    if (fused) {
      launch_draft_root_fused(x->xd, next_tok, m, B, R, n, H, root_state, root_tok, frag_planes(x->pl_y, B), x->d_aug_len, x->st, Rs);
    } else {
      launch_draft_root(x->xd, next_tok, m, B, R, H, x->d_rootx, root_state, root_tok, x->d_aug_len, x->st, Rs);
    }
  }
  for (int b = 0; b < B; ++b) x->aug_ub[b] += n;
  if (x->dyn_on) {
    draft_expand_dynamic(x, B, m, tree_tokens, fused);
    return finish(x, "draft_tree");
  }
  // expansion, level by level; a tree deeper than the head (e.g. a prompt chain) is not expanded
  if (t.max_depth <= c.draft_depths) {
    for (int j = 0; j < t.max_depth; ++j) {
      const int n_lvl = t.lvl_off[j + 1] - t.lvl_off[j];
      if (n_lvl == 0) break;
      const int rows = B * n_lvl;
      auto rank = [&] {   // top-k of every row and with it the tokens of the nodes' children
        Scope s(x, KC_TOPK);
        launch_topk(x->z, c.vocab, c.vocab, rows, t.kmax[j], x->cand, x->topk_ids, x->st,
                    TopkChildren{x->d_lvl_nodes + t.lvl_off[j], x->d_first_child, x->d_n_child, x->d_rank, m, n_lvl, R, tree_tokens});
      };
      if (fused) {
        // depth j: (AD2 over the parent's state and the node's token embedding, then) FC_j; the FC's partial tiles
        // and bias go straight into the head norm
        const FragPlanes A = frag_planes(x->a_norm, rows), Y = frag_planes(x->pl_y, rows), Cc = frag_planes(x->d_cat, rows);
        int sp;
        if (j == 0) {
          sp = gemm_fast(x, KC_GEMM_DRAFT, Y, x->w.fc0_w, rows, H, H);
        } else {
          const int* nodes = x->d_lvl_nodes + t.lvl_off[j];
          { Scope s(x, KC_DRAFT_MISC);
            launch_draft_level(x->d_state, tree_tokens, nodes, x->d_parent, n_lvl, B, R, H, x->w.lm_head, c.vocab,
                               x->w.ad2.norm, c.rms_eps, A, Y, Cc, x->st); }
          AdGateArgs g;
          memset(&g, 0, sizeof(g));
          g.x = x->d_state; g.ldx = H; g.out = x->d_state; g.ldo = H;
          g.nodes = nodes; g.parent = x->d_parent; g.n_lvl = n_lvl; g.R = R; g.m = m;
          g.cat = Cc;
          run_ad_fused(x, x->w.ad2, A, Y, rows, g);
          sp = gemm_fast(x, KC_GEMM_DRAFT, Cc, x->fc_w[j], rows, H, 2 * H);
        }
        { Scope s(x, KC_RMSNORM);
          launch_reduce_add_norm(x->d_g, H, x->partial, sp, (size_t)rows * H, H, x->w.head_norm, c.rms_eps, A,
                                 rows, H, x->st, j == 0 ? x->w.fc0_b : x->fc_b[j]); }
        lm_head_fast(x, A, rows, x->z);
        capture_draft_logits(x, j, rows);
        rank();
        continue;
      }
      if (j == 0) {
        run_fc(x, x->d_rootx, H, x->w.fc0_w, x->w.fc0_b, x->d_g, rows);
      } else {
        const int* nodes = x->d_lvl_nodes + t.lvl_off[j];
        { Scope s(x, KC_DRAFT_MISC);
          launch_draft_gather(x->d_state, tree_tokens, nodes, x->d_parent, n_lvl, B, R, H, x->w.lm_head, c.dtype,
                              c.vocab, x->d_xs, x->d_e, x->d_cat, x->st); }
        run_ad(x, x->w.ad2, x->d_xs, x->d_e, rows, x->d_state, AdNodes{nodes, n_lvl, R, 0, x->d_cat});
        run_fc(x, x->d_cat, 2 * H, x->fc_w[j], x->fc_b[j], x->d_g, rows);
      }
      run_head(x, x->d_g, rows);
      capture_draft_logits(x, j, rows);
      rank();
    }
  }
  return finish(x, "draft_tree");
}

int verify_tree(clover_ctx* x, int32_t batch, const int32_t* tree_tokens, float* logits, float* hidden) {
  if (!x || !tree_tokens || !logits || !hidden) return fail(x, CLOVER_E_NULL, "null argument");
  int rc = check_batch(x, batch);
  if (rc) return rc;
  const clover_config& c = x->cfg;
  const TreeHost& t = x->tree;
  const int B = batch, R = x->R, H = x->H;
  const int n_nodes = x->dyn_on ? x->dyn.N : t.n;
  // topology tables: one static tree for all sequences, or the tables draft_tree wrote per sequence
  const int* depth_tab = x->dyn_on ? x->dyn.t_depth : x->d_depth;
  const unsigned long long* anc_tab = x->dyn_on ? x->dyn.t_anc : x->d_anc;
  const int* iv_tab = !x->interval ? nullptr : x->dyn_on ? x->dyn.t_iv : x->d_iv;
  const int topo_stride = x->dyn_on ? R : 0;
  for (int b = 0; b < B; ++b)
    if (x->len_ub[b] + n_nodes > c.max_seq) return fail(x, CLOVER_E_CAPACITY, "sequence could exceed max_seq (call clover_seq_len to refresh the bound)");
  const RowMap rm{B, R, n_nodes, nullptr};
  const int M = (B - 1) * R + n_nodes;
  const AttnPlan plan = plan_attention(x, x->len_ub.data(), rm, M, false);
  start_pass(x, tree_tokens, hidden, rm, M, rope_rows(x, x->d_seq_len, depth_tab, topo_stride));
  for (int l = 0; l < c.n_layers; ++l)
    run_layer(x, x->layers[l], hidden, rm, M, x->kc + (size_t)l * x->k_layer_elems * x->kv_esz,
              x->vc + (size_t)l * x->v_layer_elems * x->kv_esz, x->d_seq_len, anc_tab,
              l + 1 < c.n_layers ? x->layers[l + 1].attn_norm : x->w.final_norm, plan, topo_stride, iv_tab);
  if (x->fast) {
    lm_head_fast(x, frag_planes(x->a_norm, M), M, logits);
  } else {
    lm_head_generic(x, hidden, x->w.final_norm, M, logits);
  }
  return finish(x, "verify_tree");
}

int accept_and_compact(clover_ctx* x, int32_t batch, const int32_t* tree_tokens, const float* logits,
                       const float* hidden, int32_t* m, int32_t* acc_idx, int32_t* new_tokens, float* hid_acc,
                       int32_t* next_tok) {
  if (!x || !tree_tokens || !logits || !hidden || !m || !acc_idx || !new_tokens || !hid_acc || !next_tok)
    return fail(x, CLOVER_E_NULL, "null argument");
  int rc = check_batch(x, batch);
  if (rc) return rc;
  rc = accept_common(x, batch, tree_tokens, logits, hidden, nullptr, nullptr, m, acc_idx, new_tokens, hid_acc, next_tok);
  if (rc) return rc;
  x->m_upper = std::min((x->dyn_on ? x->dyn.D : x->tree.max_depth) + 1, x->R);
  for (int b = 0; b < batch; ++b) x->len_ub[b] += x->m_upper;
  return CLOVER_OK;
}

int accept_and_compact_sampled(clover_ctx* x, int32_t batch, const int32_t* tree_tokens, const float* logits,
                               const float* hidden, float temperature, const float* uniforms, int32_t* m,
                               int32_t* acc_idx, int32_t* new_tokens, float* hid_acc, int32_t* next_tok) {
  if (!x || !tree_tokens || !logits || !hidden || !uniforms || !m || !acc_idx || !new_tokens || !hid_acc || !next_tok)
    return fail(x, CLOVER_E_NULL, "null argument");
  int rc = check_batch(x, batch);
  if (rc) return rc;
  if (!(temperature > 0.f) || !(temperature < 1e6f)) return fail(x, CLOVER_E_SHAPE, "temperature must be positive (use accept_and_compact for temperature 0)");
  rc = accept_common(x, batch, tree_tokens, logits, hidden, nullptr, nullptr, m, acc_idx, new_tokens, hid_acc, next_tok,
                     temperature, uniforms);
  if (rc) return rc;
  x->m_upper = std::min((x->dyn_on ? x->dyn.D : x->tree.max_depth) + 1, x->R);
  for (int b = 0; b < batch; ++b) x->len_ub[b] += x->m_upper;
  return CLOVER_OK;
}

int clover_accept_forced(clover_ctx* x, int32_t batch, const int32_t* tree_tokens, const float* logits,
                         const float* hidden, const int32_t* n_rows, const int32_t* forced_next, int32_t* m,
                         int32_t* acc_idx, int32_t* new_tokens, float* hid_acc, int32_t* next_tok) {
  if (!x || !tree_tokens || !logits || !hidden || !n_rows || !forced_next || !m || !acc_idx || !new_tokens ||
      !hid_acc || !next_tok)
    return fail(x, CLOVER_E_NULL, "null argument");
  int rc = check_batch(x, batch);
  if (rc) return rc;
  if (x->dyn_on || !x->tree.is_chain) return fail(x, CLOVER_E_TREE, "clover_accept_forced needs a chain-shaped tree");
  rc = accept_common(x, batch, tree_tokens, logits, hidden, n_rows, forced_next, m, acc_idx, new_tokens, hid_acc, next_tok);
  if (rc) return rc;
  x->m_upper = x->tree.n;
  for (int b = 0; b < batch; ++b) x->len_ub[b] += x->tree.n;
  return CLOVER_OK;
}

int clover_prefill(clover_ctx* x, int32_t b, const int32_t* tokens, int32_t n, float* logits_last, float* hid_last,
                   int32_t* next_tok_out) {
  if (!x || !tokens || !logits_last || !hid_last) return fail(x, CLOVER_E_NULL, "null argument");
  const clover_config& c = x->cfg;
  if (b < 0 || b >= c.max_batch) return fail(x, CLOVER_E_SHAPE, "sequence index out of range");
  if (n < 1) return fail(x, CLOVER_E_SHAPE, "a prompt has at least one token");
  if (x->len_ub[b] + n > c.max_seq || x->aug_ub[b] + n - 1 > c.max_seq)
    return fail(x, CLOVER_E_CAPACITY, "prompt would exceed max_seq (call clover_seq_len to refresh the bound)");
  const int H = x->H;
  const PassBufs bufs(x);
  const int P = x->rows;
  int* len_b = x->d_seq_len + b;
  int* aug_len_b = x->d_aug_len + b;
  float* xres = x->d_xs;   // residual stream of the pass (the draft head's staging buffers are idle here)
  for (int c0 = 0; c0 < n; c0 += P) {
    const int M = std::min(P, n - c0);
    const bool last = c0 + M == n;
    const RowMap rm{1, P, M, nullptr};
    // ---- target: embedding, layers with causal attention (no mask table: a chain), K/V in place ----
    start_pass(x, tokens + c0, xres, rm, M, rope_rows(x, len_b));
    const AttnPlan plan = plan_attention(x, &x->len_ub[b], rm, M, true);
    for (int l = 0; l < c.n_layers; ++l)
      run_layer(x, x->layers[l], xres, rm, M, x->kc + (size_t)l * x->k_layer_elems * x->kv_esz,
                x->vc + (size_t)l * x->v_layer_elems * x->kv_esz, len_b, nullptr,
                l + 1 < c.n_layers ? x->layers[l + 1].attn_norm : nullptr, plan, 0, nullptr, b);
    { Scope s(x, KC_DRAFT_MISC); launch_add_scalar(len_b, M, x->st); }
    x->len_ub[b] += M;
    if (last) {
      // LM head on the last row only; its hidden state is the hand-off row
      if (x->fast) {
        lm_head_fast(x, norm_planes(x, xres + (size_t)(M - 1) * H, x->w.final_norm, 1), 1, logits_last);
      } else {
        lm_head_generic(x, xres + (size_t)(M - 1) * H, x->w.final_norm, 1, logits_last);
      }
      hipMemcpyAsync(hid_last, xres + (size_t)(M - 1) * H, (size_t)H * sizeof(float), hipMemcpyDeviceToDevice, x->st);
      if (next_tok_out) {
        { Scope s(x, KC_TOPK); launch_topk(logits_last, c.vocab, c.vocab, 1, 1, x->cand, x->topk_ids, x->st); }
        hipMemcpyAsync(next_tok_out, x->topk_ids, sizeof(int), hipMemcpyDeviceToDevice, x->st);
      }
    }
    // ---- draft side: position i pairs with token i+1 (all but the prompt's last position, whose follow-up token
    // does not exist yet): Attention Decoder 1, then the Augmenting Block over its own cache ----
    const int Md = last ? M - 1 : M;
    if (Md > 0) {
      const RowMap rd{1, P, Md, nullptr};
      { Scope s(x, KC_EMBED);
        launch_pass_start(PassStart{x->w.lm_head, tokens + c0 + 1, c.vocab, x->d_e, H, H, rd, rope_rows(x, aug_len_b), nullptr, 0.f, {}},
                          c.dtype, x->st); }
      run_ad(x, x->w.ad1, xres, x->d_e, Md, x->xd);
      if (x->fast) norm_planes(x, x->xd, x->aug[0].attn_norm, Md);
      const AttnPlan plan_d = plan_attention(x, &x->aug_ub[b], rd, Md, true);
      for (int l = 0; l < c.aug_layers; ++l)
        run_layer(x, x->aug[l], x->xd, rd, Md, x->aug_kc + (size_t)l * x->k_layer_elems * x->kv_esz,
                  x->aug_vc + (size_t)l * x->v_layer_elems * x->kv_esz, aug_len_b, nullptr,
                  l + 1 < c.aug_layers ? x->aug[l + 1].attn_norm : nullptr, plan_d, 0, nullptr, b);
      { Scope s(x, KC_DRAFT_MISC); launch_add_scalar(aug_len_b, Md, x->st); }
      x->aug_ub[b] += Md;
    }
  }
  if (x->only_prefills) x->m_upper = 1;
  return finish(x, "clover_prefill");
}

int clover_set_page_table(clover_ctx* x, const int32_t* table_host) {
  if (!x) return fail(x, CLOVER_E_NULL, "null argument");
  if (!table_host) {   // back to the identity mapping
    x->kv.pages = nullptr;
    return CLOVER_OK;
  }
  const int n = x->cfg.max_batch * x->kv.T;
  std::vector<char> seen((size_t)n, 0);
  for (int i = 0; i < n; ++i) {
    const int pg = table_host[i];
    if (pg < 0 || pg >= n || seen[pg]) return fail(x, CLOVER_E_SHAPE, "page table must be a permutation of 0 .. max_batch * max_seq / 32 - 1");
    seen[pg] = 1;
  }
  hipError_t e = hipMemcpyAsync(x->d_pages, table_host, (size_t)n * sizeof(int), hipMemcpyHostToDevice, x->st);
  if (e == hipSuccess) e = hipStreamSynchronize(x->st);
  if (e != hipSuccess) return fail(x, CLOVER_E_HIP, std::string("page table upload: ") + hipGetErrorString(e));
  x->kv.pages = x->d_pages;
  return CLOVER_OK;
}

int clover_seq_len(clover_ctx* x, int32_t* out_host) {
  if (!x || !out_host) return fail(x, CLOVER_E_NULL, "null argument");
  const int B = x->cfg.max_batch;
  std::vector<int> aug(B);
  int err = 0;
  hipError_t e = hipMemcpyAsync(out_host, x->d_seq_len, B * sizeof(int), hipMemcpyDeviceToHost, x->st);
  if (e == hipSuccess) e = hipMemcpyAsync(aug.data(), x->d_aug_len, B * sizeof(int), hipMemcpyDeviceToHost, x->st);
  if (e == hipSuccess) e = hipMemcpyAsync(&err, x->d_err, sizeof(int), hipMemcpyDeviceToHost, x->st);
  if (e == hipSuccess) e = hipStreamSynchronize(x->st);
  if (e != hipSuccess) return fail(x, CLOVER_E_HIP, std::string("clover_seq_len: ") + hipGetErrorString(e));
  for (int b = 0; b < B; ++b) { x->len_ub[b] = out_host[b]; x->aug_ub[b] = aug[b]; }
  if (err) return fail(x, CLOVER_E_STATE, "a kernel refused to write past max_seq");
  return CLOVER_OK;
}

int clover_read_kv(clover_ctx* x, int32_t stack, int32_t layer, int32_t b, int32_t slot0, int32_t n_slots,
                   float* k_out_host, float* v_out_host) {
  if (!x || !k_out_host || !v_out_host) return fail(x, CLOVER_E_NULL, "null argument");
  const clover_config& c = x->cfg;
  const int nl = stack == 0 ? c.n_layers : c.aug_layers;
  if (stack < 0 || stack > 1 || layer < 0 || layer >= nl || b < 0 || b >= c.max_batch || slot0 < 0 || n_slots < 0 ||
      slot0 + n_slots > c.max_seq)
    return fail(x, CLOVER_E_SHAPE, "clover_read_kv: index out of range");
  const size_t n = (size_t)n_slots * c.n_kv_heads * c.head_dim;
  if (2 * n > (size_t)x->rows * c.vocab) return fail(x, CLOVER_E_SHAPE, "clover_read_kv: too many slots at once");
  if (n == 0) return CLOVER_OK;
  const char* kbase = (stack == 0 ? x->kc : x->aug_kc) + (size_t)layer * x->k_layer_elems * x->kv_esz;
  const char* vbase = (stack == 0 ? x->vc : x->aug_vc) + (size_t)layer * x->v_layer_elems * x->kv_esz;
  launch_read_kv(kbase, vbase, x->kvdtype, x->kv, b, slot0, n_slots, x->z, x->z + n, x->st);
  hipError_t e = hipMemcpyAsync(k_out_host, x->z, n * sizeof(float), hipMemcpyDeviceToHost, x->st);
  if (e == hipSuccess) e = hipMemcpyAsync(v_out_host, x->z + n, n * sizeof(float), hipMemcpyDeviceToHost, x->st);
  if (e == hipSuccess) e = hipStreamSynchronize(x->st);
  if (e != hipSuccess) return fail(x, CLOVER_E_HIP, std::string("clover_read_kv: ") + hipGetErrorString(e));
  return CLOVER_OK;
}

int clover_write_kv(clover_ctx* x, int32_t stack, int32_t layer, int32_t b, int32_t slot0, int32_t n_slots,
                    const float* k_in_host, const float* v_in_host) {
  if (!x || !k_in_host || !v_in_host) return fail(x, CLOVER_E_NULL, "null argument");
  const clover_config& c = x->cfg;
  const int nl = stack == 0 ? c.n_layers : c.aug_layers;
  if (stack < 0 || stack > 1 || layer < 0 || layer >= nl || b < 0 || b >= c.max_batch || slot0 < 0 || n_slots < 0 ||
      slot0 + n_slots > c.max_seq)
    return fail(x, CLOVER_E_SHAPE, "clover_write_kv: index out of range");
  const size_t n = (size_t)n_slots * c.n_kv_heads * c.head_dim;
  if (2 * n > (size_t)x->rows * c.vocab) return fail(x, CLOVER_E_SHAPE, "clover_write_kv: too many slots at once");
  if (n == 0) return CLOVER_OK;
  char* kbase = (stack == 0 ? x->kc : x->aug_kc) + (size_t)layer * x->k_layer_elems * x->kv_esz;
  char* vbase = (stack == 0 ? x->vc : x->aug_vc) + (size_t)layer * x->v_layer_elems * x->kv_esz;
  hipError_t e = hipMemcpyAsync(x->z, k_in_host, n * sizeof(float), hipMemcpyHostToDevice, x->st);
  if (e == hipSuccess) e = hipMemcpyAsync(x->z + n, v_in_host, n * sizeof(float), hipMemcpyHostToDevice, x->st);
  if (e == hipSuccess) {
    launch_write_kv(kbase, vbase, x->kvdtype, x->kv, b, slot0, n_slots, x->z, x->z + n, x->st);
    e = hipStreamSynchronize(x->st);   // the host arrays and the staging area are free again on return
  }
  if (e != hipSuccess) return fail(x, CLOVER_E_HIP, std::string("clover_write_kv: ") + hipGetErrorString(e));
  return CLOVER_OK;
}

int clover_set_seq_len(clover_ctx* x, const int32_t* len_host, const int32_t* aug_len_host) {
  if (!x || !len_host || !aug_len_host) return fail(x, CLOVER_E_NULL, "null argument");
  const int B = x->cfg.max_batch;
  for (int b = 0; b < B; ++b)
    if (len_host[b] < 0 || len_host[b] > x->cfg.max_seq || aug_len_host[b] < 0 || aug_len_host[b] > x->cfg.max_seq)
      return fail(x, CLOVER_E_CAPACITY, "clover_set_seq_len: length outside [0, max_seq]");
  hipError_t e = hipMemcpyAsync(x->d_seq_len, len_host, B * sizeof(int), hipMemcpyHostToDevice, x->st);
  if (e == hipSuccess) e = hipMemcpyAsync(x->d_aug_len, aug_len_host, B * sizeof(int), hipMemcpyHostToDevice, x->st);
  if (e == hipSuccess) e = hipStreamSynchronize(x->st);
  if (e != hipSuccess) return fail(x, CLOVER_E_HIP, std::string("clover_set_seq_len: ") + hipGetErrorString(e));
  for (int b = 0; b < B; ++b) { x->len_ub[b] = len_host[b]; x->aug_ub[b] = aug_len_host[b]; }
  return CLOVER_OK;
}

int clover_capture_draft_logits(clover_ctx* x, float* dev_out, size_t capacity_floats) {
  if (!x) return CLOVER_E_NULL;
  x->draft_capture = dev_out;
  x->draft_capture_floats = dev_out ? capacity_floats : 0;
  return CLOVER_OK;
}

int clover_profile_enable(clover_ctx* x, int32_t on) {
  if (!x) return CLOVER_E_NULL;
  x->prof = on != 0;
  return CLOVER_OK;
}

int clover_profile_collect(clover_ctx* x, double* ms, int64_t* launches, int32_t n_classes) {
  if (!x || !ms || !launches) return fail(x, CLOVER_E_NULL, "null argument");
  if (n_classes < KC_COUNT) return fail(x, CLOVER_E_SHAPE, "n_classes too small");
  for (int i = 0; i < n_classes; ++i) { ms[i] = 0.0; launches[i] = 0; }
  hipError_t e = hipStreamSynchronize(x->st);
  if (e != hipSuccess) return fail(x, CLOVER_E_HIP, hipGetErrorString(e));
  for (ProfEvent& ev : x->prof_events) {
    float t = 0.f;
    if (hipEventElapsedTime(&t, ev.a, ev.b) == hipSuccess) { ms[ev.cls] += t; launches[ev.cls] += 1; }
    x->prof_pool.push_back(ev);
  }
  x->prof_events.clear();
  return CLOVER_OK;
}

int clover_path_info(clover_ctx* x) {
  if (!x) return CLOVER_E_NULL;
  return (x->fast ? 1 : 0) | (x->attn_fast ? 2 : 0);
}

int clover_kernel_class_count(void) { return KC_COUNT; }
const char* clover_kernel_class_name(int32_t cls) { return (cls >= 0 && cls < KC_COUNT) ? kClassNames[cls] : ""; }

const char* clover_last_error(clover_ctx* x) { return x ? x->err.c_str() : ""; }
const char* clover_last_global_error(void) { return g_err.c_str(); }

// ---- operator entry points ----
// Their limits belong to the interface and stay fixed; the kernel's own choices (tile, K ranges) vary underneath.

// K ranges of a narrow output with a long K, for the paths that require them: ranges of at least four steps (256 columns,
// 128 from 65 rows on) of 128-column tiles that fill most of the chip.  0: the shape has none.
static int op_gemm_k_ranges(int M, int N, int K) {
  const int st = M > 64 ? 128 : 256, wgs_n = (N / 32 + 3) / 4, NS = K / st;
  if (M > 128 || K % st != 0 || N % 32 != 0) return 0;
  int best = 0;
  for (int d = 1; d <= NS; ++d)
    if (NS % d == 0 && wgs_n * d <= 256 && NS / d >= 4) best = d;
  return best > 1 && wgs_n * best >= (M > 64 ? 160 : 224) ? best : 0;
}
// Partial tiles [M, N] that the scratch size counts; the kernel never gets more K ranges than this.
static int op_gemm_counted_parts(int M, int N, int K) {
  if (M <= 64 && N % 32 == 0) return (K + 511) / 512;
  int parts = op_gemm_k_ranges(M, N, K);
  const int tiles = (N + 255) / 256 * (M > 128 ? 2 : 1);
  for (int d = 1; d <= K / 512; ++d)
    if (K / 64 % d == 0 && tiles * d <= 256) parts = std::max(parts, d);
  const int cols = N % 32 == 0 && N >= 8192 ? 128 : 64, steps = K / (M <= 64 ? 128 : M <= 128 ? 64 : 32);
  int s = 1;
  while ((N + cols - 1) / cols * s < 256 && s * 8 <= steps && (size_t)s * M * 32 <= (size_t)K * 2) s *= 2;
  return std::max(parts, s);
}
// [packed weight copy][activation planes][partial tiles].  counted: with M rows of planes and the counted partial tiles;
// total: what the launch uses, whole row blocks of planes and its own K ranges.
struct OpGemmScratch { size_t planes, partial, total, counted; int kp; };
static OpGemmScratch op_gemm_scratch(int M, int N, int K) {
  OpGemmScratch o;
  const int parts = op_gemm_counted_parts(M, N, K);
  o.kp = tile_gemm_pick_k_parts(M, N, K);
  if (o.kp > parts) o.kp = 1;
  o.planes = align256((size_t)N * K * 2);
  o.partial = o.planes + align256((size_t)((M + 15) / 16 * 16) * K * 4);
  o.total = 256 + o.partial + align256((size_t)o.kp * M * N * sizeof(float));
  o.counted = 256 + o.planes + align256((size_t)M * K * 4) + align256((size_t)parts * M * N * sizeof(float));
  return o;
}
size_t clover_op_gemm_scratch_bytes(int32_t M, int32_t N, int32_t K) {
  if (M < 1 || N < 1 || K < 1 || M > 256 || !mfma_shape_ok(N, K)) return 256;
  const OpGemmScratch o = op_gemm_scratch(M, N, K);
  return std::max(o.counted, o.total);
}

int clover_op_gemm(int32_t path, int32_t dtype, const float* X, const void* W, float* Y, int32_t ldy, int32_t M,
                   int32_t N, int32_t K, void* scratch, size_t scratch_bytes, void* hip_stream) {
  return op_gemm_impl(path, dtype, X, W, Y, ldy, M, N, K, scratch, scratch_bytes, hip_stream);
}

int clover_op_gemm_static(int32_t path, int32_t dtype, const float* X, const void* W, float* Y, int32_t ldy, int32_t M,
                          int32_t N, int32_t K, void* hip_stream) {
  if (path != 0 && path != 1 && path != 3 && path != 5)
    return fail(nullptr, CLOVER_E_SHAPE, "clover_op_gemm_static: path must be 0, 1, 3 or 5 (the shared buffer keeps no copy between calls)");
  const bool mfma = M >= 1 && N >= 1 && K >= 1 && M <= 256 && mfma_shape_ok(N, K);
  const OpGemmScratch o = mfma ? op_gemm_scratch(M, N, K) : OpGemmScratch{};
  if (o.counted > CLOVER_STATIC_SCRATCH_BYTES)
    return fail(nullptr, CLOVER_E_CAPACITY, "clover_op_gemm_static: M, N, K need more than CLOVER_STATIC_SCRATCH_BYTES of scratch");
  void* ptr = nullptr;
  const int rc = static_scratch_ptr(&ptr);
  if (rc) return rc;
  return op_gemm_impl(path, dtype, X, W, Y, ldy, M, N, K, ptr, kStaticScratch, hip_stream);
}

size_t clover_op_swiglu_scratch_bytes(int32_t M, int32_t F, int32_t K) {
  if (M < 1 || F < 1 || K < 1) return 256;
  return 256 + align256((size_t)2 * F * K * 2) + align256((size_t)((M + 15) / 16 * 16) * K * 4);
}
int clover_op_swiglu(const float* X, const void* Wg, const void* Wu, void* planes, int32_t M, int32_t F, int32_t K,
                     void* scratch, size_t scratch_bytes, void* hip_stream) {
  if (!X || !Wg || !Wu || !planes || !scratch) return fail(nullptr, CLOVER_E_NULL, "null argument");
  if (M < 1 || M > 1024 || F < 1 || K < 1 || F % 32 != 0 || !mfma_shape_ok(F, K)) return fail(nullptr, CLOVER_E_SHAPE, "shape not supported by the MFMA GEMM");
  if (scratch_bytes < clover_op_swiglu_scratch_bytes(M, F, K)) return fail(nullptr, CLOVER_E_CAPACITY, "scratch too small");
  hipStream_t st = (hipStream_t)hip_stream;
  launch_pack_gate_up(Wg, Wu, scratch, F, K, st);
  TileGemm g;
  memset(&g, 0, sizeof(g));
  g.X = frag_planes((char*)scratch + align256((size_t)2 * F * K * 2), M);
  launch_split_planes(X, K, g.X, M, K, st);
  g.W = (const bf16_t*)scratch;
  g.out = frag_planes(planes, M);
  g.M = M; g.N = F; g.K = K; g.epi = 1; g.k_parts = 1;
  launch_gemm_tile(g, st);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(nullptr, CLOVER_E_HIP, hipGetErrorString(e));
  return CLOVER_OK;
}

static int op_gemm_tile(int epi, int M, int N, int K, int k_parts, const int32_t* out, TileForm& f) {
  if (!out) return fail(nullptr, CLOVER_E_NULL, "null argument");
  if (epi < 0 || epi > 1 || M < 1 || N < 1 || K < 1 || !mfma_shape_ok(N, K) || k_parts < 0 || k_parts > TILE_MAX_K_PARTS ||
      (k_parts > 0 && K / 32 % k_parts != 0) || (epi == 1 && k_parts > 1))
    return fail(nullptr, CLOVER_E_SHAPE, "shape not supported by the MFMA GEMM");
  f = tile_gemm_form(M, N, K, epi, k_parts == 0 && epi == 0 && M <= 256 ? op_gemm_scratch(M, N, K).kp : k_parts);
  return CLOVER_OK;
}
int clover_op_gemm_form(int32_t epi, int32_t M, int32_t N, int32_t K, int32_t k_parts, int32_t form[5]) {
  TileForm f;
  const int rc = op_gemm_tile(epi, M, N, K, k_parts, form, f);
  if (rc) return rc;
  form[0] = f.rb; form[1] = (f.wb + 1) / 2; form[2] = f.row_tiles; form[3] = f.k_parts; form[4] = f.stages;
  return CLOVER_OK;
}
int clover_op_gemm_tile_columns(int32_t epi, int32_t M, int32_t N, int32_t K, int32_t k_parts, int32_t* columns) {
  TileForm f;
  const int rc = op_gemm_tile(epi, M, N, K, k_parts, columns, f);
  if (rc) return rc;
  *columns = 16 * f.wb;
  return CLOVER_OK;
}

}  // extern "C"

namespace {
int op_gemm_impl(int32_t path, int32_t dtype, const float* X, const void* W, float* Y, int32_t ldy, int32_t M,
                 int32_t N, int32_t K, void* scratch, size_t scratch_bytes, void* hip_stream) {
  if (!X || !W || !Y || !scratch) return fail(nullptr, CLOVER_E_NULL, "null argument");
  if (M < 1 || N < 1 || K < 1 || ldy < N) return fail(nullptr, CLOVER_E_SHAPE, "bad GEMM shape");
  hipStream_t st = (hipStream_t)hip_stream;
  if (path == 0) {
    launch_gemm_generic(X, K, W, nullptr, dtype, Y, ldy, M, N, K, 0, st);
  } else {
    if (dtype != CLOVER_DTYPE_BF16 || M > 256 || !mfma_shape_ok(N, K))
      return fail(nullptr, CLOVER_E_SHAPE, "shape not supported by the MFMA GEMM");
    if (path >= 3 && path != 7) {
      if (M > 128 || K % (M > 64 ? 128 : 256) != 0 || ldy % 4 != 0)
        return fail(nullptr, CLOVER_E_SHAPE, "shape not supported over the whole K");
      if (path >= 5 && op_gemm_k_ranges(M, N, K) == 0)
        return fail(nullptr, CLOVER_E_SHAPE, "shape not supported over K ranges");
    }
    const OpGemmScratch o = op_gemm_scratch(M, N, K);
    if (scratch_bytes < std::max(o.counted, o.total)) return fail(nullptr, CLOVER_E_CAPACITY, "scratch too small");
    // the weight copy is made once per scratch buffer contents, so repeated calls with the same W measure the GEMM
    // alone (the even paths skip it)
    if (path & 1) launch_pack_weight(W, scratch, N, K, 0, N, st);
    TileGemm g;
    memset(&g, 0, sizeof(g));
    g.X = frag_planes((char*)scratch + o.planes, M);
    launch_split_planes(X, K, g.X, M, K, st);
    g.W = (const bf16_t*)scratch;
    g.M = M; g.N = N; g.K = K; g.epi = 0;
    if (path == 3 || path == 4) {
      g.Y = Y; g.ldy = ldy; g.k_parts = 1;
      launch_gemm_tile(g, st);
    } else {
      g.Y = (float*)((char*)scratch + o.partial); g.ldy = N; g.split_stride = (size_t)M * N;
      g.k_parts = o.kp;
      launch_gemm_tile(g, st);
      launch_reduce(g.Y, g.k_parts, g.split_stride, N, nullptr, dtype, Y, ldy, M, N, 0, st);
    }
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(nullptr, CLOVER_E_HIP, hipGetErrorString(e));
  return CLOVER_OK;
}

}  // namespace
