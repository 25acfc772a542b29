// Dynamic (score-pruned) draft tree: the kernels between the draft head's LM-head passes.
//
// Candidates of one sequence are numbered in creation order: 0 = root, then the depth-1 candidates in rank
// order, then for every depth the children of the expanded candidates in (expansion slot, rank) order, so the
// id of a candidate encodes its depth, the slot of its parent in that depth's frontier and its rank.  A
// candidate's score is the sum of the draft log-probabilities along its root path.  Per depth the best
// candidates (score descending, lower id first) are expanded; at the end the best n_nodes - 1 candidates
// (score descending, shallower first, lower id first) become the tree, numbered breadth-first (depth, parent's
// number, rank), and the per-sequence topology tables the verification pass reads are written.
#include "clover_internal.h"

#include <climits>

namespace clv {

namespace {

__device__ __forceinline__ float d_wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ float d_wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
// order-preserving 64-bit key of (value, id): larger value first, then the smaller id
__device__ __forceinline__ unsigned long long d_key(float v, int id) {
  v = v + 0.0f;
  unsigned u = __float_as_uint(v);
  u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return ((unsigned long long)u << 32) | (unsigned long long)(0xFFFFFFFFu - (unsigned)id);
}
__device__ __forceinline__ float d_key_value(unsigned long long key) {
  const unsigned u = (unsigned)(key >> 32);
  return __uint_as_float((u & 0x80000000u) ? (u & 0x7FFFFFFFu) : ~u);
}
constexpr int DY_CHUNK = 2048;
constexpr int DY_EPT = DY_CHUNK / 256;

// stage 1: per 2048-wide chunk of a row of logits, its k best (value, id) keys, its maximum and the sum of
// exp(value - maximum) (the pieces of the row's log-sum-exp)
__global__ __launch_bounds__(256) void topk_lse_stage1_kernel(const float* __restrict__ z, int ldz, int V, int k,
                                                              unsigned long long* __restrict__ cand,
                                                              float* __restrict__ aux, float scale) {
  __shared__ unsigned long long red[2][4];
  __shared__ float fred[4];
  const int chunk = blockIdx.x, row = blockIdx.y, chunks = gridDim.x;
  unsigned long long key[DY_EPT];
  float val[DY_EPT];
  float mx = -INFINITY;
#pragma unroll
  for (int e = 0; e < DY_EPT; ++e) {
    const int id = chunk * DY_CHUNK + e * 256 + threadIdx.x;
    val[e] = id < V ? z[(size_t)row * ldz + id] * scale : -INFINITY;
    key[e] = id < V ? d_key(val[e], id) : 0ull;
    mx = fmaxf(mx, val[e]);
  }
  mx = d_wave_max(mx);
  if ((threadIdx.x & 63) == 0) fred[threadIdx.x >> 6] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(fred[0], fred[1]), fmaxf(fred[2], fred[3]));
  __syncthreads();
  float sm = 0.f;
#pragma unroll
  for (int e = 0; e < DY_EPT; ++e) sm += val[e] == -INFINITY ? 0.f : expf(val[e] - mx);
  sm = d_wave_sum(sm);
  if ((threadIdx.x & 63) == 0) fred[threadIdx.x >> 6] = sm;
  __syncthreads();
  if (threadIdx.x == 0) {
    aux[((size_t)row * chunks + chunk) * 2] = mx;
    aux[((size_t)row * chunks + chunk) * 2 + 1] = fred[0] + fred[1] + fred[2] + fred[3];
  }
  for (int r = 0; r < k; ++r) {
    unsigned long long best = 0ull;
#pragma unroll
    for (int e = 0; e < DY_EPT; ++e) best = key[e] > best ? key[e] : best;
    best = block_max_key(best, red, r);
#pragma unroll
    for (int e = 0; e < DY_EPT; ++e)
      if (key[e] == best) key[e] = 0ull;
    if (threadIdx.x == 0) cand[((size_t)row * chunks + chunk) * 16 + r] = best;
  }
}

// stage 2: the row's log-sum-exp (chunks merged in chunk order by one thread, so the sum does not depend on the launch
// shape) and, for a dynamic tree, its k best entries as the children of its candidate
__global__ __launch_bounds__(256) void topk_lse_stage2_kernel(const unsigned long long* __restrict__ cand,
                                                              const float* __restrict__ aux, int chunks, int k,
                                                              float* __restrict__ out_lse, DynTree to, int j, const int* __restrict__ m) {
  __shared__ unsigned long long red[2][4];
  const int row = blockIdx.x;
  const int total = chunks * k;
  unsigned long long key[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int idx = e * 256 + threadIdx.x;
    key[e] = idx < total ? cand[((size_t)row * chunks + idx / k) * 16 + idx % k] : 0ull;
  }
  // (the terms by all threads into the LDS, their sum in order by one: as a loop over global memory this was the kernel's
  // 16 us)
  __shared__ float fred[4], term[256];
  float M = -INFINITY;
  for (int c = threadIdx.x; c < chunks; c += 256) M = fmaxf(M, aux[((size_t)row * chunks + c) * 2]);
  M = d_wave_max(M);
  if ((threadIdx.x & 63) == 0) fred[threadIdx.x >> 6] = M;
  __syncthreads();
  M = fmaxf(fmaxf(fred[0], fred[1]), fmaxf(fred[2], fred[3]));
  float S = 0.f;
  for (int c0 = 0; c0 < chunks; c0 += 256) {
    const int c = c0 + threadIdx.x;
    if (c < chunks) term[threadIdx.x] = aux[((size_t)row * chunks + c) * 2 + 1] * expf(aux[((size_t)row * chunks + c) * 2] - M);
    __syncthreads();
    if (threadIdx.x == 0)
      for (int i = 0; i < min(256, chunks - c0); ++i) S += term[i];
    __syncthreads();
  }
  __shared__ int ids[16];
  __shared__ float vals[16], lse;
  if (threadIdx.x == 0) out_lse[row] = lse = M + logf(S);
  if (!to.cand_tok) return;   // (uniform)
  for (int r = 0; r < k; ++r) {
    unsigned long long best = 0ull;
#pragma unroll
    for (int e = 0; e < 8; ++e) best = key[e] > best ? key[e] : best;
    best = block_max_key(best, red, r);
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (key[e] == best) key[e] = 0ull;
    if (threadIdx.x == 0) {
      ids[r] = (int)(0xFFFFFFFFu - (unsigned)(best & 0xFFFFFFFFull));
      vals[r] = d_key_value(best);
    }
  }
  __syncthreads();
  // children of the candidate that this row ranked: token, cumulative score, parent
  const int b = row / to.F[j], r = row - b * to.F[j], i = threadIdx.x;
  if (i >= to.topk || m[b] < 1) return;
  const int par = j == 0 ? 0 : to.frontier[((size_t)b * CLOVER_MAX_DEPTH + j) * DYN_MAX_FRONT + r];
  const int cid = to.off[j + 1] + r * to.topk + i;
  const size_t o = (size_t)b * to.C;
  to.cand_tok[o + cid] = ids[i];
  to.cand_score[o + cid] = (j == 0 ? 0.f : to.cand_score[o + par]) + (vals[i] - lse);
  to.cand_par[o + cid] = par;
}

// A score that is no number (its logits were none, or infinite) ranks as minus infinity: every candidate then has a place of its
// own in the order, behind its parent, and no more candidates are kept than there are nodes.
__device__ __forceinline__ float rank_score(float s) { return s == s ? s : -INFINITY; }

// frontier of depth j: the F[j] best of its candidates (score descending, lower id first), in that order
__global__ __launch_bounds__(256) void dyn_frontier_kernel(DynTree t, int j, const int* __restrict__ m) {
  __shared__ float sc[DYN_MAX_CAND];
  const int b = blockIdx.x, tid = threadIdx.x;
  if (m[b] < 1) return;
  const int n = t.off[j + 1] - t.off[j];
  const size_t o = (size_t)b * t.C;
  if (tid < n) sc[tid] = rank_score(t.cand_score[o + t.off[j] + tid]);
  __syncthreads();
  if (tid >= n) return;
  int better = 0;
#pragma unroll 8
  for (int u = 0; u < n; ++u) better += (sc[u] > sc[tid] || (sc[u] == sc[tid] && u < tid)) ? 1 : 0;
  if (better < t.F[j]) t.frontier[((size_t)b * CLOVER_MAX_DEPTH + j) * DYN_MAX_FRONT + better] = t.off[j] + tid;
}

// selection of the tree and its breadth-first numbering; per-sequence topology tables.  One workgroup per sequence, a chain of steps
// over the LDS; every count is a loop of independent reads, unrolled (150 candidates, 40 nodes, 4 depths: 31 us with dependent reads
// and the labels numbered by one thread, 11 so).
__global__ __launch_bounds__(DYN_MAX_CAND) void dyn_finalize_kernel(DynTree t, int R, const int* __restrict__ m,
                                                                   int* __restrict__ tree_tokens) {
  __shared__ float sc[DYN_MAX_CAND];
  __shared__ int par[DYN_MAX_CAND], key[DYN_MAX_CAND], nid[DYN_MAX_CAND];
  __shared__ int n_child[CLOVER_MAX_NODES], first_child[CLOVER_MAX_NODES];
  __shared__ unsigned long long anc[CLOVER_MAX_NODES][2];
  __shared__ int sub[CLOVER_MAX_NODES], ent[CLOVER_MAX_NODES];   // subtree size, enter label
  __shared__ int level_count;
  const int b = blockIdx.x, c = threadIdx.x;
  if (m[b] < 1) return;
  const size_t o = (size_t)b * t.C;
  const bool live = c < t.C;
  int my_dep = 0;
  if (live) {
    for (int j = 1; j <= t.D; ++j) my_dep += c >= t.off[j] ? 1 : 0;
    sc[c] = c == 0 ? INFINITY : rank_score(t.cand_score[o + c]);
    par[c] = c == 0 ? 0 : t.cand_par[o + c];
  }
  if (c < CLOVER_MAX_NODES) { n_child[c] = 0; first_child[c] = INT_MAX; anc[c][0] = anc[c][1] = 0ull; }
  if (c == 0) nid[0] = 0;   // (read by other threads in front of the next barrier)
  __syncthreads();
  int keep = 0;
  if (live) {
    int better = 0;   // candidates (the root included) that come before this one: higher scores, among equals shallower ones, then
#pragma unroll 8          // lower ids -- which are in order of depth
    for (int u = 0; u < t.C; ++u) better += sc[u] > sc[c] || (sc[u] == sc[c] && u < c) ? 1 : 0;
    keep = better < t.N ? 1 : 0;
  }
  int base = 1;
  for (int j = 1; j <= t.D; ++j) {
    if (c == 0) level_count = 0;
    const bool here = live && my_dep == j;
    const int mine = here && keep ? nid[par[c]] * 16 + (c - t.off[j]) % t.topk : INT_MAX;
    if (here) key[c] = mine;
    __syncthreads();
    if (here && keep) {
      int pos = 0;
#pragma unroll 8
      for (int u = t.off[j]; u < t.off[j + 1]; ++u) pos += key[u] < mine ? 1 : 0;
      nid[c] = base + pos;
      atomicAdd(&level_count, 1);
    }
    __syncthreads();
    base += level_count;
    __syncthreads();
  }
  // tables
  const size_t ro = (size_t)b * R;
  if (live && keep) {
    const int node = nid[c];
    const int pn = c == 0 ? -1 : nid[par[c]];
    tree_tokens[ro + node] = t.cand_tok[o + c];
    t.t_parent[ro + node] = pn;
    t.t_rank[ro + node] = c == 0 ? 0 : (c - t.off[my_dep]) % t.topk;
    t.t_depth[ro + node] = my_dep;
    t.t_keep[ro + node] = c;
    if (c > 0) { atomicAdd(&n_child[pn], 1); atomicMin(&first_child[pn], node); }
  }
  if (c == 0) anc[0][0] = 1ull;
  for (int j = 1; j <= t.D; ++j) {
    __syncthreads();
    if (live && keep && my_dep == j) {
      const int node = nid[c], pn = nid[par[c]];
      anc[node][0] = anc[pn][0];
      anc[node][1] = anc[pn][1];
      anc[node][node >> 6] |= 1ull << (node & 63);
    }
  }
  __syncthreads();
  // interval labels of a depth-first numbering (the linear-size form of the mask): the size of a subtree counts the nodes whose
  // path holds its root; a node enters behind its parent and its earlier siblings' subtrees, depth by depth
  if (c < t.N) {
    int size = 0;
#pragma unroll 8
    for (int v = 0; v < t.N; ++v) size += (int)(anc[v][c >> 6] >> (c & 63) & 1ull);
    sub[c] = size;
  }
  if (c == 0) ent[0] = 0;
  for (int j = 1; j <= t.D; ++j) {
    __syncthreads();
    if (live && keep && my_dep == j) {
      const int node = nid[c], pn = nid[par[c]];
      int e = ent[pn] + 1;
      for (int s = first_child[pn]; s < node; ++s) e += sub[s];
      ent[node] = e;
    }
  }
  __syncthreads();
  if (c < t.N) {
    t.t_n_child[ro + c] = n_child[c];
    t.t_first_child[ro + c] = n_child[c] ? first_child[c] : 0;
    t.t_anc[(ro + c) * 2] = anc[c][0];
    t.t_anc[(ro + c) * 2 + 1] = anc[c][1];
    t.t_iv[(ro + c) * 2] = ent[c];
    t.t_iv[(ro + c) * 2 + 1] = ent[c] + sub[c] - 1;
  }
}

// Verification at a temperature > 0, in three launches.
//   walk   one wavefront per sequence: at node u with p = softmax(logits[u] / T), the children (one per lane) are tried
//          in index order, child i accepted when uniforms[u][i] < p(token) / (1 - mass of the children already refused)
//   mass   where none is accepted (or u is a leaf) the next token is drawn from what is left of p (refused tokens
//          removed): its mass per chunk of 2048 tokens, one workgroup each
//   pick   inverts the cumulative sum in token order with uniforms[u][16]: the chunk first, then the token in it
// Sums are carried in double precision.  What bounds it is one sequence's row of V exponentials in double precision: a
// single workgroup that summed the row and searched it took 290 us at V = 128256; spread over 63 workgroups the row
// is a few us and the search reads one chunk again.
constexpr int SAMPLE_CHUNK = 2048;   // tokens per chunk, 8 adjacent ones per thread
__global__ __launch_bounds__(64) void sample_walk_kernel(
    const float* __restrict__ logits, int V, const float* __restrict__ lse, float inv_temp, const int* __restrict__ tokens,
    const int* __restrict__ first_child, const int* __restrict__ n_child, int child_stride, int R,
    const float* __restrict__ uniforms, int* __restrict__ m, int* __restrict__ acc_idx, int* __restrict__ new_tokens,
    int* __restrict__ next_tok, int* __restrict__ seq_len) {
  const int b = blockIdx.x, lane = threadIdx.x;
  const size_t o = (size_t)b * R;
  first_child += (size_t)b * child_stride;
  n_child += (size_t)b * child_stride;
  int u = 0, len = 1;
  if (lane == 0) acc_idx[o] = 0;
  for (;;) {   // (uniform: every lane takes the same decisions)
    const int c0 = first_child[u], nk = min(n_child[u], CLOVER_MAX_RANK);
    const double l = (double)lse[o + u];
    int x = -1;
    double px = 0.0, un = 1.0;
    if (lane < nk) {
      x = tokens[o + c0 + lane];
      if (x >= 0 && x < V) px = exp((double)(logits[(o + u) * (size_t)V + x] * inv_temp) - l);
      un = (double)uniforms[(o + u) * 17 + lane];
    }
    double refused = 0.0;
    int accepted = -1;
    for (int i = 0; i < nk; ++i) {
      const double pi = __shfl(px, i, 64);
      if (__shfl(un, i, 64) < pi / fmax(1.0 - refused, 1e-300)) { accepted = i; break; }
      refused += pi;
    }
    if (accepted < 0 || len >= R) break;
    const int t = __shfl(x, accepted, 64);
    u = c0 + accepted;
    if (lane == 0) {
      acc_idx[o + len] = u;
      new_tokens[o + len - 1] = t;
      next_tok[o + len - 1] = t;
    }
    ++len;
  }
  if (lane == 0) {
    m[b] = len;
    seq_len[b] += len;   // (launch_accept_move subtracts it again)
  }
}

// what is left of p at the last accepted node of a sequence: p without the node's children
struct SampleRest {
  const float* zr;
  double l;
  float inv_temp;
  int nk, kid[CLOVER_MAX_RANK];
  __device__ __forceinline__ SampleRest(const float* logits, int V, const float* lse, float inv_t, const int* tokens,
                                        const int* first_child, const int* n_child, size_t o, int u) {
    zr = logits + (o + u) * (size_t)V;
    l = (double)lse[o + u];
    inv_temp = inv_t;
    nk = min(n_child[u], CLOVER_MAX_RANK);
    const int c0 = first_child[u];
#pragma unroll
    for (int i = 0; i < CLOVER_MAX_RANK; ++i) kid[i] = i < nk ? tokens[o + c0 + i] : -1;
  }
  __device__ __forceinline__ double at(int t) const {
    bool refused = false;
#pragma unroll
    for (int i = 0; i < CLOVER_MAX_RANK; ++i) refused = refused || kid[i] == t;
    return refused ? 0.0 : exp((double)(zr[t] * inv_temp) - l);
  }
};
__device__ __forceinline__ double d_wave_scan(double v) {   // inclusive
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const double w = __shfl_up(v, d, 64);
    if ((int)(threadIdx.x & 63) >= d) v += w;
  }
  return v;
}
__global__ __launch_bounds__(256) void sample_mass_kernel(
    const float* __restrict__ logits, int V, const float* __restrict__ lse, float inv_temp, const int* __restrict__ tokens,
    const int* __restrict__ first_child, const int* __restrict__ n_child, int child_stride, int R, const int* __restrict__ m,
    const int* __restrict__ acc_idx, double* __restrict__ mass) {
  __shared__ double part[4];
  const int b = blockIdx.y, tid = threadIdx.x;
  const size_t o = (size_t)b * R;
  const SampleRest rest(logits, V, lse, inv_temp, tokens, first_child + (size_t)b * child_stride, n_child + (size_t)b * child_stride, o,
                        acc_idx[o + m[b] - 1]);
  const int t0 = blockIdx.x * SAMPLE_CHUNK + tid * 8;
  double mine = 0.0;
#pragma unroll
  for (int e = 0; e < 8; ++e)
    if (t0 + e < V) mine += rest.at(t0 + e);
  const double incl = d_wave_scan(mine);
  if ((tid & 63) == 63) part[tid >> 6] = incl;
  __syncthreads();
  if (tid == 0) mass[(size_t)b * gridDim.x + blockIdx.x] = ((part[0] + part[1]) + part[2]) + part[3];
}
__global__ __launch_bounds__(256) void sample_pick_kernel(
    const float* __restrict__ logits, int V, const float* __restrict__ lse, float inv_temp, const int* __restrict__ tokens,
    const int* __restrict__ first_child, const int* __restrict__ n_child, int child_stride, int R,
    const float* __restrict__ uniforms, const int* __restrict__ m, const int* __restrict__ acc_idx,
    const double* __restrict__ mass, int chunks, int* __restrict__ new_tokens, int* __restrict__ next_tok) {
  __shared__ double part[4], s_before, s_target;
  __shared__ int s_chunk, s_first, s_last, s_pick;
  const int b = blockIdx.x, tid = threadIdx.x, len = m[b];
  const size_t o = (size_t)b * R;
  const int u = acc_idx[o + len - 1];
  const SampleRest rest(logits, V, lse, inv_temp, tokens, first_child + (size_t)b * child_stride, n_child + (size_t)b * child_stride, o, u);
  // At every level the choice is the first of those with mass whose running sum exceeds the target: one chunk, one thread,
  // one token, whatever the rounding of sums taken in different orders.
  if (tid < 64) {   // the chunk: prefix sums of 64 chunks at a time, in chunk order
    const double* mb = mass + (size_t)b * chunks;
    double total = 0.0;
    for (int c0 = 0; c0 < chunks; c0 += 64) total += __shfl(d_wave_scan(c0 + tid < chunks ? mb[c0 + tid] : 0.0), 63, 64);
    const double target = (double)uniforms[(o + u) * 17 + 16] * total;
    double run = 0.0, before = 0.0;
    int chunk = -1;
    for (int c0 = 0; c0 < chunks && chunk < 0; c0 += 64) {   // (uniform over the wavefront)
      const double mine = c0 + tid < chunks ? mb[c0 + tid] : 0.0, incl = d_wave_scan(mine);
      const unsigned long long beyond = __ballot(mine > 0.0 && run + incl > target);
      if (beyond) {
        const int lane = __ffsll(beyond) - 1;
        const double upto = __shfl(incl, max(lane - 1, 0), 64);
        chunk = c0 + lane;
        before = lane > 0 ? run + upto : run;
      }
      run += __shfl(incl, 63, 64);
    }
    if (tid == 0) { s_chunk = chunk; s_before = before; s_target = target; s_first = 256; s_last = 0; s_pick = V - 1; }
  }
  __syncthreads();
  const int chunk = s_chunk;
  if (chunk >= 0) {   // uniform over the workgroup
    const int t0 = chunk * SAMPLE_CHUNK + tid * 8;
    const double target = s_target;
    double p[8], mine = 0.0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      p[e] = t0 + e < V ? rest.at(t0 + e) : 0.0;
      mine += p[e];
    }
    const double incl = d_wave_scan(mine);
    if ((tid & 63) == 63) part[tid >> 6] = incl;
    __syncthreads();
    double run = s_before;
    for (int w = 0; w < (tid >> 6); ++w) run += part[w];
    if (mine > 0.0) {
      if (run + incl > target) atomicMin(&s_first, tid);
      atomicMax(&s_last, tid);
    }
    const double upto = __shfl_up(incl, 1, 64);
    if ((tid & 63) > 0) run += upto;
    __syncthreads();
    if (tid == (s_first < 256 ? s_first : s_last)) {   // (the last one where rounding leaves the target at the chunk's end)
      int pick = -1, last = 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        run += p[e];
        if (p[e] > 0.0) {
          last = e;
          if (pick < 0 && run > target) pick = e;
        }
      }
      s_pick = t0 + (pick >= 0 ? pick : last);
    }
    __syncthreads();
  }
  if (tid == 0) {
    new_tokens[o + len - 1] = s_pick;
    next_tok[o + len - 1] = s_pick;
  }
}

}  // namespace

int sample_chunks(int V) { return (V + SAMPLE_CHUNK - 1) / SAMPLE_CHUNK; }
void launch_accept_sample(const float* logits, int V, const float* lse, float inv_temp, const int* tokens,
                          const int* first_child, const int* n_child, int child_stride, int B, int R,
                          const float* uniforms, int* m, int* acc_idx, int* new_tokens, int* next_tok, int* seq_len, double* mass,
                          hipStream_t st) {
  const int chunks = sample_chunks(V);
  sample_walk_kernel<<<B, 64, 0, st>>>(logits, V, lse, inv_temp, tokens, first_child, n_child, child_stride, R, uniforms, m, acc_idx,
                                       new_tokens, next_tok, seq_len);
  sample_mass_kernel<<<dim3(chunks, B), 256, 0, st>>>(logits, V, lse, inv_temp, tokens, first_child, n_child, child_stride, R, m,
                                                      acc_idx, mass);
  sample_pick_kernel<<<B, 256, 0, st>>>(logits, V, lse, inv_temp, tokens, first_child, n_child, child_stride, R, uniforms, m, acc_idx,
                                        mass, chunks, new_tokens, next_tok);
}

void launch_topk_lse(const float* z, int ldz, int V, int rows, int k, void* cand, float* aux, float* out_lse, hipStream_t st,
                     float scale, const DynTree* to, int j, const int* m) {
  if (rows <= 0) return;
  const int chunks = (V + DY_CHUNK - 1) / DY_CHUNK;
  topk_lse_stage1_kernel<<<dim3(chunks, rows), 256, 0, st>>>(z, ldz, V, k, (unsigned long long*)cand, aux, scale);
  topk_lse_stage2_kernel<<<rows, 256, 0, st>>>((const unsigned long long*)cand, aux, chunks, k, out_lse, to ? *to : DynTree{}, j, m);
}
void launch_dyn_frontier(const DynTree& t, int j, int B, const int* m, hipStream_t st) {
  dyn_frontier_kernel<<<B, 256, 0, st>>>(t, j, m);
}
void launch_dyn_finalize(const DynTree& t, int B, int R, const int* m, int* tree_tokens, hipStream_t st) {
  dyn_finalize_kernel<<<B, DYN_MAX_CAND, 0, st>>>(t, R, m, tree_tokens);
}

}  // namespace clv
