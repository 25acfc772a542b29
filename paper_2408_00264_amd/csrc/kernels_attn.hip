// Tree-masked decode attention on the gfx950 matrix cores (head_dim 128).
//
// For one sequence and one KV head, the G query heads that share it and the N tree nodes form
// G*N query rows; they attend to the L cached keys (all visible) and to the N tree keys, of which
// node u sees exactly those on its own root path (one bit per tree node in anc[u]).  Without a mask table
// (anc == null) the nodes form a chain of any length -- a prompt chunk: node u sees tree keys 0..u, and the key tiles
// behind a node group's last row are skipped.  With interval labels (iv: enter and exit of a depth-first numbering,
// two integers per node) tree key w is visible to node u iff enter[w] <= enter[u] <= exit[w]; the labels of the tree
// keys sit in the LDS behind the stage buffers, so the test is two integer compares against LDS values.
//
// Work split: a workgroup = (sequence, KV head, group of 32 to 128 nodes, range of 32-key tiles); its wavefronts are 16 nodes
// each of the G query heads.  K and V^T tiles are staged once per workgroup in LDS and shared by the wavefronts; with several
// ranges every split writes an un-normalised partial (O, reference, running sum) and a small kernel merges them with the
// usual log-sum-exp weights, with one range the workgroup writes the finished rows.
//
// What bounds it: the waits between the steps of a tile (matrix pipe 69 % busy over the 2048-row passes of an 8192-token prompt,
// two workgroups to a CU, 42 % with one, 96 nodes at 8192 keys), so what counts is wavefronts in flight (120 registers and 66 KB of LDS: two workgroups of eight to a
// CU), independent work inside a wavefront (scores of the next tile beside the probabilities of this one) and no exchange
// between lanes.  A launch of few tiles is mostly its first ones: Q, then the tiles that are in no cache, are requested before
// anything is waited for (64 nodes at 1024 keys: scores of the first tile 5 us after the launch's start, 2.7 for two more tiles, 1.9
// for the results).  8B shape, 8 KV heads, us per launch: 64 nodes at 1024 keys 12.6, 96 at 8192 45, 8 x 32 ragged to 2048
// 30, one row at 1024 7.6, prompts in 2048-row passes 342 (8192 tokens, average).  Two blocks of 16 nodes per wavefront (half the
// LDS reads) need 220 registers and with them half the wavefronts: 574 there.  Reading fragments two pairs ahead by
// scheduling barriers: 360.
//
// MFMA mapping (v_mfma_f32_16x16x32_bf16, D[i][j] += sum_k A[i][k] B[j][k]):
//   scores   S^T[key][row] : A = K tile  (16 keys x 32 d),  B = Q (16 rows x 32 d)
//   output   O^T[d][row]   : A = V^T tile (16 d x 32 keys), B = P (16 rows x 32 keys)
// A lane owns one query row in both products (j = lane%16), so the soft-max statistics and the
// rescaling of O never leave the lane, and the eight probabilities a lane computes for the keys
// 8*(lane/16)..+7 of a tile are exactly the B fragment of the second product.
//
// Precision: a random-init stack amplifies bf16 rounding ~20x over 32 layers, so Q, K, V and P are
// all carried as hi + lo bf16 pairs and each product takes three MFMAs (hi*hi, hi*lo, lo*hi).  The
// caches already hold K and V^T as (hi, lo) planes.
#include "clover_internal.h"

#include <algorithm>
#include <cstdlib>
#include <type_traits>

namespace clv {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

union Frag {
  u32x4 u;
  bf16x8 v;
};

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
// (a, b) -> packed hi pair and packed lo pair (round to nearest even through v_cvt_pk_bf16_f32), hi + lo == value to 16
// mantissa bits: six instructions per pair
__device__ __forceinline__ void a_split2(float a, float b, unsigned& hi, unsigned& lo) {
  const f32x2_t v = {a, b};
  const bf16x2_t h = __builtin_convertvector(v, bf16x2_t);
  const bf16x2_t l = __builtin_convertvector(v - __builtin_convertvector(h, f32x2_t), bf16x2_t);
  hi = __builtin_bit_cast(unsigned, h);
  lo = __builtin_bit_cast(unsigned, l);
}

constexpr int AT_D = 128;         // head dim
constexpr int AT_TK = KV_PAGE;    // keys per tile = one page of the caches
// (template parameters: WM wavefronts per query head, MB blocks of 16 nodes per wavefront; a workgroup covers 16 MB WM nodes)
// A staged tile lies in the LDS fragment by fragment: 1 KB blocks in which lane l's 16 bytes sit at l * 16, exactly what
// one 16x32 MFMA operand read takes (a contiguous KB: the LDS's full 256 B/clk).  K: blocks [plane][tt][ks] (16 keys of
// sub-tile tt, head-dim columns 32 ks ..), V^T: blocks [plane][db] (head-dim rows 16 db .., the 32 keys).
constexpr int AT_FRAG = 512;                  // bf16 elements of a fragment block
constexpr int AT_KSTAGE = 16 * AT_FRAG, AT_VSTAGE = 16 * AT_FRAG;   // one staged tile: 16 KB of K, 16 KB of V^T
constexpr int AT_NKB = 2, AT_NVB = 2;         // K and V^T buffers: tile i in buffers i % 2 (four of each, requested three tiles ahead:
                                              // 0.7 to 1 us slower in every launch from 3 to 26 tiles a workgroup)
constexpr int AT_LDS_EL = AT_NKB * AT_KSTAGE + AT_NVB * AT_VSTAGE;
constexpr float LOG2E = 1.44269504088896f;
constexpr float AT_SLACK = 8.f;               // log2 of how far a score may exceed the reference of the soft-max
constexpr int AT_MAX_IV = CLOVER_MAX_NODES_INTERVAL;   // interval labels of the tree keys kept in the LDS

// Wait until at most N of this wavefront's vector-memory loads are outstanding (the vmcnt field of s_waitcnt: bits 3:0
// and 15:14; the other counters are left alone).
template <int N>
__device__ __forceinline__ void wait_staging() {
  static_assert(N >= 0 && N < 64, "vmcnt has six bits");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

template <int G, int WM, int MB>
__global__ __launch_bounds__(64 * G * WM) void attn_mfma_kernel(AttnParams p) {
  constexpr int NODES = 16 * MB * WM;   // nodes per workgroup
  extern __shared__ __attribute__((aligned(16))) bf16_t sm[];  // [2][AT_KSTAGE] [2][AT_VSTAGE] [AT_MAX_IV] labels
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int l16 = lane & 15, g4 = lane >> 4;
  const bool chain = p.anc == nullptr && p.iv == nullptr;
  // Grid: KV heads (ids 8 apart share an XCD), then the node groups that read the same tiles, then the units.  A chain's last nodes
  // see most keys: its node groups are outermost, the last ones first, so that the short ones fill the gaps at the end.
  const int kvh = blockIdx.x, ng = chain ? (int)gridDim.z - 1 - (int)blockIdx.z : (int)blockIdx.y;
  const int unit = chain ? blockIdx.y : blockIdx.z;
  int b, split;
  bool whole;   // the sequence has one range: no partial results
  if (p.plan.tab) {
    const unsigned ent = p.plan.unit[unit];
    b = (int)(ent & 255u); split = (int)(ent >> 8 & 127u); whole = (ent >> 15) != 0;
  } else {
    b = unit / p.plan.most; split = unit - b * p.plan.most; whole = p.plan.most == 1;
  }
  const RowMap& rm = p.rm;
  const int t0 = split * p.plan.tiles;
  const int head = kvh * G + wave % G;
  const int node0 = ng * NODES + (wave / G) * MB * 16;   // this wavefront's first node

  // ---- staging: global -> LDS without a stop in registers.  A wavefront instruction moves one fragment block, a contiguous KB of
  // the cache, which holds the 16 bytes that the MFMA operand layout wants of lane l at l * 16 (K: key 8 (l%16 / 4) + 4 tt +
  // l%16 % 4, columns 32 ks + 8 (l / 16) ..; V^T: row 16 db + l % 16, keys 8 (l / 16) ..).  The 16 blocks of a K and of a V^T
  // tile are dealt to the workgroup's wavefronts.  Key tile t of this sequence is page pages[b * T + t] of the paged caches: K
  // and V^T of (page, KV head) are 16 contiguous KB each.  An address is a uniform base plus the lane's 32-bit offset, so staging costs no vector-ALU instruction.  The compiler is not told that these loads write the LDS (it would wait for all of
  // them before every LDS read that follows): the waits before the barriers below are written by hand.
  constexpr int NT = 64 * G * WM, NW = G * WM;
  constexpr int FPW = 16 / NW;          // K blocks and V^T blocks per wavefront and tile
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const unsigned lane_off = (unsigned)lane * 16u;
  bf16_t* const k_lds = sm;
  bf16_t* const v_lds = sm + AT_NKB * AT_KSTAGE;
  const KVLayout& kv = p.kv;
  // Page numbers: lane l holds the page of tile t0 + 64 r + l of this split, read 64 tiles at a time (a table read per tile
  // would have to be a vector load -- the compiler must assume that the staging statements write memory -- and its wait
  // would drain the staging loads in flight).  page_of(i) then is a lane read: no memory, no wait.
  int pgv;
  auto read_pages = [&](int i) __attribute__((always_inline)) {   // for tiles i .. i + 63 of the split
    const int lp = (b + kv.b0) * kv.T + min(t0 + i + lane, kv.T - 1);
    pgv = kv.pages ? kv.pages[lp] : lp;
  };
  auto page_of = [&](int i) __attribute__((always_inline)) -> int { return __builtin_amdgcn_readlane(pgv, i & 63); };
  read_pages(0);
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)sm;   // LDS byte address of sm
  auto stage = [&](const bf16_t* cache, int page, int at /* LDS element */) __attribute__((always_inline)) {
    const bf16_t* src = cache + ((size_t)page * kv.n_kv + kvh) * (size_t)(2 * KV_PAGE * AT_D);   // K and V^T blocks are equal
#pragma unroll
    for (int j = 0; j < FPW; ++j) {
      const int f = wave_u * FPW + j;
      lds_load16<false>((gbyte_ptr)(src + f * AT_FRAG), lane_off, lds0 + 2u * (unsigned)(at + f * AT_FRAG));
    }
  };
  auto stage_k = [&](int buf, int page) __attribute__((always_inline)) { stage(p.k, page, buf * AT_KSTAGE); };
  auto stage_v = [&](int buf, int page) __attribute__((always_inline)) { stage(p.v, page, AT_NKB * AT_KSTAGE + buf * AT_VSTAGE); };
  // ---- Q fragments (already scaled and split by the RoPE kernel) and masks: requested in front of the first tiles, which are
  // not in any cache and would hold them up (loads return in order), and before the lengths are known.  Rows behind the last
  // node read some row's, or what an earlier call left there, and are multiplied along; their results are never stored and
  // `limit` does not ask them.
  Frag qh[MB][4], ql[MB][4];
  unsigned long long a0[MB], a1[MB];
  int my_enter[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int node = min(node0 + mb * 16 + l16, rm.n - 1);
    const size_t qo = ((size_t)b * rm.R + node) * p.ldq + head * AT_D + g4 * 8, mo = 2 * ((size_t)b * p.anc_stride + node);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      qh[mb][ks].u = *(const u32x4*)(p.q_hi + qo + ks * 32);
      ql[mb][ks].u = *(const u32x4*)(p.q_lo + qo + ks * 32);
    }
    const bool bits = !chain && !p.iv;
    a0[mb] = bits ? p.anc[mo] : 0ull;
    a1[mb] = bits ? p.anc[mo + 1] : 0ull;
    my_enter[mb] = p.iv ? p.iv[mo] : 0;
  }
  __builtin_amdgcn_sched_barrier(0);
  // The first tiles are requested before anything else is waited for (their addresses need the page table only:
  // keys past the cache are clamped and masked later), so their HBM latency overlaps the loads of the lengths,
  // the masks and Q.
  stage_k(0, page_of(0));
  if (p.plan.tiles > 1) stage_k(1, page_of(1));   // (used if the range has a second tile)
  stage_v(0, page_of(0));
  const int nv = rm.n_valid ? min(rm.n_valid[b], rm.n) : rm.n;
  const int L = p.base_len[b];
  if (ng * NODES >= nv || L + nv > p.max_seq) {  // whole workgroup
    wait_staging<0>();   // no staging load may land in the LDS after the workgroup has given it back
    return;
  }
  const int total = L + nv;
  int2* kiv = (int2*)(sm + AT_LDS_EL);   // [AT_MAX_IV] (enter, exit) of the tree keys; published by the first barrier
  if (p.iv)
    for (int w = tid; w < nv; w += NT) kiv[w] = *(const int2*)(p.iv + 2 * ((size_t)b * p.anc_stride + w));
  const bool work = __builtin_amdgcn_readfirstlane(node0) < nv;   // (a wavefront without nodes only helps with the staging)
  unsigned long long valid[MB];   // lanes whose row is a node
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) valid[mb] = __builtin_amdgcn_ballot_w64(node0 + mb * 16 + l16 < nv);
  const int open = L + (chain ? ng * NODES : 0);
  const int n_tiles = ((chain ? min(total, L + ng * NODES + NODES) : total) + AT_TK - 1) / AT_TK;
  const int n = min(n_tiles, t0 + p.plan.tiles) - t0;   // tiles of this split (<= 0: none)
  f32x4 O[8][MB];
#pragma unroll
  for (int db = 0; db < 8; ++db)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) O[db][mb] = (f32x4){0.f, 0.f, 0.f, 0.f};
  // Running reference of the soft-max in units of log2: m2 is what the probabilities so far are relative to (not necessarily
  // the largest score, see below), ms the same with 0 for "none yet"; l_run this lane's share of the running sum.
  float m2[MB], ms[MB], l_run[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) { m2[mb] = -INFINITY; ms[mb] = 0.f; l_run[mb] = 0.f; }

  // ---- the steps of a key tile.  scores: S^T = K Q^T (matrix pipe); probabilities: exp2 of the scores relative to m2, as hi/lo
  // fragments (vector ALU); output: O^T += V^T P (matrix pipe); limit: masks, and a new reference if a score asks for it. ----
  auto scores = [&](int kbuf, f32x4 (&sc)[2][MB]) __attribute__((always_inline)) {
    const bf16_t* kb = k_lds + kbuf * AT_KSTAGE + lane * 8;
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) sc[tt][mb] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        Frag kh, kl;
        kh.u = *(const u32x4*)(kb + (tt * 4 + ks) * AT_FRAG);
        kl.u = *(const u32x4*)(kb + (8 + tt * 4 + ks) * AT_FRAG);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          sc[tt][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kl.v, qh[mb][ks].v, sc[tt][mb], 0, 0, 0);
          sc[tt][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kh.v, ql[mb][ks].v, sc[tt][mb], 0, 0, 0);
          sc[tt][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kh.v, qh[mb][ks].v, sc[tt][mb], 0, 0, 0);
        }
      }
  };
  auto probabilities = [&](const f32x4 (&sc)[2][MB], Frag (&ph)[MB], Frag (&pl)[MB]) __attribute__((always_inline)) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      float pe[8], psum = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) { pe[e] = __builtin_amdgcn_exp2f(fmaf(sc[e >> 2][mb][e & 3], LOG2E, -ms[mb])); psum += pe[e]; }
      l_run[mb] += psum;
      unsigned h, l;
      a_split2(pe[0], pe[1], h, l); ph[mb].u.x = h; pl[mb].u.x = l;
      a_split2(pe[2], pe[3], h, l); ph[mb].u.y = h; pl[mb].u.y = l;
      a_split2(pe[4], pe[5], h, l); ph[mb].u.z = h; pl[mb].u.z = l;
      a_split2(pe[6], pe[7], h, l); ph[mb].u.w = h; pl[mb].u.w = l;
    }
  };
  auto output = [&](int vbuf, const Frag (&ph)[MB], const Frag (&pl)[MB]) __attribute__((always_inline)) {
    const bf16_t* vb = v_lds + vbuf * AT_VSTAGE + lane * 8;
#pragma unroll
    for (int db = 0; db < 8; ++db) {
      Frag vh, vl;
      vh.u = *(const u32x4*)(vb + db * AT_FRAG);
      vl.u = *(const u32x4*)(vb + (8 + db) * AT_FRAG);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        O[db][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vl.v, ph[mb].v, O[db][mb], 0, 0, 0);
        O[db][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vh.v, pl[mb].v, O[db][mb], 0, 0, 0);
        O[db][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vh.v, ph[mb].v, O[db][mb], 0, 0, 0);
      }
    }
  };
  auto limit = [&](int t, f32x4 (&sc)[2][MB]) __attribute__((always_inline)) {
    // Uniform: some key of the tile may be hidden from some row (keys in front of `open` are visible to every row).
    if ((t + 1) * AT_TK > open) {
      const int w0 = t * AT_TK + 8 * g4 - L;   // the lane's keys are slots L + w0 .. + 7: new rows w0 .. where not negative
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        unsigned seen = 0u;   // bit e: the lane's e-th key is visible to its row
        if (chain) {
          seen = (1u << max(0, min(8, node0 + mb * 16 + l16 - w0 + 1))) - 1u;
        } else if (!p.iv) {   // (no bits behind the last node)
          const int lo = max(0, min(8, -w0)), w = max(w0, 0);
          const unsigned long long a = w < 64 ? (a0[mb] >> w) | (w > 0 ? a1[mb] << (64 - w) : 0ull) : w < 128 ? a1[mb] >> (w - 64) : 0ull;
          seen = (unsigned)(a << lo) | ((1u << lo) - 1u);
        } else {
#pragma unroll 1
          for (int e = 0; e < 8; ++e) {
            const int wn = w0 + e;
            bool vis = wn < 0;
            if (wn >= 0 && wn < nv) { const int2 ke = kiv[wn]; vis = ke.x <= my_enter[mb] && my_enter[mb] <= ke.y; }
            if (vis) seen |= 1u << e;
          }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (!(seen >> e & 1u)) sc[e >> 2][mb][e & 3] = -INFINITY;
      }
    }
    // The reference moves only when some score exceeds it by a factor of 2^AT_SLACK (the first visible scores exceed "none"):
    // probabilities up to that factor above one are as exact in floating point as those below one, and the exchange between
    // the lanes of a row and the rescaling drop out of nearly every tile.
    // Rows behind the last node have no say: what an earlier call left in them would decide when the valid rows beside them are
    // rescaled, and with that their last bits.
    float tmax[MB];
    unsigned long long above = 0ull;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      tmax[mb] = sc[0][mb][0];
#pragma unroll
      for (int e = 1; e < 8; ++e) tmax[mb] = fmaxf(tmax[mb], sc[e >> 2][mb][e & 3]);
      above |= __builtin_amdgcn_ballot_w64(tmax[mb] * LOG2E > m2[mb] + AT_SLACK) & valid[mb];
    }
    if (above != 0ull) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        float t2 = fmaxf(tmax[mb], __shfl_xor(tmax[mb], 16, 64));
        t2 = fmaxf(t2, __shfl_xor(t2, 32, 64)) * LOG2E;
        const float m_new = fmaxf(m2[mb], t2);
        ms[mb] = m_new == -INFINITY ? 0.f : m_new;
        const float corr = __builtin_amdgcn_exp2f(m2[mb] - ms[mb]);   // exp2(-inf) = 0 on the first visible tile
        m2[mb] = m_new;
        l_run[mb] *= corr;
#pragma unroll
        for (int db = 0; db < 8; ++db) O[db][mb] *= corr;
      }
    }
  };

  // ---- the loop over this range's key tiles: the scores of tile i + 1 (matrix pipe) are computed beside the probabilities of
  // tile i (vector ALU), so K runs one tile ahead of V^T.  Requested at the top of iteration i: K tile i + 2 into the buffer of
  // tile i (its scores were computed in iteration i - 1, every wavefront is past that barrier), V^T tile i + 1.  Both are
  // complete, and visible to every wavefront, at the barrier that ends iteration i: each wavefront waits for its own
  // staging loads first. ----
  if (n > 0) {  // uniform over the workgroup
    f32x4 sa[2][MB], sb[2][MB];
    Frag ph[MB], pl[MB];
    wait_staging<0>();
    __syncthreads();
    if (work) { scores(0, sa); limit(t0, sa); }
    __syncthreads();   // K buffer 0 is overwritten from here on
    for (int i = 0; i + 1 < n; ++i) {
      const int page1 = page_of(i + 1);
      if (i + 2 < n) {
        if (((i + 2) & 63) == 0) read_pages(i + 2);
        stage_k(i & 1, page_of(i + 2));
      }
      stage_v((i + 1) & 1, page1);
      if (work) {
        scores((i + 1) & 1, sb);
        probabilities(sa, ph, pl);
        output(i & 1, ph, pl);
        limit(t0 + i + 1, sb);
#pragma unroll
      for (int tt = 0; tt < 2; ++tt)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) sa[tt][mb] = sb[tt][mb];
      }
      wait_staging<0>();
      __syncthreads();
    }
    if (work) { probabilities(sa, ph, pl); output((n - 1) & 1, ph, pl); }
  }

  wait_staging<0>();   // (a range without tiles still has its first staging loads in flight)
  // ---- one range of keys: the finished rows as planes; several: the partial result of this range ----
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int node = node0 + mb * 16 + l16;
    float lsum = l_run[mb];
    lsum += __shfl_xor(lsum, 16, 64);
    lsum += __shfl_xor(lsum, 32, 64);
    if (node >= nv) continue;
    const size_t row = (size_t)b * rm.R + node;
    if (whole) {
#pragma unroll
      for (int db = 0; db < 8; ++db) {
        const f32x4 v = O[db][mb];
        frag_store4(p.out, (int)row, head * AT_D + db * 16 + 4 * g4, v[0] / lsum, v[1] / lsum, v[2] / lsum, v[3] / lsum);
      }
      continue;
    }
    const size_t prow = ((size_t)split * p.rows_total + row) * p.n_q + head;
#pragma unroll
    for (int db = 0; db < 8; ++db) {
      const f32x4 v = O[db][mb];
      *(float4*)(p.o_part + prow * AT_D + db * 16 + 4 * g4) = make_float4(v[0], v[1], v[2], v[3]);
    }
    if (g4 == 0) {
      p.ml_part[prow * 2] = m2[mb];
      p.ml_part[prow * 2 + 1] = lsum;
    }
  }
}

// merge the ranges of one (row, head): out = sum_s 2^{m_s - M} O_s / sum_s 2^{m_s - M} l_s, as planes.
// One thread owns four adjacent channels of one head; the (m, l) pairs and the partial rows of all ranges are requested before
// the first is used.  The number of ranges is rounded up to one of a few compile-time counts (the last range again, weight 0).
constexpr int MG_HEADS = 8;   // heads per workgroup (32 threads each)
constexpr int MG_MAXS = 16;   // >= the largest number of ranges that attn_plan picks
template <int NS>
__device__ __forceinline__ void merge_ranges(const float* __restrict__ o, const float* __restrict__ ml_p, size_t stride, int ns,
                                             const FragPlanes& out, int row, int col) {
  float2 ml[NS];
  float4 v[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) ml[s] = *(const float2*)(ml_p + (size_t)min(s, ns - 1) * stride * 2);
#pragma unroll
  for (int s = 0; s < NS; ++s) v[s] = *(const float4*)(o + (size_t)min(s, ns - 1) * stride * AT_D);
  float M = -INFINITY;
#pragma unroll
  for (int s = 0; s < NS; ++s) M = fmaxf(M, ml[s].x);
  float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
  float den = 0.f;
#pragma unroll
  for (int s = 0; s < NS; ++s) {  // in range order
    const float wgt = s >= ns || ml[s].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml[s].x - M);
    den += wgt * ml[s].y;
    num.x += wgt * v[s].x; num.y += wgt * v[s].y; num.z += wgt * v[s].z; num.w += wgt * v[s].w;
  }
  frag_store4(out, row, col, num.x / den, num.y / den, num.z / den, num.w / den);
}
struct MergeArgs {
  const float *o_part, *ml_part;
  int rows_total, n_q, most, tab;
  FragPlanes out;
  RowMap rm;
  unsigned char ranges[ATTN_TAB];
};
__global__ __launch_bounds__(MG_HEADS * 32) void attn_merge_kernel(MergeArgs p) {
  const int i = blockIdx.x, b = blockIdx.y;
  const int head = blockIdx.z * MG_HEADS + (threadIdx.x >> 5), d4 = (threadIdx.x & 31) * 4;
  const int ns = p.tab ? (int)p.ranges[b] : p.most;
  const RowMap& rm = p.rm;
  const int nv = rm.n_valid ? min(rm.n_valid[b], rm.n) : rm.n;
  if (ns == 1 || i >= nv || head >= p.n_q) return;   // (one range: the attention kernel has written the rows)
  const size_t row = (size_t)b * rm.R + i;
  const size_t stride = (size_t)p.rows_total * p.n_q;   // (row, head) pairs per range
  const size_t pr0 = row * p.n_q + head;
  const float *o = p.o_part + pr0 * AT_D + d4, *ml = p.ml_part + pr0 * 2;
  if (ns <= 4) merge_ranges<4>(o, ml, stride, ns, p.out, (int)row, head * AT_D + d4);
  else if (ns <= 8) merge_ranges<8>(o, ml, stride, ns, p.out, (int)row, head * AT_D + d4);
  else if (ns <= 12) merge_ranges<12>(o, ml, stride, ns, p.out, (int)row, head * AT_D + d4);
  else merge_ranges<16>(o, ml, stride, ns, p.out, (int)row, head * AT_D + d4);
}

bool attn_mfma_supported(int head_dim, int n_q, int n_kv, int max_seq) {
  const int g = n_q / n_kv;
  return head_dim == AT_D && (g == 1 || g == 2 || g == 4 || g == 8) && max_seq % KV_PAGE == 0 && max_seq >= KV_PAGE &&
         max_seq / KV_PAGE <= 4096;
}

template <int G, int WM, int MB>
static void launch_attn_one(const AttnParams& p, dim3 grid, hipStream_t st) {
  constexpr size_t lds = (size_t)AT_LDS_EL * sizeof(bf16_t) + AT_MAX_IV * sizeof(int2);
  static OncePerDevice once;
  allow_dynamic_lds(once, (const void*)attn_mfma_kernel<G, WM, MB>, (int)lds);
  attn_mfma_kernel<G, WM, MB><<<grid, 64 * G * WM, lds, st>>>(p);
}

// Nodes per workgroup: with one or two query heads per KV head 64 or 128 where they are there, so that up to eight
// wavefronts share a staged tile (32 heads of their own K/V, us: 64 nodes at 512 keys 13.6 -> 11.2, 128 nodes at 1500 keys
// 36.6 -> 22.7, a 2048-token prompt 224 -> 122; 16 KV heads, 8 x 60 nodes at 700 keys 41.1 -> 32.5)
static int group_nodes(int g, int n) { return g == 1 && n > 64 ? 128 : g <= 2 && n > 32 ? 64 : 32; }

AttnPlan attn_plan(const int* keys, int B, int n, int n_kv, int n_q, bool chain, int max_ranges) {
  const int nodes = group_nodes(n_q / n_kv, n), per_unit = n_kv * ((n + nodes - 1) / nodes);
  int most_keys = 0;
  for (int b = 0; b < B; ++b) most_keys = std::max(most_keys, keys[b]);
  const int n_tiles = (most_keys + AT_TK - 1) / AT_TK;
  // Key splits by estimated time, in us, fitted to every split count of 283 launches over sequences of equal length (8 and 32 KV
  // heads, groups of 1 to 8 heads, 1 to 16 sequences, 1 to 128 nodes, 8 to 8192 keys, prompts to 2000 tokens; on average 1.7 %
  // behind the best; over 20 batches of unequal ones 2.1 %, most of it 8 x 32 nodes with 32 KV heads, 84.5 where 3 splits take 71.3).
  // A key tile adds 1.0 to a lone workgroup of a compute unit that has 16 nodes, 1.2 to one with all 32, 2.0 to 2.5 to two of those
  // together (8192 keys; what a launch takes besides is left out): 1.05 here, and two count as twice one, which keeps a second
  // workgroup for where it pays.  Splitting at all costs the merge launch and the traffic of the partial results, 2 + 0.2 per MB (32 heads, 8 KV
  // heads: one node at 133 keys unsplit 14.9, in 3 splits 10.4; 64 nodes at 100 keys 17.1 and 15.3, at 1024 keys 52 and 19 in 12;
  // 128 nodes at 8192 keys 59.4 in 8, 55.5 in 16).  Where most keys are the launch's own new rows the workgroups' tiles grow from
  // one to all, so a split shortens only the last of them: 1.5 and 5.2 + 0.4 there (200 tokens unsplit 17.0, in 4 splits 20.9).
  // With equally many ranges for all sequences the longest one would set every workgroup's tiles and the short ones' workgroups
  // would idle; ranges of equal length give the short ones fewer.  Sequences of 32 nodes between 256 and 2048 keys, us: 8 of them
  // 37 -> 30, 16 of them 63 -> 46; 2 x 40 nodes at 238 and 1252 keys 16.6 -> 13.8.
  const int only = tune_int("CLOVER_ATTN_SPLITS", 0), limit = std::min(max_ranges, MG_MAXS);
  const double mb = (double)n * n_q * AT_D * 4e-6;   // of a range's partial results
  const bool fresh = chain && 2 * n > most_keys;
  const double tile = fresh ? 1.5 : 1.05, merge = fresh ? 5.2 : 2.0, per_mb = fresh ? 0.4 : 0.2;
  const bool table = B <= ATTN_TAB;
  AttnPlan plan{{n_tiles, B, 1, 0, {}}, {}};
  double best = 1e30;
  const int step = (n_tiles + 255) / 256;   // (long caches: 256 lengths of a range are looked at)
  for (int c = n_tiles; c >= std::min(2, n_tiles) && (n_tiles + c - 1) / c <= limit; c -= step) {
    const int most = (n_tiles + c - 1) / c;
    int units = 0, parts = 0;
    for (int b = 0; b < B; ++b) {
      const int r = ((keys[b] + AT_TK - 1) / AT_TK + c - 1) / c;
      units += r;
      parts += r > 1 ? r : 0;
    }
    const bool tab = table && units <= ATTN_TAB && units != B * most;   // (equally many ranges each need no table)
    if (!tab) { units = B * most; parts = most > 1 ? units : 0; }
    const double t = tile * c * ((units * per_unit + 255) / 256) + (most > 1 ? merge + per_mb * mb * parts : 0.0);
    if (only > 0 ? most <= only : t < best) { best = t; plan.tiles = c; plan.n_units = units; plan.most = most; plan.tab = tab; }
  }
  if (plan.tab) {
    int u = 0;
    for (int b = 0; b < B; ++b) {
      const int r = ((keys[b] + AT_TK - 1) / AT_TK + plan.tiles - 1) / plan.tiles;
      plan.ranges[b] = (unsigned char)r;
      for (int s = 0; s < r; ++s) plan.unit[u++] = (unsigned short)(b | s << 8 | (r == 1 ? 0x8000 : 0));
    }
  }
  return plan;
}

void launch_attn_mfma(AttnParams p, const AttnPlan& plan, hipStream_t st) {
  p.plan = plan;
  const int g = p.n_q / p.n_kv, nodes = group_nodes(g, p.rm.n);
  const unsigned groups = (unsigned)((p.rm.n + nodes - 1) / nodes), units = (unsigned)p.plan.n_units;
  const bool chain = p.anc == nullptr && p.iv == nullptr;
  const dim3 grid((unsigned)p.n_kv, chain ? units : groups, chain ? groups : units);
  switch (g) {
    case 1:
      if (nodes == 128) launch_attn_one<1, 8, 1>(p, grid, st);
      else if (nodes == 64) launch_attn_one<1, 4, 1>(p, grid, st);
      else launch_attn_one<1, 2, 1>(p, grid, st);
      break;
    case 2: if (nodes == 64) launch_attn_one<2, 4, 1>(p, grid, st); else launch_attn_one<2, 2, 1>(p, grid, st); break;
    case 4: launch_attn_one<4, 2, 1>(p, grid, st); break;
    default: launch_attn_one<8, 1, 2>(p, grid, st); break;
  }
  if (p.plan.most > 1) {
    MergeArgs m{p.o_part, p.ml_part, p.rows_total, p.n_q, p.plan.most, p.plan.tab, p.out, p.rm, {}};
    std::copy(plan.ranges, plan.ranges + ATTN_TAB, m.ranges);
    attn_merge_kernel<<<dim3(p.rm.n, p.rm.B, (p.n_q + MG_HEADS - 1) / MG_HEADS), MG_HEADS * 32, 0, st>>>(m);
  }
}

}  // namespace clv
