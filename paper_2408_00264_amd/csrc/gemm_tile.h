// The MFMA GEMM of every pass on gfx950 (bf16 weights in fragment order, activations as FragPlanes, fp32 accumulation):
//
//   EPI 0:  Y[M,N]      = X[M,K] * W[N,K]^T                   (fp32; over k_parts ranges of K: partial tiles)
//   EPI 1:  out[M,F]    = planes of silu(X Wg^T) * (X Wu^T)    (the SwiGLU projection)
//   EPI 3:  q, k, v     = X * W^T, q and k rotated, k and v into the caches (the QKV projection; k_parts ranges of K are summed
//                         inside the launch by the workgroups that have them, exchange.h)
//
// What bounds it: up to 16 rows the weight stream from HBM, above ~150 rows the matrix pipe (hi + lo planes are two
// matrix instructions per fragment pair; from 512 rows on its power: it is busy 82 to 90 % of the time at 1.9 to 2.2 GHz,
// and nothing but products runs at 2.25), and in between the read requests that a compute unit has in flight: by counters (the sum
// of their latencies / its busy cycles) about 145 at one row of gate+up, 135 at 23, 120 at 64, 110 at 80 and 96, 90 to 95 at 133 and
// 256, whatever the stage buffers hold beyond 16 KB; 1000 clocks each at one row, nearly all of them weights, 700 at 64, where half
// are activations out of the L2.  So what counts is lines per compute unit.
//
// Shape.  A workgroup of four wavefronts (2 x 2, one per SIMD; up to 16 rows 1 x 4) owns 32 RB rows x 16 WB columns (RB 1 to 5 and 8); a wavefront RB x WB / 2
// products of 16 x 16.  Both operands go global -> LDS directly, 32 columns of K per stage, as 1 KB blocks that are
// contiguous in global memory too (one load instruction each), NBUF stages deep: the loads of stage s + NBUF are issued
// while stage s is multiplied.  In flight per workgroup (mostly one to a compute unit): NBUF stages of 2 KB per 16 rows and
// 1 KB per 16 columns, 60 to 108 KB for tiles of up to 64 rows and 128 columns (and 32 x 192, 96 x 96), else 120 to 160.  The fragments
// of stage s + 1 are read from the LDS into the other of two register sets meanwhile, so a stage costs one barrier and
// no wait that is not already over.  Every operand byte crosses the L1 once per workgroup.
//
// Measured (8B shapes, weights from HBM, us per launch by kernel trace in passes of two layers; in brackets by events the
// kernels it replaced, which read row-major planes: K-slice and panel form up to 64 rows, 128-row panel and 128 x 256
// tiles above):
//   rows        1          23         64         80         133    256
//   gate+up     35.0 (43)  37.7 (49)  44.8 (55)  50.6 (80)  69.8   83.4 (101)
//   down        18.9 (21)  20.4       25.4 (30)  27.2 (36)  36.3   51.4 (57)
//   QKV          9.7 (12)  11.2       14.9 (18)  16.2 (27)  20.5   25.7 (34)   (EPI 0; EPI 3 at 64 rows: 18.6, of which, by clock in
//                the kernel, 1.1 the partial tile's way out, 1.5 the meeting, 1.2 the parts' way in, 1.3 rotation and stores)
//   Wo           6.6        8.8       11.1       12.9       15.8   20.6
//   LM head    154        170        177        187        229    365
// The same kernel on row-major planes (64-byte row pieces): gate+up 64.4 at 64 rows, 69.5 at 80, 107 at 256.
// Many rows, tiles of up to 160 / of 256 rows (and half the staged bytes per product): gate+up 179 / 154 at 512, 351 / 306
// at 1024, 701 / 605 at 2048, LM head 777 / 663 at 512, 3106 / 2713 at 2048, down 322 / 302 at 2048, QKV 159 / 137.
//
// RB, WB and the K ranges are chosen per launch (pick_tile).
#pragma once
#include "clover_internal.h"
#include "exchange.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace clv {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

namespace {

union Frag {
  u32x4 u;
  bf16x8 v;
};

constexpr int TL_KST = 32;            // K columns per stage: one k-tile

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

__device__ __forceinline__ unsigned t_rn(float a) { return (unsigned)__builtin_bit_cast(unsigned short, (__bf16)a); }

// (a, b) as packed hi and lo pairs (v_cvt_pk_bf16_f32, round to nearest even)
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void t_split2(float a, float b, unsigned& hi, unsigned& lo) {
  const f32x2 v = {a, b};
  const bf16x2 h = __builtin_convertvector(v, bf16x2);
  hi = __builtin_bit_cast(unsigned, h);
  lo = __builtin_bit_cast(unsigned, __builtin_convertvector(v - __builtin_convertvector(h, f32x2), bf16x2));
}

// acc += A B^T with the accumulator tied to one accumulation-register tuple for the whole kernel.  (Written through the
// builtin, the register allocator gives a fifth of the products of a loop trip a destination that differs from its
// source and moves the registers back; those moves are vector-ALU instructions and do not overlap the matrix pipe.)
__device__ __forceinline__ void mfma_acc(f32x4& acc, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}

// this wavefront's staging loads but the youngest N have landed and its LDS reads are done; then the workgroup meets
template <int N>
__device__ __forceinline__ void wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(N) : "memory");
}

// RB 0: the form for up to 16 rows: one row block, the four wavefronts side by side on its columns, 64 columns of K per
// stage.  (As RB 1, half of the activation loads would fetch the same row block again: gate+up at one row 40 us of which
// the weights alone take 36 and the activations 11.)
// WB: weight blocks (16 columns) of a workgroup.
template <int RB, int WB>
struct TileShape {
  static constexpr bool ONE = RB == 0;
  static constexpr int KS = ONE ? 2 : 1;               // 32-column steps per stage
  static constexpr int RBT = ONE ? 1 : 2 * RB;         // row blocks of the workgroup
  static constexpr int RBW = ONE ? 1 : RB;             // row and column blocks of a wavefront
  static constexpr int CBW = ONE ? (WB + 3) / 4 : (WB + 1) / 2;
  static constexpr int XF = KS * RBT * 2, WF = KS * WB;   // fragment blocks of a stage: activations (hi, lo), weights
  static constexpr int WREST = WF % 4;                 // weight blocks that the four wavefronts share in their last load
  static constexpr int STAGE = (XF + WF) * 1024;       // bytes
  static constexpr int NBUF = std::min(6, 160 * 1024 / STAGE);   // (12 for the narrow tiles measured 2 % slower)
  static constexpr int EPI_LD = WB * 16 + (WB % 2 ? 32 : 16);    // EPI 1: LDS row stride of the finished planes (bytes): an odd number of 16-byte pieces
  static constexpr int LDS = std::max(NBUF * STAGE, 2 * RBT * 16 * EPI_LD);
};

// ---- results over several ranges of K, finished by the workgroups of the ranges together ----
constexpr int DEVICE_SCOPE = 16;   // cache policy (sc1): a store is visible to, and a load sees, the whole device
struct DeviceWord {
  unsigned* p;
  __device__ __forceinline__ unsigned add(unsigned v) const { return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
  __device__ __forceinline__ unsigned load() const { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
  __device__ __forceinline__ void store(unsigned v) const { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
  __device__ __forceinline__ bool swap(unsigned from, unsigned to) const {
    return __hip_atomic_compare_exchange_strong(p, &from, to, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
};
// A member's share of a tile's blocks of 16 x 16: the column blocks member, member + S ... of all row blocks, dealt to its wavefronts by
// row block, and with one or two row blocks also by column.  (No division, and one row block per wavefront up to 64 rows: what
// is done behind the meeting is a chain of instructions that nothing else hides, about 2 ns each.)
struct Walk {
  int r_step, c_step, r, c, c0;
  __device__ __forceinline__ Walk(int rows, int wave, int S, int member) {
    const int lg = rows > 2 ? 2 : rows - 1;
    r_step = 1 << lg;
    r = wave & (r_step - 1);
    c_step = S << (2 - lg);
    c = c0 = member + S * (wave >> lg);
  }
  __device__ __forceinline__ void next(int n, int cols) {   // behind n blocks of a row block
    c += n * c_step;
    const bool row_done = c >= cols;
    c = row_done ? c0 : c;
    r += row_done ? r_step : 0;
  }
};

// One row of the QKV projection's result: where it belongs.  (All that has to be loaded is loaded here: behind the first store a load
// would wait for the stores in front of it.)
struct QkvRow {
  int m, b, i, nv, L, page;
  bool here;
  __device__ __forceinline__ void request(const QkvOut& o, int row, int M) {
    here = row < M;
    m = min(row, M - 1);
    b = o.rm.B == 1 ? 0 : m / o.rm.R;
    i = m - b * o.rm.R;
    nv = o.rm.n_valid ? o.rm.n_valid[b] : o.rm.n;
    L = o.base_len[b];
  }
  __device__ __forceinline__ void request_page(const QkvOut& o) {   // (waits for the length)
    page = (b + o.kv.b0) * o.kv.T + min((L + i) / KV_PAGE, o.kv.T - 1);
    if (o.kv.pages) page = o.kv.pages[page];
  }
  __device__ __forceinline__ bool on(const QkvOut& o) const {
    const int n = min(nv, o.rm.n);
    if (i >= n) return false;
    if (L + n <= o.kv.max_seq) return true;
    atomicOr(o.err_flag, 1);   // would overrun the cache: refuse, flag
    return false;
  }
};
// 16 columns of it, four to a lane: of a head in rotary order (lanes 0 .. 31 the first half's, 32 .. 63 the second's), or of v.
struct QkvBlock {
  int blk;
  float4 c, s;   // (v has no use for them)
  static __device__ __forceinline__ int per_head_log2(const QkvOut& o) { return o.d == 128 ? 3 : 2; }   // blocks of a head
  __device__ __forceinline__ void request(const QkvOut& o, const QkvRow& row, int blk_, int g4) {
    blk = blk_;
    const int half = o.d / 2, ii = (blk & ((1 << per_head_log2(o)) - 1)) * 8 + 4 * (g4 & 1);
    c = *(const float4*)(o.cos_t + (size_t)row.m * half + ii);
    s = *(const float4*)(o.sin_t + (size_t)row.m * half + ii);
  }
  static __device__ __forceinline__ void planes4(bf16_t* hi, bf16_t* lo, const float (&v)[4]) {
    uint2 h, l;
    t_split2(v[0], v[1], h.x, l.x);
    t_split2(v[2], v[3], h.y, l.y);
    *(uint2*)hi = h;
    *(uint2*)lo = l;
  }
  __device__ __forceinline__ void put(const QkvOut& o, const QkvRow& row, const f32x4& v, int g4) const {
    const int lg = per_head_log2(o), hh = blk >> lg, j = blk & ((1 << lg) - 1), n_kv = o.kv.n_kv, pos = (row.L + row.i) % KV_PAGE;
    const size_t page = (size_t)row.page * n_kv, block = 2 * KV_PAGE * o.d;   // (two planes: KVLayout)
    if (hh >= o.n_q + n_kv) {
      if (!row.on(o)) return;
      const int col = j * 16 + 4 * g4;
      bf16_t* at = o.vc + (page + (hh - o.n_q - n_kv)) * block + (col >> 4) * 512 + ((pos >> 3) * 16 + (col & 15)) * 8 + (pos & 7);
#pragma unroll
      for (int r = 0; r < 4; r += 2) {
        unsigned h, l;
        t_split2(v[r], v[r + 1], h, l);
        at[8 * r] = (bf16_t)h;
        at[8 * r + 8] = (bf16_t)(h >> 16);
        at[8 * r + KV_PAGE * o.d] = (bf16_t)l;
        at[8 * r + 8 + KV_PAGE * o.d] = (bf16_t)(l >> 16);
      }
      return;
    }
    const int col = j * 8 + 4 * (g4 & 1) + (g4 >> 1) * (o.d / 2);
    // the pair of a lane's column is in the lane 32 further or back (same row: both are here or neither)
    const float sgn = g4 < 2 ? -1.f : 1.f, cs[4] = {c.x, c.y, c.z, c.w}, sn[4] = {s.x, s.y, s.z, s.w};
    float out[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[r]), __float_as_uint(v[r]), false, false);
      out[r] = v[r] * cs[r] + sgn * __uint_as_float(g4 < 2 ? sw[1] : sw[0]) * sn[r];
    }
    if (!row.on(o)) return;
    if (hh >= o.n_q) {
      bf16_t* at = o.kc + (page + (hh - o.n_q)) * block + ((pos >> 2) & 1) * 16 * o.d + ((pos >> 3) * 4 + (pos & 3)) * 8 +
                   (col >> 5) * 512 + ((col >> 3) & 3) * 128 + (col & 7);
      planes4(at, at + KV_PAGE * o.d, out);
    } else {
      const size_t at = (size_t)row.m * o.ldq + hh * o.d + col;
      if (o.q_hi) {
#pragma unroll
        for (int r = 0; r < 4; ++r) out[r] *= o.q_scale;
        planes4(o.q_hi + at, o.q_lo + at, out);
      } else {
        *(float4*)(o.q + at) = make_float4(out[0], out[1], out[2], out[3]);
      }
    }
  }
};

// The blocks of a member's share that come next: what they need besides their sums (epi 3).
template <int EPI> using TileArgs = std::conditional_t<EPI == 3, TileGemmQkv, TileGemm>;
template <int EPI, int NB>
struct Pending {
  __device__ __forceinline__ Pending(const TileGemm&, int, int, int, int, int, int, int) {}
  __device__ __forceinline__ void request() {}
};
template <int NB>
struct Pending<3, NB> {
  const TileGemmQkv& p;
  const int row0, col0, l16, g4, rows_here, cols_here;   // first row and column block of the tile; row and column blocks that it has
  Walk walk;
  QkvRow row;
  QkvBlock blk[NB];
  __device__ __forceinline__ Pending(const TileGemmQkv& p_, int row0_, int tile, int WB, int member, int wave, int l16_, int g4_)
      : p(p_), row0(row0_), col0(tile * WB), l16(l16_), g4(g4_), rows_here(min(p_.row_blocks, (p_.M - row0_ + 15) / 16)),
        cols_here(min(WB, p_.N / 16 - tile * WB)), walk(rows_here, wave, p_.k_parts, member) {}
  __device__ __forceinline__ void request() {
    row.request(p.qkv, row0 + walk.r * 16 + l16, p.M);
#pragma unroll
    for (int i = 0; i < NB; ++i) blk[i].request(p.qkv, row, col0 + walk.c + i * walk.c_step, g4);
  }
};

// NT: non-temporal loads, for weights that no other workgroup reads (gate+up at 64 rows 47.0 -> 44.6 us; where row tiles
// share them it costs: 256 rows 96.5 -> 100).
template <int RB, int WB, int EPI, bool NT>
__global__ __launch_bounds__(256, 1) void gemm_tile_kernel(TileArgs<EPI> p) {
  using T = TileShape<RB, WB>;
  constexpr int XF = T::XF, WF = T::WF, WREST = T::WREST, STAGE = T::STAGE, NBUF = T::NBUF;
  constexpr int KS = T::KS, RBT = T::RBT, RBW = T::RBW, CBW = T::CBW;
  constexpr int XL = XF / 4, WL = (WF + 3) / 4, L = XL + WL;   // staging loads per wavefront and stage
  constexpr int NRS = 2 * RBW + CBW, NR = KS * NRS;            // fragments a wavefront reads per step and stage
  constexpr int MMS = 2 * RBW * CBW, MM = KS * MMS;            // matrix instructions per wavefront, step and stage
  static_assert(T::LDS <= 160 * 1024 && (NBUF - 2) * L <= 63, "stage buffers exceed the LDS or the load counter");
  extern __shared__ __attribute__((aligned(16))) char sm[];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int l16 = lane & 15, g4 = lane >> 4;
  const int wr = T::ONE ? 0 : wave & 1, wc = T::ONE ? wave : wave >> 1;
  // first column block of the wavefront, and the first that it stores: where the blocks do not divide, the last wavefronts' begin
  // earlier and the overlap is computed twice
  const int wb0 = min(wc * CBW, WB - CBW), wown = wc * CBW;
  // workgroup id -> (row tile, column tile, K range): ids 8 apart share an XCD (dealt round-robin), so the row tiles
  // of the same columns are neighbours in that XCD's own order and find the weights in its L2
  const int rt = (p.M + 16 * RBT - 1) / (16 * RBT);
  int rh = 0, unit = (int)blockIdx.x;
  if (rt > 1) {
    const int xcd = (int)blockIdx.x & 7, j = (int)blockIdx.x >> 3;
    rh = j % rt;
    unit = (j / rt) * 8 + xcd;
  }
  int part, tile;
  bool together = false;   // the ranges of a tile on one XCD
  if constexpr (EPI == 3) together = p.k_parts > 1 && !p.spread;
  if (together) {
    // The workgroups that exchange partial tiles share an XCD: they meet in its L2 (8 of 32 KB each: 1.8 us, on different XCDs 5.5).
    // Each XCD has a range of adjacent tiles and the ranges of K are interleaved, stage by stage, so the whole launch still walks
    // the matrix side by side (33 MB streamed so 6.6 us, with contiguous ranges 7.4).
    const int tiles = p.n_units / p.k_parts, xcd = (int)blockIdx.x & 7, j = (int)blockIdx.x >> 3, q = j / p.k_parts;
    part = j - q * p.k_parts;
    rh = q % rt;
    tile = xcd * tiles / 8 + q / rt;
    if (tile >= (xcd + 1) * tiles / 8) return;
  } else {
    if (unit >= p.n_units) return;   // (grid rounded up to whole XCD rows; uniform over the workgroup)
    part = unit % p.k_parts;
    tile = unit / p.k_parts;
  }
  const int NS = p.K / (TL_KST * KS) / p.k_parts;      // stages of this workgroup's K range
  const int kt0 = EPI == 3 ? part * KS : part * NS * KS;
  const int row0 = rh * 16 * RBT;

  // ---- exchange: what the first blocks of the workgroup's share need besides their sums is requested in front of everything else
  // (tiles of up to 128 rows have the registers to keep it) ----
  constexpr int NB = 2;   // blocks at a time
  constexpr bool EARLY = RB <= 4;
  Pending<EPI, NB> next(p, row0, tile, WB, part, wave, l16, g4);
  if (EPI == 3 && EARLY && p.k_parts > 1) next.request();

  // ---- staging: activation block f of a stage = (row block f / 2, plane f % 2), weight block c = 16 rows of W (epi 1:
  // 8 gate and the 8 up rows of the same F columns, so that a lane pair (l, l + 32) ends up with both factors).  Row
  // blocks past the matrix read its last one again: an output row depends on its own activation row only, and rows
  // >= M are never stored (nor need the rows that pad the last block hold numbers).
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)sm;
  const unsigned lane16 = (unsigned)lane * 16u;
  const size_t xstage = (size_t)p.X.mb * 2048;          // bytes of a 32-column step of all rows
  const int n_wb = p.N / (EPI == 1 ? 8 : 16);           // weight blocks of 16 rows
  const size_t wstage = (size_t)n_wb * 1024;            // bytes of a 32-column step of the whole matrix
  // A load's address is the stage's (one scalar pair each for activations and weights, advanced once per stage) plus the
  // load's own 32-bit lane offset: between two matrix instructions of 16 clocks a wavefront has issue slots for two more
  // instructions, and a load with 64-bit address arithmetic of its own took six (512 rows of the LM head 738 -> 715 us).
  unsigned xoff[XL], woff[WL];
#pragma unroll
  for (int j = 0; j < XL; ++j) {
    const int f = (j * 4 + wave) >> 1, rblk = min(row0 / 16 + f % RBT, p.X.mb - 1);
    xoff[j] = lane16 + (unsigned)(f / RBT) * (unsigned)xstage + (unsigned)rblk * 2048u + (unsigned)(wave & 1) * 1024u;
  }
#pragma unroll
  for (int i = 0; i < WL; ++i) {   // (the last load: 16 WREST lanes of every wavefront take the blocks that are left, piece after piece)
    const bool rest = WREST > 0 && i == WL - 1;
    const int pc = rest ? min(wave * 16 * WREST + lane, 64 * WREST - 1) : wave * 64 + lane, f = i * 4 + (pc >> 6), c = min(tile * WB + f % WB, n_wb - 1);
    woff[i] = (unsigned)(pc & 63) * 16u + (unsigned)(f / WB) * (unsigned)wstage + (unsigned)c * 1024u;
  }
  const char* xp = (const char*)p.X.p + (size_t)kt0 * xstage;   // the stage that is requested next
  const char* wp = (const char*)p.W + (size_t)kt0 * wstage;
  const unsigned ldsw = lds0 + (unsigned)wave * 1024u;
  // The last load's destination and lanes.  (Two wavefronts used to stage the last blocks a second time, and a line that is loaded
  // twice costs its share of the kernel.  64 rows, both in tiles of 96 columns, six blocks a stage: gate+up of 11008 channels 45.4 ->
  // 40.9 us, QKV 16.7 -> 15.6.)
  const unsigned wlast = (unsigned)__builtin_amdgcn_readfirstlane((XF + (WL - 1) * 4) * 1024 + wave * (WREST * 256 - 1024));
  const unsigned long long some_lanes = (1ull << (16 * WREST)) - 1ull;
  // Load j of the stage at (xp, wp), M0 set in front of it: at least one instruction (or the no-op) has to lie in between.
  // Contract: each load has one set_m0 of its own, with no other load and no jump in between.  The load cannot say that it
  // reads M0, so nothing but that order -- kept, both are volatile -- and the absence of compiler-made writes of M0 carries
  // the address; tests/test_kernel_waits.py looks for both in the machine code.
  auto set_m0 = [&](auto jc, unsigned buf) __attribute__((always_inline)) {
    constexpr int j = decltype(jc)::value, i = j - XL;
    const unsigned base = ldsw + buf, last = wlast;
    if constexpr (j < XL) asm volatile("s_add_u32 m0, %0, %1" : : "s"(base), "n"(j * 4096) : "m0", "scc");
    else if constexpr (i * 4 + 3 < WF) asm volatile("s_add_u32 m0, %0, %1" : : "s"(base), "n"((XF + i * 4) * 1024) : "m0", "scc");
    else asm volatile("s_add_u32 m0, %0, %1" : : "s"(base), "s"(last) : "m0", "scc");
  };
  auto load = [&](auto jc, auto nopc) __attribute__((always_inline)) {
    constexpr int j = decltype(jc)::value;
    if constexpr (decltype(nopc)::value) asm volatile("s_nop 0");
    if constexpr (j < XL) {
      const unsigned off = xoff[j];
      const gbyte_ptr src = (gbyte_ptr)xp;
      asm volatile("global_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(src));
    } else {
      const unsigned off = woff[j - XL];
      const gbyte_ptr src = (gbyte_ptr)wp;
      if constexpr (WREST > 0 && j == L - 1) {   // (every lane is active here: the kernel's control flow is uniform)
        if constexpr (NT) asm volatile("s_mov_b64 exec, %2\n\tglobal_load_lds_dwordx4 %0, %1 nt\n\ts_mov_b64 exec, -1" : : "v"(off), "s"(src), "s"(some_lanes));
        else asm volatile("s_mov_b64 exec, %2\n\tglobal_load_lds_dwordx4 %0, %1\n\ts_mov_b64 exec, -1" : : "v"(off), "s"(src), "s"(some_lanes));
      } else if constexpr (NT) asm volatile("global_load_lds_dwordx4 %0, %1 nt" : : "v"(off), "s"(src));
      else asm volatile("global_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(src));
    }
  };
  const size_t n_between = EPI == 3 ? p.k_parts : 1, xstep = n_between * KS * xstage, wstep = n_between * KS * wstage;
  // (xp, wp) from stage t to t + 1, or not behind the last one: that one is requested again, into a buffer that nothing reads
  // any more; those loads hit the cache, and a loop without conditions keeps the accumulators in place -- with separate
  // code for the last NBUF stages the allocator moved all of them at every hand-over
  auto advance = [&](int t) __attribute__((always_inline)) {
    const bool more = t + 1 < NS;
    xp += more ? xstep : 0;
    wp += more ? wstep : 0;
  };

  f32x4 acc[CBW][RBW];
#pragma unroll
  for (int c = 0; c < CBW; ++c)
#pragma unroll
    for (int rb = 0; rb < RBW; ++rb) acc[c][rb] = (f32x4){0.f, 0.f, 0.f, 0.f};
  // (the wait states between the write of an accumulator and the first matrix instruction, which the compiler does not see)
#pragma unroll
  for (int c = 0; c < CBW; ++c)
#pragma unroll
    for (int rb = 0; rb < RBW; ++rb) asm volatile("" : "+a"(acc[c][rb]));
  asm volatile("s_nop 7" ::: "memory");

  Frag fa[NR], fb[NR];   // per step: [2 rb + plane], then [2 RBW + column block]
  const char* const xrd = sm + wr * RBW * 2048 + l16 * 64 + ((g4 ^ ((0 - (l16 >> 2)) & 3)) * 16);
  const char* const wrd = sm + (XF + wb0) * 1024 + lane * 16;
  auto read1 = [&](Frag (&f)[NR], auto rc, unsigned buf) __attribute__((always_inline)) {
    constexpr int k = decltype(rc)::value / NRS, r = decltype(rc)::value % NRS;
    if constexpr (r < 2 * RBW) f[k * NRS + r].u = *(const u32x4*)(xrd + buf + (k * RBT * 2 + r) * 1024);
    else f[k * NRS + r].u = *(const u32x4*)(wrd + buf + (k * WB + r - 2 * RBW) * 1024);
  };
  // Order of a stage's products: lo plane, then hi plane of the same output block back to back (the second takes the sum and
  // the weights that the first has just used).  Long launches are bound by power -- the clock falls to what the matrix
  // pipe's switching allows -- and this order needs the least: 2.25 PFLOP/s at 2.25 GHz in a loop of nothing but
  // products of 8 x 8 blocks, against 2.06 at 2.07 GHz with all of the lo plane in front of the hi plane and 1.89 at 1.84 for
  // 32 x 32 x 16 products (probes/mfma_order.hip; in the kernel: 512 rows of the LM head 731 -> 700 us, 1024 of down 168 -> 159).
  auto mm = [&](const Frag (&f)[NR], auto mc) __attribute__((always_inline)) {
    constexpr int k = decltype(mc)::value / MMS, m = decltype(mc)::value % MMS, rb = m / (2 * CBW), c = m / 2 % CBW, lo = 1 - m % 2;
    mfma_acc(acc[c][rb], f[k * NRS + 2 * RBW + c].v, f[k * NRS + 2 * rb + lo].v);
  };

  // ---- prologue: NBUF stages requested, the fragments of the first one read ----
#pragma unroll
  for (int t = 0; t < NBUF; ++t) {
    static_for<0, L>([&](auto jc) { set_m0(jc, (unsigned)(t * STAGE)); load(jc, std::true_type{}); });
    advance(t);
  }
  wait_barrier<(NBUF - 2) * L>();
  static_for<0, NR>([&](auto rc) { read1(fa, rc, 0u); });
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory");   // buffer 0 may be overwritten

  // One stage: its products from `f`; between them, one per product or two, the reads of the next stage's fragments
  // into `fn` and the loads of stage s + NBUF into the buffer that stage s was read from in the previous stage.
  unsigned cur = 0;   // byte offset of stage s's buffer
  auto stage = [&](const Frag (&f)[NR], Frag (&fn)[NR], int s) __attribute__((always_inline)) {
    const unsigned nxt = cur + STAGE == (unsigned)(NBUF * STAGE) ? 0u : cur + STAGE;
    constexpr int O = NR + 2 * L, SPAN = MM - MM / 8;   // operations: reads, then (M0, load) pairs
    static_for<0, MM>([&](auto mc) {
      constexpr int m = decltype(mc)::value, o0 = std::min((m * O + SPAN - 1) / SPAN, O);
      mm(f, mc);
      static_for<o0, std::min(((m + 1) * O + SPAN - 1) / SPAN, O)>([&](auto oc) {
        constexpr int o = decltype(oc)::value, j = (o - NR) / 2;
        if constexpr (o < NR) read1(fn, oc, nxt);   // (behind the last stage: bytes of an older one, never used)
        else if constexpr ((o - NR) % 2 == 0) set_m0(std::integral_constant<int, j>{}, cur);
        else load(std::integral_constant<int, j>{}, std::bool_constant<(o - 1 >= o0)>{});   // M0 in the same gap: no-op
      });
    });
    advance(s + NBUF);
    wait_barrier<(NBUF - 2) * L>();
    cur = nxt;
  };
  int s = 0;
  for (; s + 1 < NS; s += 2) {
    stage(fa, fb, s);
    stage(fb, fa, s + 1);
  }
  if (s < NS) stage(fa, fb, s);
  wait_barrier<0>();   // no load may land in the LDS once it is used for the results, or given back

  // (the compiler does not know that the asm statements are matrix instructions, so the wait states between the last
  // of them and the first read of an accumulator are spelled out: 8 are needed, and the statements that follow the no-op
  // take every accumulator, so that no read can be moved in front of it)
  asm volatile("s_nop 15" ::: "memory");
#pragma unroll
  for (int c = 0; c < CBW; ++c)
#pragma unroll
    for (int rb = 0; rb < RBW; ++rb) asm volatile("" : "+a"(acc[c][rb]));
  // ---- epilogue: lane holds rows rb*16 + l16 of the wavefront's tile, columns 4*g4 .. 4*g4+3 of each block ----
  if (EPI == 1) {
    // Lanes 0..31 hold the gate, 32..63 the up factors of the same 8 columns: one half-wavefront swap of two row blocks
    // leaves both factors of the first block in the lower lanes and of the second in the upper ones.  The finished
    // planes pass through the LDS so that they leave as whole pieces of the fragment order.
    constexpr int LD = T::EPI_LD, PLANE = RBT * 16 * LD;
    const int up = lane >> 5, cl = (g4 & 1) * 4;
#pragma unroll
    for (int c = 0; c < CBW; ++c)
#pragma unroll
      for (int rb = 0; rb < RBW; rb += 2) {
        const int rb2 = rb + 1 < RBW ? rb + 1 : rb;
        unsigned h[4], l[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[c][rb][r]), __float_as_uint(acc[c][rb2][r]), false, false);
          const float g = __uint_as_float(sw[0]), u = __uint_as_float(sw[1]);
          const float o = g / (1.0f + expf(-g)) * u;
          h[r] = t_rn(o);
          l[r] = t_rn(o - __uint_as_float(h[r] << 16));
        }
        if (rb + up < RBW && wb0 + c >= wown) {
          char* dst = sm + ((wr * RBW + rb + up) * 16 + l16) * LD + ((wb0 + c) * 8 + cl) * 2;
          *(uint2*)dst = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
          *(uint2*)(dst + PLANE) = make_uint2(l[0] | (l[1] << 16), l[2] | (l[3] << 16));
        }
      }
    __syncthreads();
    // pieces of 8 columns, in pairs where their number is even (and a tile starts at an even piece): 16 rows x 32 bytes of a KB
    // block per half wavefront, else x 16
    constexpr int PP = WB % 2 ? 1 : 2, PL = PP - 1;   // pieces side by side; their bits of an index
    for (int i = tid; i < WB * RBT * 32; i += 256) {
      const int q = i & PL, r = (i >> PL) & 15, plane = (i >> (PL + 4)) & 1, rb = (i >> (PL + 5)) % RBT, pc = (i >> (PL + 5)) / RBT * PP + q;
      const int row = rb * 16 + r, m = row0 + row, col = (tile * WB + pc) * 8;
      if (m < p.M && col < p.N)
        *(u32x4*)(p.out.p + frag_at(p.out, m, col) + plane * 512) = *(const u32x4*)(sm + plane * PLANE + row * LD + pc * 16);
    }
  } else if constexpr (EPI == 3) {
    if (p.k_parts == 1) {
      // the wavefront's blocks through its part of the LDS, as many columns at a time as fit, so that what is done with a block is
      // there once (unrolled over 64 accumulators it did not fit the registers)
      constexpr int CP = std::min(CBW, T::LDS / 4096 / RBW);
      char* const mine = sm + wave * (CP * RBW * 1024) + lane * 16;
      static_for<0, (CBW + CP - 1) / CP>([&](auto pc) {
        constexpr int c0 = decltype(pc)::value * CP, nc = std::min(CP, CBW - c0);
#pragma unroll
        for (int c = 0; c < nc; ++c)
#pragma unroll
          for (int rb = 0; rb < RBW; ++rb) *(f32x4*)(mine + (rb * nc + c) * 1024) = acc[c0 + c][rb];
#pragma unroll 1
        for (int rb = 0; rb < RBW; ++rb) {
          const int m = row0 + (wr * RBW + rb) * 16 + l16;
          if (m >= p.M) break;
          QkvRow row;
          row.request(p.qkv, m, p.M);
          row.request_page(p.qkv);
#pragma unroll 2
          for (int c = 0; c < nc; ++c) {
            const int blk = tile * WB + wb0 + c0 + c;
            if (blk * 16 >= p.N || wb0 + c0 + c < wown) continue;
            QkvBlock b;
            b.request(p.qkv, row, blk, g4);
            b.put(p.qkv, row, *(const f32x4*)(mine + (rb * nc + c) * 1024), g4);
          }
        }
      });
      return;
    }
    // Several ranges of K: the partial tile into memory, block by block; the workgroups of the other ranges do the same; then each
    // of them sums and finishes its share of the tile's blocks.
    const int S = p.k_parts, tiles = p.n_units / S, U = p.row_blocks * WB;
    const auto parts = __builtin_amdgcn_make_buffer_rsrc(p.part + (size_t)(rh * tiles + tile) * S * U * 256, 0, S * U * 1024, 0x00027000);
#pragma unroll
    for (int c = 0; c < CBW; ++c)
#pragma unroll
      for (int rb = 0; rb < RBW; ++rb) {
        const int r = wr * RBW + rb;
        if (row0 + r * 16 + l16 < p.M && wb0 + c >= wown)
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[c][rb]), parts, lane16, ((part * U + r * WB) + wb0 + c) * 1024, DEVICE_SCOPE);
      }
    // (stores of device scope: once the counter says so, every compute unit's loads of device scope see them)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    unsigned* const todo = (unsigned*)sm;
    if (tid == 0) *todo = meet(DeviceWord{p.meet + (size_t)(rh * tiles + tile) * MEET_STRIDE}, (unsigned)S, (unsigned)part, p.polls);
    if (!EARLY) next.request();
    __syncthreads();
    // (its own share; those of members that did not wait, if it came last)
    auto finish = [&](auto nc) __attribute__((always_inline)) {
      constexpr int NS = decltype(nc)::value;   // >= S: a load behind the last part returns zeros
      unsigned left = __builtin_amdgcn_readfirstlane(*todo);
      for (int who = part;;) {
        if (left >> who & 1u) {
          f32x4 q[NB][NS];
          auto fetch = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
              const int c = next.walk.c + i * next.walk.c_step;
              const unsigned off = next.walk.r < next.rows_here && c < next.cols_here ? (unsigned)(next.walk.r * WB + c) * 1024u + lane16 : 0x70000000u;
#pragma unroll
              for (int s = 0; s < NS; ++s) q[i][s] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(parts, off + (unsigned)(s * U) * 1024u, 0, DEVICE_SCOPE));
            }
          };
          fetch();
          while (next.walk.r < next.rows_here) {
            f32x4 v[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i) {
              v[i] = q[i][0];
#pragma unroll
              for (int s = 1; s < NS; ++s) v[i] += q[i][s];
            }
            QkvRow row = next.row;
            QkvBlock blk[NB];
            const int c_now = next.walk.c, c_step = next.walk.c_step;
#pragma unroll
            for (int i = 0; i < NB; ++i) blk[i] = next.blk[i];
            // what is next is requested in front of the stores: a load behind them would wait for them
            next.walk.next(NB, next.cols_here);
            next.request();
            fetch();
            row.request_page(p.qkv);
            if (row.here) {
#pragma unroll
              for (int i = 0; i < NB; ++i)
                if (c_now + i * c_step < next.cols_here) blk[i].put(p.qkv, row, v[i], g4);
            }
          }
        }
        left &= ~(1u << who);
        if (left == 0u) return;
        who = __builtin_ctz(left);
        next.walk = Walk(next.rows_here, wave, S, who);
        next.request();
      }
    };
    if (S <= 4) finish(std::integral_constant<int, 4>{});
    else finish(std::integral_constant<int, TILE_MAX_K_PARTS>{});
  } else {
#pragma unroll
    for (int c = 0; c < CBW; ++c) {
      const int blk = tile * WB + wb0 + c;
      if (blk * 16 >= p.N || wb0 + c < wown) continue;
      const int col = blk * 16 + 4 * g4;
#pragma unroll
      for (int rb = 0; rb < RBW; ++rb) {
        const int m = row0 + (wr * RBW + rb) * 16 + l16;
        const f32x4 v = acc[c][rb];
        if (m < p.M) *(float4*)(p.Y + part * p.split_stride + (size_t)m * p.ldy + col) = make_float4(v[0], v[1], v[2], v[3]);
      }
    }
  }
}

template <int RB, int WB, int EPI, bool NT>
void launch_tile_one(const TileArgs<EPI>& g, int wgs, hipStream_t st) {
  constexpr int lds = TileShape<RB, WB>::LDS;
  static OncePerDevice once;
  allow_dynamic_lds(once, (const void*)gemm_tile_kernel<RB, WB, EPI, NT>, lds);
  gemm_tile_kernel<RB, WB, EPI, NT><<<wgs, 256, lds, st>>>(g);
}
template <int EPI, bool NT>
void launch_tile_many(const TileArgs<EPI>& g, int rb, int wb, int wgs, hipStream_t st) {   // rb 3..5, wb 8, 12, 14, 16; rb 3, wb 6
#define CLV_TL(RB_)                                                   \
  if (wb == 8) launch_tile_one<RB_, 8, EPI, NT>(g, wgs, st);          \
  else if (wb == 12) launch_tile_one<RB_, 12, EPI, NT>(g, wgs, st);   \
  else if (wb == 14) launch_tile_one<RB_, 14, EPI, NT>(g, wgs, st);   \
  else launch_tile_one<RB_, 16, EPI, NT>(g, wgs, st);
  if (rb == 3 && wb == 6) launch_tile_one<3, 6, EPI, NT>(g, wgs, st);
  else if (rb == 3) { CLV_TL(3) } else if (rb == 4) { CLV_TL(4) } else { CLV_TL(5) }
#undef CLV_TL
}
template <int EPI>
void launch_tile_big(const TileArgs<EPI>& g, int wb, int wgs, hipStream_t st) {   // rb 8 (always several row tiles): wb 12, 14, 16
  if (wb == 12) launch_tile_one<8, 12, EPI, false>(g, wgs, st);
  else if (wb == 14) launch_tile_one<8, 14, EPI, false>(g, wgs, st);
  else launch_tile_one<8, 16, EPI, false>(g, wgs, st);
}
template <int EPI>
void launch_tile_few(const TileArgs<EPI>& g, int rb, int wb, int wgs, hipStream_t st) {    // rb 0: wb 8, 12; rb 1: wb 6, 7, 8, 12; rb 2: wb 6, 7, 8, 12, 16
  if (rb == 0) {
    if constexpr (EPI != 3) {   // (few rows over one range of K: the QKV projection leaves rotation and stores to a second launch)
      if (wb == 8) launch_tile_one<0, 8, EPI, true>(g, wgs, st);
      else launch_tile_one<0, 12, EPI, true>(g, wgs, st);
    } else g_not_launched = "no such form of the QKV projection";
  } else if (rb == 1 && wb == 6) launch_tile_one<1, 6, EPI, true>(g, wgs, st);
  else if (rb == 1 && wb == 7) launch_tile_one<1, 7, EPI, true>(g, wgs, st);
  else if (rb == 1 && wb == 8) launch_tile_one<1, 8, EPI, true>(g, wgs, st);
  else if (rb == 1) launch_tile_one<1, 12, EPI, true>(g, wgs, st);
  else if (wb == 6) launch_tile_one<2, 6, EPI, true>(g, wgs, st);
  else if (wb == 7) launch_tile_one<2, 7, EPI, true>(g, wgs, st);
  else if (wb == 8) launch_tile_one<2, 8, EPI, true>(g, wgs, st);
  else if (wb == 12) launch_tile_one<2, 12, EPI, true>(g, wgs, st);
  else launch_tile_one<2, 16, EPI, true>(g, wgs, st);
}

// one form of the kernel; which of them, pick_tile (kernels_tile.hip)
template <int EPI>
void launch_tile(const TileArgs<EPI>& g, const TileForm& t, int wgs, hipStream_t st) {
  if (t.rb == 8) launch_tile_big<EPI>(g, t.wb, wgs, st);
  else if (t.rb < 3) launch_tile_few<EPI>(g, t.rb, t.wb, wgs, st);
  else if (t.row_tiles > 1) launch_tile_many<EPI, false>(g, t.rb, t.wb, wgs, st);
  else launch_tile_many<EPI, true>(g, t.rb, t.wb, wgs, st);
}

}  // namespace
}  // namespace clv
