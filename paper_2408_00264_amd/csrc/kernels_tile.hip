// The MFMA GEMM of every pass on gfx950 (bf16 weights in fragment order, activations as FragPlanes, fp32 accumulation):
//
//   EPI 0:  Y[M,N]      = X[M,K] * W[N,K]^T                   (fp32; over k_parts ranges of K: partial tiles)
//   EPI 1:  out[M,F]    = planes of silu(X Wg^T) * (X Wu^T)    (the SwiGLU projection)
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
//   QKV          9.7 (12)  11.2       14.9 (18)  16.2 (27)  20.5   25.7 (34)
//   Wo           6.6        8.8       11.1       12.9       15.8   20.6
//   LM head    154        170        177        187        229    365
// The same kernel on row-major planes (64-byte row pieces): gate+up 64.4 at 64 rows, 69.5 at 80, 107 at 256.
// Many rows, tiles of up to 160 / of 256 rows (and half the staged bytes per product): gate+up 179 / 154 at 512, 351 / 306
// at 1024, 701 / 605 at 2048, LM head 777 / 663 at 512, 3106 / 2713 at 2048, down 322 / 302 at 2048, QKV 159 / 137.
//
// RB, WB and the K ranges are chosen per launch (pick_tile).
#include "clover_internal.h"

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
constexpr int TL_CUS = 256;

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

__device__ __forceinline__ unsigned t_rn(float a) { return (unsigned)__builtin_bit_cast(unsigned short, (__bf16)a); }

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

// NT: non-temporal loads, for weights that no other workgroup reads (gate+up at 64 rows 47.0 -> 44.6 us; where row tiles
// share them it costs: 256 rows 96.5 -> 100).
template <int RB, int WB, int EPI, bool NT>
__global__ __launch_bounds__(256, 1) void gemm_tile_kernel(TileGemm p) {
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
  if (unit >= p.n_units) return;   // (grid rounded up to whole XCD rows; uniform over the workgroup)
  const int part = unit % p.k_parts, tile = unit / p.k_parts;
  const int NS = p.K / (TL_KST * KS) / p.k_parts;      // stages of this workgroup's K range
  const int kt0 = part * NS * KS;
  const int row0 = rh * 16 * RBT;

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
  const size_t xstep = KS * xstage, wstep = KS * wstage;
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
void launch_tile_one(const TileGemm& g, int wgs, hipStream_t st) {
  constexpr int lds = TileShape<RB, WB>::LDS;
  static OncePerDevice once;
  allow_dynamic_lds(once, (const void*)gemm_tile_kernel<RB, WB, EPI, NT>, lds);
  gemm_tile_kernel<RB, WB, EPI, NT><<<wgs, 256, lds, st>>>(g);
}
template <int EPI, bool NT>
void launch_tile_many(const TileGemm& g, int rb, int wb, int wgs, hipStream_t st) {   // rb 3..5, wb 8, 12, 14, 16; rb 3, wb 6
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
void launch_tile_big(const TileGemm& g, int wb, int wgs, hipStream_t st) {   // rb 8 (always several row tiles): wb 12, 14, 16
  if (wb == 12) launch_tile_one<8, 12, EPI, false>(g, wgs, st);
  else if (wb == 14) launch_tile_one<8, 14, EPI, false>(g, wgs, st);
  else launch_tile_one<8, 16, EPI, false>(g, wgs, st);
}
template <int EPI>
void launch_tile_few(const TileGemm& g, int rb, int wb, int wgs, hipStream_t st) {    // rb 0: wb 8, 12; rb 1: wb 6, 7, 8, 12; rb 2: wb 6, 7, 8, 12, 16
  if (rb == 0 && wb == 8) launch_tile_one<0, 8, EPI, true>(g, wgs, st);
  else if (rb == 0) launch_tile_one<0, 12, EPI, true>(g, wgs, st);
  else if (rb == 1 && wb == 6) launch_tile_one<1, 6, EPI, true>(g, wgs, st);
  else if (rb == 1 && wb == 7) launch_tile_one<1, 7, EPI, true>(g, wgs, st);
  else if (rb == 1 && wb == 8) launch_tile_one<1, 8, EPI, true>(g, wgs, st);
  else if (rb == 1) launch_tile_one<1, 12, EPI, true>(g, wgs, st);
  else if (wb == 6) launch_tile_one<2, 6, EPI, true>(g, wgs, st);
  else if (wb == 7) launch_tile_one<2, 7, EPI, true>(g, wgs, st);
  else if (wb == 8) launch_tile_one<2, 8, EPI, true>(g, wgs, st);
  else if (wb == 12) launch_tile_one<2, 12, EPI, true>(g, wgs, st);
  else launch_tile_one<2, 16, EPI, true>(g, wgs, st);
}

struct TilePick { int rb, wb, kp; };

// Tile and K ranges of a launch by estimated time, in clocks.  A stage of a workgroup takes the longest of its matrix
// instructions, of its 1 KB loads at 40 B/clk (what is left of the load path's 55 beside the LDS reads) and of an HBM
// round trip shared by the stages in flight; rounds of workgroups over the compute units times stages, against the time
// of the weight stream at 5.3 TB/s (fourth-power mean: near the crossing the two do not overlap freely), + start and
// end of each round, + the partial tiles, written here and read by the consumer.  Over 50 launches (the five 8B shapes at
// ten row counts from 23 to 256, up to 63 combinations of tile and ranges each) the choice is the best or within 5 % of it,
// except Wo at 112 rows (8 %: 22.2 us with its consumer against 20.6 with two row tiles of 96).  So few rows take narrow tiles
// (the weight stream needs every compute unit), 256 rows of gate+up 2 x 128 tiles of 128 rows x 224 columns (one whole
// round, where 256-column tiles leave 32 compute units idle), 80 rows one row tile of 96.
// More than 256 rows over 1024 columns of K or more also have tiles of 256 rows (256 accumulators and 200 other registers a
// lane with 256 columns; 128 columns were slower than 128 x 256 at every shape), a stage there costs 260 + 20.6 clocks per product
// (2 % to 8 % off over 40 forms at 512, 1024 and 2048 rows; the choice is the best or within 4 % of it there and in 60 launches
// at twelve odd row counts from 343 to 1533, but for QKV at 459 rows, 13 %, and at 623 and Wo at 747, 5 to 7 %), and a
// round ends with the XCD that has most row tiles (Wo at 1024 rows: 264 workgroups of 96 x 192, 33 of them on one XCD, 114 us;
// 256 of 128 x 128 58).
// kp_fixed > 0 fixes the K ranges.
TilePick pick_tile(int M, int N, int K, int epi, int kp_fixed) {
  static const int cbs[5] = {3, 4, 6, 7, 8};
  const bool one = M <= 16;
  M = (M + 31) / 32 * 32;   // the K ranges (and with them the size of the partial tiles) depend on this only
  const int blocks = epi == 1 ? N / 8 : N / 16;
  const double stream = (double)blocks * 32.0 * K / 2450.0;
  const int rb_lo = M > 64 ? 3 : M / 32, rb_hi = M > 64 ? 5 : M / 32, KT = K / TL_KST;
  const int only_rb = tune_int("CLOVER_TILE_RB", 0), only_cb = tune_int("CLOVER_TILE_CB", 0), only_kp = tune_int("CLOVER_TILE_KP", 0);
  const bool many = M > 256 && K >= 1024;
  TilePick best{rb_lo, 8, 1};
  double best_t = 1e30;
  for (int rb = rb_lo; rb <= (many ? 8 : rb_hi); ++rb)
    for (int cb : cbs) {
      if (rb == 6 || rb == 7) continue;
      if ((only_rb > 0 && rb != only_rb) || (only_cb > 0 && cb != only_cb)) continue;
      // (up to 32 rows a tile of 256 columns is slower than one of 192 however the rounds fall: LM head 176 against 166 us)
      if ((rb == 1 && cb > 6) || (rb == 2 && cb == 7) || (rb > 3 && cb == 3) || (rb == 8 && cb == 4)) continue;
      const int rt = (M + 32 * rb - 1) / (32 * rb), tiles = (blocks + 2 * cb - 1) / (2 * cb);
      const int nbuf = std::min(6, 160 / (4 * rb + 2 * cb));
      const double products = rb * cb * 2 * 19.0 + (many ? 260.0 + rb * cb * 1.6 : 0.0);
      const double stage = std::max(std::max(products, (4 * rb + 2 * cb) * 1024 / 40.0), 4300.0 / nbuf);
      for (int kp = 1; kp <= TILE_MAX_K_PARTS; ++kp) {
        // (row tiles of the same columns stay on one XCD: its 32 compute units bound the round, not the 256 of all eight)
        const int rounds = many ? ((tiles * kp + 7) / 8 * rt + TL_CUS / 8 - 1) / (TL_CUS / 8) : (rt * tiles * kp + TL_CUS - 1) / TL_CUS;
        if (kp_fixed > 0 ? kp != kp_fixed : KT % kp != 0 || (kp > 1 && (KT / kp < 8 || rounds > 1))) continue;
        if (kp_fixed <= 0 && only_kp > 0 && kp != only_kp) continue;
        const double work = rounds * (KT / kp) * stage, a = work * work, b = stream * stream;
        const double t = std::sqrt(std::sqrt(a * a + b * b)) + rounds * 5000.0 + (kp > 1 ? kp * (double)M * N * 8.0 / 2300.0 : 0.0);
        if (t < best_t) { best_t = t; best = TilePick{rb, 2 * cb, kp}; }
      }
    }
  // Up to 16 rows over the whole K: the one-row-block form (gate+up 41 -> 36 us, LM head 165 -> 157 at one row).  Over K
  // ranges its 64-column stages are too coarse for 8 to 16 of them (QKV 10.9 -> 12.7, Wo and down 13.5 -> 14.0).
  if (one && best.kp == 1 && best.wb != 6) best.rb = 0;
  // Seven column blocks instead of eight where one round of workgroups still holds them: more compute units share the lines that
  // are loaded.  gate+up of 14336 channels, 224 -> 256 workgroups: 23 rows 38.5 -> 37.5 us, 64 rows 46.9 -> 45.8; 80 and 96 rows gain
  // less than half a percent, and one row, bound by the weight stream itself, loses one.
  if ((best.rb == 1 || best.rb == 2) && best.wb == 8 && M <= 32 * best.rb && (blocks + 6) / 7 * best.kp <= TL_CUS && tune_int("CLOVER_TILE_WB7", 1)) best.wb = 7;
  return best;
}

}  // namespace

// N: rows of W (epi 1: the FFN width F), N % 16 == 0, K % 64 == 0
int tile_gemm_pick_k_parts(int M, int N, int K) { return pick_tile(M, N, K, 0, 0).kp; }

TileForm tile_gemm_form(int M, int N, int K, int epi, int k_parts) {
  const TilePick t = pick_tile(M, N, K, epi, epi == 1 ? 1 : k_parts);
  const int rows = t.rb == 0 ? 16 : 32 * t.rb;
  return TileForm{t.rb, t.wb, (M + rows - 1) / rows, t.kp, K / (t.rb == 0 ? 2 * TL_KST : TL_KST) / t.kp};
}

void launch_gemm_tile(const TileGemm& g_in, hipStream_t st) {
  TileGemm g = g_in;
  if (g.k_parts < 1 || g.epi == 1) g.k_parts = 1;
  const TileForm t = tile_gemm_form(g.M, g.N, g.K, g.epi, g.k_parts);
  const int blocks = g.epi == 1 ? g.N / 8 : g.N / 16, rt = t.row_tiles;
  g.n_units = (blocks + t.wb - 1) / t.wb * g.k_parts;
  const int wgs = rt > 1 ? (g.n_units + 7) / 8 * 8 * rt : g.n_units;
  auto go = [&](auto epic) {
    constexpr int EPI = decltype(epic)::value;
    if (t.rb == 8) launch_tile_big<EPI>(g, t.wb, wgs, st);
    else if (t.rb < 3) launch_tile_few<EPI>(g, t.rb, t.wb, wgs, st);
    else if (rt > 1) launch_tile_many<EPI, false>(g, t.rb, t.wb, wgs, st);
    else launch_tile_many<EPI, true>(g, t.rb, t.wb, wgs, st);
  };
  if (g.epi == 1) go(std::integral_constant<int, 1>{});
  else go(std::integral_constant<int, 0>{});
}

// ------------------------------------------------------------------------------------------
// weights in fragment order, once at init
// ------------------------------------------------------------------------------------------
namespace {
// one 16-byte piece per thread: row block nb of src becomes block nb0 + nb of a matrix of n_wb row blocks;
// GU: block b of the packed matrix is 8 rows of src, then the same 8 of src2
template <bool GU>
__global__ void pack_weight_kernel(const bf16_t* __restrict__ src, const bf16_t* __restrict__ src2, bf16_t* __restrict__ dst,
                                   size_t pieces, int K, int nb0, int n_wb) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= pieces) return;
  const int lane = (int)(idx & 63), r = lane & 15, KT = K / 32;
  const size_t blk = idx >> 6, nb = blk / KT;
  const int kt = (int)(blk % KT), k = kt * 32 + (lane >> 4) * 8;
  const bf16_t* from = GU ? (r < 8 ? src : src2) + (nb * 8 + (r & 7)) * K : src + (nb * 16 + r) * K;
  *(u32x4*)(dst + (((size_t)kt * n_wb + nb0 + nb) * 64 + lane) * 8) = *(const u32x4*)(from + k);
}
}  // namespace
void launch_pack_weight(const void* src, void* dst, int N, int K, int row0, int n_rows, hipStream_t st) {
  const size_t pieces = (size_t)N * K / 8;
  pack_weight_kernel<false><<<(unsigned)((pieces + 255) / 256), 256, 0, st>>>((const bf16_t*)src, nullptr, (bf16_t*)dst, pieces, K,
                                                                              row0 / 16, n_rows / 16);
}
void launch_pack_gate_up(const void* gate, const void* up, void* dst, int F, int K, hipStream_t st) {
  const size_t pieces = (size_t)2 * F * K / 8;
  pack_weight_kernel<true><<<(unsigned)((pieces + 255) / 256), 256, 0, st>>>((const bf16_t*)gate, (const bf16_t*)up, (bf16_t*)dst, pieces, K,
                                                                             0, F / 8);
}

}  // namespace clv
