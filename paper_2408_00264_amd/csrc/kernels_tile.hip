// Which form of the MFMA GEMM (gemm_tile.h) a launch takes, and the packing of its weights.
#include "clover_internal.h"

#include <algorithm>
#include <cmath>

namespace clv {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

void launch_tile_plain(const TileGemm& g, const TileForm& t, int wgs, hipStream_t st);
void launch_tile_swiglu(const TileGemm& g, const TileForm& t, int wgs, hipStream_t st);
void launch_tile_qkv(const TileGemmQkv& g, const TileForm& t, int wgs, hipStream_t st);

namespace {

constexpr int TL_KST = 32, TL_CUS = 256;   // K columns per stage; compute units

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

static int tiles_of(const TileForm& t, int N) { return (N / 16 + t.wb - 1) / t.wb; }
// workgroups of an XCD that has the ranges of its tiles together
static int wgs_per_xcd(const TileForm& t, int N) { return (tiles_of(t, N) + 7) / 8 * t.row_tiles * t.k_parts; }

// Measured by whole verify passes, one launch and two in turn, us a layer (profiles/qkv_joint_sweep.txt).
//
// With MFMA attention, one launch - two: 48 and 64 rows over three or four ranges -0.4 to -3.2 of 54 to 365 (4096 channels, 64 rows -1.6 of
// 138, with 32 KV heads -2.0), 33 rows and up to 32 -2.1 to +0.4.  Two ranges: up to 32 rows -2.1 to +0.7, above +0.4 to +4.4
// (4096 channels, 32 KV heads, 128 rows +3.6 of 185): a member has half the tile to finish.  65 to 128 rows in one row tile: -3.6 to 0
// where a range has 16 stages or more, +0.5 to +1.5 where it has fewer (1024, 1280 and 1536 channels).  More row tiles: -2.0 to
// +1.2 (4096 channels, 8 KV heads, 128 rows +1.1).  Above 128 rows, and ranges on different XCDs: +3.7 to -2.9, and 256 rows and more the
// same or slower.  Five to eight ranges, which few rows have: a step of 23 rows 0.8 % slower.
//
// Without it (heads of 64, groups other than 1, 2, 4, 8), where the second launch writes q in fp32; one launch and two: 2048 channels, 32
// heads of 64 over 8: one row 64.8 and 63.8, 16 66.5 and 66.0, 32 73.7 and 73.1, 33 79.9 and 80.3, 64 88.1 and 90.9, 256 167 and 173, a prompt
// of 1024 824 and 849; 3584 channels, 28 heads of 128 over 4 (at 64 rows seven ranges on different XCDs): 122.2 and 121.1, 129.3 and
// 128.5, 138.8 and 138.8, 145.5 and 146.4, 163.9 and 167.5, 422 and 422, 1919 and 1947.
bool tile_gemm_qkv_joins(int M, int N, int K, int k_parts, bool mfma_attention, TileForm* form) {
  if (mfma_attention && (M > 128 || k_parts > 4 || k_parts < (M <= 32 ? 2 : 3))) return false;
  if (!mfma_attention && M <= 32) return false;
  const TileForm t = *form = tile_gemm_form(M, N, K, 0, k_parts);
  if (k_parts > 1 && tiles_of(t, N) * t.row_tiles > TILE_MEETINGS) return false;
  return !mfma_attention || (t.row_tiles == 1 && wgs_per_xcd(t, N) <= TL_CUS / 8 && (M <= 64 || t.stages >= 16));
}
size_t tile_gemm_exchange_bytes(const TileForm& t, int M, int N) {
  if (t.k_parts < 2) return 0;
  return (size_t)t.row_tiles * tiles_of(t, N) * t.k_parts * std::min(2 * t.rb, (M + 15) / 16) * t.wb * 1024;
}

void launch_gemm_tile(const TileGemm& g_in, hipStream_t st) {
  TileGemm g = g_in;
  if (g.k_parts < 1 || g.epi == 1) g.k_parts = 1;
  const TileForm t = tile_gemm_form(g.M, g.N, g.K, g.epi, g.k_parts);
  const int blocks = g.epi == 1 ? g.N / 8 : g.N / 16, rt = t.row_tiles;
  g.n_units = (blocks + t.wb - 1) / t.wb * g.k_parts;
  const int wgs = rt > 1 ? (g.n_units + 7) / 8 * 8 * rt : g.n_units;
  (g.epi == 1 ? launch_tile_swiglu : launch_tile_plain)(g, t, wgs, st);
}

void launch_gemm_qkv(const TileGemmQkv& g_in, const TileForm& t, hipStream_t st) {
  TileGemmQkv g = g_in;
  const int rt = t.row_tiles, tiles = tiles_of(t, g.N), per_xcd = wgs_per_xcd(t, g.N);
  g.k_parts = t.k_parts;
  g.n_units = tiles * g.k_parts;
  g.row_blocks = std::min(2 * t.rb, (g.M + 15) / 16);
  g.spread = per_xcd > TL_CUS / 8;   // (a member of a second round would keep those of the first waiting)
  int wgs = rt > 1 ? (g.n_units + 7) / 8 * 8 * rt : g.n_units;
  if (g.k_parts > 1 && !g.spread) wgs = 8 * per_xcd;
  launch_tile_qkv(g, t, wgs, st);
}

// ------------------------------------------------------------------------------------------
// weights in fragment order, once at init
// ------------------------------------------------------------------------------------------
namespace {
// one 16-byte piece per thread: row block nb of src becomes block nb0 + nb of a matrix of n_wb row blocks;
// GU: block b of the packed matrix is 8 rows of src, then the same 8 of src2
template <bool GU>
__global__ void pack_weight_kernel(const bf16_t* __restrict__ src, const bf16_t* __restrict__ src2, bf16_t* __restrict__ dst,
                                   size_t pieces, int K, int nb0, int n_wb, int rotary_d) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= pieces) return;
  const int lane = (int)(idx & 63), r = lane & 15, KT = K / 32;
  const size_t blk = idx >> 6, nb = blk / KT;
  const int kt = (int)(blk % KT), k = kt * 32 + (lane >> 4) * 8;
  size_t row = nb * 16 + r;
  if (rotary_d) {   // block j of a head: rows 8j .. of its first half, then of its second
    const size_t per_head = rotary_d / 16, h = nb / per_head, j = nb % per_head;
    row = h * rotary_d + j * 8 + (r & 7) + (r >> 3) * (rotary_d / 2);
  }
  const bf16_t* from = GU ? (r < 8 ? src : src2) + (nb * 8 + (r & 7)) * K : src + row * K;
  *(u32x4*)(dst + (((size_t)kt * n_wb + nb0 + nb) * 64 + lane) * 8) = *(const u32x4*)(from + k);
}
}  // namespace
void launch_pack_weight(const void* src, void* dst, int N, int K, int row0, int n_rows, hipStream_t st, int rotary_d) {
  const size_t pieces = (size_t)N * K / 8;
  pack_weight_kernel<false><<<(unsigned)((pieces + 255) / 256), 256, 0, st>>>((const bf16_t*)src, nullptr, (bf16_t*)dst, pieces, K,
                                                                              row0 / 16, n_rows / 16, rotary_d);
}
void launch_pack_gate_up(const void* gate, const void* up, void* dst, int F, int K, hipStream_t st) {
  const size_t pieces = (size_t)2 * F * K / 8;
  pack_weight_kernel<true><<<(unsigned)((pieces + 255) / 256), 256, 0, st>>>((const bf16_t*)gate, (const bf16_t*)up, (bf16_t*)dst, pieces, K,
                                                                             0, F / 8, 0);
}

}  // namespace clv
