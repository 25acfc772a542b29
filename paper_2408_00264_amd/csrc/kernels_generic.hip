// Plain fp32-ALU kernels of the Clover-2 speculative step: every stage that is not a large
// contraction, plus simple (slow, shape-agnostic) GEMM and attention used for fp32 models and
// as the on-device cross-check of the MFMA path.
#include "clover_internal.h"

#include <algorithm>
#include <type_traits>

namespace clv {

// ------------------------------------------------------------------------------------------
// small device helpers
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ float bf16_to_f32(bf16_t u) { return __uint_as_float(((unsigned)u) << 16); }
// round to nearest even through the hardware conversion (v_cvt_pk_bf16_f32)
__device__ __forceinline__ bf16_t f32_to_bf16(float f) { return __builtin_bit_cast(unsigned short, (__bf16)f); }
__device__ __forceinline__ float ldf(const float* p, size_t i) { return p[i]; }
__device__ __forceinline__ float ldf(const bf16_t* p, size_t i) { return bf16_to_f32(p[i]); }
__device__ __forceinline__ void stf(float* p, size_t i, float v) { p[i] = v; }
__device__ __forceinline__ void stf(bf16_t* p, size_t i, float v) { p[i] = f32_to_bf16(v); }
// KV-cache elements: fp32, or a (hi, lo) pair of bf16 planes `plane` elements apart
__device__ __forceinline__ float ldkv(const float* p, size_t i, size_t) { return p[i]; }
__device__ __forceinline__ float ldkv(const bf16_t* p, size_t i, size_t plane) {
  return bf16_to_f32(p[i]) + bf16_to_f32(p[i + plane]);
}
__device__ __forceinline__ void stkv(float* p, size_t i, size_t, float v) { p[i] = v; }
__device__ __forceinline__ void stkv(bf16_t* p, size_t i, size_t plane, float v) {
  const bf16_t h = f32_to_bf16(v);
  p[i] = h;
  p[i + plane] = f32_to_bf16(v - bf16_to_f32(h));
}
__device__ __forceinline__ void mvkv(float* p, size_t dst, size_t src, size_t) { p[dst] = p[src]; }
__device__ __forceinline__ void mvkv(bf16_t* p, size_t dst, size_t src, size_t plane) {
  p[dst] = p[src];
  p[dst + plane] = p[src + plane];
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
// sum over a 256-thread block; `red` is 4 floats of LDS.  All threads get the result.
__device__ __forceinline__ float block_sum_256(float v, float* red) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

// ------------------------------------------------------------------------------------------
// RMSNorm: out = x * rsqrt(mean(x^2) + eps) * gain      (one block per row)
// ------------------------------------------------------------------------------------------
template <typename WT>
__global__ void rmsnorm_kernel(const float* __restrict__ x, int ldx, const WT* __restrict__ gain, float eps,
                               float* __restrict__ out, int ldo, int H) {
  __shared__ float red[4];
  const size_t row = blockIdx.x;
  const float* xr = x + row * ldx;
  float ss = 0.f;
  for (int c = threadIdx.x; c < H; c += 256) { float v = xr[c]; ss += v * v; }
  ss = block_sum_256(ss, red);
  const float scale = 1.0f / sqrtf(ss / (float)H + eps);
  for (int c = threadIdx.x; c < H; c += 256) out[row * ldo + c] = xr[c] * scale * ldf(gain, c);
}

void launch_rmsnorm(const float* x, int ldx, const void* gain, int wdtype, float eps, float* out, int ldo, int H,
                    int rows, hipStream_t st) {
  if (rows <= 0) return;
  if (wdtype == 0)
    rmsnorm_kernel<float><<<rows, 256, 0, st>>>(x, ldx, (const float*)gain, eps, out, ldo, H);
  else
    rmsnorm_kernel<bf16_t><<<rows, 256, 0, st>>>(x, ldx, (const bf16_t*)gain, eps, out, ldo, H);
}

// ------------------------------------------------------------------------------------------
// RoPE on q and k (half-split pairing), K rows and transposed V columns into the cache; q stays in fp32.  For fp32 models, and for few
// rows of bf16 models whose heads have no MFMA attention: there the QKV GEMM leaves partial tiles, heads of q and k in rotary order
// (launch_pack_weight).  (Those could take the kernel below as well; us a layer with it / with this one, 2048 channels, 32 heads of 64
// over 8: one row 64.2 / 62.2, 16 rows 67.3 / 66.3.)
// blocks [0, n*hc): 256 (head, pair) items of one row; then blocks of 8 (head,dim) lines of V^T
// ------------------------------------------------------------------------------------------
template <typename KT>
__device__ __forceinline__ float qkv_at(const float* __restrict__ p, int nsp, size_t sps) {   // the sum of the ranges, in their order
  if constexpr (std::is_same<KT, float>::value) return *p;
  float q[TILE_MAX_K_PARTS], v = 0.f;
#pragma unroll
  for (int j = 0; j < TILE_MAX_K_PARTS; ++j) q[j] = j < nsp ? p[(size_t)j * sps] : 0.f;
#pragma unroll
  for (int j = 0; j < TILE_MAX_K_PARTS; ++j) v += q[j];
  return v;
}
template <typename KT>
__global__ void rope_kv_write_kernel(const float* __restrict__ qkv, int ldqkv, int nsp, size_t sps, const float* __restrict__ cos_t,
                                     const float* __restrict__ sin_t, float* __restrict__ q_out, int ldq,
                                     KT* __restrict__ kc, KT* __restrict__ vc, KVLayout kv,
                                     const int* __restrict__ base_len, int n_q, RowMap rm, int* err_flag, int hc) {
  constexpr bool ROTARY = !std::is_same<KT, float>::value;   // order of a head's columns
  const int b = blockIdx.y;
  const int nv = rows_valid(rm, b);
  const int L = base_len[b];
  const int d = kv.d, half = d / 2, n_kv = kv.n_kv;
  if (L + nv > kv.max_seq) {  // would overrun the cache: refuse, flag
    if (threadIdx.x == 0 && blockIdx.x == 0) atomicOr(err_flag, 1);
    return;
  }
  if ((int)blockIdx.x < rm.n * hc) {
    const int i = blockIdx.x / hc;
    if (i >= nv) return;
    const int idx = (blockIdx.x % hc) * 256 + threadIdx.x;
    if (idx >= (n_q + n_kv) * half) return;
    const size_t row = (size_t)b * rm.R + i;
    const int hh = idx / half, ii = idx - hh * half;
    const float c = cos_t[row * half + ii], s = sin_t[row * half + ii];
    const float* src = qkv + row * ldqkv + hh * d + (ROTARY ? (ii >> 3) * 16 + (ii & 7) : ii);
    const float x1 = qkv_at<KT>(src, nsp, sps), x2 = qkv_at<KT>(src + (ROTARY ? 8 : half), nsp, sps);
    const float o1 = x1 * c - x2 * s, o2 = x2 * c + x1 * s;
    if (hh < n_q) {
      q_out[row * ldq + hh * d + ii] = o1;
      q_out[row * ldq + hh * d + ii + half] = o2;
    } else {
      const size_t base = kv_k_at(kv, b, L + i, hh - n_q);
      stkv(kc, base + kv_k_col(kv, ii), kv.plane, o1);
      stkv(kc, base + kv_k_col(kv, ii + half), kv.plane, o2);
    }
  } else {
    const int vb = blockIdx.x - rm.n * hc;
    const int voff = (n_q + n_kv) * d;
    for (int idx = threadIdx.x; idx < 8 * rm.n; idx += blockDim.x) {
      const int node = idx % rm.n, e = vb * 8 + idx / rm.n;
      if (node >= nv || e >= n_kv * d) continue;
      const float v = qkv_at<KT>(qkv + ((size_t)b * rm.R + node) * ldqkv + voff + e, nsp, sps);
      stkv(vc, kv_v_at(kv, b, e / d, e % d, L + node), kv.plane, v);
    }
  }
}

// The same operation in front of the MFMA attention, for launches whose QKV GEMM does not do it itself (heads of q and k in rotary order,
// q as pre-scaled bf16 planes, bf16-plane caches), vectorised: a thread of the first blocks rotates four adjacent channels of one head
// (float4 loads of every partial, issued before anything else is waited for; 8-byte plane stores); the last blocks transpose 64 nodes x
// 32 channels of V through LDS so that the partials are read along the channels and V^T is written along the nodes.
__device__ __forceinline__ void planes4(bf16_t* hi, bf16_t* lo, size_t off, const float (&o)[4]) {
  unsigned h[4], l[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const bf16_t hb = f32_to_bf16(o[r]);
    h[r] = hb;
    l[r] = f32_to_bf16(o[r] - bf16_to_f32(hb));
  }
  *(uint2*)(hi + off) = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
  *(uint2*)(lo + off) = make_uint2(l[0] | (l[1] << 16), l[2] | (l[3] << 16));
}
// The K ranges are counted at compile time here and in reduce_add_norm_kernel: every load of a thread is requested in
// straight-line code before the first is used.  With a runtime count the two halves of a pair were one round trip to memory
// after the other, and most of the instructions were branches around loads of ranges that do not exist.  us per launch:
// reduce_add_norm of 512 rows x 2 ranges 12.5 -> 10.0, 1024 x 1 17.9 -> 14.2, 2048 x 1 31.9 -> 26.2; rope_kv_planes of one row
// x 8 ranges 5.6 -> 5.1, 64 x 4 5.2 -> 5.1, 512 x 2 10.8 -> 10.4.
template <int NS>
struct Partials4 {
  float4 q[NS];
  __device__ __forceinline__ void request(const float* __restrict__ p, size_t sps) {
#pragma unroll
    for (int s = 0; s < NS; ++s) q[s] = *(const float4*)(p + (size_t)s * sps);
  }
  __device__ __forceinline__ float4 add_to(float4 v) const {   // in range order
#pragma unroll
    for (int s = 0; s < NS; ++s) { v.x += q[s].x; v.y += q[s].y; v.z += q[s].z; v.w += q[s].w; }
    return v;
  }
  __device__ __forceinline__ float4 sum() const { return add_to(make_float4(0.f, 0.f, 0.f, 0.f)); }
};
template <>
struct Partials4<0> {
  __device__ __forceinline__ void request(const float*, size_t) {}
  __device__ __forceinline__ float4 add_to(float4 v) const { return v; }
};
template <int NS>
__global__ __launch_bounds__(256) void rope_kv_planes_kernel(const float* __restrict__ qkv, int ldqkv, size_t sps,
                                                             const float* __restrict__ cos_t, const float* __restrict__ sin_t,
                                                             bf16_t* __restrict__ kc, bf16_t* __restrict__ vc, KVLayout kv,
                                                             const int* __restrict__ base_len, int n_q, RowMap rm,
                                                             int* err_flag, int qk_blocks, bf16_t* __restrict__ q_hi,
                                                             bf16_t* __restrict__ q_lo, int ldq, float q_scale) {
  __shared__ float tile[64][33];
  const int b = blockIdx.y, tid = threadIdx.x;
  const int d = kv.d, half = d / 2, n_kv = kv.n_kv;
  if ((int)blockIdx.x < qk_blocks) {
    // four of a head's channels in rotary order (launch_pack_weight) to a thread, so that the partials are read as they lie; the
    // channels that are rotated with them are two lanes away
    const int quads = d / 4, per_row = (n_q + n_kv) * quads;
    const int idx = blockIdx.x * 256 + tid;
    const int i = idx / per_row, rem = idx - i * per_row, hh = rem / quads, p4 = rem - hh * quads, ii = (p4 >> 2) * 8 + (p4 & 1) * 4;
    const bool second = p4 & 2;
    const size_t row = (size_t)b * rm.R + min(i, rm.n - 1);
    Partials4<NS> p;
    p.request(qkv + row * ldqkv + rem * 4, sps);
    const float4 c = *(const float4*)(cos_t + row * half + ii), s = *(const float4*)(sin_t + row * half + ii);
    const int nv = rows_valid(rm, b), L = base_len[b];
    if (L + nv > kv.max_seq) {  // would overrun the cache: refuse, flag
      if (tid == 0 && blockIdx.x == 0) atomicOr(err_flag, 1);
      return;
    }
    if (i >= nv) return;   // (four adjacent lanes have one row)
    const float4 v = p.sum();
    const float x[4] = {v.x, v.y, v.z, v.w}, cs[4] = {c.x, c.y, c.z, c.w}, sn[4] = {s.x, s.y, s.z, s.w};
    float o[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float y = __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x[r]), 0x4e, 0xf, 0xf, false));   // quad_perm 2 3 0 1
      o[r] = second ? x[r] * cs[r] + y * sn[r] : x[r] * cs[r] - y * sn[r];
    }
    const int col = ii + (second ? half : 0);
    if (hh < n_q) {
#pragma unroll
      for (int r = 0; r < 4; ++r) o[r] *= q_scale;
      planes4(q_hi, q_lo, row * ldq + hh * d + col, o);
    } else {
      planes4(kc, kc + kv.plane, kv_k_at(kv, b, L + i, hh - n_q) + kv_k_col(kv, col), o);
    }
  } else {
    const int n_eb = n_kv * d / 32;
    const int vblk = blockIdx.x - qk_blocks, eb = vblk % n_eb, nb0 = (vblk / n_eb) * 64;
    const int voff = (n_q + n_kv) * d + eb * 32;
    Partials4<NS> p[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int f = tid + 256 * j, node = min(nb0 + f / 8, rm.n - 1), e4 = (f % 8) * 4;
      p[j].request(qkv + ((size_t)b * rm.R + node) * ldqkv + voff + e4, sps);
    }
    const int nv = rows_valid(rm, b), L = base_len[b];
    if (L + nv > kv.max_seq) return;  // (flagged by the first block)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int f = tid + 256 * j, e4 = (f % 8) * 4;
      const float4 v = p[j].sum();
      tile[f / 8][e4] = v.x; tile[f / 8][e4 + 1] = v.y; tile[f / 8][e4 + 2] = v.z; tile[f / 8][e4 + 3] = v.w;
    }
    __syncthreads();
    const int nl = tid % 64, node = nb0 + nl;
    if (node >= nv) return;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int e = tid / 64 + 4 * j;
      const float val = tile[nl][e];
      const size_t at = kv_v_at(kv, b, (eb * 32 + e) / d, (eb * 32 + e) % d, L + node);
      const bf16_t hb = f32_to_bf16(val);
      vc[at] = hb;
      vc[at + kv.plane] = f32_to_bf16(val - bf16_to_f32(hb));
    }
  }
}

void launch_rope_kv_planes(const float* qkv, int ldqkv, int splits, size_t split_stride, const float* cos_t, const float* sin_t, bf16_t* k_cache,
                           bf16_t* v_cache, KVLayout kv, const int* base_len, int n_q, RowMap rm, int* err_flag, bf16_t* q_hi, bf16_t* q_lo,
                           int ldq, float q_scale, hipStream_t st) {
  const int per_row = (n_q + kv.n_kv) * (kv.d / 4);
  const int qk_blocks = (rm.n * per_row + 255) / 256;
  const int v_blocks = (kv.n_kv * kv.d / 32) * ((rm.n + 63) / 64);
  with_count<1, TILE_MAX_K_PARTS>(splits, [&](auto nc) {
    rope_kv_planes_kernel<decltype(nc)::value><<<dim3(qk_blocks + v_blocks, rm.B), 256, 0, st>>>(
        qkv, ldqkv, split_stride, cos_t, sin_t, k_cache, v_cache, kv, base_len, n_q, rm, err_flag, qk_blocks, q_hi, q_lo, ldq, q_scale);
  });
}
template <typename KT>
static void launch_rope_kv_one(const float* qkv, int ldqkv, int splits, size_t split_stride, const float* cos_t, const float* sin_t, float* q_out,
                               int ldq, KT* k_cache, KT* v_cache, KVLayout kv, const int* base_len, int n_q, RowMap rm, int* err_flag,
                               hipStream_t st) {
  const int vblocks = (kv.n_kv * kv.d + 7) / 8;
  const int hc = ((n_q + kv.n_kv) * (kv.d / 2) + 255) / 256;
  rope_kv_write_kernel<KT><<<dim3(rm.n * hc + vblocks, rm.B), 256, 0, st>>>(qkv, ldqkv, splits, split_stride, cos_t, sin_t, q_out, ldq, k_cache,
                                                                            v_cache, kv, base_len, n_q, rm, err_flag, hc);
}
void launch_rope_kv_write(const float* qkv, int ldqkv, const float* cos_t, const float* sin_t, float* q_out, int ldq, float* k_cache,
                          float* v_cache, KVLayout kv, const int* base_len, int n_q, RowMap rm, int* err_flag, hipStream_t st) {
  launch_rope_kv_one(qkv, ldqkv, 1, 0, cos_t, sin_t, q_out, ldq, k_cache, v_cache, kv, base_len, n_q, rm, err_flag, st);
}
void launch_rope_kv_parts(const float* qkv, int ldqkv, int splits, size_t split_stride, const float* cos_t, const float* sin_t, float* q_out,
                          int ldq, bf16_t* k_cache, bf16_t* v_cache, KVLayout kv, const int* base_len, int n_q, RowMap rm, int* err_flag,
                          hipStream_t st) {
  if (splits > TILE_MAX_K_PARTS) { g_not_launched = "no kernel for this count of partial results"; return; }
  launch_rope_kv_one(qkv, ldqkv, splits, split_stride, cos_t, sin_t, q_out, ldq, k_cache, v_cache, kv, base_len, n_q, rm, err_flag, st);
}

// ------------------------------------------------------------------------------------------
// tree-masked attention.  Keys: cached slots [0,L) all visible,
// then the rm.n new rows at slots L+w, visible iff bit w of the row's ancestor mask is set.
// anc == null: the rows form a chain (row i sees new rows 0..i), any number of rows.
// iv != null: new row w is visible to row i iff enter[w] <= enter[i] <= exit[w] (interval labels, two ints per node).
// ------------------------------------------------------------------------------------------
// Over caches of two bf16 planes, for heads that the MFMA attention does not take (fp32 caches: attn_fp32_kernel below): one wavefront per
// (row, query head), results as planes.  What bounds it: memory round trips.  A lane fetches its key's row and its channel's 64 values
// in pieces of four that are all requested before the first is used.
// Tiles that are hidden from a row altogether are not loaded, and a chain's row ends with its own tile (heads of 64, 1000 tokens in one
// pass: 1300 -> 730 us a layer).
__device__ __forceinline__ float4 ldkv4(const bf16_t* p, size_t i, size_t plane) {
  const uint2 h = *(const uint2*)(p + i), l = *(const uint2*)(p + i + plane);
  return make_float4(__uint_as_float(h.x << 16) + __uint_as_float(l.x << 16),
                     __uint_as_float(h.x & 0xFFFF0000u) + __uint_as_float(l.x & 0xFFFF0000u),
                     __uint_as_float(h.y << 16) + __uint_as_float(l.y << 16),
                     __uint_as_float(h.y & 0xFFFF0000u) + __uint_as_float(l.y & 0xFFFF0000u));
}
template <int D>
__global__ __launch_bounds__(64) void attn_generic_kernel(const float* __restrict__ q, int ldq, const bf16_t* __restrict__ kc,
                                                          const bf16_t* __restrict__ vc, KVLayout kv, const int* __restrict__ base_len,
                                                          const unsigned long long* __restrict__ anc, int n_q,
                                                          FragPlanes planes, RowMap rm, int anc_stride, const int* __restrict__ iv) {
  __shared__ __attribute__((aligned(16))) float qs[D];
  __shared__ __attribute__((aligned(16))) float ps[64];
  const int h = blockIdx.x, i = blockIdx.y, b = blockIdx.z, lane = threadIdx.x;
  const int nv = rows_valid(rm, b);
  if (i >= nv) return;
  const int n_kv = kv.n_kv;
  const int L = base_len[b];
  if (L + nv > kv.max_seq) return;
  const size_t row = (size_t)b * rm.R + i;
  const bool chain = anc == nullptr && iv == nullptr;
  const bool bits = anc != nullptr && iv == nullptr;
  const unsigned long long a0 = bits ? anc[2 * ((size_t)b * anc_stride + i)] : 0ull;
  const unsigned long long a1 = bits ? anc[2 * ((size_t)b * anc_stride + i) + 1] : 0ull;
  const int my_enter = iv ? iv[2 * ((size_t)b * anc_stride + i)] : 0;
  const int g = h / (n_q / n_kv);
  const float scale = 1.0f / sqrtf((float)D);
  for (int c = lane; c < D; c += 64) qs[c] = q[row * ldq + h * D + c] * scale;
  __syncthreads();
  float mrun = -INFINITY, lrun = 0.f, o[D / 64];
#pragma unroll
  for (int u = 0; u < D / 64; ++u) o[u] = 0.f;
  const int total = L + (chain ? i + 1 : rm.n);   // (a chain's row sees nothing behind itself)
  const int ntiles = (total + 63) / 64;
  for (int t = 0; t < ntiles; ++t) {
    const int s = t * 64 + lane;
    bool vis = s < L;
    if (!vis && s < total) {
      const int w = s - L;
      if (chain) vis = true;
      else if (iv) vis = iv[2 * ((size_t)b * anc_stride + w)] <= my_enter && my_enter <= iv[2 * ((size_t)b * anc_stride + w) + 1];
      else vis = ((w < 64 ? (a0 >> w) : (a1 >> (w - 64))) & 1ull) != 0ull;
    }
    if (__builtin_amdgcn_ballot_w64(vis) == 0ull) continue;   // uniform: nothing of a hidden tile is loaded
    // (slots of the tile behind the cache's last page are read from the last page and never used)
    const size_t kr = kv_k_at(kv, b, min(s, kv.max_seq - 1), g);
    float4 kx[D / 4];
#pragma unroll
    for (int c = 0; c < D / 4; ++c)   // (kv_k_col(4 c), at compile time)
      kx[c] = ldkv4(kc, kr + (c >> 3) * 512 + ((c >> 1) & 3) * 128 + (c & 1) * 4, kv.plane);
    float4 vx[16];
    auto load_v = [&](int u) __attribute__((always_inline)) {   // channel lane + 64 u of the tile's two pages
#pragma unroll
      for (int pg = 0; pg < 2; ++pg) {
        const size_t at = kv_v_at(kv, b, g, lane + 64 * u, min(t * 64 + pg * KV_PAGE, kv.max_seq - KV_PAGE));
#pragma unroll
        for (int c = 0; c < 8; ++c) vx[pg * 8 + c] = ldkv4(vc, at + (c >> 1) * 128 + (c & 1) * 4, kv.plane);
      }
    };
    load_v(0);
    float acc = 0.f;
#pragma unroll
    for (int c = 0; c < D / 4; ++c) {
      const float4 qv = *(const float4*)(qs + c * 4);
      acc += qv.x * kx[c].x; acc += qv.y * kx[c].y; acc += qv.z * kx[c].z; acc += qv.w * kx[c].w;
    }
    const float sc = vis ? acc : -INFINITY;
    const float mnew = fmaxf(mrun, wave_max(sc));
    if (mnew == -INFINITY) continue;  // uniform across the wave (every visible score is)
    const float p = vis ? expf(sc - mnew) : 0.f;
    const float corr = (mrun == -INFINITY) ? 0.f : expf(mrun - mnew);
    lrun = lrun * corr + wave_sum(p);
#pragma unroll
    for (int u = 0; u < D / 64; ++u) o[u] *= corr;
    mrun = mnew;
    __syncthreads();
    ps[lane] = p;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < D / 64; ++u) {
      if (u > 0) load_v(u);
#pragma unroll
      for (int c = 0; c < 16; ++c) {   // (a hidden key's value, or an unwritten slot's, has no part in the sum whatever it holds)
        const float4 pj = *(const float4*)(ps + c * 4);
        o[u] += pj.x != 0.f ? pj.x * vx[c].x : 0.f;
        o[u] += pj.y != 0.f ? pj.y * vx[c].y : 0.f;
        o[u] += pj.z != 0.f ? pj.z * vx[c].z : 0.f;
        o[u] += pj.w != 0.f ? pj.w * vx[c].w : 0.f;
      }
    }
  }
  const float inv = 1.0f / lrun;
#pragma unroll
  for (int u = 0; u < D / 64; ++u) {
    const int c = h * D + 64 * u + lane;
    const float v = o[u] * inv;
    bf16_t* dst = planes.p + frag_at(planes, (int)row, c);
    const bf16_t hb = f32_to_bf16(v);
    dst[0] = hb;
    dst[512] = f32_to_bf16(v - bf16_to_f32(hb));
  }
}

// The same over fp32 caches, a workgroup of one to four wavefronts that share a row's key tiles.  What bounds it: memory round trips,
// and the load path of a compute unit, which takes a clock or more per line that an instruction touches.  So a page of K, [32][D],
// and of V^T, [D][32], is read as it lies, a KB per instruction: D / 4 lanes have a key's row and add their products up between them, 8
// lanes have a channel's 32 positions and add theirs up once, at the end.  (With a lane per key, and per channel, 64 lines per
// instruction and one wavefront, us per launch, 4 heads of 64: 16 nodes at 64 keys 7.3 -> 5.6, by events 64 nodes at 300 15.8 -> 9.5, 16 at
// 900 31 -> 12.5; 8 heads of 128: 16 nodes at 300 keys 19.3 -> 12.6, at 2000 95 -> 32, 128 at 2000 235 -> 77.)
// Wavefronts of a row and head: as many as the chip has idle SIMDs for (one / two / four, 8 heads of 128 at 300 keys: 512 rows x heads
// 24.8, 16.9, 15.1, 1024 29.2, 22.2, 25.7; at 2000 keys 107, 65, 45 and 119, 77, 79).
constexpr int AF_WAVES = 4;   // most wavefronts of a row and head
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {   // v + the lane's that CTRL names, all of which have one
  return v + __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float sum_of_8(float v) { return dpp_add<0x141>(dpp_add<0x4e>(dpp_add<0xb1>(v))); }   // quad_perm, quad_perm, row_half_mirror
template <int D>
__global__ __launch_bounds__(64 * AF_WAVES) void attn_fp32_kernel(const float* __restrict__ q, int ldq, const float* __restrict__ kc,
                                                                  const float* __restrict__ vc, KVLayout kv, const int* __restrict__ base_len,
                                                                  const unsigned long long* __restrict__ anc, int n_q, float* __restrict__ out,
                                                                  int ldo, RowMap rm, int anc_stride, const int* __restrict__ iv) {
  constexpr int LPK = D / 4, KPI = 64 / LPK, NP = D / 8;   // lanes of a key, keys of a load, loads of a page
  __shared__ __attribute__((aligned(16))) float ps_all[AF_WAVES][64];
  __shared__ float all_m[AF_WAVES], all_l[AF_WAVES], all_o[AF_WAVES][D];
  const int h = blockIdx.x, i = blockIdx.y, b = blockIdx.z, lane = threadIdx.x & 63, waves = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float* const ps = ps_all[wave];
  const size_t row = (size_t)b * rm.R + i;
  const bool chain = anc == nullptr && iv == nullptr, bits = anc != nullptr && iv == nullptr;
  const int nv = rows_valid(rm, b), L = base_len[b];
  const unsigned long long a0 = bits ? anc[2 * ((size_t)b * anc_stride + i)] : 0ull;
  const unsigned long long a1 = bits ? anc[2 * ((size_t)b * anc_stride + i) + 1] : 0ull;
  const int my_enter = iv ? iv[2 * ((size_t)b * anc_stride + i)] : 0;
  const int x = lane % LPK, key = KPI * x + lane / LPK;   // the lane's four channels of q and k; its key of a tile for the soft-max
  float4 qv = *(const float4*)(q + row * ldq + h * D + 4 * x);
  if (i >= nv || L + nv > kv.max_seq) return;   // (whole workgroup)
  const float scale = 1.0f / sqrtf((float)D);
  qv.x *= scale; qv.y *= scale; qv.z *= scale; qv.w *= scale;
  const int g = h / (n_q / kv.n_kv);
  float mrun = -INFINITY, lrun = 0.f, o[NP];   // o: channel 8 c + lane / 8, the lane's positions only
#pragma unroll
  for (int c = 0; c < NP; ++c) o[c] = 0.f;
  const int total = L + (chain ? i + 1 : rm.n);   // (a chain's row sees nothing behind itself)
  const int ntiles = (total + 63) / 64;
  for (int t = wave; t < ntiles; t += waves) {
    const int s = t * 64 + key;
    bool vis = s < L;
    if (!vis && s < total) {
      const int w = s - L;
      if (chain) vis = true;
      else if (iv) vis = iv[2 * ((size_t)b * anc_stride + w)] <= my_enter && my_enter <= iv[2 * ((size_t)b * anc_stride + w) + 1];
      else vis = ((w < 64 ? (a0 >> w) : (a1 >> (w - 64))) & 1ull) != 0ull;
    }
    if (__builtin_amdgcn_ballot_w64(vis) == 0ull) continue;   // uniform: nothing of a hidden tile is loaded
    // (a page behind the cache's last one is read from there and never used)
    const size_t at[2] = {kv_block(kv, b, t * 64, g) + lane * 4, kv_block(kv, b, min(t * 64 + KV_PAGE, kv.max_seq - 1), g) + lane * 4};
    float4 kx[2][NP], vx[2][NP];
#pragma unroll
    for (int pg = 0; pg < 2; ++pg)
#pragma unroll
      for (int c = 0; c < NP; ++c) kx[pg][c] = *(const float4*)(kc + at[pg] + c * 256);
    auto load_v = [&](int pg) __attribute__((always_inline)) {
#pragma unroll
      for (int c = 0; c < NP; ++c) vx[pg][c] = *(const float4*)(vc + at[pg] + c * 256);
    };
    load_v(0);
    if (D == 64) load_v(1);
    float sc = -INFINITY;
#pragma unroll
    for (int pg = 0; pg < 2; ++pg)
#pragma unroll
      for (int c = 0; c < NP; ++c) {   // keys KPI (NP pg + c) ..: every lane of a key ends up with its score
        const float4 k4 = kx[pg][c];
        float v = dpp_add<0x140>(sum_of_8(qv.x * k4.x + qv.y * k4.y + qv.z * k4.z + qv.w * k4.w));   // row_mirror
        if (D == 128) v += __shfl_xor(v, 16, 64);
        sc = x == NP * pg + c ? v : sc;
      }
    if (D != 64) load_v(1);
    sc = vis ? sc : -INFINITY;
    const float mnew = fmaxf(mrun, wave_max(sc));
    if (mnew == -INFINITY) {   // uniform across the wave: every visible score is, or no number, which fmaxf leaves out
      lrun = vis && sc != sc ? sc : lrun;
      continue;
    }
    const float p = vis ? expf(sc - mnew) : 0.f;
    const float corr = (mrun == -INFINITY) ? 0.f : expf(mrun - mnew);
    mrun = mnew;
    // (the wavefront's own LDS words, which it accesses in order; only the compiler has to keep to it)
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
    ps[key] = p;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
    lrun = lrun * corr + p;   // (the lane's share)
#pragma unroll
    for (int c = 0; c < NP; ++c) o[c] *= corr;
#pragma unroll
    for (int pg = 0; pg < 2; ++pg) {
      const float4 pj = *(const float4*)(ps + pg * KV_PAGE + (lane & 7) * 4);
#pragma unroll
      for (int c = 0; c < NP; ++c) {   // (a hidden key's value, or an unwritten slot's, has no part in the sum whatever it holds)
        const float4 v4 = vx[pg][c];
        o[c] += pj.x != 0.f ? pj.x * v4.x : 0.f;
        o[c] += pj.y != 0.f ? pj.y * v4.y : 0.f;
        o[c] += pj.z != 0.f ? pj.z * v4.z : 0.f;
        o[c] += pj.w != 0.f ? pj.w * v4.w : 0.f;
      }
    }
  }
  // the wavefronts' results relative to the largest of their references, in their order
  lrun = wave_sum(lrun);
#pragma unroll
  for (int c = 0; c < NP; ++c) {
    o[c] = sum_of_8(o[c]);
    if ((lane & 7) == 0) all_o[wave][8 * c + lane / 8] = o[c];
  }
  if (lane == 0) { all_m[wave] = mrun; all_l[wave] = lrun; }
  __syncthreads();
  float m = -INFINITY, l = 0.f;
  for (int w = 0; w < waves; ++w) m = fmaxf(m, all_m[w]);
  for (int c = threadIdx.x; c < D; c += blockDim.x) {
    float v = 0.f;
    l = 0.f;
    for (int w = 0; w < waves; ++w) {
      if (all_m[w] == -INFINITY && all_l[w] == 0.f) continue;   // (saw no key; its sum is no number if it saw one whose score is none)
      const float f = expf(all_m[w] - m);
      l += f * all_l[w];
      v += f * all_o[w][c];
    }
    out[row * ldo + h * D + c] = v * (1.0f / l);
  }
}

void launch_attn_generic(const float* q, int ldq, const void* k_cache, const void* v_cache, int kvdtype, KVLayout kv,
                         const int* base_len, const unsigned long long* anc, int n_q, float* out, int ldo,
                         FragPlanes planes, RowMap rm, hipStream_t st, int anc_stride, const int* iv) {
  const dim3 grid(n_q, rm.n, rm.B);
  auto go = [&](auto dc) {   // head_dim is 64 or 128
    constexpr int D = decltype(dc)::value;
    if (kvdtype == 0) {
      const size_t wgs = (size_t)n_q * rm.n * rm.B;
      const int waves = tune_int("CLOVER_AF_WAVES", wgs <= 512 ? 4 : wgs <= 1024 ? 2 : 1);
      attn_fp32_kernel<D><<<grid, 64 * waves, 0, st>>>(q, ldq, (const float*)k_cache, (const float*)v_cache, kv, base_len, anc, n_q, out, ldo,
                                                       rm, anc_stride, iv);
    } else {
      attn_generic_kernel<D><<<grid, 64, 0, st>>>(q, ldq, (const bf16_t*)k_cache, (const bf16_t*)v_cache, kv, base_len, anc, n_q, planes, rm,
                                                  anc_stride, iv);
    }
  };
  if (kv.d == 64) go(std::integral_constant<int, 64>{});
  else go(std::integral_constant<int, 128>{});
}

// ------------------------------------------------------------------------------------------
// generic GEMM: Y[M,N] (+)= X[M,K] W[N,K]^T (+ bias), 64x64x16 LDS tiles, 4x4 per thread
// ------------------------------------------------------------------------------------------
template <typename WT>
__global__ __launch_bounds__(256) void gemm_generic_kernel(const float* __restrict__ X, int ldx,
                                                           const WT* __restrict__ W, const WT* __restrict__ bias,
                                                           float* __restrict__ Y, int ldy, int M, int N, int K,
                                                           int mode) {
  __shared__ float Xs[16][68];
  __shared__ float Ws[16][68];
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int bm = blockIdx.y * 64, bn = blockIdx.x * 64;
  float acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;
  for (int k0 = 0; k0 < K; k0 += 16) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int idx = tid + j * 256, r = idx >> 4, kk = idx & 15;
      const bool kin = (k0 + kk) < K;
      Xs[kk][r] = (kin && bm + r < M) ? X[(size_t)(bm + r) * ldx + k0 + kk] : 0.f;
      Ws[kk][r] = (kin && bn + r < N) ? ldf(W, (size_t)(bn + r) * K + k0 + kk) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      float a[4], w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = Xs[kk][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) w[j] = Ws[kk][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] += a[i] * w[j];
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = bm + ty * 4 + i;
    if (m >= M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = bn + tx * 4 + j;
      if (n >= N) continue;
      float v = acc[i][j];
      if (bias) v += ldf(bias, n);
      float* y = Y + (size_t)m * ldy + n;
      *y = (mode == 1) ? (*y + v) : v;
    }
  }
}

// The same product for launches that give the tiles above no chip to fill: one wavefront per 16 rows x 4 columns, its
// lanes split K (four adjacent columns each), the 64 sums are exchanged so that every lane ends with one output.  What
// bounds a 16 x 256 x 256 product in 64 x 64 tiles is a chain of 16 K steps with two barriers and a memory round trip
// each on 4 workgroups, 22 us; here it is one round trip on 64 wavefronts, 4 us.  Beyond that its loads bound it, 20
// loads of 16 bytes per 256 multiply-adds of a lane, out of the L2: 64 x 4096 x 14336 198 us (the tiles 1960).
constexpr int GS_ROWS = 16, GS_COLS = 4, GS_WAVES = 4;
__device__ __forceinline__ float4 ldw4(const float* w) { return *(const float4*)w; }
__device__ __forceinline__ float4 ldw4(const bf16_t* w) {
  const uint2 u = *(const uint2*)w;
  return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u), __uint_as_float(u.y << 16),
                     __uint_as_float(u.y & 0xFFFF0000u));
}
// Sums over the lanes of a wavefront without the LDS: 2 O values per lane become one per lane, each step halving the values
// and adding the two lanes that differ in bit O (for O = 4: and in the bits below, which are summed over anyway).
template <int O>
__device__ __forceinline__ float add_halves(float a, float b) {   // lanes without bit O: the pair's sum of a, with it: of b
  const unsigned ua = __float_as_uint(a), ub = __float_as_uint(b);
  if constexpr (O == 32) { const auto s = __builtin_amdgcn_permlane32_swap(ua, ub, false, false); return __uint_as_float(s[0]) + __uint_as_float(s[1]); }
  else { const auto s = __builtin_amdgcn_permlane16_swap(ua, ub, false, false); return __uint_as_float(s[0]) + __uint_as_float(s[1]); }
}
template <int O>
__device__ __forceinline__ float add_pair(float v) {   // the partner: O 8 row_ror:8, 4 row_half_mirror, 2 and 1 quad_perm
  constexpr int ctrl = O == 8 ? 0x128 : O == 4 ? 0x141 : O == 2 ? 0x4E : 0xB1;
  return v + __uint_as_float(__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), ctrl, 0xF, 0xF, true));
}
template <int O>
__device__ __forceinline__ void exchange_sums(float* v, int lane) {
#pragma unroll
  for (int i = 0; i < O; ++i) {
    if constexpr (O >= 16) {
      v[i] = add_halves<O>(v[i], v[i + O]);
    } else {
      const float a = add_pair<O>(v[i]), b = add_pair<O>(v[i + O]);
      v[i] = (lane & O) ? b : a;
    }
  }
  if constexpr (O > 1) exchange_sums<O / 2>(v, lane);
}
// One launch takes up to three products over the same rows and K (blocks of the second behind those of the first), sums the
// squares of its rows on the way where a product's input is to be normalised (RMSNorm's factor belongs to the row and is
// applied to the finished sums, its gain to the weights), and for SwiGLU computes two gate and the two up columns that belong
// to them in one wavefront: a fp32 step of 16 rows is a chain of launches of 3 to 4 us each, whatever they do (87 -> 52 of
// them, 351 -> 188 us of kernels, with the attention above).
struct SmallArgs {
  SmallGemm g[3];
  int first[3];       // first column block of each product
  int M, K, mode, swiglu;
  float eps;
};
template <typename WT, bool NORM, bool SWIGLU>
__global__ __launch_bounds__(64 * GS_WAVES) void gemm_small_kernel(SmallArgs a) {
  __shared__ float part[2][GS_WAVES][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6, cb = blockIdx.x, m0 = blockIdx.y * GS_ROWS, M = a.M, K = a.K;
  const int which = SWIGLU ? 0 : cb >= a.first[2] ? 2 : cb >= a.first[1] ? 1 : 0;
  const SmallGemm g = a.g[which];
  const float* const X = g.X;
  const WT* const W = (const WT*)g.W;
  const int N = g.N, n0 = (cb - (SWIGLU ? 0 : a.first[which])) * (SWIGLU ? 2 : GS_COLS);
  const WT* wrow[GS_COLS];
#pragma unroll
  for (int c = 0; c < GS_COLS; ++c)
    wrow[c] = SWIGLU ? (c < 2 ? W : (const WT*)a.g[1].W) + (size_t)min(n0 + (c & 1), N - 1) * K : W + (size_t)min(n0 + c, N - 1) * K;
  float acc[64], ss[GS_ROWS];   // [column][row], sums of squares
#pragma unroll
  for (int i = 0; i < 64; ++i) acc[i] = 0.f;
#pragma unroll
  for (int r = 0; r < GS_ROWS; ++r) ss[r] = 0.f;
  for (int k0 = wave * 256; k0 < K; k0 += waves * 256) {
    const int k = k0 + lane * 4, kc = min(k, K - 4);   // (K % 4 == 0; lanes past K multiply zeros)
    const bool in = k < K;
    float4 w[GS_COLS], x[GS_ROWS], gn;
#pragma unroll
    for (int c = 0; c < GS_COLS; ++c) w[c] = ldw4(wrow[c] + kc);
    if (NORM && g.gain) gn = ldw4((const WT*)g.gain + kc);
#pragma unroll
    for (int r = 0; r < GS_ROWS; ++r) x[r] = *(const float4*)(X + (size_t)min(m0 + r, M - 1) * g.ldx + kc);
    if (!in) {
#pragma unroll
      for (int c = 0; c < GS_COLS; ++c) w[c] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int r = 0; r < GS_ROWS; ++r) x[r] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if (NORM && g.gain) {   // uniform
#pragma unroll
      for (int c = 0; c < GS_COLS; ++c) { w[c].x *= gn.x; w[c].y *= gn.y; w[c].z *= gn.z; w[c].w *= gn.w; }
#pragma unroll
      for (int r = 0; r < GS_ROWS; ++r) ss[r] += x[r].x * x[r].x + x[r].y * x[r].y + x[r].z * x[r].z + x[r].w * x[r].w;
    }
#pragma unroll
    for (int c = 0; c < GS_COLS; ++c)
#pragma unroll
      for (int r = 0; r < GS_ROWS; ++r) {
        float v = acc[c * GS_ROWS + r];
        v += x[r].x * w[c].x; v += x[r].y * w[c].y; v += x[r].z * w[c].z; v += x[r].w * w[c].w;
        acc[c * GS_ROWS + r] = v;
      }
  }
  exchange_sums<32>(acc, lane);   // lane's sum: column lane / 16, row lane % 16
  const int m = m0 + (lane & 15), n = n0 + (SWIGLU ? (lane >> 4) & 1 : lane >> 4);
  float v = acc[0];
  if (NORM && g.gain) {   // the same for the 16 sums of squares: lane's row is lane % 16
    exchange_sums<8>(ss, lane);
    ss[0] = add_halves<16>(ss[0], ss[0]);
    ss[0] = add_halves<32>(ss[0], ss[0]);
  }
  if (waves > 1) {   // uniform: the wavefronts' sums, in their order
    part[0][wave][lane] = v;
    part[1][wave][lane] = ss[0];
    __syncthreads();
    if (wave > 0) return;
    for (int w = 1; w < waves; ++w) { v += part[0][w][lane]; ss[0] += part[1][w][lane]; }
  }
  if (NORM && g.gain) {
    v *= 1.0f / sqrtf(ss[0] / (float)K + a.eps);
  }
  if (SWIGLU) {   // lanes 0 .. 31 hold the gate, 32 .. 63 the up factor of the same output
    const float u = __uint_as_float(__builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false)[1]);
    v = v / (1.0f + expf(-v)) * u;
    if (lane >= 32) return;
  }
  if (m >= M || n >= N) return;
  if (g.bias) v += ldf((const WT*)g.bias, n);
  float* y = g.Y + (size_t)m * g.ldy + n;
  *y = a.mode == 1 ? *y + v : v;
}

// Up to three 64 x 64 tiles to a compute unit (half of that at K of 256, where the tile kernel's K chain is short): the tile
// kernel takes its K chain's time whether a compute unit has one tile or three.  us, this kernel and the tiles: 1 x 14336 x 4096
// 50 / 397, 256 x 4096 x 4096 (256 tiles) 201 / 483, 512 x 4096 x 1024 (512) 94 / 110, 1000 x 2816 x 1024 (704) 131 / 146,
// 1000 x 4096 x 1024 (1024) 180 / 169; K of 256: 512 x 2816 (352) 27.5 / 28.9, 512 x 4096 (512) 35 / 29.
// (16-byte loads: rows of X and W must start on 16 bytes, 8 for bf16 weights.)
static bool gemm_small_ok(const SmallGemm& g, int wdtype, int M, int K) {
  const size_t walign = wdtype == 0 ? 15 : 7;
  return (size_t)((g.N + 63) / 64) * ((M + 63) / 64) < (K > 256 ? 768 : 384) && K % 4 == 0 && g.ldx % 4 == 0 &&
         ((uintptr_t)g.X & 15) == 0 && ((uintptr_t)g.W & walign) == 0 && ((uintptr_t)g.gain & walign) == 0;
}
// Wavefronts that share a block's K.  Few blocks: a round trip per 1024 columns of K instead of one per 256 (64 x 1024 x 4096:
// one 20.7 us, two 18.5, four 19.9; 16 x 1024 x 4096: 18.2, 11.9, 9.1).  Many: the exchange of the 64 sums, which every wavefront
// does for itself, is paid for in throughput (128 x 1024 x 1024: 11.8, 13.0, 12.9; 256 x 4096 x 1024: 48, 53, 76).
static int small_waves(long blocks, int K) { return std::min(blocks <= 512 ? 4 : blocks <= 1024 ? 2 : 1, (K + 255) / 256); }
static int small_blocks(const SmallGemm* g, int n, bool swiglu) {
  if (swiglu) return (g[0].N + 1) / 2;
  int blocks = 0;
  for (int i = 0; i < n; ++i) blocks += (g[i].N + GS_COLS - 1) / GS_COLS;
  return blocks;
}
template <typename WT>
static void launch_small_one(const SmallArgs& a, bool norm, dim3 grid, hipStream_t st) {
  const int nt = 64 * small_waves((long)grid.x * grid.y, a.K);
  if (a.swiglu && norm) gemm_small_kernel<WT, true, true><<<grid, nt, 0, st>>>(a);
  else if (a.swiglu) gemm_small_kernel<WT, false, true><<<grid, nt, 0, st>>>(a);
  else if (norm) gemm_small_kernel<WT, true, false><<<grid, nt, 0, st>>>(a);
  else gemm_small_kernel<WT, false, false><<<grid, nt, 0, st>>>(a);
}
// Is the joint launch faster than what it replaces?  It saves launches and their round trips, and pays with a fifth of its
// vector work for the squares, which every block sums for itself, and for SwiGLU with a second matrix that streams through the
// L2 for every row block.  In units of blocks times columns of K, the crossings lie at (us, joint and separate):
//   norm in front of one product    6 M   1024 wide: 128 x 2816 24.9 / 25.1, 128 x 4096 32.1 / 30.0; 4096: 48 x 2816 45.2 / 39.9
//   norm and three products        26 M   1024: 512 rows 85 / 96, 1024 rows 165 / 171; 4096, GQA: 64 rows 85.5 / 97, 128 rows 160 / 153
//   norm, two products and SwiGLU  16 M   1024: 64 x 4096 33.8 / 38.7, 128 x 4096 61.7 / 59.6; 4096: 16 x 4096 33 / 50, 48 x 4096 98 / 93
bool gemm_small_joins(const SmallGemm* g, int n, bool swiglu, int wdtype, int M, int K) {
  for (int i = 0; i < n; ++i)
    if (!gemm_small_ok(g[i], wdtype, M, K)) return false;
  const double work = (double)small_blocks(g, n, swiglu) * ((M + GS_ROWS - 1) / GS_ROWS) * K;
  return work <= (swiglu ? 16e6 : n == 1 ? 6e6 : 26e6);
}
void launch_gemm_small(const SmallGemm* g, int n, bool swiglu, int wdtype, int M, int K, int mode, float eps, hipStream_t st) {
  SmallArgs a{};
  bool norm = false;
  for (int i = 0, blocks = 0; i < 3; ++i) {
    a.first[i] = i < n ? blocks : 1 << 30;
    if (i >= n) continue;
    a.g[i] = g[i];
    norm = norm || g[i].gain;
    blocks += small_blocks(&g[i], 1, false);
  }
  const int blocks = small_blocks(g, n, swiglu);
  if (M <= 0 || blocks <= 0) return;
  a.M = M; a.K = K; a.mode = mode; a.swiglu = swiglu; a.eps = eps;
  const dim3 grid(blocks, (M + GS_ROWS - 1) / GS_ROWS);
  if (wdtype == 0) launch_small_one<float>(a, norm, grid, st);
  else launch_small_one<bf16_t>(a, norm, grid, st);
}

void launch_gemm_generic(const float* X, int ldx, const void* W, const void* bias, int wdtype, float* Y, int ldy,
                         int M, int N, int K, int mode, hipStream_t st) {
  if (M <= 0 || N <= 0) return;
  const SmallGemm g{X, ldx, W, bias, nullptr, Y, ldy, N};
  if (gemm_small_ok(g, wdtype, M, K)) return launch_gemm_small(&g, 1, false, wdtype, M, K, mode, 0.f, st);
  dim3 grid((N + 63) / 64, (M + 63) / 64);
  if (wdtype == 0)
    gemm_generic_kernel<float><<<grid, 256, 0, st>>>(X, ldx, (const float*)W, (const float*)bias, Y, ldy, M, N, K, mode);
  else
    gemm_generic_kernel<bf16_t><<<grid, 256, 0, st>>>(X, ldx, (const bf16_t*)W, (const bf16_t*)bias, Y, ldy, M, N, K,
                                                      mode);
}

__global__ void swiglu_kernel(const float* __restrict__ g, const float* __restrict__ u, float* __restrict__ h,
                              size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    const float a = g[i];
    h[i] = a / (1.0f + expf(-a)) * u[i];
  }
}
void launch_swiglu(const float* g, const float* u, float* h, size_t n, hipStream_t st) {
  if (n == 0) return;
  swiglu_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(g, u, h, n);
}

// ------------------------------------------------------------------------------------------
// Attention-Decoder gate: per head cos(q_h, k_h) scales v_h, residual add of x
// ------------------------------------------------------------------------------------------
__global__ void ad_gate_kernel(const float* __restrict__ x, int ldx, const float* __restrict__ q,
                               const float* __restrict__ k, const float* __restrict__ v, int H, int heads,
                               float* __restrict__ out, AdNodes to) {
  const size_t row = blockIdx.x;
  size_t orow = row;
  if (to.nodes) {
    const int b = (int)row / to.n_lvl, r = (int)row - b * to.n_lvl;
    orow = (size_t)b * to.R + to.nodes[(size_t)b * to.stride + r];
  }
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, hd = H / heads;
  for (int h = wave; h < heads; h += 4) {
    const size_t o = row * H + (size_t)h * hd;
    float qq = 0.f, kk = 0.f, qk = 0.f;
    for (int c = lane; c < hd; c += 64) {
      const float a = q[o + c], bb = k[o + c];
      qq += a * a; kk += bb * bb; qk += a * bb;
    }
    qq = wave_sum(qq); kk = wave_sum(kk); qk = wave_sum(qk);
    const float att = qk / (fmaxf(sqrtf(qq), 1e-8f) * fmaxf(sqrtf(kk), 1e-8f));
    for (int c = lane; c < hd; c += 64) {
      const float r = x[row * ldx + h * hd + c] + att * v[o + c];
      out[orow * H + h * hd + c] = r;
      if (to.cat) to.cat[row * 2 * H + h * hd + c] = r;
    }
  }
}
void launch_ad_gate(const float* x, int ldx, const float* q, const float* k, const float* v, int H, int heads,
                    float* out, int rows, hipStream_t st, AdNodes to) {
  if (rows <= 0) return;
  ad_gate_kernel<<<rows, 256, 0, st>>>(x, ldx, q, k, v, H, heads, out, to);
}

// ------------------------------------------------------------------------------------------
// top-k by (value desc, id asc).  Keys are 64-bit: order-preserving image of the float in the high
// word, ~id in the low word, so an unsigned max picks the larger value and, among equals, the
// smaller id.  Stage 1: one block per 2048-wide chunk; stage 2: one block per row merges.
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ unsigned long long topk_key(float v, int id) {
  v = v + 0.0f;  // -0 -> +0 so that equal values compare equal
  unsigned u = __float_as_uint(v);
  u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return ((unsigned long long)u << 32) | (unsigned long long)(0xFFFFFFFFu - (unsigned)id);
}
// Thread i's child of the node that row `row` of a depth expands: where its token goes and which of the row's ranked ids it is.
// (Looked up in front of the ranking: a chain of loads that costs nothing there.)
struct ChildSlot {
  int* at = nullptr;
  int rank = 0;
  __device__ __forceinline__ ChildSlot(const TopkChildren& to, int row) {
    if (!to.tokens) return;
    const int b = row / to.n_lvl, u = to.nodes[row - b * to.n_lvl];
    if ((int)threadIdx.x >= to.n_child[u] || to.m[b] < 1) return;
    const int c = to.first_child[u] + (int)threadIdx.x;
    at = to.tokens + (size_t)b * to.R + c;
    rank = to.rank[c];
  }
};

constexpr int TOPK_CHUNK = 2048;
constexpr int TOPK_EPT = TOPK_CHUNK / 256;
int topk_chunks(int V) { return (V + TOPK_CHUNK - 1) / TOPK_CHUNK; }

__global__ __launch_bounds__(256) void topk_stage1_kernel(const float* __restrict__ z, int ldz, int V, int k,
                                                          unsigned long long* __restrict__ cand, int* __restrict__ out_ids,
                                                          TopkChildren to) {
  __shared__ unsigned long long red[2][4];
  __shared__ int ids[16];
  const int chunk = blockIdx.x, row = blockIdx.y, chunks = gridDim.x;
  const ChildSlot child(to, row);
  unsigned long long key[TOPK_EPT];
#pragma unroll
  for (int e = 0; e < TOPK_EPT; ++e) {
    const int id = chunk * TOPK_CHUNK + e * 256 + threadIdx.x;
    const float v = id < V ? z[(size_t)row * ldz + id] : 0.f;
    key[e] = id < V ? topk_key(v, id) : 0ull;
  }
  for (int r = 0; r < k; ++r) {
    unsigned long long best = 0ull;
#pragma unroll
    for (int e = 0; e < TOPK_EPT; ++e) best = key[e] > best ? key[e] : best;
    best = block_max_key(best, red, r);
#pragma unroll
    for (int e = 0; e < TOPK_EPT; ++e)
      if (key[e] == best) key[e] = 0ull;
    if (threadIdx.x == 0) {
      if (out_ids) out_ids[row * 16 + r] = ids[r] = (int)(0xFFFFFFFFu - (unsigned)(best & 0xFFFFFFFFull));   // the only chunk
      else cand[((size_t)row * chunks + chunk) * 16 + r] = best;
    }
  }
  if (!to.tokens) return;   // (uniform)
  __syncthreads();
  if (child.at) *child.at = ids[child.rank];
}

// stage 1 for k = 1 (the target's argmax over every row): one wavefront per chunk, 16-byte loads, the 64-bit key only for
// the exchange between lanes.  Bound by reading the logits: 256 rows x 128256 are 131 MB, 49 us through the kernel above
// (16128 workgroups of 8 KB with two barriers each).
__global__ __launch_bounds__(256) void argmax_stage1_kernel(const float* __restrict__ z, int ldz, int V, int chunks,
                                                            unsigned long long* __restrict__ cand) {
  const int lane = threadIdx.x & 63, chunk = blockIdx.x * 4 + (threadIdx.x >> 6), row = blockIdx.y;
  if (chunk >= chunks) return;
  const float* zr = z + (size_t)row * ldz;
  float4 v[TOPK_CHUNK / 256];
#pragma unroll
  for (int e = 0; e < TOPK_CHUNK / 256; ++e)   // (V % 4 == 0: a piece is inside or outside as a whole)
    v[e] = *(const float4*)(zr + min(chunk * TOPK_CHUNK + (e * 64 + lane) * 4, V - 4));
  unsigned best = 0u;
  int id = -1;   // none yet: a NaN of all ones has the key 0 and is a value all the same
#pragma unroll
  for (int e = 0; e < TOPK_CHUNK / 256; ++e) {
    const int i0 = chunk * TOPK_CHUNK + (e * 64 + lane) * 4;
    const float f[4] = {v[e].x, v[e].y, v[e].z, v[e].w};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const unsigned u = (unsigned)(topk_key(f[r], 0) >> 32);
      if (i0 < V && (u > best || id < 0)) { best = u; id = i0 + r; }   // ids ascend: the smallest of equals stays
    }
  }
  unsigned long long key = id >= 0 ? ((unsigned long long)best << 32) | (unsigned long long)(0xFFFFFFFFu - (unsigned)id) : 0ull;
  key = wave_max_key(key);
  if (lane == 0) cand[((size_t)row * chunks + chunk) * 16] = key;
}

__global__ __launch_bounds__(256) void topk_stage2_kernel(const unsigned long long* __restrict__ cand, int chunks,
                                                          int k, int* __restrict__ out_ids, TopkChildren to) {
  __shared__ unsigned long long red[2][4];
  __shared__ int ids[16];
  const int row = blockIdx.x;
  const ChildSlot child(to, row);
  const int total = chunks * k;  // <= 63*16 for V <= 129024; loop handles more
  unsigned long long key[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int idx = e * 256 + threadIdx.x;
    key[e] = idx < total ? cand[((size_t)row * chunks + idx / k) * 16 + idx % k] : 0ull;
  }
  for (int r = 0; r < k; ++r) {
    unsigned long long best = 0ull;
#pragma unroll
    for (int e = 0; e < 8; ++e) best = key[e] > best ? key[e] : best;
    best = block_max_key(best, red, r);
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (key[e] == best) key[e] = 0ull;
    if (threadIdx.x == 0) out_ids[row * 16 + r] = ids[r] = (int)(0xFFFFFFFFu - (unsigned)(best & 0xFFFFFFFFull));
  }
  if (!to.tokens) return;   // (uniform)
  __syncthreads();
  if (child.at) *child.at = ids[child.rank];
}

void launch_topk(const float* z, int ldz, int V, int rows, int k, void* cand, int* out_ids, hipStream_t st, TopkChildren to) {
  if (rows <= 0) return;
  const int chunks = topk_chunks(V);  // chunks * k <= 2048 is checked at init (vocab <= 262144)
  if (chunks == 1) {   // (a vocabulary of up to 2048: nothing to merge)
    topk_stage1_kernel<<<dim3(1, rows), 256, 0, st>>>(z, ldz, V, k, (unsigned long long*)cand, out_ids, to);
    return;
  }
  if (k == 1 && V % 4 == 0 && ldz % 4 == 0 && ((uintptr_t)z & 15) == 0)
    argmax_stage1_kernel<<<dim3((chunks + 3) / 4, rows), 256, 0, st>>>(z, ldz, V, chunks, (unsigned long long*)cand);
  else
    topk_stage1_kernel<<<dim3(chunks, rows), 256, 0, st>>>(z, ldz, V, k, (unsigned long long*)cand, nullptr, TopkChildren{});
  topk_stage2_kernel<<<rows, 256, 0, st>>>((const unsigned long long*)cand, chunks, k, out_ids, to);
}

// ------------------------------------------------------------------------------------------
// draft-tree bookkeeping
// ------------------------------------------------------------------------------------------
template <typename WT>
__global__ void draft_gather_kernel(const float* __restrict__ state, const int* __restrict__ tokens,
                                    const int* __restrict__ lvl_nodes, const int* __restrict__ parent, int n_lvl,
                                    int R, int H, const WT* __restrict__ lm_head, int vocab, float* __restrict__ xs,
                                    float* __restrict__ e, float* __restrict__ cat, int nodes_stride, int parent_stride) {
  const int r = blockIdx.x, b = blockIdx.y;
  const int u = lvl_nodes[(size_t)b * nodes_stride + r], p = parent[(size_t)b * parent_stride + u];
  int t = tokens[(size_t)b * R + u];
  t = t < 0 ? 0 : (t >= vocab ? vocab - 1 : t);
  const size_t row = (size_t)b * n_lvl + r;
  for (int c = threadIdx.x; c < H; c += blockDim.x) {
    xs[row * H + c] = state[((size_t)b * R + p) * H + c];
    const float ev = ldf(lm_head, (size_t)t * H + c);
    e[row * H + c] = ev;
    cat[row * 2 * H + H + c] = ev;
  }
}
void launch_draft_gather(const float* state, const int* tokens, const int* lvl_nodes, const int* parent, int n_lvl,
                         int B, int R, int H, const void* lm_head, int wdtype, int vocab, float* xs, float* e,
                         float* cat, hipStream_t st, int nodes_stride, int parent_stride) {
  if (n_lvl <= 0) return;
  dim3 grid(n_lvl, B);
  if (wdtype == 0)
    draft_gather_kernel<float><<<grid, 256, 0, st>>>(state, tokens, lvl_nodes, parent, n_lvl, R, H,
                                                     (const float*)lm_head, vocab, xs, e, cat, nodes_stride, parent_stride);
  else
    draft_gather_kernel<bf16_t><<<grid, 256, 0, st>>>(state, tokens, lvl_nodes, parent, n_lvl, R, H,
                                                      (const bf16_t*)lm_head, vocab, xs, e, cat, nodes_stride, parent_stride);
}

__global__ void draft_root_kernel(const float* __restrict__ a, const int* __restrict__ next_tok,
                                  const int* __restrict__ m, int R, int H, float* __restrict__ root_x,
                                  float* __restrict__ state, int* __restrict__ tokens, int* __restrict__ aug_len, int Rs) {
  const int b = blockIdx.x;
  const int mb = min(m[b], R);
  for (int c = threadIdx.x; c < H; c += blockDim.x) {
    const float v = mb >= 1 ? a[((size_t)b * R + mb - 1) * H + c] : 0.f;
    root_x[(size_t)b * H + c] = v;
    state[((size_t)b * Rs) * H + c] = v;
  }
  if (threadIdx.x == 0) {
    if (mb >= 1) tokens[(size_t)b * Rs] = next_tok[(size_t)b * R + mb - 1];
    aug_len[b] += max(m[b], 0);
  }
}
void launch_draft_root(const float* a, const int* next_tok, const int* m, int B, int R, int H, float* root_x,
                       float* state, int* tokens, int* aug_len, hipStream_t st, int Rs) {
  draft_root_kernel<<<B, 256, 0, st>>>(a, next_tok, m, R, H, root_x, state, tokens, aug_len, Rs ? Rs : R);
}

__global__ void add_scalar_kernel(int* __restrict__ p, int v) { *p += v; }
void launch_add_scalar(int* p, int v, hipStream_t st) { add_scalar_kernel<<<1, 1, 0, st>>>(p, v); }

__global__ void fill_i32_kernel(int* p, int v, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}
void launch_fill_i32(int* p, int v, int n, hipStream_t st) {
  if (n > 0) fill_i32_kernel<<<(n + 255) / 256, 256, 0, st>>>(p, v, n);
}

// ------------------------------------------------------------------------------------------
// greedy acceptance walk (one thread per sequence; the tree has at most 128 nodes)
// ------------------------------------------------------------------------------------------
__global__ void accept_walk_kernel(const int* __restrict__ argmax, const int* __restrict__ tokens,
                                   const int* __restrict__ first_child, const int* __restrict__ n_child, int n_nodes,
                                   int B, int R, const int* __restrict__ n_forced,
                                   const int* __restrict__ forced_next, int* __restrict__ m,
                                   int* __restrict__ acc_idx, int* __restrict__ new_tokens,
                                   int* __restrict__ next_tok, int* __restrict__ seq_len, int child_stride) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  const size_t o = (size_t)b * R;
  first_child += (size_t)b * child_stride;
  n_child += (size_t)b * child_stride;
  int len, bonus;
  if (n_forced) {
    len = min(max(n_forced[b], 0), n_nodes);
    if (len == 0) { m[b] = 0; return; }
    for (int i = 0; i < len; ++i) acc_idx[o + i] = i;
    const int f = forced_next[b];
    bonus = f >= 0 ? f : argmax[(o + len - 1) * 16];
  } else {
    int u = 0;
    len = 1;
    acc_idx[o] = 0;
    for (;;) {
      const int t = argmax[(o + u) * 16];
      int found = -1;
      const int c0 = first_child[u], c1 = c0 + n_child[u];
      for (int c = c0; c < c1; ++c)
        if (tokens[o + c] == t) { found = c; break; }
      bonus = t;
      if (found < 0 || len >= R) break;
      u = found;
      acc_idx[o + len++] = u;
    }
  }
  for (int j = 1; j < len; ++j) {
    const int t = tokens[o + acc_idx[o + j]];
    new_tokens[o + j - 1] = t;
    next_tok[o + j - 1] = t;
  }
  new_tokens[o + len - 1] = bonus;
  next_tok[o + len - 1] = bonus;
  m[b] = len;
  seq_len[b] += len;   // (launch_accept_move subtracts it again)
}
void launch_accept_walk(const int* argmax, const int* tokens, const int* first_child, const int* n_child, int n_nodes,
                        int B, int R, const int* n_forced, const int* forced_next, int* m, int* acc_idx,
                        int* new_tokens, int* next_tok, int* seq_len, hipStream_t st, int child_stride) {
  accept_walk_kernel<<<(B + 63) / 64, 64, 0, st>>>(argmax, tokens, first_child, n_child, n_nodes, B, R, n_forced,
                                                   forced_next, m, acc_idx, new_tokens, next_tok, seq_len, child_stride);
}

// ------------------------------------------------------------------------------------------
// What an accept call moves once the walk has written m and acc_idx and added m to the lengths, in one launch: blocks y < n_layers
// compact the K/V rows of a layer, slot L+i <- slot L+acc_idx[i], ascending i (a thread owns one cache column for all rows,
// so the in-place moves of a column are ordered without any barrier); the others gather one accepted hidden row each.
// ------------------------------------------------------------------------------------------
template <typename KT>
__global__ void accept_move_kernel(KT* __restrict__ kc, KT* __restrict__ vc, KVLayout kv, int n_layers, size_t layer_elems,
                                   const int* __restrict__ len, const int* __restrict__ m, const int* __restrict__ acc_idx,
                                   int R, const float* __restrict__ hidden, int H, float* __restrict__ hid_acc) {
  const int b = blockIdx.z, mb = m[b];
  if ((int)blockIdx.y >= n_layers) {
    const int i = blockIdx.y - n_layers;
    if (i >= mb) return;
    const int a = acc_idx[(size_t)b * R + i];
    if (a < 0 || a >= R) return;
    for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < H; c += gridDim.x * blockDim.x)
      hid_acc[((size_t)b * R + i) * H + c] = hidden[((size_t)b * R + a) * H + c];
    return;
  }
  const int col = blockIdx.x * blockDim.x + threadIdx.x, layer = blockIdx.y;
  if (col >= kv.n_kv * kv.d || mb <= 0) return;
  const int L = len[b] - mb;
  if (L + mb > kv.max_seq) return;
  KT* kbase = kc + (size_t)layer * layer_elems;
  KT* vbase = vc + (size_t)layer * layer_elems;
  const int head = col / kv.d, dim = col % kv.d;
  for (int i = 0; i < mb; ++i) {
    const int a = acc_idx[(size_t)b * R + i];
    if (a == i || a < 0 || L + a >= kv.max_seq) continue;
    mvkv(kbase, kv_k_at(kv, b, L + i, head) + kv_k_col(kv, dim), kv_k_at(kv, b, L + a, head) + kv_k_col(kv, dim), kv.plane);
    mvkv(vbase, kv_v_at(kv, b, head, dim, L + i), kv_v_at(kv, b, head, dim, L + a), kv.plane);
  }
}
void launch_accept_move(void* k_cache, void* v_cache, int kvdtype, KVLayout kv, int n_layers, size_t layer_elems, const int* len,
                        const int* m, const int* acc_idx, int B, int R, int max_rows, const float* hidden, int H, float* hid_acc,
                        hipStream_t st) {
  const dim3 grid((kv.n_kv * kv.d + 255) / 256, n_layers + max_rows, B);
  if (kvdtype == 0)
    accept_move_kernel<float><<<grid, 256, 0, st>>>((float*)k_cache, (float*)v_cache, kv, n_layers, layer_elems, len, m, acc_idx, R, hidden, H, hid_acc);
  else
    accept_move_kernel<bf16_t><<<grid, 256, 0, st>>>((bf16_t*)k_cache, (bf16_t*)v_cache, kv, n_layers, layer_elems, len, m, acc_idx, R, hidden, H, hid_acc);
}

template <typename KT>
__global__ void read_kv_kernel(const KT* __restrict__ kc, const KT* __restrict__ vc, KVLayout kv, int b, int slot0,
                               int n_slots, float* __restrict__ k_out, float* __restrict__ v_out) {
  const int width = kv.n_kv * kv.d;
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)n_slots * width) return;
  const int s = (int)(idx / width), col = (int)(idx % width);
  k_out[idx] = ldkv(kc, kv_k_at(kv, b, slot0 + s, col / kv.d) + kv_k_col(kv, col % kv.d), kv.plane);
  v_out[idx] = ldkv(vc, kv_v_at(kv, b, col / kv.d, col % kv.d, slot0 + s), kv.plane);
}
void launch_read_kv(const void* k_cache, const void* v_cache, int kvdtype, KVLayout kv, int b, int slot0, int n_slots,
                    float* k_out, float* v_out, hipStream_t st) {
  const size_t n = (size_t)n_slots * kv.n_kv * kv.d;
  if (n == 0) return;
  const unsigned blocks = (unsigned)((n + 255) / 256);
  if (kvdtype == 0)
    read_kv_kernel<float><<<blocks, 256, 0, st>>>((const float*)k_cache, (const float*)v_cache, kv, b, slot0, n_slots,
                                                  k_out, v_out);
  else
    read_kv_kernel<bf16_t><<<blocks, 256, 0, st>>>((const bf16_t*)k_cache, (const bf16_t*)v_cache, kv, b, slot0,
                                                   n_slots, k_out, v_out);
}

template <typename KT>
__global__ void write_kv_kernel(KT* __restrict__ kc, KT* __restrict__ vc, KVLayout kv, int b, int slot0, int n_slots,
                                const float* __restrict__ k_in, const float* __restrict__ v_in) {
  const int width = kv.n_kv * kv.d;
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)n_slots * width) return;
  const int s = (int)(idx / width), col = (int)(idx % width);
  stkv(kc, kv_k_at(kv, b, slot0 + s, col / kv.d) + kv_k_col(kv, col % kv.d), kv.plane, k_in[idx]);
  stkv(vc, kv_v_at(kv, b, col / kv.d, col % kv.d, slot0 + s), kv.plane, v_in[idx]);
}
void launch_write_kv(void* k_cache, void* v_cache, int kvdtype, KVLayout kv, int b, int slot0, int n_slots,
                     const float* k_in, const float* v_in, hipStream_t st) {
  const size_t n = (size_t)n_slots * kv.n_kv * kv.d;
  if (n == 0) return;
  const unsigned blocks = (unsigned)((n + 255) / 256);
  if (kvdtype == 0)
    write_kv_kernel<float><<<blocks, 256, 0, st>>>((float*)k_cache, (float*)v_cache, kv, b, slot0, n_slots, k_in, v_in);
  else
    write_kv_kernel<bf16_t><<<blocks, 256, 0, st>>>((bf16_t*)k_cache, (bf16_t*)v_cache, kv, b, slot0, n_slots, k_in,
                                                    v_in);
}

// ------------------------------------------------------------------------------------------
// split-bf16 planes and partial-sum consumers
// ------------------------------------------------------------------------------------------
__global__ void split_planes_kernel(const float* __restrict__ x, int ldx, FragPlanes out, int K) {
  const int row = blockIdx.y;
  const int c = (blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (c >= K) return;
  const f32x4_any v = *(const f32x4_any*)(x + (size_t)row * ldx + c);
  frag_store4(out, row, c, v[0], v[1], v[2], v[3]);
}
void launch_split_planes(const float* x, int ldx, FragPlanes out, int rows, int K, hipStream_t st) {
  if (rows <= 0) return;
  split_planes_kernel<<<dim3((K / 4 + 255) / 256, rows), 256, 0, st>>>(x, ldx, out, K);
}

template <typename WT>
__global__ void reduce_kernel(const float* __restrict__ P, int splits, size_t sps, int ldp, const WT* __restrict__ bias,
                              float* __restrict__ Y, int ldy, int N, int mode) {
  const size_t row = blockIdx.y;
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= N) return;
  float v = 0.f;
  for (int s = 0; s < splits; ++s) v += P[s * sps + row * ldp + c];
  if (bias) v += ldf(bias, c);
  float* y = Y + row * ldy + c;
  *y = mode == 1 ? *y + v : v;
}
void launch_reduce(const float* P, int splits, size_t split_stride, int ldp, const void* bias, int wdtype, float* Y,
                   int ldy, int M, int N, int mode, hipStream_t st) {
  if (M <= 0) return;
  dim3 grid((N + 255) / 256, M);
  if (wdtype == 0)
    reduce_kernel<float><<<grid, 256, 0, st>>>(P, splits, split_stride, ldp, (const float*)bias, Y, ldy, N, mode);
  else
    reduce_kernel<bf16_t><<<grid, 256, 0, st>>>(P, splits, split_stride, ldp, (const bf16_t*)bias, Y, ldy, N, mode);
}

// total over the block of every thread's v; `red` holds a float per wavefront
__device__ __forceinline__ float block_sum_up_to_1024(float v, float* red) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < 16; ++w)
    if (w * 64 < (int)blockDim.x) tot += red[w];
  return tot;
}

// Start of a pass, one block per row (b, i): out = table[tok] where the row is valid, with a gain its RMSNorm as planes, and the
// row's rotary table at position base_len[b] + (depth ? depth[i] : i).  Three small launches' work; what bounds it is the chain
// token -> table row -> norm, with the angles' arithmetic beside it.
template <typename WT, int PC>
__global__ __launch_bounds__(1024) void pass_start_kernel(PassStart p) {
  __shared__ float red[16];
  const RowMap& rm = p.rm;
  const int b = blockIdx.y, i = blockIdx.x;
  const size_t row = (size_t)b * rm.R + i;
  const bool valid = i < rows_valid(rm, b);
  const int H = p.H, c0 = threadIdx.x * 4, step = blockDim.x * 4;
  float4 keep[PC], gn[PC];
  float ss = 0.f;
  if (valid) {
    int t = p.tok[row];
    t = t < 0 ? 0 : (t >= p.vocab ? p.vocab - 1 : t);
    const WT* src = (const WT*)p.table + (size_t)t * H;
    auto copy = [&](int c) -> float4 {
      const float4 v = ld4_any(src + c);
      *(f32x4_any*)(p.out + row * p.ldo + c) = (f32x4_any){v.x, v.y, v.z, v.w};
      ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
      return v;
    };
#pragma unroll
    for (int it = 0; it < PC; ++it) {
      const int c = c0 + it * step;
      if (c < H) {
        if (p.gain) gn[it] = ld4_any((const WT*)p.gain + c);
        keep[it] = copy(c);
      }
    }
    if (PC > 1)
      for (int c = c0 + PC * step; c < H; c += step) copy(c);
  }
  rope_row(p.rope, b, i, row);
  if (!p.gain || !valid) return;   // (uniform)
  const float tot = block_sum_up_to_1024(ss, red);
  const float scale = 1.0f / sqrtf(tot / (float)H + p.eps);
  auto emit = [&](int c, float4 v, float4 g4) {
    frag_store4(p.planes, (int)row, c, v.x * scale * g4.x, v.y * scale * g4.y, v.z * scale * g4.z, v.w * scale * g4.w);
  };
#pragma unroll
  for (int it = 0; it < PC; ++it) {
    const int c = c0 + it * step;
    if (c < H) emit(c, keep[it], gn[it]);
  }
  if (PC > 1)
    for (int c = c0 + PC * step; c < H; c += step) emit(c, ld4_any(p.out + row * p.ldo + c), ld4_any((const WT*)p.gain + c));   // written by this same thread above
}
void launch_pass_start(const PassStart& p, int wdtype, hipStream_t st) {
  const dim3 grid(p.rm.n, p.rm.B);
  const int threads = std::min(1024, (p.H / 4 + 63) / 64 * 64);
  if (wdtype == 0) {
    if (p.H <= 4096) pass_start_kernel<float, 1><<<grid, threads, 0, st>>>(p);
    else pass_start_kernel<float, 2><<<grid, threads, 0, st>>>(p);
  } else {
    if (p.H <= 4096) pass_start_kernel<bf16_t, 1><<<grid, threads, 0, st>>>(p);
    else pass_start_kernel<bf16_t, 2><<<grid, threads, 0, st>>>(p);
  }
}

// One block of up to 1024 threads per row: residual add of the partial tiles over NS ranges of K (all requested at once,
// summed in range order), then RMSNorm written as planes in fragment order.  A thread keeps PC float4 of the new row in
// registers across the block-wide sum of squares; rows wider than PC * 4096 re-read the rest.
template <int NS, int PC>
__global__ __launch_bounds__(1024) void reduce_add_norm_kernel(float* __restrict__ x, int ldx,
                                                               const float* __restrict__ P, size_t sps, int ldp,
                                                               const bf16_t* __restrict__ gain, float eps,
                                                               FragPlanes out, int H, const bf16_t* __restrict__ bias) {
  __shared__ float red[16];
  const size_t row = blockIdx.x;
  float* xr = x + row * ldx;
  const float* pr = P + row * ldp;
  const int c0 = threadIdx.x * 4, step = blockDim.x * 4;
  float4 keep[PC], gn[PC];
  Partials4<NS> q[PC];
#pragma unroll
  for (int it = 0; it < PC; ++it) {  // (static indices: the kept pieces live in registers)
    const int c = c0 + it * step;
    if (c < H) {
      q[it].request(pr + c, sps);
      keep[it] = bias ? ld4_any(bias + c) : *(const float4*)(xr + c);
      if (gain) gn[it] = ld4_any(gain + c);
    }
  }
  float ss = 0.f;
  auto put = [&](int c, float4 v) {
    if (NS > 0 || bias) *(float4*)(xr + c) = v;
    ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
  };
#pragma unroll
  for (int it = 0; it < PC; ++it) {
    const int c = c0 + it * step;
    if (c < H) { keep[it] = q[it].add_to(keep[it]); put(c, keep[it]); }
  }
  if (PC > 1)
    for (int c = c0 + PC * step; c < H; c += step) {
      Partials4<NS> r;
      r.request(pr + c, sps);
      put(c, r.add_to(bias ? ld4_any(bias + c) : *(const float4*)(xr + c)));
    }
  if (!gain) return;
  const float tot = block_sum_up_to_1024(ss, red);
  const float scale = 1.0f / sqrtf(tot / (float)H + eps);
  auto emit = [&](int c, float4 v, float4 g4) {
    frag_store4(out, (int)row, c, v.x * scale * g4.x, v.y * scale * g4.y, v.z * scale * g4.z, v.w * scale * g4.w);
  };
#pragma unroll
  for (int it = 0; it < PC; ++it) {
    const int c = c0 + it * step;
    if (c < H) emit(c, keep[it], gn[it]);
  }
  if (PC > 1)
    for (int c = c0 + PC * step; c < H; c += step) emit(c, *(const float4*)(xr + c), ld4_any(gain + c));  // written by this same thread above
}
// splits <= TILE_MAX_K_PARTS; gain and bias are bf16
void launch_reduce_add_norm(float* x, int ldx, const float* P, int splits, size_t split_stride, int ldp,
                            const void* gain, float eps, FragPlanes out, int rows, int H,
                            hipStream_t st, const void* bias) {
  if (rows <= 0) return;
  with_count<0, TILE_MAX_K_PARTS>(splits, [&](auto nc) {
    constexpr int NS = decltype(nc)::value;
    const int threads = std::min(1024, (H / 4 + 63) / 64 * 64);
    if (H <= 4096)
      reduce_add_norm_kernel<NS, 1><<<rows, threads, 0, st>>>(x, ldx, P, split_stride, ldp, (const bf16_t*)gain, eps, out, H, (const bf16_t*)bias);
    else
      reduce_add_norm_kernel<NS, 2><<<rows, threads, 0, st>>>(x, ldx, P, split_stride, ldp, (const bf16_t*)gain, eps, out, H, (const bf16_t*)bias);
  });
}

}  // namespace clv
