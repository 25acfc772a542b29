// Does the ORDER of a tile's matrix products change their rate?  (stand-alone; no part of the library)
// Every wavefront of 256 workgroups of four (one wavefront per SIMD) multiplies one fixed pair of operands over and over into
// 8 x 8 blocks of 16 x 16 accumulators, as the GEMM's 256 x 256 tile does for one 32-column step: 8 blocks of rows with a hi
// and a lo plane, 8 blocks of columns.  Orders: the block's lo and hi product back to back; all lo products, then all hi; the
// same work as 32 x 32 x 16 products (4 x 4 blocks).  Random operands: the switching of the pipe is what counts.
// Clock: shader clocks (s_memtime) over the 100 MHz reference (s_memrealtime), both read on the device.
//   hipcc -O3 --offload-arch=gfx950 -o /tmp/mfma_order paper_2408_00264_amd/csrc/probes/mfma_order.hip && /tmp/mfma_order
#include <hip/hip_runtime.h>
#include <cstdio>
#include <vector>
#define CK(x) do { hipError_t e = (x); if (e != hipSuccess) { printf("HIP error %s at line %d\n", hipGetErrorString(e), __LINE__); return 1; } } while (0)
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

template <int ORDER>
__global__ __launch_bounds__(256, 1) void probe(const bf16x8* src, float* out, unsigned long long* clocks, int iters) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  bf16x8 a[16], b[8];   // [row block][lo, hi], [column block]
  for (int i = 0; i < 16; ++i) a[i] = src[(wave * 24 + i) * 64 + lane];
  for (int i = 0; i < 8; ++i) b[i] = src[(wave * 24 + 16 + i) * 64 + lane];
  float s = 0.f;
  unsigned long long t0 = 0, r0 = 0;
  auto start = [&] { __syncthreads(); t0 = __builtin_readcyclecounter(); r0 = __builtin_amdgcn_s_memrealtime(); };
  if constexpr (ORDER < 2) {
    f32x4 acc[64];
#pragma unroll
    for (int i = 0; i < 64; ++i) acc[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
    start();
    for (int it = 0; it < iters; ++it) {
#pragma unroll
      for (int m = 0; m < 128; ++m) {
        const int blk = ORDER == 0 ? m / 2 : m % 64, plane = ORDER == 0 ? m % 2 : m / 64, rb = blk / 8, cb = blk % 8;
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[blk]) : "v"(b[cb]), "v"(a[2 * rb + plane]));
      }
    }
    asm volatile("s_nop 15\n\ts_nop 7" : : : "memory");
#pragma unroll
    for (int i = 0; i < 64; ++i) s += acc[i][0] + acc[i][1] + acc[i][2] + acc[i][3];
  } else {
    f32x16 acc[16];
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[i][j] = 0.f;
    start();
    for (int it = 0; it < iters; ++it) {
#pragma unroll
      for (int m = 0; m < 64; ++m) {   // 4 x 4 blocks of 32 x 32, two planes, two halves of the 32 columns of K
        const int blk = m / 4, k = m % 4, rb = blk / 4, cb = blk % 4;
        asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc[blk]) : "v"(b[2 * cb + (k & 1)]), "v"(a[4 * rb + k]));
      }
    }
    asm volatile("s_nop 15\n\ts_nop 15" : : : "memory");
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
      for (int j = 0; j < 16; ++j) s += acc[i][j];
  }
  const unsigned long long t1 = __builtin_readcyclecounter(), r1 = __builtin_amdgcn_s_memrealtime();
  out[blockIdx.x * 256 + threadIdx.x] = s;
  if (threadIdx.x == 0) { clocks[2 * blockIdx.x] = t1 - t0; clocks[2 * blockIdx.x + 1] = r1 - r0; }
}

template <int ORDER>
static int run(const char* name, const bf16x8* src, float* out, unsigned long long* clocks) {
  const int iters = 20000;
  hipEvent_t e0, e1;
  CK(hipEventCreate(&e0)); CK(hipEventCreate(&e1));
  for (int rep = 0; rep < 3; ++rep) {
    CK(hipEventRecord(e0));
    probe<ORDER><<<256, 256>>>(src, out, clocks, iters);
    CK(hipEventRecord(e1));
    CK(hipEventSynchronize(e1));
  }
  float ms = 0.f;
  CK(hipEventElapsedTime(&ms, e0, e1));
  unsigned long long c[512];
  CK(hipMemcpy(c, clocks, sizeof(c), hipMemcpyDeviceToHost));
  double cyc = 0, ref = 0;
  for (int i = 0; i < 256; ++i) { cyc += c[2 * i]; ref += c[2 * i + 1]; }
  const double flop = 256.0 * 4 * iters * 128 * 2 * 16 * 16 * 32;
  printf("%-44s %8.3f ms  %5.2f PFLOP/s  %5.2f GHz  %5.2f clocks per 16 x 16 x 32 product\n", name, ms, flop / ms * 1e-12, cyc / ref * 0.1,
         cyc / 256 / iters / 128);
  return 0;
}

int main() {
  std::vector<unsigned short> h(4 * 24 * 64 * 8);
  unsigned x = 12345;
  for (auto& v : h) {   // +-[0.5, 1), random mantissas
    x = x * 1664525u + 1013904223u;
    v = (unsigned short)(((x >> 16) & 0x8000u) | 0x3F00u | ((x >> 9) & 0x7Fu));
  }
  bf16x8* src; float* out; unsigned long long* clocks;
  CK(hipMalloc(&src, h.size() * 2)); CK(hipMalloc(&out, 256 * 256 * 4)); CK(hipMalloc(&clocks, 512 * 8));
  CK(hipMemcpy(src, h.data(), h.size() * 2, hipMemcpyHostToDevice));
  return run<0>("lo and hi product of a block back to back", src, out, clocks) || run<1>("all lo products, then all hi products", src, out, clocks) ||
         run<2>("32 x 32 x 16 products", src, out, clocks);
}
