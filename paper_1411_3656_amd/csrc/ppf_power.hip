// Detection after the filter bank: the power |X[m][k]|^2 of every bin summed
// over K consecutive spectra, in the epilogue of the fused FP32 kernel (or
// of the FFT pass of the two-pass form), so the spectra never reach HBM.
// Each thread owns the same bins of every spectrum it transforms, so the
// sum stays in registers; tiles start at multiples of K.

#include "ppf_engine.h"

namespace ppf {

typedef hipError_t (*PowerFn)(const PlanDev&, const BatchArgs&, const float*, int, hipStream_t, float*, int);

template <int N>
static PowerFn power_for_taps(int TP) {
  switch (TP) {
    case 1: return &fused_launch<N, 1, false, true>;
    case 2: if constexpr (fused_ok(N, 2)) return &fused_launch<N, 2, false, true>; else return nullptr;
    case 4: if constexpr (fused_ok(N, 4)) return &fused_launch<N, 4, false, true>; else return nullptr;
    case 8: if constexpr (fused_ok(N, 8)) return &fused_launch<N, 8, false, true>; else return nullptr;
    case 16: if constexpr (fused_ok(N, 16)) return &fused_launch<N, 16, false, true>; else return nullptr;
    default: return nullptr;
  }
}

static PowerFn power_fn(int N, int TP) {
  switch (N) {
    case 16: return power_for_taps<16>(TP);
    case 32: return power_for_taps<32>(TP);
    case 64: return power_for_taps<64>(TP);
    case 128: return power_for_taps<128>(TP);
    case 256: return power_for_taps<256>(TP);
    case 512: return power_for_taps<512>(TP);
    case 1024: return power_for_taps<1024>(TP);
    case 2048: return power_for_taps<2048>(TP);
    case 4096: return power_for_taps<4096>(TP);
    case 8192: return power_for_taps<8192>(TP);
    case 16384: return power_for_taps<16384>(TP);
    default: return nullptr;
  }
}

static PowerFn fft_power_fn(int N) {
  switch (N) {
    case 16: return &fused_launch<16, 1, true, true>;
    case 32: return &fused_launch<32, 1, true, true>;
    case 64: return &fused_launch<64, 1, true, true>;
    case 128: return &fused_launch<128, 1, true, true>;
    case 256: return &fused_launch<256, 1, true, true>;
    case 512: return &fused_launch<512, 1, true, true>;
    case 1024: return &fused_launch<1024, 1, true, true>;
    case 2048: return &fused_launch<2048, 1, true, true>;
    case 4096: return &fused_launch<4096, 1, true, true>;
    case 8192: return &fused_launch<8192, 1, true, true>;
    case 16384: return &fused_launch<16384, 1, true, true>;
    default: return nullptr;
  }
}

// A group's K spectra are summed in order by one workgroup, so few groups leave
// most of the chip idle. Then each group is cut into parts: the kernels above
// sum the parts (K / parts spectra each) side by side into a buffer, and this
// kernel adds a group's parts, out[g][c] = sum_i part[g * parts + i][c]. It
// reads at most 2 MiB (16 at N = 16384), from cache, and is bound by its launch
// and the latency of a few loads: lanes (tx) take four neighbouring bins each,
// rows (ty) of the workgroup every Y-th part, and the rows' sums meet in LDS in
// a fixed order. 64 spectra in one group, T = 8: N = 256 39.0 -> 10.0 us, 1024
// 56.0 -> 11.3, 4096 224 -> 21, 16384 829 -> 29; the sums' error against 64
// bits falls (1.2e-7 -> 0.7e-7 of the power at N = 1024).
__global__ void __launch_bounds__(256) ppf_power_parts_kernel(const float4* part, float4* out, int n4, int parts) {
  __shared__ float4 red[256];
  const int L = blockDim.x, Y = blockDim.y;
  const int tx = threadIdx.x, ty = threadIdx.y;
  const int c = (int)blockIdx.y * L + tx;      // the grid covers n4 exactly
  const float4* src = part + (long long)blockIdx.x * parts * n4 + c;
  float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
  for (int i = ty; i < parts; i += Y) {
    const float4 v = src[(long long)i * n4];
    a.x += v.x;
    a.y += v.y;
    a.z += v.z;
    a.w += v.w;
  }
  red[ty * L + tx] = a;
  for (int h = Y / 2; h > 0; h /= 2) {
    __syncthreads();
    if (ty < h) {
      const float4 v = red[(ty + h) * L + tx];
      a.x += v.x;
      a.y += v.y;
      a.z += v.z;
      a.w += v.w;
      red[ty * L + tx] = a;
    }
  }
  if (ty == 0) out[(long long)blockIdx.x * n4 + c] = a;
}

// Groups and parts together stay within these many, where a launch keeps every
// CU busy: with twice as many, cutting groups in two lost up to 15% (N = 1024,
// T = 8, 512 groups of 16: 26.6 us whole, 30.6 cut), here it gains from the
// first cut on (256 groups 19.6 -> 18.8; N = 2048, 128 groups 35.9 -> 24.2;
// N = 4096 70.0 -> 48.8; N = 16384 330 -> 228).
// At N = 128 half as many: the T = 8 kernel has one workgroup of eight tiles on a CU
// (2048 groups of 24 22.0 us whole, 24.8 cut in two).
static long long power_slots(int N) {
  return (long long)device_cus() * (N == 128 ? 8 : (N < 2048 ? 2048 / N : 1));
}

size_t power_parts_bytes(int N) { return (size_t)power_slots(N) * N * sizeof(float); }

int power_parts(int N, long long M, int K) {
  const long long groups = M / K;
  long long most = power_slots(N) / groups;
  if (most > 1024) most = 1024;                // the summing kernel's serial length
  if (most > K) most = K;
  if (most < 2) return 1;
  int parts = (int)most;
  while (parts > 1 && K % parts) --parts;
  // A part saves the serial work of K - K / parts spectra, 0.4 us + N / 1300 each,
  // and costs a launch. N = 1024: K = 4 5.7 us whole, 10.0 cut, K = 6 13.3, 10.1;
  // N = 256: K = 4 6.1, 9.9, K = 16 11.5, 9.9; N = 2048: K = 2 8.6, 9.8, K = 4
  // 11.7, 10.2. Up to N = 1024 most kernels compute four spectra per step, and
  // halves that give CUs a second workgroup have to save two steps (N = 1024,
  // K = 10: 128 groups 14.4 whole, 12.9 cut; 171 14.7, 16.9; 256 groups, K = 12
  // 16.0, 17.8; K = 14 18.9, 18.4; K = 16 20.0, 19.0).
  if (parts == 2 && N <= 1024 && groups * 4 > power_slots(N) && (K + 3) / 4 - (K / 2 + 3) / 4 < 2) return 1;
  return (long long)(K - K / parts) * (N + 512) >= 15 * 512 ? parts : 1;
}

hipError_t launch_power_parts(const float* part, float* out, int N, long long groups, int parts, hipStream_t st) {
  const int n4 = N / 4;
  const int L = n4 < 64 ? n4 : 64;
  int Y = 256 / L;
  while (Y > 1 && Y > parts) Y /= 2;
  hipLaunchKernelGGL(ppf_power_parts_kernel, dim3((unsigned)groups, (unsigned)(n4 / L)), dim3(L, Y), 0, st,
                     (const float4*)part, (float4*)out, n4, parts);
  return hipGetLastError();
}

hipError_t launch_fused_power(const PlanDev& pd, const BatchArgs& a, float* pout, int K, hipStream_t st) {
  PowerFn f = power_fn(pd.N, pd.TP);
  if (!f) return hipErrorInvalidValue;
  return f(pd, a, pd.coef, pd.T, st, pout, K);
}

hipError_t launch_fft_power(const PlanDev& pd, const void* in, float* pout, long long M, int K, hipStream_t st) {
  PowerFn f = fft_power_fn(pd.N);
  if (!f) return hipErrorInvalidValue;
  BatchArgs a{in, in, 0, nullptr, M};
  return f(pd, a, pd.ones, 1, st, pout, K);
}

}  // namespace ppf
