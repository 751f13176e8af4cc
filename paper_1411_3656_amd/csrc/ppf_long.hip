// Fused FIR + FFT kernels for tap windows that are too large for the layout
// of the fused kernel in ppf_engine.h (17 to 32 taps at N = 64 to 1024, 5 to
// 16 at N = 2048, 5 to 8 at N = 4096): one pass over HBM.
//
// The fused kernel of ppf_engine.h gives the FIR the layout of the FFT: a
// lane owns the R channels j + e*W that it transforms, and its tap window of
// R * T complex values is what bounds it. Here the FIR has a layout of its
// own: a lane owns C <= R channels and computes B = R / C consecutive spectra
// of them per step, so the window is C * (T + B) values, and the T
// coefficients of a channel are read once for B spectra. With C < R the B * N
// presums of a step go through LDS to the lanes that transform them: lane l
// of the N / C lanes of a group takes elements j + e * N/R of spectrum fb,
// fb = l / (N/R), j = l % (N/R). From there on the group FFT (radix 8) and
// the stores are those of the fused kernel.

#include "ppf_engine.h"

namespace ppf {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

// N channels, C per lane in the FIR, R elements per lane in the FFT, TP tap
// slots, PF blocks loaded ahead, G groups (tiles) per workgroup; CL keeps
// the coefficients in LDS; IT is the stored input type.
template <int N, int C, int R, int TP, int PF, int G, bool CL, int IT>
struct LongEngine {
  static constexpr int B = R / C;              // spectra per step
  static constexpr int W1 = N / C;             // lanes of a group
  static constexpr int WF = N / R;             // lanes of one spectrum's transform
  static constexpr int Q = TP + PF;            // ring slots
  static constexpr int NT = W1 * G;
  static constexpr int GG = G * B;             // transforms per workgroup
  static constexpr int SB = in_bytes(IT);
  // N >= 512 (2 waves per SIMD): a step's blocks are loaded after the FIR of
  // the step before, into the slots it has finished with, so the loads run
  // under its transforms. Loaded at the start of the step that uses them
  // they measured 0.959 ms at N = 512, T = 32 (after: 0.876), 1.036 (0.992)
  // at N = 1024 and 1.190 (0.950) at N = 2048, T = 16; with 3 waves per SIMD
  // or narrower groups the early loads are as fast or faster (N = 64: 0.867,
  // after: 0.892).
  static constexpr bool LATE = N >= 512;
  static constexpr bool WS = WF <= 64;         // transforms within one wavefront
  static constexpr bool HW = W1 <= 64;         // hand-over within one wavefront
  static constexpr bool DB = !WS && 2 * GG * N * 8 + (CL ? TP * N * 4 : 0) <= 80 * 1024;
  using Fft = GroupFft<N, R, R, GG, 1, DB, false, false, WS>;
  // WS: hand-over rows of their own, two sets where waves of one group pass
  // a barrier at it (the next step's writes then meet finished reads). The
  // rows are padded so that the 16-lane transforms of N = 64 read distinct banks.
  static constexpr int HS = N + (WF < 32 ? 16 : 0);
  static constexpr int NH = WS && C < R ? (HW ? 1 : 2) : 0;
  static constexpr size_t hand_bytes() { return (size_t)NH * GG * HS * sizeof(v2f); }
  static constexpr size_t coef_bytes() { return CL ? (size_t)TP * N * sizeof(float) : 0; }
  static constexpr size_t lds_bytes() { return Fft::lds_bytes() + hand_bytes() + coef_bytes(); }
  static_assert(Q % B == 0 && Q >= TP + B - 1, "ring size");
  static_assert(!CL || (TP / 4 * N) % NT == 0, "whole passes over the coefficients");
  static_assert(W1 >= 64, "a wavefront works on one tile");

  Fft fft;
  v2f* hand;
  int g, l, fb, fj;
  int d, hp;
  float hreg[CL ? 1 : TP][C];
  uint32_t hl;
  uint32_t loff, soff;
  v2f ring[Q][C];
  TileArgs a;
  int m0, ng, niter, vb_lo, vb_hi;

  __device__ __forceinline__ void init(float* smem, const float* coef, const v2f* tw, int d_) {
    const int tid = threadIdx.x;
    g = __builtin_amdgcn_readfirstlane(tid / W1);
    l = tid % W1;
    fb = l / WF;
    fj = l % WF;
    if constexpr (WF >= 64) fb = __builtin_amdgcn_readfirstlane(fb);
    d = d_;
    hp = 0;
    fft.init(smem, g * B + fb, fj, tw);
    hand = (v2f*)((char*)smem + Fft::lds_bytes());
    if constexpr (CL) {
      // all loads in flight at once: a loop that waits for each took 17 us,
      // more than a short batch's transforms
      v4f* cl = (v4f*)((char*)smem + Fft::lds_bytes() + hand_bytes());
#pragma unroll
      for (int k = 0; k < TP / 4 * N / NT; ++k) {
        const int i = tid + k * NT, t = i / N, c = i % N;
        v4f h4;
#pragma unroll
        for (int q = 0; q < 4; ++q) h4[q] = coef[(4 * t + q) * N + c];
        cl[i] = h4;
      }
      __syncthreads();
      hl = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) v4f*)(cl + l);
    } else {
#pragma unroll
      for (int t = 0; t < TP; ++t)
#pragma unroll
        for (int c = 0; c < C; ++c) hreg[t][c] = coef[t * N + l + c * W1];
    }
    loff = (uint32_t)(l * SB);
    soff = (uint32_t)((fb * N + fj) * (int)sizeof(v2f));
  }

  // CL: the coefficients of four taps are one 16-byte LDS element of the
  // channel, read through a base refreshed every step (so that the reads are
  // not hoisted into registers)
  __device__ __forceinline__ v4f hcoef4(uint32_t base, int t, int c) const {
    return *(const __attribute__((address_space(3))) v4f*)(uintptr_t)(base + (uint32_t)(((t / 4) * N + c * W1) * 16));
  }

  // Blocks outside [vb_lo, vb_hi) are the zero padding of the first taps, or
  // feed only spectra beyond the tile: an empty range reads zeros.
  __device__ __forceinline__ void load(v2f (&dst)[C], int vb) {
    const bool ok = vb >= vb_lo && vb < vb_hi;
    const __amdgpu_buffer_rsrc_t rs = block_rsrc(block_addr<N, SB>(a, ok ? vb - d : 0), ok ? N * SB : 0);
    constexpr int aux = kNtLoads ? kAuxNt : 0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const uint32_t so = (uint32_t)(c * W1 * SB);
      if constexpr (IT == 0) {
        dst[c] = buf_load<aux>(rs, loff, so);
      } else if constexpr (IT == 1) {
        dst[c].x = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, loff, so, aux));
      } else {
        dst[c].x = __builtin_bit_cast(float, (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(rs, loff, so, aux));
      }
    }
  }
  // FP16 / int8 slots hold the stored bits until the step that first reads them
  __device__ __forceinline__ void widen(v2f (&slot)[C]) {
    if constexpr (IT != 0) {
#pragma unroll
      for (int c = 0; c < C; ++c) {
        const uint32_t w = __builtin_bit_cast(uint32_t, slot[c].x);
        slot[c] = IT == 1 ? widen_c16(w) : widen_ci8(w);
      }
    }
  }

  __device__ __forceinline__ static void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }

  // B presums of channel c handed to the transforms' lanes
  __device__ __forceinline__ void exchange(const v2f (&u)[B][C], v2f (&v)[1][R]) {
    if constexpr (WS) {
      v2f* hb = hand + hp * (GG * HS);
#pragma unroll
      for (int b = 0; b < B; ++b)
#pragma unroll
        for (int c = 0; c < C; ++c) hb[(g * B + b) * HS + l + c * W1] = u[b][c];
      if constexpr (HW) wave_fence(); else __syncthreads();
#pragma unroll
      for (int e = 0; e < R; ++e) v[0][e] = hb[(g * B + fb) * HS + fj + e * WF];
      if constexpr (NH > 1) hp ^= 1;
      if constexpr (HW) wave_fence();
    } else {
      if constexpr (!DB) __syncthreads();       // the planes are free
      v2f* pl0 = (v2f*)fft.lds + (DB ? fft.par * (GG * Fft::PL) : 0);
#pragma unroll
      for (int b = 0; b < B; ++b)
#pragma unroll
        for (int c = 0; c < C; ++c) pl0[(g * B + b) * Fft::PL + swz64(l + c * W1)] = u[b][c];
      __syncthreads();
      const v2f* pl = pl0 + (g * B + fb) * Fft::PL;
#pragma unroll
      for (int e = 0; e < R; ++e) v[0][e] = pl[swz64(fj + e * WF)];
      if constexpr (DB) fft.par ^= 1;
    }
  }

  // one step (B spectra from it on) at ring phase K, then the next
  template <int K>
  __device__ __forceinline__ void steps(int base) {
    if constexpr (K < Q) {
      const int it = base + K;
      if (it < niter) {
        if constexpr (!LATE) {
#pragma unroll
          for (int b = 0; b < B; ++b) load(ring[(K + Q - B + b) % Q], m0 + it + Q - B + b);
        }
#pragma unroll
        for (int b = 0; b < B; ++b) widen(ring[(K + TP - 1 + b) % Q]);
        v2f u[B][C];
        uint32_t hb = hl;
        if constexpr (CL) asm volatile("" : "+v"(hb));
        v4f h4[C];
#pragma unroll
        for (int t = 0; t < TP; ++t)
#pragma unroll
          for (int c = 0; c < C; ++c) {
            if (CL && t % 4 == 0) h4[c] = hcoef4(hb, t, c);
            const float h = CL ? h4[c][t % 4] : hreg[CL ? 0 : t][c];
#pragma unroll
            for (int b = 0; b < B; ++b) {
              const v2f x = ring[(K + b + t) % Q][c];
              if (t == 0) {
                u[b][c].x = h * x.x;
                u[b][c].y = h * x.y;
              } else {
                u[b][c].x = fmaf(h, x.x, u[b][c].x);
                u[b][c].y = fmaf(h, x.y, u[b][c].y);
              }
            }
          }
        if constexpr (LATE) {
#pragma unroll
          for (int b = 0; b < B; ++b) load(ring[(K + b) % Q], m0 + it + Q + b);
        }
        v2f v[1][R];
        if constexpr (C == R) {
#pragma unroll
          for (int e = 0; e < R; ++e) v[0][e] = u[0][e];
        } else {
          exchange(u, v);
        }
        fft.run(v);
        const int left = ng - it;              // spectra beyond the tile fall outside the range
        const int rows = left < 0 ? 0 : (left < B ? left : B);
        const __amdgpu_buffer_rsrc_t rs =
            block_rsrc(a.out + (long long)(m0 + it) * N, rows * N * (int)sizeof(v2f));
#pragma unroll
        for (int e = 0; e < R; ++e) buf_store<kAuxNt>(v[0][e], rs, soff, (uint32_t)(e * WF * (int)sizeof(v2f)));
        steps<K + B>(base);
      }
    }
  }

  __device__ __forceinline__ void run(const TileArgs& a_, int m0_, int ng_, int niter_) {
    a = a_;
    m0 = m0_;
    ng = ng_;
    niter = niter_;
    vb_lo = m0 > d ? m0 : d;
    vb_hi = ng > 0 ? m0 + ng + TP - 1 : m0;
#pragma unroll
    for (int s = 0; s < Q; ++s)
#pragma unroll
      for (int c = 0; c < C; ++c) { ring[s][c].x = 0.f; ring[s][c].y = 0.f; }
#pragma unroll
    for (int s = 0; s < (LATE ? Q : Q - B); ++s) load(ring[s], m0 + s);
#pragma unroll
    for (int s = 0; s < TP - 1; ++s) widen(ring[s]);
    for (int base = 0; base < niter; base += Q) steps<0>(base);
  }
};

template <int N, int C, int R, int TP, int PF, int G, bool CL, int IT>
__global__ void __launch_bounds__((N / C) * G)
__attribute__((amdgpu_waves_per_eu(N == 64 ? 3 : 2)))
ppf_long_kernel(FusedParams p) {
  using Eng = LongEngine<N, C, R, TP, PF, G, CL, IT>;
  extern __shared__ float smem[];
  if ((int)blockIdx.x >= p.nblocks) {
    history_block(p.hist, (int)blockIdx.x - p.nblocks);
    return;
  }
  const int lb = xcd_remap(blockIdx.x, p.nblocks);
  const int blk_m0 = lb * G * p.S;
  if (blk_m0 >= p.M) return;                                   // whole block idle
  Eng eng;
  eng.init(smem, p.coef, p.tw, p.d);
  const int m0 = blk_m0 + eng.g * p.S;
  const int rem = p.M - m0;
  const int ng = rem <= 0 ? 0 : (rem < p.S ? rem : p.S);       // this group's spectra
  const int brem = p.M - blk_m0;
  const int niter = brem < p.S ? brem : p.S;                   // uniform over the block
  TileArgs a{p.x0, p.x1, p.x1, p.out, p.h0, p.h0};
  eng.run(a, m0, ng, niter);
}

// Layouts, measured at 2^28 FP32 samples (in brackets what they replaced).
// R = 8 transforms take fewer, wider stages (512 = 8*8*8) and read the
// coefficients once for more spectra, at 2 waves per SIMD; R = 4 fits 3.
//   T = 32 (two passes), N = 64: R = 4 0.879 ms, R = 8 0.974 (1.507)
//     N = 128: R = 4 0.936, R = 8 0.869 (1.538)
//     N = 256: R = 4 0.932, R = 8 0.863 (2.174)
//     N = 512: R = 4 1.199 (coefficients in LDS 1.265), R = 8 0.876 (1.629)
//     N = 1024: R = 4 1.291, two channels per lane and R = 8 0.992 (1.723)
//   N = 2048, T = 16: four channels per lane 0.953 ms (two passes 1.709)
//   N = 2048, T = 8: 0.812 ms, coefficients in LDS 0.834 (8 channels per
//     lane without a hand-over, loads at the start of the step: 0.932)
//   N = 4096, T = 8: eight channels per lane, no hand-over 0.878 ms (four
//     over 1024 threads, radix 4, ten barriers per spectrum: 1.084).
// Where the coefficients (T * C registers per lane) do not fit beside the
// window they are in LDS. With 16 taps or fewer at N <= 1024 the fused kernel's
// window fits and it is as fast at N = 64 (T = 16: 0.787 against 0.860) and N =
// 1024 (T = 8: 0.810 against 0.805 to 1.058). Not so with 16 taps at N = 128, 256
// and 512, where radix 8 and four tiles per slot measured 0.81, 0.84 and 0.875
// against the fused kernel's 0.88, 0.87 and 0.942; no such kernels are built.
constexpr int long_C(int N) { return N == 4096 ? 8 : (N == 2048 ? 4 : (N == 1024 ? 2 : 1)); }
constexpr int long_R(int N) { return N == 64 ? 4 : 8; }
constexpr int long_PF(int N) { return long_R(N) / long_C(N); }   // a step's blocks
constexpr int long_G(int N) { return N >= 256 ? 1 : 256 / N; }   // 256 lanes or more
constexpr bool long_CL(int N, int TP) { return N >= 1024 && !(N == 2048 && TP == 8); }

template <int N, int C, int R, int TP, int PF, int G, bool CL, int IT>
hipError_t long_launch(const PlanDev& pd, const float* coef, int T, const BatchArgs& a0, hipStream_t st) {
  using Eng = LongEngine<N, C, R, TP, PF, G, CL, IT>;
  auto kern = &ppf_long_kernel<N, C, R, TP, PF, G, CL, IT>;
  static const int occ = [&] {
    KernelInfo ki{(const void*)kern, Eng::NT, G, Eng::lds_bytes()};
    return occupancy(ki);
  }();
  for (long long s0 = 0; s0 < a0.M; s0 += kMaxLaunchSpectra) {
    const long long k = a0.M - s0 < kMaxLaunchSpectra ? a0.M - s0 : kMaxLaunchSpectra;
    const BatchArgs a = sub_batch(a0, N, Eng::SB, s0, k);
    // one tile per resident group (4 or 8 measured no faster), whole steps.
    // Small batches take one-step tiles: a step is bound by its FIR on one
    // CU (3.7 us at N = 1024), the re-reads of the tap window come from cache
    const long long slots = (long long)device_cus() * occ * G;
    long long S = (a.M + slots - 1) / slots;
    S = (S + Eng::B - 1) / Eng::B * Eng::B;
    const long long nblocks = (a.M + S * G - 1) / (S * G);
    FusedParams p{};
    p.x0 = (const v2f*)a.x0;
    p.x1 = (const v2f*)a.x1;
    p.out = (v2f*)a.out;
    p.coef = coef;
    p.tw = (const v2f*)pd.tw;
    p.h0 = (int)a.h0;
    p.M = (int)a.M;
    p.S = (int)S;
    p.d = TP - T;
    p.nblocks = (int)nblocks;
    const long long hb = history_blocks(a.hist, Eng::NT);
    if (hb > 0) p.hist = *a.hist;
    hipLaunchKernelGGL(kern, dim3((unsigned)(nblocks + hb)), dim3(Eng::NT), Eng::lds_bytes(), st, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int N, int TP, int IT>
hipError_t long_batch(const PlanDev& pd, const BatchArgs& a, hipStream_t st) {
  return long_launch<N, long_C(N), long_R(N), TP, long_PF(N), long_G(N), long_CL(N, TP), IT>(pd, pd.coef, pd.T, a, st);
}

typedef hipError_t (*LongFn)(const PlanDev&, const BatchArgs&, hipStream_t);

template <int N, int TP>
LongFn long_for_type(int it) {
  switch (it) {
    case 0: return &long_batch<N, TP, 0>;
    case 1: return &long_batch<N, TP, 1>;
    case 2: return &long_batch<N, TP, 2>;
    default: return nullptr;
  }
}

// supported shapes; fused_by_long (ppf_engine.h) names those of the fused path
LongFn long_fn(int N, int TP, int it) {
  if (TP == 8 && N == 4096) return fused_by_long(4096, 8) ? long_for_type<4096, 8>(it) : nullptr;
  if (TP == 8) return N == 2048 ? long_for_type<2048, 8>(it) : nullptr;
  if (TP == 16) return N == 2048 ? long_for_type<2048, 16>(it) : nullptr;
  if (TP != 32) return nullptr;
  switch (N) {
    case 64: return long_for_type<64, 32>(it);
    case 128: return long_for_type<128, 32>(it);
    case 256: return long_for_type<256, 32>(it);
    case 512: return long_for_type<512, 32>(it);
    case 1024: return long_for_type<1024, 32>(it);
    default: return nullptr;
  }
}

}  // namespace

// Shortest batch of a two-pass shape taken in one launch. A workgroup reads
// T + B - 1 blocks and all coefficients for its first step, which takes the
// same time however few spectra there are; two passes spread a short batch
// over more CUs. FP32 input, us in one launch and in two passes: N = 512,
// T = 17: 1 spectrum 8.9, 6.7; 256 9.4, 8.4; 600 9.6, 9.8. N = 1024: 1 11.9,
// 7.5; 256 13.9, 10.1; 512 14.3, 12.2; 600 14.4, 14.7. N = 2048, T = 16: 64 13.5,
// 8.5; 256 14.7, 11.3; 400 14.8, 14.7; 512 15.1, 15.9. FP16 and int8 input, whose
// FIR pass converts as it loads: N = 512: 1 8.8, 8.3; 4 9.0, 9.0; N = 1024,
// T = 17: 1 11.5, 9.4; 12 11.9, 11.2; 16 11.9, 11.7 (T = 32: no more than 0.2 apart up to
// 32); N = 2048: 64 10.9, 10.3; 128 11.2, 11.4 (int8 11.8, 11.4). Up to N = 256 one
// launch is as fast from one spectrum on.
int long_min_spectra(int N, int in_type) {
  switch (N) {
    case 512: return in_type == 0 ? 512 : 1;
    case 1024: return in_type == 0 ? 576 : 16;
    case 2048: return in_type == 0 ? 400 : 128;
    default: return 1;
  }
}

bool long_available(int N, int TP) { return long_fn(N, TP, 0) != nullptr; }

hipError_t launch_long(const PlanDev& pd, const BatchArgs& a, hipStream_t st) {
  LongFn f = long_fn(pd.N, pd.TP, pd.in_type);
  if (!f) return hipErrorInvalidValue;
  return f(pd, a, st);
}

// The FFT pass of those shorter batches at N = 512 and 1024: this file's kernel
// with a single tap of one. Its radix is that of the one-launch kernels, so that a
// spectrum has the same bits in either form (launch_fft's is 4 there), and it is
// faster: N = 512, 16 spectra, both passes 8.4 -> 7.4 us; 256 9.1 -> 8.4; N = 1024,
// 256 10.3 -> 10.1.
bool long_fft_available(int N) { return N == 512 || N == 1024; }

hipError_t launch_long_fft(const PlanDev& pd, const void* in, void* out, long long M, hipStream_t st) {
  const BatchArgs a{in, in, 0, out, M};
  switch (pd.N) {
    case 512: return long_launch<512, 8, 8, 1, 1, 4, false, 0>(pd, pd.ones, 1, a, st);
    case 1024: return long_launch<1024, 8, 8, 1, 1, 2, false, 0>(pd, pd.ones, 1, a, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ppf
