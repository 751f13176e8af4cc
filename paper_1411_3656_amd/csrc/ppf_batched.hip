// Fused FIR + FFT for N = 4096 with 9 to 16 taps and N = 8192 with 2 to 8: one
// pass over HBM for shapes whose tap window (up to 512 KiB) fits neither the
// registers nor the LDS of a CU.
//
// N = 4096. A workgroup computes a batch of B = 8 consecutive spectra at a time, and
// no tap window outlives it. Lane l of 512 owns the channels l + 512 e,
// e < 8 (the first radix-8 stage's elements). It takes them in two halves:
// the B presums of four channels are accumulated in registers while the
// T + B - 1 blocks that they need stream past, each block read once per
// batch; those of the first half wait in LDS (128 KiB) until the second half
// is done. Then the B transforms follow, each on the presums of both halves.
//
// A block is so read by three consecutive batches, 23 blocks for 8 spectra.
// Consecutive batches run at the same time on the CUs of one XCD, and each
// takes its blocks in three groups of eight, starting with another group
// than its neighbours (group -q mod 3 for batch q): group g of batch q is
// blocks 8 (q + g) .. 8 (q + g) + 7, so at any time the three batches that
// share a group of blocks read the same one, and two of the three reads are
// L2 hits (HBM traffic measured: 2.31 GB read, 2.15 GB written at 2^28
// samples; 2.15 each is the least).
//
// N = 4096, T = 16, 2^28 FP32 samples: 1.117 ms, two passes 1.769 (int8 input
// at 2^27: 0.445, 0.909). Counters: the VALU is busy 48% of the cycles and the LDS
// 35%, and waves wait for instructions in flight 34% of their time, so it is the
// serial chain of the FIR and four pairs of transforms with their barriers, at 2
// waves per SIMD, that bounds it. One transform at a time took 1.196 ms; twiddles
// from the global table 1.796; the next batch's coefficients loaded under the
// last transforms 1.139; without the rotated order, in which equal blocks would
// also have equal bits wherever they stand in the batch, 1.142.

#include "ppf_engine.h"

namespace ppf {
namespace {

// Workgroup w runs on XCD w % 8; an XCD takes a contiguous range of batches,
// its workgroups in turn, so that the batches running at once on it are
// neighbours. This workgroup's: q0, q0 + step, .. below q1.
__device__ __forceinline__ bool batch_range(const FusedParams& p, int B, int& q0, int& step, int& q1) {
  const int nb = (p.M + B - 1) / B;
  const int xcds = p.nblocks < 8 ? p.nblocks : 8;
  const int x = (int)blockIdx.x % xcds, k = (int)blockIdx.x / xcds;
  step = (p.nblocks - x + xcds - 1) / xcds;                  // workgroups of this XCD, after `before` of others
  const int before = x * (p.nblocks / xcds) + (x < p.nblocks % xcds ? x : p.nblocks % xcds);
  q0 = (int)((long long)nb * before / p.nblocks) + k;
  q1 = (int)((long long)nb * (before + step) / p.nblocks);
  return q0 < q1;
}

template <int IT>
struct BatchedEngine {
  static constexpr int N = 4096, TP = 16, R = 8, C = 4, B = 8, NT = 512;
  static constexpr int SB = in_bytes(IT);
  // two transforms share each barrier; the second one's plane is the parked
  // presums of the first two spectra, which the first pair has read
  using Fft = GroupFft<N, R, R, 1, 2, false, false>;
  static constexpr size_t plane_bytes() { return (size_t)N * sizeof(v2f); }
  static constexpr size_t park_bytes() { return (size_t)B * C * NT * sizeof(v2f); }
  static constexpr size_t lds_bytes() { return plane_bytes() + park_bytes(); }
  static_assert(Fft::lds_bytes() == 2 * plane_bytes() && 2 * C * NT * sizeof(v2f) == plane_bytes(), "planes");

  Fft fft;
  v2f* park;
  TileArgs a;
  int l, d, M;
  uint32_t loff, soff;
  float h[TP][C];
  v2f acc[B][C];
  static constexpr int D = 4;        // blocks loaded ahead (8 spill)
  static_assert(B % D == 0, "a block keeps its slot across groups");
  v2f xr[D][C];

  struct Batch {
    int m, lo, hi;       // first spectrum, blocks the batch reads
  };
  __device__ __forceinline__ Batch batch(int q, bool any) const {
    Batch t;
    t.m = q * B;
    t.lo = t.m > d ? t.m : d;
    const int ng = M - t.m < B ? M - t.m : B;
    t.hi = any ? t.m + ng + TP - 1 : t.m;
    return t;
  }

  // block k of the batch, channels of half p
  __device__ __forceinline__ void load(v2f (&dst)[C], const Batch& t, int k, int p) const {
    const int vb = t.m + k;
    const bool ok = vb >= t.lo && vb < t.hi;
    const __amdgpu_buffer_rsrc_t rs = block_rsrc(block_addr<N, SB>(a, ok ? vb - d : 0), ok ? N * SB : 0);
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const uint32_t so = (uint32_t)((p * C + c) * NT * SB);
      if constexpr (IT == 0) {
        dst[c] = buf_load<0>(rs, loff, so);
      } else if constexpr (IT == 1) {
        dst[c].x = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, loff, so, 0));
      } else {
        dst[c].x = __builtin_bit_cast(float, (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(rs, loff, so, 0));
      }
    }
  }
  __device__ __forceinline__ v2f widened(v2f s) const {
    if constexpr (IT == 0) return s;
    const uint32_t w = __builtin_bit_cast(uint32_t, s.x);
    return IT == 1 ? widen_c16(w) : widen_ci8(w);
  }

  // group G's blocks into the presums, each slot then refilled from group gn
  // of half pn of batch tn
  template <int G>
  __device__ __forceinline__ void group(const Batch& t, int p, const Batch& tn, int gn, int pn) {
#pragma unroll
    for (int j = 0; j < B; ++j) {
      constexpr int last = TP + B - 2;
      if (G * B + j <= last) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
          const v2f x = widened(xr[j % D][c]);
#pragma unroll
          for (int b = 0; b < B; ++b) {
            const int t = G * B + j - b;
            if (t >= 0 && t < TP) {
              acc[b][c].x = fmaf(h[t][c], x.x, acc[b][c].x);
              acc[b][c].y = fmaf(h[t][c], x.y, acc[b][c].y);
            }
          }
        }
      }
      if (j + D < B) load(xr[j % D], t, G * B + j + D, p);
      else load(xr[j % D], tn, gn * B + j + D - B, pn);
    }
  }

  // coefficients of a half (buffer loads: one lane offset, scalar offsets)
  __device__ __forceinline__ void coefs(const FusedParams& p, int half) {
    const __amdgpu_buffer_rsrc_t rc = block_rsrc(p.coef + half * C * NT, (TP * N - half * C * NT) * 4);
#pragma unroll
    for (int s = 0; s < TP; ++s)
#pragma unroll
      for (int c = 0; c < C; ++c)
        h[s][c] = __builtin_bit_cast(
            float, __builtin_amdgcn_raw_buffer_load_b32(rc, (uint32_t)l * 4u, (uint32_t)((s * N + c * NT) * 4), 0));
  }

  // batches q0, q0 + step, .. below q1; G0 is the group that each half
  // begins with
  template <int G0>
  __device__ __forceinline__ void run(const FusedParams& p, float* smem, int q0, int step, int q1) {
    constexpr int G1 = (G0 + 1) % 3, G2 = (G0 + 2) % 3;
    l = threadIdx.x;
    d = p.d;
    M = p.M;
    a = TileArgs{p.x0, p.x1, p.x1, p.out, p.h0, p.h0};
    loff = (uint32_t)(l * SB);
    soff = (uint32_t)(l * (int)sizeof(v2f));
    fft.init(smem, 0, l, p.tw);
    park = (v2f*)((char*)smem + plane_bytes()) + l;
    Batch t = batch(q0, true);
#pragma unroll
    for (int j = 0; j < D; ++j) load(xr[j], t, G0 * B + j, 0);
    for (int q = q0; q < q1; q += step) {
      const Batch tn = batch(q + step, q + step < q1);
#pragma nounroll
      for (int half = 0; half < 2; ++half) {
        coefs(p, half);
#pragma unroll
        for (int b = 0; b < B; ++b)
#pragma unroll
          for (int c = 0; c < C; ++c) acc[b][c].x = acc[b][c].y = 0.f;
        group<G0>(t, half, t, G1, half);
        group<G1>(t, half, t, G2, half);
        group<G2>(t, half, half == 0 ? t : tn, G0, 1 - half);
        if (half == 0) {
#pragma unroll
          for (int b = 0; b < B; ++b)
#pragma unroll
            for (int c = 0; c < C; ++c) park[(b * C + c) * NT] = acc[b][c];   // read by this lane only
        }
      }
      const int ng = M - t.m < B ? M - t.m : B;
#pragma unroll
      for (int b = 0; b < B; b += 2) {
        if (b < ng) {
          v2f v[2][R];
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int c = 0; c < C; ++c) {
              v[i][c] = park[((b + i) * C + c) * NT];
              v[i][C + c] = acc[b + i][c];
            }
          fft.run(v);
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const __amdgpu_buffer_rsrc_t rs =
                block_rsrc(a.out + (long long)(t.m + b + i) * N, b + i < ng ? N * (int)sizeof(v2f) : 0);
#pragma unroll
            for (int e = 0; e < R; ++e) buf_store<kAuxNt>(v[i][e], rs, soff, (uint32_t)(e * NT * (int)sizeof(v2f)));
          }
        }
      }
      __syncthreads();   // the planes, which hold parked presums next
      t = tn;
    }
  }
};

template <int IT>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
ppf_batched_kernel(FusedParams p) {
  using Eng = BatchedEngine<IT>;
  extern __shared__ float smem[];
  int q0, step, q1;
  if (!batch_range(p, Eng::B, q0, step, q1)) return;
  Eng eng;
  // group -k mod 3 first, k the workgroup's place on its XCD
  const int k = (int)blockIdx.x / 8 % 3;
  if (k == 0) eng.template run<0>(p, smem, q0, step, q1);
  else if (k == 1) eng.template run<2>(p, smem, q0, step, q1);
  else eng.template run<1>(p, smem, q0, step, q1);
}

// --------------------------------------------------------------------------
// N = 8192 with 2 to 8 taps
// --------------------------------------------------------------------------

// The same for N = 8192, whose transform alone fills a 64 KiB plane: four
// spectra at a time, the presums of two of them waiting in LDS (the first in
// the exchange plane itself) and of two in registers. A lane owns the
// channels l + 512 e, e < 16, and takes PC of them at a time through the
// T + 3 blocks in order. A coefficient register is reloaded for the next PC
// channels as soon as the last spectrum has used it, and D blocks are loaded
// ahead; the first part's come under the last transform of the batch before.
// Neighbouring batches run at the same time on one XCD and read a part of a
// block (16 KiB) within a few of each other's steps, so most of its reads
// hit L2 without a rotated order.
//
// 2^28 FP32 samples: T = 8 1.320 ms, T = 4 1.175, T = 2 1.084 (four-step form
// in two passes 1.807, 1.779, 1.862); int8 input at 2^27, T = 8: 0.481
// (0.806). Eight channels per part spill at T = 8 (1.538 ms); 16 taps take
// 1.697, no faster than two passes. N = 16384 does not fit: its transform
// needs the registers of the spectrum that waits (2.22 ms, two passes 1.77).
template <int N, int TP, int IT>
struct LargeEngine {
  static constexpr int NT = 512, R = N / NT;
  static constexpr int NP = 2, NR = 2, B = NP + NR;           // spectra that wait in LDS, in registers
  static constexpr int PC = 4;              // channels per part
  static constexpr int PARTS = R / PC;
  static constexpr int D = 3;               // blocks loaded ahead
  static constexpr int NB = (TP + B - 1 + D - 1) / D * D;    // block steps of a part
  static constexpr int SB = in_bytes(IT);
  using Fft = GroupFft<N, R, R, 1, 1, false, false>;
  static constexpr size_t lds_bytes() { return (size_t)NP * N * sizeof(v2f); }
  static_assert(Fft::lds_bytes() == (size_t)N * sizeof(v2f), "one plane");

  Fft fft;
  v2f* park;
  TileArgs a;
  int l, d, M;
  uint32_t loff, soff;
  const float* coef;
  float h[TP][PC];
  v2f xr[D][PC];
  v2f wait[NR][R];       // presums that wait in registers

  struct Batch {
    int m, lo, hi;       // first spectrum, blocks the batch reads
  };
  __device__ __forceinline__ Batch batch(int q, bool any) const {
    Batch t;
    t.m = q * B;
    t.lo = t.m > d ? t.m : d;
    const int ng = M - t.m < B ? M - t.m : B;
    t.hi = any ? t.m + ng + TP - 1 : t.m;
    return t;
  }
  // block k of the batch, channels of part p
  __device__ __forceinline__ void load(v2f (&dst)[PC], const Batch& t, int k, int p) const {
    const int vb = t.m + k;
    const bool ok = vb >= t.lo && vb < t.hi;
    const __amdgpu_buffer_rsrc_t rs = block_rsrc(block_addr<N, SB>(a, ok ? vb - d : 0), ok ? N * SB : 0);
#pragma unroll
    for (int c = 0; c < PC; ++c) {
      const uint32_t so = (uint32_t)((p * PC + c) * NT * SB);
      if constexpr (IT == 0) {
        dst[c] = buf_load<0>(rs, loff, so);
      } else if constexpr (IT == 1) {
        dst[c].x = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, loff, so, 0));
      } else {
        dst[c].x = __builtin_bit_cast(float, (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(rs, loff, so, 0));
      }
    }
  }
  __device__ __forceinline__ v2f widened(v2f s) const {
    if constexpr (IT == 0) return s;
    const uint32_t w = __builtin_bit_cast(uint32_t, s.x);
    return IT == 1 ? widen_c16(w) : widen_ci8(w);
  }
  // tap t of part p (buffer loads: one lane offset, scalar offsets)
  __device__ __forceinline__ void coefs(int t, int p) {
    const __amdgpu_buffer_rsrc_t rc = block_rsrc(coef, TP * N * 4);
#pragma unroll
    for (int c = 0; c < PC; ++c)
      h[t][c] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                              rc, (uint32_t)l * 4u, (uint32_t)((t * N + (p * PC + c) * NT) * 4), 0));
  }

  // coefficients and first blocks of a batch's first part
  __device__ __forceinline__ void begin(const Batch& t) {
#pragma unroll
    for (int s = 0; s < TP; ++s) coefs(s, 0);
#pragma unroll
    for (int k = 0; k < D; ++k) load(xr[k], t, k, 0);
  }

  template <int P>
  __device__ __forceinline__ void part(const Batch& t) {
    if constexpr (P < PARTS) {
      constexpr bool more = P + 1 < PARTS;
      v2f acc[B][PC];
#pragma unroll
      for (int k = 0; k < NB; ++k) {
        if (k < TP + B - 1) {
#pragma unroll
          for (int c = 0; c < PC; ++c) {
            const v2f x = widened(xr[k % D][c]);
#pragma unroll
            for (int b = 0; b < B; ++b) {
              const int s = k - b;
              if (s == 0) {
                acc[b][c].x = h[0][c] * x.x;
                acc[b][c].y = h[0][c] * x.y;
              } else if (s > 0 && s < TP) {
                acc[b][c].x = fmaf(h[s][c], x.x, acc[b][c].x);
                acc[b][c].y = fmaf(h[s][c], x.y, acc[b][c].y);
              }
            }
          }
        }
        if (k + D < NB) load(xr[k % D], t, k + D, P);
        else if (more) load(xr[k % D], t, k + D - NB, P + 1);
        if (more && k >= B - 1 && k < TP + B - 1) coefs(k - (B - 1), P + 1);
      }
      if constexpr (P == 0) __syncthreads();           // the last batch's transforms are done with the planes
#pragma unroll
      for (int c = 0; c < PC; ++c) {
#pragma unroll
        for (int b = 0; b < NP; ++b) park[b * N + (P * PC + c) * NT] = acc[b][c];   // read by this lane only
#pragma unroll
        for (int b = 0; b < NR; ++b) {
          // computed here: a sum used only under a condition below would be
          // moved there, with all the samples and coefficients it needs
          asm volatile("" : "+v"(acc[NP + b][c].x), "+v"(acc[NP + b][c].y));
          wait[b][P * PC + c] = acc[NP + b][c];
        }
      }
      part<P + 1>(t);
    }
  }

  __device__ __forceinline__ void run(const FusedParams& p, float* smem, int q0, int step, int q1) {
    l = threadIdx.x;
    d = p.d;
    M = p.M;
    coef = p.coef;
    a = TileArgs{p.x0, p.x1, p.x1, p.out, p.h0, p.h0};
    loff = (uint32_t)(l * SB);
    soff = (uint32_t)(l * (int)sizeof(v2f));
    park = (v2f*)smem + l;
    Batch t = batch(q0, true);
    begin(t);
    for (int q = q0; q < q1; q += step) {
      const Batch tn = batch(q + step, q + step < q1);
      // a fresh base per batch: its loads are the same for every batch and
      // would be hoisted out of the loop, all parts' at once
      asm volatile("" : "+s"(coef));
      part<0>(t);
      // the register twiddles live only through the transforms: a fresh base
      // keeps their loads here
      const v2f* tw = p.tw;
      asm volatile("" : "+s"(tw));
      fft.init(smem, 0, l, tw);
      const int ng = M - t.m < B ? M - t.m : B;
#pragma unroll
      for (int b = 0; b < B; ++b) {
        if (b == B - 1) begin(tn);   // under the last transform
        if (b < ng) {
          v2f v[1][R];
#pragma unroll
          for (int e = 0; e < R; ++e) v[0][e] = b < NP ? park[b * N + e * NT] : wait[b < NP ? 0 : b - NP][e];
          fft.run(v);
          const __amdgpu_buffer_rsrc_t rs = block_rsrc(a.out + (long long)(t.m + b) * N, N * (int)sizeof(v2f));
#pragma unroll
          for (int e = 0; e < R; ++e) buf_store<kAuxNt>(v[0][e], rs, soff, (uint32_t)(e * NT * (int)sizeof(v2f)));
        }
      }
      t = tn;
    }
  }
};

template <int N, int TP, int IT>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
ppf_large_kernel(FusedParams p) {
  using Eng = LargeEngine<N, TP, IT>;
  extern __shared__ float smem[];
  int q0, step, q1;
  if (!batch_range(p, Eng::B, q0, step, q1)) return;
  Eng eng;
  eng.run(p, smem, q0, step, q1);
}

template <int N, typename Eng>
hipError_t batched_launch(void (*kern)(FusedParams), const PlanDev& pd, const BatchArgs& a0, hipStream_t st) {
  static const int occ = [&] {
    KernelInfo ki{(const void*)kern, Eng::NT, 1, Eng::lds_bytes()};
    return occupancy(ki);
  }();
  for (long long s0 = 0; s0 < a0.M; s0 += kMaxLaunchSpectra) {
    const long long k = a0.M - s0 < kMaxLaunchSpectra ? a0.M - s0 : kMaxLaunchSpectra;
    const BatchArgs a = sub_batch(a0, N, Eng::SB, s0, k);
    const long long nb = (a.M + Eng::B - 1) / Eng::B;
    long long grid = (long long)device_cus() * occ;
    if (grid > nb) grid = nb;
    FusedParams p{};
    p.x0 = (const v2f*)a.x0;
    p.x1 = (const v2f*)a.x1;
    p.out = (v2f*)a.out;
    p.coef = pd.coef;
    p.tw = (const v2f*)pd.tw;
    p.h0 = (int)a.h0;
    p.M = (int)a.M;
    p.d = pd.TP - pd.T;
    p.nblocks = (int)grid;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(Eng::NT), Eng::lds_bytes(), st, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

typedef hipError_t (*BatchedFn)(const PlanDev&, const BatchArgs&, hipStream_t);

template <int IT>
hipError_t launch_4096(const PlanDev& pd, const BatchArgs& a, hipStream_t st) {
  return batched_launch<4096, BatchedEngine<IT>>(&ppf_batched_kernel<IT>, pd, a, st);
}
template <int N, int TP, int IT>
hipError_t launch_large(const PlanDev& pd, const BatchArgs& a, hipStream_t st) {
  return batched_launch<N, LargeEngine<N, TP, IT>>(&ppf_large_kernel<N, TP, IT>, pd, a, st);
}
template <int N, int IT>
BatchedFn large_fn(int TP) {
  switch (TP) {
    case 2: return &launch_large<N, 2, IT>;
    case 4: return &launch_large<N, 4, IT>;
    case 8: return &launch_large<N, 8, IT>;
    default: return nullptr;
  }
}
template <int IT>
BatchedFn batched_fn(int N, int TP) {
  switch (N) {
    case 4096: return TP == 16 ? &launch_4096<IT> : nullptr;
    case 8192: return large_fn<8192, IT>(TP);
    default: return nullptr;
  }
}

}  // namespace

// A batch takes the same time however many of the CUs have one, and two
// passes, spread over all CUs, take a time in proportion to the spectra.
// N = 4096: 33 us, and 24 us per 1000 spectra, so batches are faster where the
// last round of them leaves at most a third of the CUs without one (M = 1003:
// 34.7 us, two passes 29.9; M = 1500: 36.0, 41.3; M = 2003: 35.5, 52.4; int8 and
// FP16 input M = 1366: 33, 48).
// N = 8192: 30 to 38 us, and 62 us per 1000 spectra over some 12: from two
// fifths of a round on (M = 690: 36.8 us, two passes 56.7; M = 1023: 38.9,
// 73.3; M = 1370, two rounds: 71.5, 96.3). FP16 and int8 input with 5 to 8 taps
// take two passes in 41 us per 1000 spectra over 13: there the second and third
// rounds pay from a quarter full on (int8, T = 8: M = 1030 61.2 us, two passes 53.9;
// 1200 62.7, 57.9; 1300 62.9, 62.9; 1500 62.9, 66.3; M = 2100 92.5, 87.4; 2300 92.9,
// 91.5; later rounds M = 3080 120.3, 118.3; 3300 122.3, 146.5, as the presums
// then leave the cache). With up to 4 taps they pay as FP32 does (T = 4:
// M = 1060 53.2, 53.0).
bool batched_worth(int N, int TP, int in_type, long long M) {
  if (!batched_fn<0>(N, TP)) return false;
  const long long round = (N == 4096 ? 8ll : 4ll) * device_cus();
  const long long capacity = (M + round - 1) / round * round;
  if (N == 4096) return 3 * M >= 2 * capacity;
  if (in_type != 0 && TP == 8 && (capacity == 2 * round || capacity == 3 * round))
    return 4 * (M - (capacity - round)) >= round;
  return 5 * M >= 2 * capacity;
}

hipError_t launch_batched(const PlanDev& pd, const BatchArgs& a, hipStream_t st) {
  BatchedFn f = nullptr;
  switch (pd.in_type) {
    case 0: f = batched_fn<0>(pd.N, pd.TP); break;
    case 1: f = batched_fn<1>(pd.N, pd.TP); break;
    case 2: f = batched_fn<2>(pd.N, pd.TP); break;
  }
  if (!f) return hipErrorInvalidValue;
  return f(pd, a, st);
}

}  // namespace ppf
