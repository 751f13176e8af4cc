// Fused FIR + FFT for N = 4096 with 9 to 16 taps: one pass over HBM for a
// shape whose tap window (512 KiB) fits neither the registers nor the LDS of
// a CU.
//
// A workgroup computes a batch of B = 8 consecutive spectra at a time, and
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
// at 2^27: 0.445, 0.909). The FIR takes about 8 us of a batch's 33, bound by
// the VALU; the transforms, bound by VALU and LDS issue and their barriers,
// the rest. One transform at a time took 1.196 ms; twiddles from the global
// table 1.796; the next batch's coefficients loaded under the last
// transforms 1.139.

#include "ppf_engine.h"

namespace ppf {
namespace {

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

// Workgroup w runs on XCD w % 8 and is the w / 8th of it; an XCD takes a
// contiguous range of batches, its workgroups in turn, so that the batches
// running at once on it are neighbours.
template <int IT>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
ppf_batched_kernel(FusedParams p) {
  using Eng = BatchedEngine<IT>;
  extern __shared__ float smem[];
  const int nb = (p.M + Eng::B - 1) / Eng::B;
  const int xcds = p.nblocks < 8 ? p.nblocks : 8;
  const int x = (int)blockIdx.x % xcds, k = (int)blockIdx.x / xcds;
  const int per = (p.nblocks - x + xcds - 1) / xcds;         // workgroups of this XCD, after `before` of others
  const int before = x * (p.nblocks / xcds) + (x < p.nblocks % xcds ? x : p.nblocks % xcds);
  const int q0 = (int)((long long)nb * before / p.nblocks), q1 = (int)((long long)nb * (before + per) / p.nblocks);
  if (q0 + k >= q1) return;
  Eng eng;
  // group -k mod 3 first
  if (k % 3 == 0) eng.template run<0>(p, smem, q0 + k, per, q1);
  else if (k % 3 == 1) eng.template run<2>(p, smem, q0 + k, per, q1);
  else eng.template run<1>(p, smem, q0 + k, per, q1);
}

template <int IT>
hipError_t batched_launch(const PlanDev& pd, const BatchArgs& a0, hipStream_t st) {
  using Eng = BatchedEngine<IT>;
  auto kern = &ppf_batched_kernel<IT>;
  static const int occ = [&] {
    KernelInfo ki{(const void*)kern, Eng::NT, 1, Eng::lds_bytes()};
    return occupancy(ki);
  }();
  for (long long s0 = 0; s0 < a0.M; s0 += kMaxLaunchSpectra) {
    const long long k = a0.M - s0 < kMaxLaunchSpectra ? a0.M - s0 : kMaxLaunchSpectra;
    const BatchArgs a = sub_batch(a0, Eng::N, Eng::SB, s0, k);
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
    p.d = Eng::TP - pd.T;
    p.nblocks = (int)grid;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(Eng::NT), Eng::lds_bytes(), st, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

bool batched_available(int N, int TP) { return N == 4096 && TP == 16; }

// A batch takes 33 us however many of the CUs have one, and two passes, spread
// over all CUs, 24 us per 1000 spectra: batches are faster where the last
// round of them leaves at most a third of the CUs without one (M = 1003: 34.7
// us, two passes 29.9; M = 1500: 36.0, 41.3; M = 2003: 35.5, 52.4).
bool batched_worth(int N, int TP, long long M) {
  if (!batched_available(N, TP)) return false;
  const long long round = 8ll * device_cus();
  const long long capacity = (M + round - 1) / round * round;
  return 3 * M >= 2 * capacity;
}

hipError_t launch_batched(const PlanDev& pd, const BatchArgs& a, hipStream_t st) {
  switch (pd.in_type) {
    case 0: return batched_launch<0>(pd, a, st);
    case 1: return batched_launch<1>(pd, a, st);
    case 2: return batched_launch<2>(pd, a, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ppf
