// balance.hip - load-balance quantities computed from the expert loads:
// MaxVio (arXiv 2609.28053, Sec. 5 and Appendix E, "Balance metrics") and
// Load-Error Injection (Sec. 4, Eq. lei and its normalisation).
#include "eqb_internal.hpp"

namespace eqb {

// Maximum of f over the block (every thread receives it): within each wave,
// then over the waves.
__device__ __forceinline__ int64_t block_max_i64(int64_t f, int64_t* sh) {
  for (int off = 32; off > 0; off >>= 1) {
    const int64_t o = (int64_t)__shfl_xor((unsigned long long)f, off);
    f = o > f ? o : f;
  }
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = f;
  __syncthreads();
  int64_t m = sh[0];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w) m = sh[w] > m ? sh[w] : m;
  __syncthreads();
  return m;
}

// MaxVio = (max_e f_e) * E / (K * |B|) - 1 in binary64: the integer maximum
// is exact, the division and the subtraction round once each; NaN for an
// empty batch.
__device__ __forceinline__ double maxvio_of(int64_t m, int E, int K, int64_t n) {
  return n > 0 ? (double)(m * E) / ((double)K * (double)n) - 1.0 : __builtin_nan("");
}

// Block p < P: partition p alone; block P: the whole batch (loads summed over
// the partitions) and, with out_local_mean, the mean of the partitions'
// values over the non-empty partitions (Appendix E: Local MaxVio is computed
// per local batch and then averaged), a binary64 sum in ascending partition
// order divided by their number.
__global__ __launch_bounds__(kNBins) void max_violation_kernel(
    const int32_t* __restrict__ load, int E, int K, const PartTable pt,
    double* __restrict__ out_global, double* __restrict__ out_local, double* __restrict__ out_local_mean) {
  __shared__ int64_t sh_max[kNBins / 64];
  const int p = blockIdx.x;
  const int e = threadIdx.x;
  int64_t f = 0;
  if (e < E) {
    if (p < pt.P) {
      f = load[(int64_t)p * E + e];
    } else {
      for (int q = 0; q < pt.P; ++q) f += load[(int64_t)q * E + e];
    }
  }
  const int64_t m = block_max_i64(f, sh_max);
  const int64_t n = (p < pt.P) ? pt.off[p + 1] - pt.off[p] : pt.off[pt.P];
  if (p < pt.P) {
    if (e == 0 && out_local) out_local[p] = maxvio_of(m, E, K, n);
    return;
  }
  if (e == 0) *out_global = maxvio_of(m, E, K, n);
  if (out_local_mean == nullptr) return;
  double acc = 0.0;
  int count = 0;
  for (int q = 0; q < pt.P; ++q) {
    const int64_t nq = pt.off[q + 1] - pt.off[q];
    if (nq == 0) continue;            // block-uniform
    const int64_t mq = block_max_i64(e < E ? (int64_t)load[(int64_t)q * E + e] : 0, sh_max);
    acc += maxvio_of(mq, E, K, nq);
    ++count;
  }
  if (e == 0) *out_local_mean = count > 0 ? acc / (double)count : __builtin_nan("");
}

eqb_status launch_max_violation(const int32_t* load, int E, int K, const PartTable& pt,
                                double* out_global, double* out_local, double* out_local_mean, hipStream_t s) {
  max_violation_kernel<<<pt.P + 1, kNBins, 0, s>>>(load, E, K, pt, out_global, out_local, out_local_mean);
  return launch_status();
}

// ------------------------------------------------- Load-Error Injection --
// Block p: rho_e = f_{p,e} E / (K |B_p|) - 1 in binary64; with c > 0 the
// shared scale tanh(xi)/xi, xi = max_e |rho_e| / c (1 at xi = 0); the value
// injected into every score gradient of partition p is eta * (rho_e * scale),
// rounded once to binary32.  An empty partition injects 0.
__global__ __launch_bounds__(kNBins) void lei_residual_kernel(
    const int32_t* __restrict__ load, int E, int K, const PartTable pt, double eta, double c,
    float* __restrict__ inj) {
  __shared__ double sh_max[kNBins / 64];
  const int p = blockIdx.x;
  const int e = threadIdx.x;
  const int64_t n = pt.off[p + 1] - pt.off[p];
  double rho = 0.0;
  if (e < E && n > 0) rho = (double)((int64_t)load[(int64_t)p * E + e] * E) / ((double)K * (double)n) - 1.0;
  double a = fabs(rho);
  for (int off = 32; off > 0; off >>= 1) a = fmax(a, __shfl_xor(a, off));
  if ((e & 63) == 0) sh_max[e >> 6] = a;
  __syncthreads();
  double m = sh_max[0];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w) m = fmax(m, sh_max[w]);
  double scale = 1.0;
  if (c > 0.0) {
    const double xi = m / c;
    if (xi > 0.0) scale = tanh(xi) / xi;
  }
  if (e < E) inj[(int64_t)p * E + e] = n > 0 ? (float)(eta * (rho * scale)) : 0.0f;
}

// grad_s[t,e] += inj[p(t),e], one binary32 addition per score.  G = E/4
// lanes cover a row with one 16-byte access each; every lane handles kLeiU
// rows per step, so that many loads are in flight before the first store.
constexpr int kLeiU = 4;

template <int E>
__global__ __launch_bounds__(kBlock) void lei_inject_kernel(
    float* __restrict__ grad, const float* __restrict__ inj, int64_t T, const PartTable pt,
    int64_t rows_per_block) {
  constexpr int G = E / 4;
  constexpr int R = 64 / G;
  constexpr int ROWS = kWaves * R * kLeiU;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane % G, rr = lane / G;
  int64_t r0, r1;
  block_rows(T, rows_per_block, &r0, &r1);
  for_each_segment(r0, r1, pt, [&](int p, int64_t s0, int64_t s1) {
    const float4 d = *reinterpret_cast<const float4*>(inj + (int64_t)p * E + g * 4);
    for (int64_t base = s0; base < s1; base += ROWS) {
      float4 v[kLeiU];
#pragma unroll
      for (int u = 0; u < kLeiU; ++u) {
        const int64_t t = base + (int64_t)(u * kWaves + wave) * R + rr;
        if (t < s1) v[u] = *reinterpret_cast<const float4*>(grad + t * E + g * 4);
      }
#pragma unroll
      for (int u = 0; u < kLeiU; ++u) {
        const int64_t t = base + (int64_t)(u * kWaves + wave) * R + rr;
        if (t < s1) {
          const float4 o = make_float4(v[u].x + d.x, v[u].y + d.y, v[u].z + d.z, v[u].w + d.w);
          *reinterpret_cast<float4*>(grad + t * E + g * 4) = o;
        }
      }
    }
  });
}

// ------------------------------------- router backward with LEI ---------
// grad_z[t,e] = (g[t,e] + inj[p(t),e]) * sigmoid'(z[t,e]), where g[t,e] is
// grad_score[t,k] for e = topk_idx[t,k] and 0 for the other experts.  G = E/4
// lanes hold a row, 4 experts each, and every lane works on kBwdU rows per
// step: each load of z, store of grad_z and LDS read of a wave is then of
// consecutive bytes (512, 1,024 and 1,024) at every E.  The K mixture gradients
// of a row are scattered into a per-wave LDS row of zeros, read back 4 at a time,
// and their places zeroed again.  With K <= G lane g of a row owns pair k = g,
// and the next step's logits and pairs are loaded while a step is processed; a
// larger K reads its pairs inside the step.
//
// Bound by memory: 2E + 8K bytes read and 4E written per row.  The kernel took
// 86 VGPRs, so that only one of the two 1,024-thread blocks per CU of its grid
// ran at a time, and about 30 instructions per logit for sigmoid'.  Offsets of
// 32 bits from the segment's bases bring it under 64 VGPRs, eight waves per
// SIMD, in blocks of 512 threads.  Non-temporal loads and stores (a pass reads
// and writes each byte once) pay once both are of whole lines.  With the
// residual's launch, before -> after: E = 256, 147,456 rows 63.7 -> 48.4 us;
// E = 128, 1,000,003 rows, K = 8 191 -> 157 (5.3 TB/s); E = 64, 300,001 rows,
// K = 16 53.7 -> 29.7; E = 16, 4,000,001 rows 108 -> 88.  Four rows per step
// spill at 64 VGPRs (168 us at E = 128), two take 159; six waves per SIMD 175;
// plain stores 172 to 182.
constexpr int kBwdU = 3;
constexpr int kBwdBlock = 512, kBwdWaves = kBwdBlock / 64;
constexpr int kBwdBlocksPerCu = 2048 / kBwdBlock;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int E, bool kOnePair>
__global__ __launch_bounds__(kBwdBlock, 8) void lei_router_backward_kernel(
    const uint16_t* __restrict__ z, const int32_t* __restrict__ topk_idx, const float* __restrict__ grad_score,
    const float* __restrict__ inj, int64_t T, int K, float* __restrict__ grad_z, const PartTable pt,
    int64_t rows_per_block) {
  constexpr int G = E / 4;
  constexpr int R = 64 / G;
  constexpr uint32_t ROWS = kBwdWaves * R * kBwdU;
  __shared__ __align__(16) float sh_g[kBwdWaves][kBwdU][R][E];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane % G, rr = lane / G;
  float* my = &sh_g[wave][0][rr][0];      // row u of this lane: my + u * R * E
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  auto place = [&](int u) -> f32x4& { return *reinterpret_cast<f32x4*>(my + u * R * E + 4 * g); };
#pragma unroll
  for (int u = 0; u < kBwdU; ++u) place(u) = zero;
  lds_wave_sync();
  int64_t r0, r1;
  block_rows(T, rows_per_block, &r0, &r1);
  for_each_segment(r0, r1, pt, [&](int p, int64_t s0, int64_t s1) {
    // a segment holds at most kSegMax rows: 32-bit byte offsets from its bases
    const int64_t su = wave_uniform(s0);
    const uint16_t* seg_z = z + su * E;
    const int32_t* seg_idx = topk_idx + su * K;
    const float* seg_gs = grad_score + su * K;
    float* seg_gz = grad_z + su * E;
    const uint32_t n = (uint32_t)(s1 - s0);
    f32x4 d = zero;
    if (inj) {
      const float* di = inj + wave_uniform((int64_t)p * E);
      uint32_t o = 16u * g;
      asm volatile("" : "+v"(o));
      d = f32x4{at<const float>(di, o), at<const float>(di, o + 4), at<const float>(di, o + 8), at<const float>(di, o + 12)};
    }
    auto row_of = [&](uint32_t base, int u) -> uint32_t { return base + (uint32_t)((wave * kBwdU + u) * R + rr); };
    // logits and this lane's pair of its rows at step base
    auto load = [&](uint32_t base, u32x2 (&zw)[kBwdU], int (&e)[kBwdU], float (&gv)[kBwdU]) {
#pragma unroll
      for (int u = 0; u < kBwdU; ++u) {
        const uint32_t t = row_of(base, u);
        zw[u] = u32x2{0, 0};
        e[u] = -1;
        gv[u] = 0.0f;
        if (t < n) {
          zw[u] = __builtin_nontemporal_load(&at<const u32x2>(seg_z, (t * E + 4 * g) * 2u));
          if (kOnePair && g < K) {
            e[u] = at<const int32_t>(seg_idx, (t * K + g) * 4u);
            gv[u] = at<const float>(seg_gs, (t * K + g) * 4u);
          }
        }
      }
    };
    u32x2 zn[kBwdU];
    int en[kBwdU];
    float gn[kBwdU];
    // opaque: the first step's lane offsets, formed here rather than kept (as 64-bit
    // addresses) in registers across the segments
    uint32_t first = 0;
    asm volatile("" : "+s"(first));
    load(first, zn, en, gn);
    for (uint32_t base = first; base < n; base += ROWS) {
      u32x2 zw[kBwdU];
      int ec[kBwdU];
      float gc[kBwdU];
#pragma unroll
      for (int u = 0; u < kBwdU; ++u) {
        zw[u] = zn[u];
        ec[u] = en[u];
        gc[u] = gn[u];
      }
      if (base + ROWS < n) load(base + ROWS, zn, en, gn);
      // Logits of 32 or more take a longer form, chosen per wave and step, so that the
      // usual step has 12 instructions per sigmoid'.  Both work from the registers: with
      // one logit in a hundred above 32, 1,000,003 rows of E = 128, K = 8 take 158.1 us,
      // and 155.1 without any (computing such logits again from memory one by one, after
      // the stores, took 402; normal logits of deviation 64, most steps: 592 -> 158).
      float zmax = 0.0f;
#pragma unroll
      for (int u = 0; u < kBwdU; ++u)
        zmax = max3_abs(max3_abs(zmax, bf16_lo(zw[u].x), bf16_hi(zw[u].x)), bf16_lo(zw[u].y), bf16_hi(zw[u].y));
      const bool large = __any(zmax >= kSigmoidMax);
      // scatter the rows' mixture gradients
#pragma unroll
      for (int u = 0; u < kBwdU; ++u) {
        const uint32_t t = row_of(base, u);
        if (kOnePair) {
          if (ec[u] >= 0 && ec[u] < E) my[u * R * E + ec[u]] = gc[u];
        } else if (t < n) {
          for (int k = g; k < K; k += G) {
            const int e = at<const int32_t>(seg_idx, (t * K + k) * 4u);
            if (e >= 0 && e < E) my[u * R * E + e] = at<const float>(seg_gs, (t * K + k) * 4u);
          }
        }
      }
      lds_wave_sync();
      auto write = [&](auto wide) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kBwdU; ++u) {
          const uint32_t t = row_of(base, u);
          uint32_t w0 = zw[u].x, w1 = zw[u].y;
          // nothing of the usual form is kept, and no row begun before the last is stored: registers
          if (decltype(wide)::value) asm volatile("" : "+v"(w0), "+v"(w1)::"memory");
          const f32x4 gm = place(u);
          const float zf[4] = {bf16_lo(w0), bf16_hi(w0), bf16_lo(w1), bf16_hi(w1)};
          f32x4 o;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            o[j] = (gm[j] + d[j]) * sigmoid_prime_bf16<decltype(wide)::value>(zf[j]);
            if (decltype(wide)::value) __builtin_amdgcn_sched_barrier(0);
          }
          if (t < n) {
            __builtin_nontemporal_store(o, &at<f32x4>(seg_gz, (t * E + 4 * g) * 4u));
            // keeps the compiler from sinking the ends of both forms into one block
            if (decltype(wide)::value) asm volatile("; large logits");
            else asm volatile("; usual logits");
          }
        }
      };
      if (__builtin_expect(large, 0)) write(std::true_type{});
      else write(std::false_type{});
      if (kOnePair) lds_wave_sync();   // every place has been read
#pragma unroll
      for (int u = 0; u < kBwdU; ++u) {
        if (!kOnePair) place(u) = zero;
        else if (ec[u] >= 0 && ec[u] < E) my[u * R * E + ec[u]] = 0.0f;
      }
      lds_wave_sync();          // the next step scatters into zeros
    }
  });
}

template <int E>
static void launch_backward_e(const uint16_t* z, const int32_t* idx, const float* gs, const float* inj, int64_t T,
                              int K, float* gz, const PartTable& pt, hipStream_t s) {
  int blocks;
  int64_t rpb;
  grid_for(T, kBwdWaves * (256 / E) * kBwdU, kBwdBlocksPerCu, &blocks, &rpb);
  if (K <= E / 4)
    lei_router_backward_kernel<E, true><<<blocks, kBwdBlock, 0, s>>>(z, idx, gs, inj, T, K, gz, pt, rpb);
  else
    lei_router_backward_kernel<E, false><<<blocks, kBwdBlock, 0, s>>>(z, idx, gs, inj, T, K, gz, pt, rpb);
}

eqb_status launch_lei_router_backward(const uint16_t* z, const int32_t* idx, const float* gs, const float* inj,
                                      int64_t T, int E, int K, float* gz, const PartTable& pt, hipStream_t s) {
  switch (E) {
    case 8: launch_backward_e<8>(z, idx, gs, inj, T, K, gz, pt, s); break;
    case 16: launch_backward_e<16>(z, idx, gs, inj, T, K, gz, pt, s); break;
    case 32: launch_backward_e<32>(z, idx, gs, inj, T, K, gz, pt, s); break;
    case 64: launch_backward_e<64>(z, idx, gs, inj, T, K, gz, pt, s); break;
    case 128: launch_backward_e<128>(z, idx, gs, inj, T, K, gz, pt, s); break;
    case 256: launch_backward_e<256>(z, idx, gs, inj, T, K, gz, pt, s); break;
    default: return EQB_ERR_UNSUPPORTED;
  }
  return launch_status();
}

eqb_status launch_lei_residual(const int32_t* load, int E, int K, const PartTable& pt, double eta,
                               double c, float* inj, hipStream_t s) {
  lei_residual_kernel<<<pt.P, kNBins, 0, s>>>(load, E, K, pt, eta, c, inj);
  return launch_status();
}

template <int E>
static void launch_inject_e(float* grad, const float* inj, int64_t T, const PartTable& pt, hipStream_t s) {
  int blocks;
  int64_t rpb;
  grid_for(T, kWaves * (64 / (E / 4)) * kLeiU, 2, &blocks, &rpb);
  lei_inject_kernel<E><<<blocks, kBlock, 0, s>>>(grad, inj, T, pt, rpb);
}

eqb_status launch_lei_inject(float* grad, const float* inj, int64_t T, int E, const PartTable& pt,
                             hipStream_t s) {
  switch (E) {
    case 8: launch_inject_e<8>(grad, inj, T, pt, s); break;
    case 16: launch_inject_e<16>(grad, inj, T, pt, s); break;
    case 32: launch_inject_e<32>(grad, inj, T, pt, s); break;
    case 64: launch_inject_e<64>(grad, inj, T, pt, s); break;
    case 128: launch_inject_e<128>(grad, inj, T, pt, s); break;
    case 256: launch_inject_e<256>(grad, inj, T, pt, s); break;
    default: return EQB_ERR_UNSUPPORTED;
  }
  return launch_status();
}

}  // namespace eqb
