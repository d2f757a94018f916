// select.hip - selection steps of Algorithm 1 (arXiv 2609.28053, Appendix C):
// the all-reduce stand-in (sum of the P partition slabs), the coarse choice
// u_e, rho_e (step 3), the fine choice v_e and b_hat_e = kappa^-1(u_e, v_e)
// (steps 5-6), and the centred bias of Eq. 2.
#include "eqb_internal.hpp"

namespace eqb {

// One block per expert (and, with kLocal, per partition), one thread per bin.
// Global: the P slabs are summed first (the all-reduce) and r is the rank over
// the whole batch.  kLocal: slab p alone, with its own rank
// r_p = ceil(|B_p| K / E), written to entry [p, e]; an empty partition has no
// quantile and gets -1 without raising the status.
// Layer form (eqb_layer): `clear` zeroes the summed counters once read, and
// the loads accumulated by the route kernel (load_acc [P,E]) are copied to
// load_out and zeroed, so the workspace is left as it was found: all zero.
// Each counter is read and cleared by the same thread.
// kSlab16 (the layer, global form): the P slabs hold 16-bit counters in the
// layout of PartTable::slab16; each is read, summed and cleared as a uint16.
// images > 0 (the layer): the counts of the window's bins come from that many
// block images at win as well.
template <bool kLocal, bool kSlab16 = false>
__global__ __launch_bounds__(kNBins) void select_coarse_kernel(
    int32_t* __restrict__ hist, int P, int E, int K, int64_t r, const PartTable pt,
    int32_t* __restrict__ sel_hi, int64_t* __restrict__ rank_in_bin, int32_t* __restrict__ hist_sum,
    int32_t* __restrict__ status, bool clear = false, int32_t* __restrict__ load_acc = nullptr,
    int32_t* __restrict__ load_out = nullptr, const uint32_t* __restrict__ win = nullptr, int images = 0) {
  __shared__ int64_t sh[kNBins];
  __shared__ uint32_t sh_win[kNBins / 64][kWinBins];
  const int e = blockIdx.x, u = threadIdx.x, p = kLocal ? (int)blockIdx.y : 0;
  const int64_t out = kLocal ? (int64_t)p * E + e : e;
  if (kLocal) {
    const int64_t n = pt.off[p + 1] - pt.off[p];
    if (n == 0) {
      if (u == 0) {
        sel_hi[out] = -1;
        rank_in_bin[out] = 0;
      }
      return;
    }
    r = (n * K + E - 1) / E;
  }
  int64_t c = 0;
  if (kLocal) {
    c = hist[((int64_t)p * E + e) * kNBins + u];
  } else {
    if (images > 0) {
      // thread u reads words 4 (u % 4) .. + 3 of the pair's row of images u / 4, + 64, ..
      const int half = (e & 1) * 16;
      const uint4* src = reinterpret_cast<const uint4*>(win + (int64_t)(e >> 1) * kWinBins) + (u & 3);
      const int64_t step = win_words(E) / 4;
      uint32_t s[4] = {0, 0, 0, 0};
      auto add = [&](const uint4& v) {
        s[0] += (v.x >> half) & 0xFFFFu;
        s[1] += (v.y >> half) & 0xFFFFu;
        s[2] += (v.z >> half) & 0xFFFFu;
        s[3] += (v.w >> half) & 0xFFFFu;
      };
      int i = u >> 2;
      for (; i + 192 < images; i += 256) {
        uint4 v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = src[(i + 64 * j) * step];
#pragma unroll
        for (int j = 0; j < 4; ++j) add(v[j]);
      }
      for (; i < images; i += 64) add(src[i * step]);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
#pragma unroll
        for (int d = 4; d < 64; d <<= 1) s[j] += __shfl_xor(s[j], d);
        if ((u & 63) < 4) sh_win[u >> 6][4 * (u & 3) + j] = s[j];
      }
      __syncthreads();
      const int w = win_place(raw_hi_of_kappa(u));
      if (w >= 0) {
#pragma unroll
        for (int j = 0; j < kNBins / 64; ++j) c += sh_win[j][w];
      }
    }
    if (kSlab16) {
      uint16_t* h16 = reinterpret_cast<uint16_t*>(hist) + ((int64_t)(e >> 1) * kNBins + u) * 2 + (e & 1);
      const int64_t stride = (int64_t)E * kNBins * 2;  // one int32 slab, in 16-bit units
      int q = 0;
      for (; q + 8 <= P; q += 8) {
        uint32_t v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = h16[(q + j) * stride];
#pragma unroll
        for (int j = 0; j < 8; ++j) c += v[j];
      }
      for (; q < P; ++q) c += h16[q * stride];
      if (clear)
        for (int q2 = 0; q2 < P; ++q2) h16[q2 * stride] = 0;
    } else {
      c += slab_sum(hist + (int64_t)e * kNBins + u, P, (int64_t)E * kNBins);
      if (clear) slab_clear(hist + (int64_t)e * kNBins + u, P, (int64_t)E * kNBins);
    }
    if (hist_sum) hist_sum[(int64_t)e * kNBins + u] = (int32_t)c;
    if (load_acc) {
      for (int q = u; q < pt.P; q += kNBins) {
        load_out[(int64_t)q * E + e] = load_acc[(int64_t)q * E + e];
        load_acc[(int64_t)q * E + e] = 0;
      }
    }
  }
  const int64_t cum = block_inclusive_scan_256(c, sh);
  if (cum >= r && cum - c < r) {
    sel_hi[out] = u;
    rank_in_bin[out] = r - (cum - c);
  }
  if (u == kNBins - 1 && cum < r) {
    sel_hi[out] = -1;
    rank_in_bin[out] = 0;
    if (status) *status = EQB_DEV_RANK_EXCEEDS_COUNT;
  }
}

// Binary64 sum of val[0..E) (E <= 256, 256 threads or more) in ascending
// order.  The values are BF16 numbers: 8 significant bits each, so while their
// exponents span at most 36 every partial sum in any order is below 2^(8 + 1 +
// emax) and a multiple of 2^(emin - 7), 53 bits at most: exact, and equal to the
// ascending sum.  Then the waves sum in parallel; a wider span (or a NaN) is
// summed one by one, 256 dependent additions.  The ascending sum begins with +0, which
// makes a sum of nothing but -0 +0; so does the last addition here.
__device__ __forceinline__ double ascending_sum(const double* val, int E, double* sh, int* shx) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (wave < 4) {
    double x = tid < E ? val[tid] : 0.0;
    // biased binary64 exponents; zeros do not count
    const int ex = (int)((__double_as_longlong(x) >> 52) & 0x7FF);
    int lo = x != 0.0 ? ex : 0x7FF, hi = x != 0.0 ? ex : 0;
    for (int d = 32; d > 0; d >>= 1) {
      x += __shfl_xor(x, d);
      lo = min(lo, __shfl_xor(lo, d));
      hi = max(hi, __shfl_xor(hi, d));
    }
    if (lane == 0) {
      sh[wave] = x;
      shx[2 * wave] = lo;
      shx[2 * wave + 1] = hi;
    }
  }
  __syncthreads();
  const int lo = min(min(shx[0], shx[2]), min(shx[4], shx[6]));
  const int hi = max(max(shx[1], shx[3]), max(shx[5], shx[7]));
  if (hi - lo <= 36) return 0.0 + (((sh[0] + sh[1]) + sh[2]) + sh[3]);
  double acc = 0.0;
  for (int e = 0; e < E; ++e) acc += val[e];
  return acc;
}

// b = b_hat - mean(b_hat) (Eq. 2): the binary64 sum in ascending expert order
// divided by E, the difference in binary64, one rounding to binary32.  Called
// by every thread of a block of at least 256, thread e < E with b_hat_e.
__device__ __forceinline__ void center_block(uint32_t q, int E, float* b_next) {
  __shared__ double val[256], sh_sum[4];
  __shared__ int sh_exp[8];
  const int e = threadIdx.x;
  if (e < E) val[e] = (double)__uint_as_float(q << 16);
  __syncthreads();
  const double mean = ascending_sum(val, E, sh_sum, sh_exp) / (double)E;
  if (e < E) b_next[e] = (float)(val[e] - mean);
}

__global__ __launch_bounds__(256) void center_kernel(const uint16_t* __restrict__ q, int E,
                                                     float* __restrict__ b_next) {
  center_block(threadIdx.x < E ? q[threadIdx.x] : 0u, E, b_next);
}

// The end of a layer's fine selection: the last of its blocks to finish centres
// the bias and writes the status (an expert whose selection failed holds fewer
// counts than its rank).  A launch of its own for that took 4 to 5 us of every
// layer.  No block waits for another: each adds itself to the ticket, and the
// one that completes the count goes on.
// The blocks sit on XCDs with an L2 each.  Only b_hat passes between them, in
// agent-scope stores and loads that go past the L2s: the stores have completed
// (vmcnt) before the block's ticket is drawn.  A release and an acquire fence
// instead would write back and invalidate a whole L2 in each of the E/2 blocks
// (70.9 us per layer of 147,456 tokens, E = 256).  Everything else a block
// leaves behind, it writes alone.
struct LayerTail {
  int32_t* ticket = nullptr;   // zero before and after: finished blocks, failed ones counted above bit 16
  float* b_next = nullptr;
  int32_t* status = nullptr;
};

__device__ __forceinline__ void store_bhat(uint16_t* q, uint16_t bits) {
  __hip_atomic_store(q, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void layer_tail(const LayerTail& tail, bool failed, uint16_t* q, int E) {
  __shared__ int sh_n;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  const int bad = __syncthreads_or((int)failed) ? 1 << 16 : 0;
  if (threadIdx.x == 0)
    sh_n = bad + 1 + __hip_atomic_fetch_add(tail.ticket, bad + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  const int n = sh_n;
  if ((n & 0xFFFF) != (int)gridDim.x) return;
  if (threadIdx.x == 0) {
    __hip_atomic_store(tail.ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *tail.status = (n >> 16) ? EQB_DEV_RANK_EXCEEDS_COUNT : EQB_DEV_OK;
  }
  const int e = threadIdx.x;
  center_block(e < E ? __hip_atomic_load(q + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u, E, tail.b_next);
}

// Layer form (kTail): `hist` is cleared once summed, the selections read are
// zeroed (sel_lo is not written: it stays zero), and layer_tail follows.
template <bool kLocal, bool kTail = false>
__global__ __launch_bounds__(kNBins) void select_fine_kernel(
    int32_t* __restrict__ hist, int P, int E, const PartTable pt, int32_t* __restrict__ sel_hi,
    int64_t* __restrict__ rank_in_bin, int32_t* __restrict__ sel_lo, uint16_t* __restrict__ q_bf16,
    int32_t* __restrict__ hist_sum, int32_t* __restrict__ status, const LayerTail tail = LayerTail{}) {
  __shared__ int64_t sh[kNBins];
  const int e = blockIdx.x, v = threadIdx.x, p = kLocal ? (int)blockIdx.y : 0;
  const int64_t out = kLocal ? (int64_t)p * E + e : e;
  if (kLocal && pt.off[p + 1] == pt.off[p]) {
    if (v == 0) {
      sel_lo[out] = -1;
      q_bf16[out] = 0x7FC0;
    }
    return;
  }
  // the coarse choice is read first: its load overlaps those of the counts
  const int u = sel_hi[out];
  const int64_t rho = rank_in_bin[out];
  int64_t c = 0;
  if (kLocal) {
    c = hist[((int64_t)p * E + e) * kNBins + v];
  } else {
    c = slab_sum(hist + (int64_t)e * kNBins + v, P, (int64_t)E * kNBins);
    if (hist_sum) hist_sum[(int64_t)e * kNBins + v] = (int32_t)c;
    if (kTail) slab_clear(hist + (int64_t)e * kNBins + v, P, (int64_t)E * kNBins);
  }
  const int64_t cum = block_inclusive_scan_256(c, sh);
  const bool ok = u >= 0 && u < kNBins && rho >= 1;
  const bool failed = v == kNBins - 1 && (!ok || cum < rho);
  if (ok && cum >= rho && cum - c < rho) {
    const uint16_t bits = kappa_inv(((uint32_t)u << 8) | (uint32_t)v);
    if (kTail) {
      store_bhat(q_bf16 + out, bits);
    } else {
      sel_lo[out] = v;
      q_bf16[out] = bits;
    }
  }
  if (failed) {
    if (kTail) {
      store_bhat(q_bf16 + out, 0x7FC0);
    } else {
      sel_lo[out] = -1;
      q_bf16[out] = 0x7FC0;
      if (status) *status = EQB_DEV_RANK_EXCEEDS_COUNT;
    }
  }
  if (kTail) {
    if (v == 0) {                  // every thread read them before the scan's barrier
      sel_hi[out] = 0;
      rank_in_bin[out] = 0;
    }
    layer_tail(tail, failed, q_bf16, E);
  }
}

// The fine selection of a layer from the fine pass's per-block count images
// (steps 5-6 of Algorithm 1 with the all-reduce stand-in summing the images
// instead of partition slabs).  One block per expert pair (2m, 2m+1), 512
// threads: each wave sums every eighth image's row for the pair (one
// 16-byte load per lane: raw low bytes 4l..4l+3 of both experts), the waves'
// sums meet in LDS, and threads 256x + v then hold kappa bin v of expert
// 2m + x: raw low byte v, or v ^ 0xFF when the expert's selected coarse bin
// holds negative margins (kappa flips every bit of a negative value).  The
// scan and the choice are those of select_fine_kernel.  Image counts are
// below 2^16 and the sums below 2^31 (T < 2^31).
constexpr int kPartThreads = 512;
__global__ __launch_bounds__(kPartThreads) void select_fine_parts_kernel(
    const uint32_t* __restrict__ part, int nparts, int E, int32_t* __restrict__ sel_hi,
    int64_t* __restrict__ rank_in_bin, uint16_t* __restrict__ q_bf16, int32_t* __restrict__ hist_sum,
    const LayerTail tail) {
  constexpr int kW = kPartThreads / 64;
  __shared__ uint32_t sh[kW][2 * kNBins];   // per wave: raw bins of expert 2m, then of 2m+1
  __shared__ int sh_tot[kW];
  const int m = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t words = part_words(E);
  const uint4* src = reinterpret_cast<const uint4*>(part + (int64_t)m * kNBins) + lane;
  uint32_t lo[4] = {0, 0, 0, 0}, hi[4] = {0, 0, 0, 0};
  int b = wave;
  for (; b + 3 * kW < nparts; b += 4 * kW) {
    uint4 v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = src[(b + j * kW) * words / 4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t w[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        lo[i] += w[i] & 0xFFFFu;
        hi[i] += w[i] >> 16;
      }
    }
  }
  for (; b < nparts; b += kW) {
    const uint4 v = src[b * words / 4];
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      lo[i] += w[i] & 0xFFFFu;
      hi[i] += w[i] >> 16;
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    sh[wave][4 * lane + i] = lo[i];
    sh[wave][kNBins + 4 * lane + i] = hi[i];
  }
  __syncthreads();
  const int x = threadIdx.x >> 8, v = threadIdx.x & (kNBins - 1);
  const int e = 2 * m + x;
  const int u = sel_hi[e];
  const int64_t rho = rank_in_bin[e];
  const bool ok = u >= 0 && u < kNBins && rho >= 1;
  const bool valid_u = u >= 0 && u < kNBins;
  const int raw = (valid_u && u < 0x80) ? (v ^ 0xFF) : v;
  int c = 0;
#pragma unroll
  for (int w = 0; w < kW; ++w) c += (int)sh[w][x * kNBins + raw];
  // the fine pass counted an expert without a valid coarse choice in bin 0;
  // like the slab flush, the selection drops those counts
  if (!valid_u) c = 0;
  if (hist_sum) hist_sum[(int64_t)e * kNBins + v] = c;
  // inclusive scan over the 256 threads of expert x (waves 4x .. 4x+3)
  int y = c;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int t = __shfl_up(y, d);
    if (lane >= d) y += t;
  }
  if (lane == 63) sh_tot[wave] = y;
  __syncthreads();
  for (int w = 4 * x; w < wave; ++w) y += sh_tot[w];
  const int64_t cum = y;
  const bool failed = v == kNBins - 1 && (!ok || cum < rho);
  if (ok && cum >= rho && cum - c < rho) store_bhat(q_bf16 + e, kappa_inv(((uint32_t)u << 8) | (uint32_t)v));
  if (failed) store_bhat(q_bf16 + e, 0x7FC0);
  if (v == 0) {                    // every thread read them before the scan's barrier
    sel_hi[e] = 0;
    rank_in_bin[e] = 0;
  }
  layer_tail(tail, failed, q_bf16, E);
}

// The layer's selections: the counts sit in P * nsub slabs, all summed; the
// loads in P rows.
eqb_status launch_layer_selects(int pass, int32_t* hist, int P, int nsub, int E, int64_t r, int32_t* sel_hi,
                                int64_t* rank_in_bin, uint16_t* q_bf16, float* b_next,
                                int32_t* hist_sum, int32_t* load_acc, int32_t* load_out, int32_t* status,
                                int32_t* ticket, hipStream_t s, RouteForm form, const uint32_t* win) {
  PartTable none{};
  none.P = P;
  const int nslabs = pass == 1 ? form.slabs : P * nsub;
  if (pass == 1) {
    if (form.slab16)
      select_coarse_kernel<false, true><<<E, kNBins, 0, s>>>(hist, nslabs, E, 0, r, none, sel_hi, rank_in_bin,
                                                             hist_sum, nullptr, true, load_acc, load_out, win,
                                                             form.images);
    else
      select_coarse_kernel<false><<<E, kNBins, 0, s>>>(hist, nslabs, E, 0, r, none, sel_hi, rank_in_bin, hist_sum,
                                                       nullptr, true, load_acc, load_out, win, form.images);
    return launch_status();
  }
  select_fine_kernel<false, true><<<E, kNBins, 0, s>>>(hist, nslabs, E, none, sel_hi, rank_in_bin, nullptr, q_bf16,
                                                       hist_sum, nullptr, LayerTail{ticket, b_next, status});
  return launch_status();
}

eqb_status launch_layer_select_parts(const uint32_t* part, int nparts, int E, int32_t* sel_hi,
                                     int64_t* rank_in_bin, uint16_t* q_bf16, float* b_next,
                                     int32_t* hist_sum, int32_t* status, int32_t* ticket, hipStream_t s) {
  select_fine_parts_kernel<<<E / 2, kPartThreads, 0, s>>>(part, nparts, E, sel_hi, rank_in_bin, q_bf16, hist_sum,
                                                          LayerTail{ticket, b_next, status});
  return launch_status();
}

static eqb_status mark(void* const* marks, int i, hipStream_t s) {
  if (marks == nullptr || marks[i] == nullptr) return EQB_OK;
  return hipEventRecord(static_cast<hipEvent_t>(marks[i]), s) == hipSuccess ? EQB_OK : EQB_ERR_HIP;
}

eqb_status launch_layer(const RouteArgs& route, int64_t r, const LayerWorkspace& w, uint16_t* q_bf16,
                        float* b_next, int32_t* load_out, int32_t* hist_hi_sum, int32_t* hist_lo_sum,
                        int32_t* dev_status, void* const* marks, hipStream_t s) {
  RouteArgs a = route;
  a.load = w.load_acc;
  a.hist = w.hist_hi;
  a.pt.nsub = w.nsub;
  a.slab16_ok = true;
  eqb_status st = mark(marks, 0, s);
  if (st != EQB_OK) return st;
  a.win = w.part;                   // consumed before the fine pass stores its images there
  a.win_blocks = w.part_blocks;
  RouteForm form;
  st = launch_route(a, s, &form);
  if (st != EQB_OK) return st;
  if ((st = mark(marks, 1, s)) != EQB_OK) return st;
  const int P = a.pt.P, E = a.E;
  st = launch_layer_selects(1, w.hist_hi, P, w.nsub, E, r, w.sel_hi, w.rank_in_bin, nullptr, nullptr,
                            hist_hi_sum, w.load_acc, load_out, nullptr, nullptr, s, form, w.part);
  if (st != EQB_OK) return st;
  if ((st = mark(marks, 2, s)) != EQB_OK) return st;
  MarginArgs m;
  m.z = a.z;
  m.tau = a.tau;
  m.T = a.T;
  m.E = E;
  m.sel_hi = w.sel_hi;
  m.hist = w.hist_lo;
  m.pt = a.pt;
  m.part = w.part;
  m.part_blocks = w.part_blocks;
  int nparts = 0;
  st = launch_margin(true, m, s, &nparts);
  if (st != EQB_OK) return st;
  if ((st = mark(marks, 3, s)) != EQB_OK) return st;
  if (nparts > 0)
    st = launch_layer_select_parts(w.part, nparts, E, w.sel_hi, w.rank_in_bin, q_bf16, b_next,
                                   hist_lo_sum, dev_status, w.tickets, s);
  else
    st = launch_layer_selects(2, w.hist_lo, P, w.nsub, E, r, w.sel_hi, w.rank_in_bin, q_bf16, b_next,
                              hist_lo_sum, nullptr, nullptr, dev_status, w.tickets, s);
  if (st != EQB_OK) return st;
  return mark(marks, 4, s);
}

eqb_status launch_select(int pass, const int32_t* hist, int P, int E, int64_t r, int32_t* sel_hi,
                         int64_t* rank_in_bin, int32_t* sel_lo, uint16_t* q_bf16, float* b_next,
                         int32_t* hist_sum, int32_t* status, hipStream_t s) {
  PartTable none{};
  none.P = P;
  if (pass == 1) {
    select_coarse_kernel<false><<<E, kNBins, 0, s>>>(const_cast<int32_t*>(hist), P, E, 0, r, none, sel_hi,
                                                     rank_in_bin, hist_sum, status);
    return launch_status();
  }
  select_fine_kernel<false><<<E, kNBins, 0, s>>>(const_cast<int32_t*>(hist), P, E, none, sel_hi, rank_in_bin,
                                                 sel_lo, q_bf16, hist_sum, status);
  if (launch_status() != EQB_OK) return EQB_ERR_HIP;
  if (b_next) {
    center_kernel<<<1, 256, 0, s>>>(q_bf16, E, b_next);
    return launch_status();
  }
  return EQB_OK;
}

eqb_status launch_select_local(int pass, const int32_t* hist, int E, int K, const PartTable& pt,
                               int32_t* sel_hi, int64_t* rank_in_bin, int32_t* sel_lo, uint16_t* q_bf16,
                               int32_t* status, hipStream_t s) {
  const dim3 grid(E, pt.P);
  if (pass == 1)
    select_coarse_kernel<true><<<grid, kNBins, 0, s>>>(const_cast<int32_t*>(hist), pt.P, E, K, 0, pt, sel_hi,
                                                       rank_in_bin, nullptr, status);
  else
    select_fine_kernel<true><<<grid, kNBins, 0, s>>>(const_cast<int32_t*>(hist), pt.P, E, pt, sel_hi,
                                                     rank_in_bin, sel_lo, q_bf16, nullptr, status);
  return launch_status();
}

}  // namespace eqb
