// route.hip - Top-K routing of z + b, cutoff tau, sigmoid scores, expert
// loads, fused with the coarse counts of Algorithm 1 step 1 (arXiv
// 2609.28053, Sec. 2 Eq. 1, "Quantile Balancing", Appendix C).
//
// Fast kernel (K <= kFastKmax).  A row of E logits is spread over G lanes,
// each holding N = E/G experts as N/4 8-byte pieces; row r of a wave visits
// its pieces in the order q XOR r, so that at any step the rows of a wave
// work on different experts (and count into different LDS words).  The
// coarse counts, two margins per BF16 conversion, go to a slot-major LDS
// histogram addressed by one byte permute.  Per element the kernel forms a
// 32-bit key: the binary32 bits of s = z + b with the low byte replaced by
// 255 - e, and keeps a sorted list of its kList largest keys (one maximum and
// kList-1 medians per element).  Keys are compared as floats, so negative
// scores order correctly; the key's sum takes -0 in b as +0, so a score of
// -0 keys as +0 and the two zeros share one run of keys.
// K+1 extraction rounds then take the group maximum of the list heads with
// DPP and pop the winner (unrolled: every fan-out has its own kernel; a loop
// over K took 28.4 us where the unrolled rounds take 21 for 99,991 tokens of
// E = 128, K = 5); the largest head left is rank K+1.  A lane whose list runs
// dry is scanned once for its next key, and a row whose rounds missed a key
// is extracted again with refilled lists.  Key order is
// score order except between scores that agree in their top 24 bits.  Where the
// run of rank K's top 24 bits continues past it, its members for the ranks up to K
// are chosen among the whole run by the 16 bits that order it (the scores' low
// bytes, the indices); where neighbours among the ranks agree, their exact scores
// are recomputed from z and b and every rank takes its place by counting the
// greater ones.  A block whose bias has |b| >= 2^119 (where z + b could overflow)
// takes the exact 64-bit path for every row.
//
// Generic kernel (any K < E): K+1 rounds over exact 64-bit keys.
#include "eqb_internal.hpp"

namespace eqb {

// Widest fan-out of the fast kernel.  Every fan-out is a kernel of its own per E, 46 to
// 71 KB of code at E = 256, and no configuration here routes to more than 16 experts; neither
// LDS nor registers set the line.  65,537 tokens of E = 256: K = 16 53 us, K = 17 (generic
// kernel) 171.
constexpr int kFastKmax = 16;
// Sorted keys kept per lane: the rounds pop at most K+1 keys of a lane and
// look at one more, and a lane holds N = E/G keys in all, so min(N, K + 2)
// never runs dry.  Fewer levels cost less per element (one instruction each);
// a row whose lane does run dry is done again by the full path, so the depth
// is the one at which that happens in about 1% of rows of random logits (the
// layer of 1,000,001 tokens, E = 256: K = 13 equal at 7 and 8, K = 14 294 us at
// 7, 275 at 8, K = 16 347 and 289).
// Lanes per row.  A row costs a wave its extraction rounds and outputs once,
// whatever the lanes it is spread over, so few lanes with more experts each
// are cheaper per element until their longer lists cost more: four lanes
// instead of eight took the layer of 262,144 tokens, E = 64, K = 6 from 47.4
// to 44.6 us; at E = 128 (N = 32, lists of seven) it is even, and at E = 32 two
// lanes instead of four change nothing.
template <int E> struct FastCfg { static constexpr int G = E >= 128 ? 8 : E >= 32 ? 4 : E / 8; };
template <int E, int K>
constexpr int list_depth() {
  constexpr int G = FastCfg<E>::G, N = E / G;
  constexpr int d = G == 8 ? (K <= 8 ? 5 : K <= 11 ? 6 : K <= 13 ? 7 : 8) : G == 4 ? (K <= 4 ? 5 : K <= 6 ? 6 : K <= 8 ? 7 : K <= 14 ? 8 : 9) : 8;
  constexpr int m = N < K + 2 ? N : K + 2;
  return d < m ? d : m;
}
// Block of the fast kernel: 12 waves, three per SIMD, so that a wave may hold
// up to 168 VGPRs (with 16 waves the cap of 128 forces spills).
constexpr int kRouteBlock = 768;
constexpr int kRouteWaves = kRouteBlock / 64;

constexpr int kBiasPad = 32;           // words between the rotated bias copies beyond E

// The BF16 logit z of an extracted key.  The key holds the top 24 bits H of
// s = fl32(z + b) (low byte = expert index).  The candidate is
// zc = bf16(s_mid - b), with s_mid the middle of the 256-ulp interval of H;
// it is accepted when fl32(zc + b) reproduces H and |zc| * 64 >= |s_mid|.
// The second test gives exponent(zc) >= exponent(s) - 6, so the BF16
// neighbours of zc lie at least half a BF16 ulp of zc = 2^(exponent(s)-141)
// away, about 512 binary32 ulps of s: no other BF16 value maps to H, and zc
// is z.  s_mid is never zero, so the test also rejects both zeros (+0 and -0
// give the same sum, and which one z is decides the sign of a zero tau), and
// an infinite or NaN zc cannot reproduce the finite H.  *ok reports the
// tests; otherwise z must be read from memory.
__device__ __forceinline__ uint32_t z_from_key(int key, float b, bool* ok) {
  const uint32_t kb = (uint32_t)key;
  const float s_mid = __uint_as_float((kb & 0xFFFFFF00u) | 0x80u);
  const uint32_t zc = bf16x2_bits(s_mid - b, 0.0f);   // bits 16..31: bf16(+0) = 0
  const float zf = __uint_as_float(zc << 16);
  const uint32_t sc = __float_as_uint(zf + b);
  // bitwise, not short-circuit: a branch per test would cost more than it does
  *ok = ((sc ^ kb) < 256u) & (fabsf(zf) * 64.0f >= fabsf(s_mid));
  return zc;
}

// Coarse counts of the fast kernel for E >= 64: a slot-major packed
// histogram.  Experts e, e+1 (e = 4j + 2h, a piece of four experts starting
// at 4j and its half h) share a word, counted in its low and high 16 bits.
// Half h lives in array h (64 KiB each); inside an array, slot 63 - j of bin
// u is word u*64 + 63 - j.  The counter's byte offset h << 16 | u << 8 |
// (252 - 4j) is assembled by one byte permute: u is the raw high byte of the
// BF16 margin, 252 - 4j is byte 3 of the piece's index bytes (255 - e for
// its four experts).  With the piece order rotated per row (below), the 64
// lanes of a wave hit 64 different slots at E = 256, so 64 different LDS
// banks.  Smaller E keep the expert-major layout of hist_row, which needs
// less LDS.
template <int E> constexpr bool kSlotHist = E >= 64;
template <int E>
constexpr int fast_hist_words() { return kSlotHist<E> ? 2 * 64 * kNBins : hist_words<E>(); }

// Adds the coarse counts of a slot-major histogram to slab [E][256] (kappa
// bins) and clears it, one pair of adjacent raw bins (words 64 apart) per
// thread and step.
template <int E>
__device__ __forceinline__ void flush_hist_slots(uint32_t* sh, int32_t* __restrict__ slab) {
  constexpr int kSlots = E / 4, kItems = 2 * (kNBins / 2) * kSlots;
  for (int i = threadIdx.x; i < kItems; i += blockDim.x) {
    const int it = flush_word(i, kItems);
    const int arr = it / (kItems / 2), j = it / kSlots % (kNBins / 2), slot = 64 - kSlots + it % kSlots;
    const int w0 = arr * 16384 + 2 * j * 64 + slot;
    const uint32_t c0 = sh[w0], c1 = sh[w0 + 64];
    if (c0 | c1) {
      const int e = 4 * (63 - slot) + 2 * arr;
      const bool neg = (2 * j) & 0x80;
      const int k0 = kappa_hi_of_raw(2 * j);
      if ((c0 | c1) & 0xFFFFu) add_raw_pair(slab + e * kNBins, neg, c0 & 0xFFFFu, c1 & 0xFFFFu, k0);
      if ((c0 | c1) >> 16) add_raw_pair(slab + (e + 1) * kNBins, neg, c0 >> 16, c1 >> 16, k0);
      sh[w0] = 0;
      sh[w0 + 64] = 0;
    }
  }
}

// Adds the words c0, c1 of raw bins r, r + 1 (r even, k0 its kappa bin, neg: r of
// negative margins) of expert pair m to a slab of 16-bit counters: four adjacent
// ones, one 64-bit atomic.
__device__ __forceinline__ void add_words16(int32_t* __restrict__ slab32, int m, bool neg, int k0, uint32_t c0,
                                            uint32_t c1) {
  uint16_t* slab = reinterpret_cast<uint16_t*>(slab32);
  const int k = neg ? k0 - 1 : k0;         // k0 is even, or odd (flipped) for negative bins
  const uint64_t v = neg ? ((uint64_t)c1 | ((uint64_t)c0 << 32)) : ((uint64_t)c0 | ((uint64_t)c1 << 32));
  atomicAdd(reinterpret_cast<unsigned long long*>(slab + ((int64_t)m * kNBins + k) * 2), (unsigned long long)v);
}

// flush_hist_slots into a slab of 16-bit counters (PartTable::slab16): an LDS
// word already holds the counts of experts e and e+1 (e = 4j + 2h) for one raw
// bin, so the item's two words (raw bins 2b, 2b+1, kappa bins k, k+1 or k, k-1)
// are four adjacent 16-bit counters of the slab, added with one 64-bit atomic.
// The host uses it only where no counter can pass 65,535 (no carry between
// the fields).
template <int E>
__device__ __forceinline__ void flush_hist_slots16(uint32_t* sh, int32_t* __restrict__ slab32) {
  constexpr int kSlots = E / 4, kItems = 2 * (kNBins / 2) * kSlots;
  for (int i = threadIdx.x; i < kItems; i += blockDim.x) {
    const int it = flush_word(i, kItems);
    const int arr = it / (kItems / 2), j = it / kSlots % (kNBins / 2), slot = 64 - kSlots + it % kSlots;
    const int w0 = arr * 16384 + 2 * j * 64 + slot;
    const uint32_t c0 = sh[w0], c1 = sh[w0 + 64];
    if (c0 | c1) {
      const int m = 2 * (63 - slot) + arr;   // the pair of experts 2m, 2m+1
      add_words16(slab32, m, (2 * j) & 0x80, kappa_hi_of_raw(2 * j), c0, c1);
      sh[w0] = 0;
      sh[w0 + 64] = 0;
    }
  }
}

// The histogram byte offset of half 1 of a piece: byte 3 of its index bytes
// to byte 0, 1 to byte 2.  Volatile so that it is formed where it is used
// rather than kept in a register per piece.
__device__ __forceinline__ uint32_t half1_base(uint32_t ipk, uint32_t one16) {
  uint32_t r;
  asm volatile("v_perm_b32 %0, %1, %2, %3" : "=v"(r) : "v"(one16), "v"(ipk), "s"(0x0C060C03u));
  return r;
}

// Insert key x into the sorted list L[0] >= ... >= L[n-1] (one max, n-1 med3).
template <int n>
__device__ __forceinline__ void list_insert(int (&L)[n], int x) {
#pragma unroll
  for (int j = n - 1; j > 0; --j) L[j] = key_med3(L[j - 1], L[j], x);
  L[0] = key_max(L[0], x);
}

// Insert key x as the i-th key of a list being built (the levels below i are
// still empty): i + 1 instructions while i < n.
template <int n>
__device__ __forceinline__ void list_insert_at(int (&L)[n], int x, int i) {
  if (i >= n) {
    list_insert(L, x);
  } else if (i == 0) {
    L[0] = x;
  } else {
    L[i] = key_min(L[i - 1], x);
#pragma unroll
    for (int j = n - 1; j > 0; --j)
      if (j < i) L[j] = key_med3(L[j - 1], L[j], x);
    L[0] = key_max(L[0], x);
  }
}

template <int E, int KT>
__global__ __launch_bounds__(kRouteBlock) void route_fast_kernel(
    const uint16_t* __restrict__ z, const float* __restrict__ b, int64_t T,
    int32_t* __restrict__ topk_idx, float* __restrict__ topk_score, float* __restrict__ tau,
    int32_t* __restrict__ load, int32_t* __restrict__ hist, const PartTable pt,
    int64_t rows_per_block, uint32_t* __restrict__ win, int slabs) {
  constexpr int G = FastCfg<E>::G;      // lanes per row
  constexpr int N = E / G;              // experts per lane
  constexpr int NQ = N / 4;             // 8-byte pieces per lane and row
  constexpr int R = 64 / G;             // rows per wave
  constexpr int HSLOT = (KT + G) / G;   // rank slots per lane, ranks 0..K
  constexpr int K = KT;
  static_assert(N % 4 == 0 && N >= 8, "layout");
  static_assert(KT >= 1 && KT < E && KT <= kFastKmax, "K+1 keys exist");
  constexpr int kList = list_depth<E, KT>();

  __shared__ __align__(16) uint32_t sh_hist[fast_hist_words<E>()];
  __shared__ uint32_t sh_load[E];
  __shared__ float sh_b[E];             // b as given: exact scores and tau
  // b with -0 as +0 (the keys' sums), one copy per piece rotation.  Copies
  // sit E + 32 words apart: the rows of a wave read their rotations' copies
  // with one 16-byte read per lane, and copies E words apart (a multiple of
  // the 64 banks) would put every row's reads on the same 32 banks.
  __shared__ float sh_bk[NQ][E + kBiasPad];
  // staged rows: exact keys (first routing keys) by rank; an odd stride spreads the rows over the banks
  __shared__ uint64_t sh_rank[kRouteWaves][R][(KT + 1) | 1];
  __shared__ uint32_t sh_step;                        // next unclaimed wave step of the segment

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane % G, r = lane / G;
  // Row r of a wave visits its pieces in the order q ^ rr, so at any step the
  // rows of a wave work on different experts (distinct histogram slots).
  const int rr = r & (NQ - 1);

  // Step q of this lane covers experts ex(q) .. ex(q)+3 (piece q ^ rr), so the
  // G lanes of a row read 8*G contiguous bytes per step.  b is read from LDS,
  // four experts at a time (bias4: the keys' copy, bias4x: b as given); the
  // keys' copy is kept once per rotation, sh_bk[c][j] = b[j ^ 4Gc], so that a
  // lane reads its step q at a fixed offset from its own base.
  auto ex = [&](int q) -> int { return (q ^ rr) * 4 * G + g * 4; };
  // bytes 255 - e for the four experts of a piece (ex is a multiple of 4, no borrow)
  auto idxpk = [&](int q) -> uint32_t { return 0xFCFDFEFFu - (uint32_t)ex(q) * 0x01010101u; };
  auto bias4 = [&](int q) -> float4 { return *reinterpret_cast<const float4*>(&sh_bk[rr][q * 4 * G + g * 4]); };
  auto bias4x = [&](int q) -> float4 { return *reinterpret_cast<const float4*>(&sh_b[ex(q)]); };
  auto pick = [](const float4& v, int i) -> float { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; };

  // Rows of one step of a segment starting at zb and holding n rows: row
  // base + wave * R + r of the segment, a row past its end reading the last
  // row instead (processed as invalid: no output, no count).  Byte offsets
  // stay below 2^25; the piece index occupies bits that the row and lane
  // parts leave clear, so XOR selects piece q ^ rr.
  auto load_rows = [&](uint2 (&dst)[NQ], const uint16_t* zb, uint32_t wbase, uint32_t n) {
    uint32_t t = wbase + r;
    t = t < n ? t : n - 1;
    const uint32_t off = (t * (uint32_t)E + (uint32_t)g * 4u) * 2u + (uint32_t)rr * (8u * G);
#pragma unroll
    for (int q = 0; q < NQ; ++q) dst[q] = at<uint2>(zb, off ^ ((uint32_t)q * (8u * G)));
  };
  auto load_step = [&](uint2 (&dst)[NQ], const uint16_t* zb, uint32_t base, uint32_t n) {
    load_rows(dst, zb, base + wave * R, n);
  };

  // The first step of the block's first segment (as for_each_segment will
  // cut it) is loaded before the LDS set-up, so that its latency passes while
  // the histogram is zeroed and the bias is staged.
  int64_t r0, r1;
  block_rows(T, rows_per_block, &r0, &r1);
  uint2 buf[NQ];
  if (r0 < r1) {
    int p = 0;
    while (p < pt.P - 1 && pt.off[p + 1] <= r0) ++p;
    int64_t end = pt.off[p + 1] < r1 ? pt.off[p + 1] : r1;
    if (end - r0 > kSegMax) end = r0 + kSegMax;
    load_step(buf, z + wave_uniform(r0) * E, 0, (uint32_t)(end - r0));
  }

  static_assert(fast_hist_words<E>() % 4 == 0, "16-byte zeroing");
  // of the 64 slots of a bin the last E/4 are counted and read
  constexpr int kRow4 = kSlotHist<E> ? E / 16 : fast_hist_words<E>() / 4;
  constexpr int kRows = kSlotHist<E> ? 2 * kNBins : 1;
  for (int w = threadIdx.x; w < kRows * kRow4; w += kRouteBlock)
    reinterpret_cast<uint4*>(sh_hist)[kSlotHist<E> ? w / kRow4 * 16 + 16 - kRow4 + w % kRow4 : w] = make_uint4(0, 0, 0, 0);
  int fits = 1, bzero = 1;
  if (threadIdx.x == 0) sh_step = kRouteWaves;
  for (int e = threadIdx.x; e < E; e += kRouteBlock) {
    sh_load[e] = 0;
    const float bv = b[e];
    sh_b[e] = bv;
    const float bk = (__float_as_uint(bv) == 0x80000000u) ? 0.0f : bv;
#pragma unroll
    for (int c = 0; c < NQ; ++c) sh_bk[c][e ^ (c * 4 * G)] = bk;
    fits &= (int)(fabsf(bv) < 0x1p119f);
    bzero &= (int)(bk == 0.0f);
  }
  // |z| <= 2^128 - 2^120 for a finite BF16 z, so with |b| < 2^119 every sum
  // z + b is finite and every key is a finite float.
  const bool bias_ok = __syncthreads_and(fits) != 0;
  // With a zero bias (the starting point of the balancing loop) every score
  // is a BF16 logit, so keys that agree in their top 24 bits hold equal
  // scores (for scores of either sign the index byte then orders them by
  // magnitude: lower index first for non-negative scores, last for negative
  // ones).
  const bool keys_exact = __syncthreads_and(bzero) != 0;

  uint64_t* myrank = sh_rank[wave][r];

  // key of element (q, i) from its score
  auto key_of = [&](float score, uint32_t ipk, int i) -> int {
    return (int)__builtin_amdgcn_perm(__float_as_uint(score), ipk, 0x07060500u | (uint32_t)i);
  };

  // Rebuild a lane's sorted list from the values key(sum, index bytes, i, &in) of its
  // experts that are in and strictly below thr.
  auto rebuild = [&](const float (&zf)[N], int thr, int (&L)[kList], auto&& key) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < kList; ++j) L[j] = kKeyNone;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const float4 bq = bias4(q);
      const uint32_t ipk = idxpk(q);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        bool in = true;
        const int x = key(zf[q * 4 + i] + pick(bq, i), ipk, i, &in);
        list_insert(L, (in & key_lt(x, thr)) ? x : kKeyNone);
      }
      __builtin_amdgcn_sched_barrier(0);   // one piece's keys and biases at a time: registers
    }
  };

  // Base pointers of the current segment (at most kSegMax rows): rows are
  // addressed by a 32-bit offset from them, which the loads and stores take
  // directly next to a wave-uniform 64-bit base.
  const uint16_t* seg_z = z;
  int32_t* seg_idx = topk_idx;
  float* seg_score = topk_score;
  float* seg_tau = tau;

  // t: row index inside the current segment
  // raw holds this step's logits (loaded one step earlier); once they are
  // widened, refill(raw) issues the next step's loads into the same registers.
  // exact: std::true_type when the block's keys are exact (zero bias)
  auto process = [&](auto exact, uint2 (&raw)[NQ], uint32_t t, bool valid, auto&& refill)
                     __attribute__((always_inline)) {
    // ---- widen the logits once; build keys and the per-lane sorted list
    float4 bq = bias4(0);   // read first: its LDS latency passes during the widening
    float zf[N];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      zf[q * 4 + 0] = bf16_lo(raw[q].x);
      zf[q * 4 + 1] = bf16_hi(raw[q].x);
      zf[q * 4 + 2] = bf16_lo(raw[q].y);
      zf[q * 4 + 3] = bf16_hi(raw[q].y);
    }
    refill(raw);
    int L[kList];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      // The next piece's bias is read while this piece is inserted; the
      // scheduling barrier keeps the compiler from sinking the read to its use.
      float4 bn = bq;
      if (q + 1 < NQ) bn = bias4(q + 1);
      __builtin_amdgcn_sched_barrier(0);
      const uint32_t ipk = idxpk(q);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        list_insert_at(L, key_of(zf[q * 4 + i] + pick(bq, i), ipk, i), q * 4 + i);
      bq = bn;
    }

    // ---- extraction rounds: group maximum of the list heads, winner pops
    auto pop = [&](int M) {
      const bool win = (L[0] == M);
#pragma unroll
      for (int j = 0; j < kList - 1; ++j) L[j] = win ? L[j + 1] : L[j];
      L[kList - 1] = win ? kKeyNone : L[kList - 1];
    };
    // Rows whose ranks are staged in LDS: a run that continues past rank K, equal
    // top-24-bit keys or a list that ran dry; (slow) rows of a bias beyond 2^119.
    bool staged = false, slow = false;
    float tv = 0.0f;          // tau of this lane's row (common rows)
    int rk[HSLOT];
    uint32_t zown[HSLOT];
#pragma unroll
    for (int s = 0; s < HSLOT; ++s) {
      rk[s] = kKeyNone;
      zown[s] = 0;
    }

    int mK = kKeyNone, prev = kKeyNone;
    bool near = false;      // two adjacent extracted keys share their top 24 bits
    const int tail = L[kList - 1];   // the smallest key a lane can pop
#pragma unroll
    for (int k = 0; k <= K; ++k) {
      const int M = group_max_key<G>(L[0]);
      pop(M);
      rk[k / G] = (g == k % G) ? M : rk[k / G];
      if (k > 0) near |= ((uint32_t)(M ^ prev) < 256u);
      prev = M;
      if (k == K) mK = M;
    }
    // Rank K+1 is the largest list head left.  Whether it shares the top 24
    // bits of rank K is read off the heads directly; the rest of each list
    // is not needed past this point (a row that extends its run rebuilds
    // its lists), so the last rounds' pops only shift the entries that
    // later rounds read.
    // A lane whose list ran dry popped all of its kList keys and has no
    // head: its next key is the largest of its keys below the last one it
    // popped, found by one scan of its logits.  If that key ranks above
    // rank K, the rounds missed it and the row is extracted again; if not,
    // it is the lane's head.  A head of -inf (no key left) never matches:
    // no finite key has the top 24 bits of -inf.
    int hk = L[0];
    bool missed = false;
    if (__builtin_expect(__any(L[0] == kKeyNone), 0)) {
      const bool dry_lane = L[0] == kKeyNone;
      int nxt = kKeyNone;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const float4 bq = bias4(q);
        const uint32_t ipk = idxpk(q);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int x = key_of(zf[q * 4 + i] + pick(bq, i), ipk, i);
          nxt = key_max(nxt, key_lt(x, tail) ? x : kKeyNone);
        }
      }
      hk = dry_lane ? nxt : hk;
      missed = dry_lane && key_lt(mK, nxt);
    }
    const int head = ((uint32_t)(hk ^ mK) < 256u) ? 1 : 0;
    const int rowflag = group_max_i32<G>(missed ? 2 : head);
    // z of the experts at this lane's ranks, recovered from their keys.
    // Every slot's bias is read before any is used, so the LDS latency is
    // paid once; one wave-wide test sends the failed recoveries to memory.
    int es[HSLOT];
    bool use[HSLOT], ok[HSLOT];
    float bks[HSLOT];
#pragma unroll
    for (int s = 0; s < HSLOT; ++s) {
      use[s] = valid && s * G + g <= K;
      // below E for every key of the row; the clamp keeps a row whose
      // keys cannot be trusted (it goes slow) inside its own logits
      es[s] = use[s] ? min(255 - (rk[s] & 0xFF), E - 1) : 0;
      bks[s] = sh_bk[0][es[s]];
    }
    bool bad = false;
#pragma unroll
    for (int s = 0; s < HSLOT; ++s) {
      zown[s] = z_from_key(rk[s], bks[s], &ok[s]);
      ok[s] = ok[s] | !use[s];
      bad = bad | !ok[s];
    }
    if (__builtin_expect(__any(bad), 0)) {
      // The few failed recoveries are read one lane at a time with scalar
      // loads: their wait does not include the vector loads of the next
      // step, which are still in flight (vector loads complete in order, so
      // a vector fallback load would wait for all of them).
#pragma unroll
      for (int s = 0; s < HSLOT; ++s) {
        const uint32_t off = (t * (uint32_t)E + (uint32_t)es[s]) * 2u;   // < 2^25
        uint32_t zl = zown[s];
        uint64_t need = __ballot(!ok[s]);
        while (need) {
          const int l = __builtin_ctzll(need);
          const uint32_t o = __builtin_amdgcn_readlane(off, l);
          // the aligned word holding z (seg_z is 16-byte aligned)
          const uint32_t w = at<const uint32_t>(seg_z, o & ~3u);
          if (lane == l) zl = (w >> ((o & 2u) * 8u)) & 0xFFFFu;
          need &= need - 1;
        }
        zown[s] = zl;
      }
    }
    const bool dry = rowflag == 2;   // the rounds missed a key of a dry lane
    slow = valid && !bias_ok;
    staged = valid && !slow && (near || rowflag != 0);
    // A row is staged when adjacent ranks' keys agree in their top 24 bits
    // (their order may be wrong) or the run of rank K's top 24 bits
    // continues past it.  With exact keys such keys hold equal scores, and
    // for a non-negative rank K (every rank at or above it non-negative)
    // the index byte already orders them as the exact order does: only a
    // missed key needs the staged path.
    if constexpr (decltype(exact)::value) staged = staged && (dry || mK < 0);
    // ---- staged rows: the K + 1 keys by rank, those of rank K's run chosen and
    // the others ordered by their exact scores
    if (__builtin_expect(__any(staged), 0)) {
#pragma unroll
      for (int s = 0; s < HSLOT; ++s) {
        const int k = s * G + g;
        if (staged && k <= K) myrank[k] = (uint32_t)rk[s];
      }
      // Rows whose rounds missed a key (a lane held more of the top K+1 keys
      // than its list) are extracted again, a lane's list refilled below the last
      // rank whenever it is empty.
      const bool redo = staged && dry;
      if (__any(redo)) {
        bool need = redo;
        int M = kKeyTop;
#pragma unroll 1
        for (int k = 0; k <= K; ++k) {
          if (__any(need)) {
            if (need) rebuild(zf, M, L, [&](float score, uint32_t ipk, int i, bool*) { return key_of(score, ipk, i); });
          }
          M = group_max_key<G>(L[0]);
          pop(M);
          need = redo && L[0] == kKeyNone;
          if (redo && g == 0) myrank[k] = (uint32_t)M;
        }
        if (redo) mK = M;
      }
      // Where the run of equal top 24 bits continues past rank K, its members for
      // the ranks c..K are chosen among all of it: in a run the exact order is that
      // of the scores' low bytes (the other way for negative scores), then of the
      // indices, 16 bits that are kept as a subnormal float.  A run of any length takes
      // a list and a round per rank.  Layers of logits on a grid of quarters with a zero
      // bias, before (runs extracted to their end into a buffer, ranks ordered by one
      // lane's insertions, longer runs left to the exact 64-bit path) -> now, in us: E = 32
      // K = 16 65,537 tokens 60.0 -> 35.6, 600,000 197 -> 118; E = 64 K = 16 4,097 tokens
      // 48.9 -> 30.3; E = 16 K = 15 65,537 tokens 39.2 -> 32.8.
      const bool ext = staged && rowflag != 0;
      if (__any(ext)) {
        lds_wave_sync();
        int c = 0;
#pragma unroll
        for (int s = 0; s < HSLOT; ++s) {
          const int k = s * G + g;
          if (k <= K && ((uint32_t)myrank[k] ^ (uint32_t)mK) >= 256u) c = k + 1;
        }
        c = group_max_i32<G>(c);
        lds_wave_sync();
        const uint32_t top = ((uint32_t)mK & 0xFFFFFF00u) | (mK < 0 ? 0xFFu : 0u);
        auto run_key = [&](float score, uint32_t ipk, int i, bool* in) -> int {
          const uint32_t low = __float_as_uint(score) ^ top;     // below 256: of the run
          const int x = (int)__builtin_amdgcn_perm(low, ipk, 0x0C0C0400u | (uint32_t)i);
          *in = low < 256u;
          return x;
        };
        bool need = ext, more = false;
        int M = kKeyTop;
#pragma unroll 1
        for (int k = c; __any(ext && k <= K); ++k) {
          if (__any(need)) {
            if (need) {
              rebuild(zf, M, L, run_key);
              more = L[kList - 1] != kKeyNone;
            }
          }
          M = group_max_key<G>(L[0]);
          pop(M);
          need = ext && more && L[0] == kKeyNone;
          if (ext && g == 0 && k <= K) myrank[k] = ((uint32_t)mK & 0xFFFFFF00u) | ((uint32_t)M & 0xFFu);
        }
      }
      lds_wave_sync();
      // exact keys (z as recovered above where the rank kept its key), and each
      // one's place: how many are greater
      uint32_t ek[HSLOT], zs[HSLOT];
#pragma unroll
      for (int s = 0; s < HSLOT; ++s) {
        const int k = s * G + g;
        ek[s] = 0;
        zs[s] = zown[s];
        if (staged && k <= K) {
          const int key = (int)(uint32_t)myrank[k];
          ek[s] = min(255 - (key & 0xFF), E - 1);
          bool ok = true;
          if (key != rk[s]) zs[s] = z_from_key(key, sh_bk[0][ek[s]], &ok);
          if (!ok) zs[s] = seg_z[t * E + ek[s]];
        }
      }
      uint64_t own[HSLOT];
      uint32_t place[HSLOT];
#pragma unroll
      for (int s = 0; s < HSLOT; ++s) {
        const int k = s * G + g;
        own[s] = exact_key(__float_as_uint(__uint_as_float(zs[s] << 16) + sh_b[ek[s]]), ek[s], zs[s]);
        place[s] = 0;
        if (staged && k <= K) myrank[k] = own[s];
      }
      lds_wave_sync();
      // A rank that the next one exceeds?  4,194,304 tokens of E = 256 with ties in order
      // 1332 us without the look, 1265 with it; with more ranks a lane it does not pay
      // (E = 16, K = 15, 65,537 tokens of ties 33.0 without, 33.5 with).
      bool coll = HSLOT > 4;
      if constexpr (HSLOT <= 4) {
#pragma unroll
        for (int s = 0; s < HSLOT; ++s) {
          const int k = s * G + g;
          if (staged && k < K) coll |= myrank[k + 1] > own[s];
        }
      }
      if (__any(coll)) {
#pragma unroll
        for (int i = 0; i <= K; ++i) {
          const uint64_t x = myrank[i];
#pragma unroll
          for (int s = 0; s < HSLOT; ++s) place[s] += x > own[s];
        }
        lds_wave_sync();
#pragma unroll
        for (int s = 0; s < HSLOT; ++s) {
          if (staged && s * G + g <= K) myrank[place[s]] = own[s];
        }
        lds_wave_sync();
      }
    }

    // ---- exact 64-bit extraction for rows flagged slow
    if (__builtin_expect(__any(slow), 0)) {
      if (slow) {
        uint64_t prevk = ~0ull;
        for (int k = 0; k <= K; ++k) {
          uint64_t m = 0;
#pragma unroll
          for (int q = 0; q < NQ; ++q) {
            const float4 bq = bias4x(q);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              // rebuilt every round instead of being held in 2*N registers
              float zq = zf[q * 4 + i];
              asm volatile("" : "+v"(zq));
              const uint32_t zb = __float_as_uint(zq) >> 16;
              const uint32_t sb = __float_as_uint(zq + pick(bq, i));
              const uint64_t key = exact_key(sb, ex(q) + i, zb);
              m = (key < prevk && key > m) ? key : m;
            }
          }
          m = group_max_u64<G>(m);
          prevk = m;
          if (g == 0) myrank[k] = m;
        }
      }
      lds_wave_sync();
    }

    // ---- outputs: ranks 0..K-1, loads, tau
    const bool fromlds = staged || slow;
    if (valid && !fromlds) {
      // rank k is held by lane k % G in slot k / G; its exact score is z + b of that expert
      float tk = 0.0f;
#pragma unroll
      for (int s = 0; s < HSLOT; ++s) {
        const int k = s * G + g;
        if (k <= K) {
          const int e = 255 - (rk[s] & 0xFF);
          const uint32_t zb = zown[s];
          if (k < K) {
            at<int32_t>(seg_idx, (t * K + k) * 4u) = e;
            at<float>(seg_score, (t * K + k) * 4u) = sigmoid_fast(__uint_as_float(zb << 16));
            if (load) atomicAdd(&sh_load[e], 1u);
          } else {
            tk = __uint_as_float(zb << 16) + sh_b[e];
          }
        }
      }
      tv = tk;
    }
    // every lane of the row takes tau from the lane holding rank K
    tv = group_bcast<G, K % G>(tv, g);
    if (valid && fromlds) {
#pragma unroll
      for (int s = 0; s < HSLOT; ++s) {
        const int k = s * G + g;
        if (k < K) {
          const uint64_t v = myrank[k];
          const int e = exact_key_expert(v);
          at<int32_t>(seg_idx, (t * K + k) * 4u) = e;
          at<float>(seg_score, (t * K + k) * 4u) = sigmoid_fast(__uint_as_float(exact_key_z(v) << 16));
          if (load) atomicAdd(&sh_load[e], 1u);
        }
      }
      tv = __uint_as_float(exact_key_sbits(myrank[K]));
    }
    if (valid && g == 0) at<float>(seg_tau, t * 4u) = tv;

    // ---- coarse counts: raw high byte of bf16(tau - z), two margins per conversion
    if (hist && valid) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint32_t p = bf16x2_bits(tv - zf[q * 4 + 2 * h], tv - zf[q * 4 + 2 * h + 1]);
          if constexpr (kSlotHist<E>) {
            // byte offsets: the raw high byte of either margin becomes byte 1
            if (h == 0) {
              const uint32_t ipk = idxpk(q);
              atomicAdd(&at<uint32_t>(sh_hist, __builtin_amdgcn_perm(ipk, p, 0x0C0C0107u)), 1u);
              atomicAdd(&at<uint32_t>(sh_hist, __builtin_amdgcn_perm(ipk, p, 0x0C0C0307u)), 1u << 16);
            } else {
              const uint32_t base = half1_base(idxpk(q), 0x10000u);
              atomicAdd(&at<uint32_t>(sh_hist, __builtin_amdgcn_perm(base, p, 0x0C060104u)), 1u);
              atomicAdd(&at<uint32_t>(sh_hist, __builtin_amdgcn_perm(base, p, 0x0C060304u)), 1u << 16);
            }
          } else {
            const uint32_t row = hist_row(ex(q)) + h * kHistStride;
            atomicAdd(&sh_hist[row + ((p >> 8) & 0xFFu)], 1u);
            atomicAdd(&sh_hist[row + (p >> 24)], 1u << 16);
          }
        }
      }
    }
    __builtin_amdgcn_wave_barrier();
  };

  // The sweep is compiled twice, for exact keys (a zero bias) and for any
  // bias, so that neither carries the other's test in its per-row path.
  auto set_base = [&](int64_t s0) {
    const int64_t su = wave_uniform(s0);
    seg_z = z + su * E;
    seg_idx = topk_idx + su * K;
    seg_score = topk_score + su * K;
    seg_tau = tau + su;
  };
  // Adds the block's LDS counts (coarse bins, loads) of partition p to global
  // memory and clears them.  With an image the coarse counts stay until the
  // block's rows are done.
  auto flush_counts = [&](int p) {
    __syncthreads();
    if (hist && !win) {
      if constexpr (kSlotHist<E>) {
        if (pt.slab16) flush_hist_slots16<E>(sh_hist, count_slab(hist, pt, p, E));
        else flush_hist_slots<E>(sh_hist, count_slab(hist, pt, p, E));
      } else {
        flush_hist<E, false>(sh_hist, count_slab(hist, pt, p, E), nullptr);
      }
    }
    if (load) {
      for (int e = threadIdx.x; e < E; e += kRouteBlock) {
        const uint32_t c = sh_load[e];
        if (c) atomicAdd(&load[(int64_t)p * E + e], (int32_t)c);
        sh_load[e] = 0;
      }
    }
    if (threadIdx.x == 0) sh_step = kRouteWaves;
    __syncthreads();
  };
  auto sweep = [&](auto exact) __attribute__((always_inline)) {
  bool first = true;
  for_each_segment(r0, r1, pt, [&](int p, int64_t s0, int64_t s1) {
    set_base(s0);
    const uint32_t n = (uint32_t)(s1 - s0);
    // The next step's loads are in flight while a step is processed: a step
    // widens the rows loaded one step earlier and then reuses their registers
    // for the next step's loads, so the only wait is for loads issued a whole
    // step before.  The last step also loads (the segment's last row, clamped
    // in load_step), which keeps the loads unconditional: the registers then
    // carry over to the next step without copies.  The first segment's first
    // step was loaded before the LDS set-up.
    if (!first) load_step(buf, seg_z, 0, n);
    first = false;
    // A wave starts with step `wave` (R rows) and claims each further step
    // from an LDS counter: the SIMD serves its oldest wave first, so with a
    // fixed share per wave the waves of a SIMD finish one after another and the
    // last one runs alone (4,096 rows of E = 128 per block: the first wave
    // done after 66 us, the last after 96 us).  The claim is issued when a step
    // starts and read after the step's logits are widened, where the claimed
    // rows are loaded.
    for (uint32_t base = wave * R; base < n;) {
      uint32_t claimed = 0, next = 0;
      if (lane == 0) claimed = atomicAdd(&sh_step, 1u);
      const uint32_t t = base + r;
      process(exact, buf, t, t < n, [&](uint2 (&dst)[NQ]) {
        next = __builtin_amdgcn_readfirstlane(claimed) * (uint32_t)R;
        load_rows(dst, seg_z, next, n);
      });
      base = next;
    }
    flush_counts(p);
  });
  };
  if (keys_exact) sweep(std::true_type{});
  else sweep(std::false_type{});
  if (win) {
    // The flush's atomics, a thousand and more scattered 8-byte updates per block
    // that every block of a launch makes at the same time, took 8 us of the 42 of
    // 147,456 rows of E = 256.  Nearly all margins lie in a window of 16 of the
    // 256 bins: the block stores those as one image (8 KiB at E = 256; images of
    // all bins, 32 MiB in all, cost the selection more than they saved), and adds
    // only the rest.  Layers, before -> after (us): E = 256 K = 6 147,456 tokens
    // 64.6 -> 59.0, E = 128 K = 5 99,991 tokens 44.4 -> 39.1, K = 8 1,048,576 tokens
    // 160 -> 156.5, E = 256 K = 16 65,537 tokens 56.0 -> 54.7; E = 64 and less even.
    uint4* dst = reinterpret_cast<uint4*>(win + (int64_t)blockIdx.x * win_words(E));
    for (int i = threadIdx.x; i < (E / 2) * (kWinBins / 4); i += kRouteBlock) {
      const int m = i % (E / 2), q = i / (E / 2), raw = win_raw(4 * q);
      const uint32_t* src = sh_hist + (kSlotHist<E> ? (m & 1) * 16384 + raw * 64 + 63 - (m >> 1) : m * kHistStride + raw);
      constexpr int S = kSlotHist<E> ? 64 : 1;
      dst[m * (kWinBins / 4) + q] = make_uint4(src[0], src[S], src[2 * S], src[3 * S]);
    }
    int32_t* slab = hist + (int64_t)(blockIdx.x % (unsigned)slabs) * E * kNBins;
    // pairs of adjacent raw bins outside the window, four expert pairs at a time
    // where they lie side by side
    constexpr int kPairs = kNBins / 2 - kWinBins / 2;
    constexpr int V = kSlotHist<E> ? 4 : 1, kGroups = E / 2 / V;
    for (int i = threadIdx.x; i < kPairs * kGroups; i += kRouteBlock) {
      const int group = i % kGroups, r = 2 * outside_pair(i / kGroups);
      uint32_t c0[V], c1[V];
      int m0;                              // expert pair of c0[0]; c0[v] is of pair m0 - 2v
      if constexpr (kSlotHist<E>) {
        const int arr = group & 1, slot = 64 - E / 4 + 4 * (group >> 1);
        m0 = 2 * (63 - slot) + arr;
        const uint32_t* src = sh_hist + arr * 16384 + r * 64 + slot;
        const uint4 a = *reinterpret_cast<const uint4*>(src), c = *reinterpret_cast<const uint4*>(src + 64);
        c0[0] = a.x; c0[1] = a.y; c0[2] = a.z; c0[3] = a.w;
        c1[0] = c.x; c1[1] = c.y; c1[2] = c.z; c1[3] = c.w;
      } else {
        m0 = group;
        c0[0] = sh_hist[m0 * kHistStride + r];
        c1[0] = sh_hist[m0 * kHistStride + r + 1];
      }
      uint32_t any = 0;
#pragma unroll
      for (int v = 0; v < V; ++v) any |= c0[v] | c1[v];
      if (any == 0) continue;
      const bool neg = r & 0x80;
      const int k0 = kappa_hi_of_raw(r);
#pragma unroll
      for (int v = 0; v < V; ++v) {
        if ((c0[v] | c1[v]) == 0) continue;
        if (pt.slab16) {
          add_words16(slab, m0 - 2 * v, neg, k0, c0[v], c1[v]);
        } else {
          int32_t* row = slab + (m0 - 2 * v) * 2 * kNBins;
          if ((c0[v] | c1[v]) & 0xFFFFu) add_raw_pair(row, neg, c0[v] & 0xFFFFu, c1[v] & 0xFFFFu, k0);
          if ((c0[v] | c1[v]) >> 16) add_raw_pair(row + kNBins, neg, c0[v] >> 16, c1[v] >> 16, k0);
        }
      }
    }
  }
}

// ----------------------------------------------------------- generic ----
template <int E>
__global__ __launch_bounds__(kBlock) void route_generic_kernel(
    const uint16_t* __restrict__ z, const float* __restrict__ b, int64_t T, int K,
    int32_t* __restrict__ topk_idx, float* __restrict__ topk_score, float* __restrict__ tau,
    int32_t* __restrict__ load, int32_t* __restrict__ hist, const PartTable pt,
    int64_t rows_per_block) {
  constexpr int G = E / 8;
  constexpr int R = 64 / G;
  constexpr int ROWS = kWaves * R;
  __shared__ uint32_t sh_hist[hist_words<E>()];
  __shared__ uint32_t sh_load[E];

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane % G, rr = lane / G;
  const int e0 = g * 8;
  float bb[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) bb[j] = b[e0 + j];
  for (int w = threadIdx.x; w < hist_words<E>(); w += kBlock) sh_hist[w] = 0;
  for (int w = threadIdx.x; w < E; w += kBlock) sh_load[w] = 0;
  __syncthreads();

  int64_t r0, r1;
  block_rows(T, rows_per_block, &r0, &r1);
  for_each_segment(r0, r1, pt, [&](int p, int64_t s0, int64_t s1) {
    for (int64_t base = s0; base < s1; base += ROWS) {
      const int64_t t = base + wave * R + rr;
      const bool valid = t < s1;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (valid) v = *reinterpret_cast<const uint4*>(z + t * E + e0);
      const uint32_t w4[4] = {v.x, v.y, v.z, v.w};
      float zf[8];
      uint64_t key[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const uint32_t zb = (j & 1) ? (w4[j >> 1] >> 16) : (w4[j >> 1] & 0xFFFFu);
        zf[j] = (j & 1) ? bf16_hi(w4[j >> 1]) : bf16_lo(w4[j >> 1]);
        key[j] = exact_key(__float_as_uint(zf[j] + bb[j]), e0 + j, zb);
      }
      uint64_t prev = ~0ull;
      for (int k = 0; k <= K; ++k) {
        uint64_t m = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) m = (key[j] < prev && key[j] > m) ? key[j] : m;
        m = group_max_u64<G>(m);
        prev = m;
        if (k < K && valid && g == k % G) {
          const int e = exact_key_expert(m);   // in [0, E): the row holds E > K distinct keys
          topk_idx[t * K + k] = e;
          topk_score[t * K + k] = sigmoid_f32(__uint_as_float(exact_key_z(m) << 16));
          if (load && e >= 0 && e < E) atomicAdd(&sh_load[e], 1u);
        }
      }
      const float tv = __uint_as_float(exact_key_sbits(prev));
      if (valid && g == 0) tau[t] = tv;
      if (hist && valid) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int e = e0 + j;
          const uint32_t hr = bf16_raw_hi(__float_as_uint(tv - zf[j]));
          atomicAdd(&sh_hist[hist_row(e) + hr], hist_inc(e));
        }
      }
    }
    __syncthreads();
    if (hist) flush_hist<E, false>(sh_hist, count_slab(hist, pt, p, E), nullptr);
    if (load) {
      for (int e = threadIdx.x; e < E; e += kBlock) {
        const uint32_t c = sh_load[e];
        if (c) atomicAdd(&load[(int64_t)p * E + e], (int32_t)c);
        sh_load[e] = 0;
      }
    }
    __syncthreads();
  });
}

// ------------------------------------------------------------- launch ---
template <int E, int KT>
void launch_fast(const RouteArgs& a, hipStream_t s, RouteForm* form) {
  int blocks;
  int64_t rpb;
  grid_for(a.T, kRouteWaves * (64 / FastCfg<E>::G), 1, &blocks, &rpb);
  PartTable pt = a.pt;
  if (a.hist == nullptr && a.load == nullptr) {
    // nothing is counted per partition: one segment, where each of a block's would
    // end in barriers and start with nothing in flight (1,021 rows of E = 64 in 16
    // partitions: 13.4 us, 10.1 as one)
    pt.P = 1;
    pt.off[1] = a.T;
  }
  const bool images = a.win != nullptr && a.hist != nullptr && blocks <= a.win_blocks && rpb <= kSegMax;
  const int nslabs = pt.P * pt.nsub, slabs = images ? (nslabs < kWinSlabs ? nslabs : kWinSlabs) : nslabs;
  const int64_t slab_rows = images ? (int64_t)((blocks + slabs - 1) / slabs) * rpb : slab_rows_bound(pt, rpb);
  pt.slab16 = (kSlotHist<E> && a.hist != nullptr && a.slab16_ok && slab_rows <= kSegMax) ? 1 : 0;
  if (form) *form = RouteForm{pt.slab16 != 0, images ? blocks : 0, slabs};
  route_fast_kernel<E, KT><<<blocks, kRouteBlock, 0, s>>>(a.z, a.b, a.T, a.idx, a.score, a.tau, a.load,
                                                     a.hist, pt, rpb, images ? a.win : nullptr, slabs);
}

// Every fan-out up to kFastKmax has its own kernel, the rounds unrolled.
template <int E, int K>
eqb_status launch_route_k(const RouteArgs& a, hipStream_t s, RouteForm* form) {
  if constexpr (K <= kFastKmax && K < E) {
    if (a.K == K) {
      launch_fast<E, K>(a, s, form);
      return launch_status();
    }
    return launch_route_k<E, K + 1>(a, s, form);
  } else {
    int blocks;
    int64_t rpb;
    grid_for(a.T, kWaves * (64 / (E / 8)), 1, &blocks, &rpb);
    route_generic_kernel<E><<<blocks, kBlock, 0, s>>>(a.z, a.b, a.T, a.K, a.idx, a.score, a.tau, a.load,
                                                      a.hist, a.pt, rpb);
    return launch_status();
  }
}

template <int E>
eqb_status launch_route_e(const RouteArgs& a, hipStream_t s, RouteForm* form) {
  if (form) *form = RouteForm{false, 0, a.pt.P * a.pt.nsub};
  return launch_route_k<E, 1>(a, s, form);
}

// This file is compiled once per expert count, the objects side by side.
template eqb_status launch_route_e<EQB_ROUTE_E>(const RouteArgs& a, hipStream_t s, RouteForm* form);

}  // namespace eqb
