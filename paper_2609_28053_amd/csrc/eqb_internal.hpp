// eqb_internal.hpp - launch interfaces between the C ABI shim and the kernels.
#pragma once

#include "eqb_device.hpp"

namespace eqb {

struct RouteArgs {
  const uint16_t* z;
  const float* b;
  int64_t T;
  int E, K;
  int32_t* idx;
  float* score;
  float* tau;
  int32_t* load;
  int32_t* hist;
  PartTable pt;
  // The layer: `hist` is workspace slabs that only its own coarse selection
  // reads, so the route kernel may use 16-bit counters (PartTable::slab16).
  bool slab16_ok = false;
  // The layer: room for win_blocks images (win_words(E) words each) of the blocks'
  // coarse counts.  Where the grid fits, each block stores its window there and
  // adds only the counts outside it to `hist`, to slab block % RouteForm::slabs.
  uint32_t* win = nullptr;
  int win_blocks = 0;
};

// Slabs that the counts outside the images' windows are spread over, so that the
// coarse selection reads and clears two instead of eight (147,456 tokens of E =
// 256: 59.0 us with two, 59.8 with eight).
constexpr int kWinSlabs = 2;

// How a route launch left the coarse counts.
struct RouteForm {
  bool slab16 = false;   // `hist` holds 16-bit slabs (see PartTable)
  int images = 0;        // images at RouteArgs::win, their counts not in `hist`
  int slabs = 0;         // slabs of `hist` that may hold counts, the first ones
};

struct MarginArgs {
  const uint16_t* z;
  const float* tau;
  int64_t T;
  int E;
  const int32_t* sel_hi;   // fine pass only
  int sel_stride = 0;      // 0: one selection for all partitions; E: one per partition
  int32_t* hist;
  PartTable pt;
  // Fine pass of a layer (sel_stride 0, counts summed over partitions): room
  // for part_blocks per-block images of the LDS counts (part_words(E) words
  // each).  When the pass's grid fits (at most part_blocks blocks, at most
  // kSegMax rows per block) every block stores its counts there with plain
  // stores instead of adding them to `hist`.
  uint32_t* part = nullptr;
  int part_blocks = 0;
};

// Words of one block's image of the fine counts: for each expert pair
// (2m, 2m+1), 256 words holding the two experts' 16-bit counts of raw low
// byte j in their low and high halves.
__host__ __device__ inline int64_t part_words(int E) { return (int64_t)(E / 2) * kNBins; }
// Blocks of the coarse pass per compute unit (its LDS counts take (E/2) * 257
// words per block), and the images of all E experts a layer workspace holds:
// the image-storing pass runs at most one block per compute unit, and the
// workspace has room for one full grid of whole-row blocks on a device of up
// to 256 compute units (a larger device runs the pass with fewer, longer
// blocks; blocks of fewer experts store smaller images).
inline int margin_blocks_per_cu(int E) { return (E / 2) * kHistStride * 4 * 2 <= 160 * 1024 ? 2 : 1; }
constexpr int kPartCUs = 256;
inline int layer_part_blocks(int) { return kPartCUs; }

eqb_status launch_route(const RouteArgs& a, hipStream_t s, RouteForm* form = nullptr);
template <int E>
eqb_status launch_route_e(const RouteArgs& a, hipStream_t s, RouteForm* form);   // route.hip, one object per E
// *part_used: the number of per-block images the fine pass wrote (0 when it
// added its counts to a.hist).
eqb_status launch_margin(bool fine, const MarginArgs& a, hipStream_t s, int* part_used = nullptr);
eqb_status launch_load(const int32_t* idx, int64_t T, int K, int E, int32_t* load, const PartTable& pt,
                       hipStream_t s);
eqb_status launch_select(int pass, const int32_t* hist, int P, int E, int64_t r, int32_t* sel_hi,
                         int64_t* rank_in_bin, int32_t* sel_lo, uint16_t* q_bf16, float* b_next,
                         int32_t* hist_sum, int32_t* status, hipStream_t s);

// form: how the route launch left the pass-1 counts; win its images.
eqb_status launch_layer_selects(int pass, int32_t* hist, int P, int nsub, int E, int64_t r, int32_t* sel_hi,
                                int64_t* rank_in_bin, uint16_t* q_bf16, float* b_next,
                                int32_t* hist_sum, int32_t* load_acc, int32_t* load_out, int32_t* status,
                                int32_t* ticket, hipStream_t s, RouteForm form = RouteForm{},
                                const uint32_t* win = nullptr);
// The fine selection of a layer from the fine pass's per-block images
// (nparts of them), then the centring and status as launch_layer_selects(2).
eqb_status launch_layer_select_parts(const uint32_t* part, int nparts, int E, int32_t* sel_hi,
                                     int64_t* rank_in_bin, uint16_t* q_bf16, float* b_next,
                                     int32_t* hist_sum, int32_t* status, int32_t* ticket, hipStream_t s);

eqb_status launch_select_local(int pass, const int32_t* hist, int E, int K, const PartTable& pt,
                               int32_t* sel_hi, int64_t* rank_in_bin, int32_t* sel_lo, uint16_t* q_bf16,
                               int32_t* status, hipStream_t s);
eqb_status launch_rank_average(const uint16_t* q_bf16, int E, const PartTable& pt, double* b_avg,
                               float* b_next, hipStream_t s);
eqb_status launch_uniform_hist(const uint16_t* z, const float* tau, int64_t T, int E, const PartTable& pt,
                               float lo, float scale, int nbins, int32_t* hist, hipStream_t s);
eqb_status launch_select_uniform(const int32_t* hist, int P, int E, int nbins, int64_t r, double lo,
                                 double width, double* est, float* b_next, int32_t* status, hipStream_t s);
eqb_status launch_max_violation(const int32_t* load, int E, int K, const PartTable& pt,
                                double* out_global, double* out_local, double* out_local_mean, hipStream_t s);

eqb_status launch_lei_residual(const int32_t* load, int E, int K, const PartTable& pt, double eta,
                               double c, float* inj, hipStream_t s);
eqb_status launch_lei_router_backward(const uint16_t* z, const int32_t* idx, const float* gs, const float* inj,
                                      int64_t T, int E, int K, float* gz, const PartTable& pt, hipStream_t s);
eqb_status launch_lei_inject(float* grad, const float* inj, int64_t T, int E, const PartTable& pt,
                             hipStream_t s);

// Count slabs per partition in a layer's workspace: enough that about 8
// slabs share the blocks of a launch, so no counter receives the flush
// atomics of every block.  Only the route sweep's coarse counts use them
// when the fine pass stores per-block images, and the coarse selection reads
// and clears every slab: 8 measured faster than 16, 4, 2 or 1 at one
// partition of 147,456 tokens (1.2% against 16), and no slower on the other
// workloads.  With images (RouteForm) the route sweep uses kWinSlabs of them.
inline int layer_replicas(int P) { return P >= 8 ? 1 : 8 / P; }

// Working buffers of one layer (eqb_layer): the per-partition coarse and
// fine counts (layer_replicas(P) slabs per partition), the loads as the
// route kernel accumulates them, the selections, and (optionally) room for
// the per-block count images.  Each piece starts on a 256-byte
// boundary.  The counters (everything before the images) are zero when a
// layer starts and zero again when it ends: the selection that reads a
// counter clears it.  The images are scratch: the route sweep and after it the
// fine pass overwrite the ones their selections read.
struct LayerWorkspace {
  int nsub;               // count slabs per partition
  int32_t* hist_hi;       // [P,nsub,E,256]
  int32_t* hist_lo;       // [P,nsub,E,256]
  int32_t* load_acc;      // [P,E]
  int32_t* sel_hi;        // [E]
  int64_t* rank_in_bin;   // [E]
  int32_t* tickets;       // counters of finished blocks (kTicketBytes reserved)
  uint32_t* part;         // [part_blocks, part_words(E)] or null
  int part_blocks;
};

// Reserved for tickets.  Far more than they take: the workspace keeps the size
// that callers have allocated by.
constexpr size_t kTicketBytes = 128 << 10;

inline size_t align256(size_t n) { return (n + 255) & ~(size_t)255; }

// Bytes of a layer workspace, and its pieces carved from base (null base:
// only the size is computed).  with_part = false leaves out the fine pass's
// images (the layer then adds the fine counts to the slabs); *zero_bytes
// (nullable) receives the size of the leading part that holds the counters.
inline size_t layer_workspace(void* base, int E, int P, LayerWorkspace* w, bool with_part = true,
                              size_t* zero_bytes = nullptr) {
  const int nsub = layer_replicas(P);
  const size_t hist = align256((size_t)P * nsub * E * kNBins * sizeof(int32_t));
  const size_t load = align256((size_t)P * E * sizeof(int32_t));
  const size_t sel = align256((size_t)E * sizeof(int32_t));
  const size_t rib = align256((size_t)E * sizeof(int64_t));
  const size_t zero = 2 * hist + load + 2 * sel + rib + kTicketBytes;   // the second sel is not used
  const size_t part = with_part ? align256((size_t)layer_part_blocks(E) * part_words(E) * sizeof(uint32_t)) : 0;
  if (base && w) {
    char* p = static_cast<char*>(base);
    w->nsub = nsub;
    w->hist_hi = reinterpret_cast<int32_t*>(p);
    w->hist_lo = reinterpret_cast<int32_t*>(p + hist);
    w->load_acc = reinterpret_cast<int32_t*>(p + 2 * hist);
    w->sel_hi = reinterpret_cast<int32_t*>(p + 2 * hist + load);
    w->rank_in_bin = reinterpret_cast<int64_t*>(p + 2 * hist + load + 2 * sel);
    w->tickets = reinterpret_cast<int32_t*>(p + 2 * hist + load + 2 * sel + rib);
    w->part = with_part ? reinterpret_cast<uint32_t*>(p + zero) : nullptr;
    w->part_blocks = with_part ? layer_part_blocks(E) : 0;
  }
  if (zero_bytes) *zero_bytes = zero;
  return zero + part;
}

// eqb_layer with the workspace layout chosen by with_part (the fine pass's
// per-block images present or not; see layer_workspace).
eqb_status layer_call(const uint16_t* z, const float* b, int64_t T, int32_t E, int32_t K,
                      const int64_t* part_off, int32_t P, int32_t* topk_idx, float* topk_score, float* tau,
                      int32_t* load, uint16_t* q_bf16, float* b_next, int32_t* hist_hi_sum,
                      int32_t* hist_lo_sum, int32_t* dev_status, void* workspace, size_t workspace_bytes,
                      bool with_part, void* const* marks, void* stream);

// The whole layer on one stream: route + loads + coarse counts, coarse
// selection (clearing the coarse counts, handing the loads out), fine
// counts, fine selection (clearing the fine counts), centring and status.
// marks (nullable, 5 entries, each nullable): events recorded before the
// route kernel, after it, after the coarse selection, after the fine pass
// and at the end.
eqb_status launch_layer(const RouteArgs& route, int64_t r, const LayerWorkspace& w, uint16_t* q_bf16,
                        float* b_next, int32_t* load_out, int32_t* hist_hi_sum, int32_t* hist_lo_sum,
                        int32_t* dev_status, void* const* marks, hipStream_t s);

// Number of compute units of the current device (cached per device).
int num_cus();

// Upper bound on the grid of the streaming kernels set by eqb_set_max_blocks
// (0: none).
int max_blocks_cap();

// Blocks and rows per block for a streaming kernel over T rows: at most
// blocks_per_cu blocks per CU, each owning a contiguous range of
// ceil(T / blocks) rows (the last may be shorter), and no more than ceil(T /
// min_rows) blocks (a block's fixed costs, zeroing and flushing its LDS counts,
// then pay for more rows; just past a multiple of min_rows a block's share is up to
// half of it smaller: 1,025 rows at 1,024 are blocks of 513).  With slices > 1 every row range is
// shared by that many blocks, and *blocks counts the ranges.  The ranges are
// not rounded to whole steps: with P equal partitions and a block count that P
// divides, every partition boundary then falls on a block boundary, and no
// block pays for a second segment (a second flush and a cold restart of its
// prefetch).
inline void grid_for(int64_t T, int64_t min_rows, int blocks_per_cu, int* blocks, int64_t* rows_per_block,
                     int slices = 1) {
  int64_t max_blocks = (int64_t)num_cus() * blocks_per_cu;
  const int cap = max_blocks_cap();
  if (cap > 0 && cap < max_blocks) max_blocks = cap;
  max_blocks /= slices;
  const int64_t want = (T + min_rows - 1) / min_rows;
  int64_t nb = want < max_blocks ? want : max_blocks;
  if (nb < 1) nb = 1;
  *rows_per_block = T > 0 ? (T + nb - 1) / nb : 1;
  *blocks = (int)((T + *rows_per_block - 1) / *rows_per_block);
  if (*blocks < 1) *blocks = 1;
}

inline eqb_status launch_status() { return hipGetLastError() == hipSuccess ? EQB_OK : EQB_ERR_HIP; }

// Most rows any count slab of a route launch with static ranges receives:
// block b covers rows [b * rows_per_block, (b + 1) * rows_per_block) and adds
// partition p's rows to slab p * nsub + b % nsub, so a slab of partition p
// takes at most ceil(c_p / nsub) blocks' rows, c_p the blocks overlapping p.
inline int64_t slab_rows_bound(const PartTable& pt, int64_t rows_per_block) {
  int64_t worst = 0;
  for (int p = 0; p < pt.P; ++p) {
    if (pt.off[p + 1] <= pt.off[p]) continue;
    const int64_t b0 = pt.off[p] / rows_per_block, b1 = (pt.off[p + 1] - 1) / rows_per_block;
    const int64_t c = b1 - b0 + 1;
    const int64_t per = (c + pt.nsub - 1) / pt.nsub;
    const int64_t n = pt.off[p + 1] - pt.off[p];
    const int64_t rows = per * rows_per_block < n ? per * rows_per_block : n;
    worst = rows > worst ? rows : worst;
  }
  return worst;
}

}  // namespace eqb
