// libonebitlamb: host side of the C ABI (include/onebitlamb.h) -- context, tile tables, argument
// validation and kernel launches.  The kernels live in ob_kernels.h.
//
// Build flags that the arithmetic depends on: -ffp-contract=off (one rounding per operation) and
// hipcc's default correctly rounded fp32 divide/sqrt; never -ffast-math.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <limits>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "ob_kernels.h"
#include "ob_plan.h"
#include "onebitlamb.h"

using namespace obk;

namespace {

// 128-bit accesses per thread per array in the plain N-sized kernels: tiles of 1024 elements measured
// ~7 % faster than 4096 on MI355X (ratio and update kernels at 6.4-6.5 TB/s instead of 6.0).  The
// kernels with a per-layer barrier share the segment arrays of this tiling, so it is fixed at 1.
constexpr int U_MAIN = 1;
constexpr int U_SRV = 1;    // ... in the kernels over the single server chunk
// ... in the single-pass server kernel (zb stays in registers): the smallest of these whose tiles of
// the served chunk all fit on the device at once (more, smaller workgroups hide the W dependent
// additions per element better)
constexpr int U_SRV_RES[] = {1, 2, 4};   // (8 would need registers that cost more slots than it saves tiles)
#ifndef OB_U_RES
#define OB_U_RES 16
#endif
constexpr int U_RES = OB_U_RES;   // ... in the single-pass worker compression (z stays in registers)
// workgroups per CU the single-pass compression kernel is built for: 5 lets the instantiation with
// momentum scaling spill its layer cursor (touched only in tiles that meet a layer boundary) instead
// of dropping to 4 (measured 3 % faster; without momentum scaling the kernel fits 5 anyway)
#ifndef OB_RES_MINW
#define OB_RES_MINW 5
#endif
#ifndef OB_G_RES
#define OB_G_RES 2
#endif
constexpr int G_RES = OB_G_RES;    // the single-pass kernel issues its loads G_RES accesses at a time
constexpr int TILE_MAIN = SPAN * U_MAIN;
constexpr int TILE_SRV = SPAN * U_SRV;
constexpr int TILE_RES = SPAN * U_RES;
#ifndef OB_U_LB
#define OB_U_LB 8
#endif
constexpr int U_LB = OB_U_LB;  // ... in the fused ratio+update kernel (v_frozen and signs stay in registers)
constexpr int TILE_LB = SPAN * U_LB;
constexpr int S_LH = 6;        // spans in LDS in the LDS form of k_ratios_apply_hist
#ifndef OB_U_WU
#define OB_U_WU 8
#endif
// safety margin, in tiles, under 80 % of the device's workgroup slots for the largest layer a
// barrier kernel takes
#ifndef OB_SPLIT_MARGIN
#define OB_SPLIT_MARGIN 8
#endif
constexpr int U_WU = OB_U_WU;  // ... in the single-pass warmup kernel (u and x stay in registers and LDS)
constexpr int TILE_WU = SPAN * U_WU;
#ifndef OB_G_WU
#define OB_G_WU 1
#endif
constexpr int G_WU = OB_G_WU;        // the single-pass warmup kernel issues its loads G_WU accesses at a time

enum KernelId {
  KID_MOMENTUM_Z = 0,
  KID_COMPRESS_RESIDENT,
  KID_CHUNK_SCALE,
  KID_SIGN_PACK,
  KID_COMPRESS_DEFERRED,
  KID_SERVER_AVG,
  KID_SERVER_SCALE,
  KID_SERVER_PACK,
  KID_SERVER_RESIDENT,
  KID_RATIOS_PASS,
  KID_RATIOS_FINALIZE,
  KID_APPLY,
  KID_RATIOS_APPLY_RESIDENT,
  KID_RATIOS_APPLY_HIST,
  KID_RATIOS_APPLY_HIST_LDS,
  KID_RATIOS_APPLY_SMALL,
  KID_WARMUP_SMALL,
  KID_VARIANCE_DENSE,
  KID_RATIOS_BIG_HIST,
  KID_RATIOS_TRAIL,
  KID_MOMENTUM_DENSE,
  KID_ERROR_DENSE,
  KID_MOMENTUM_SCALE,
  KID_WARMUP_MOMENTS,
  KID_WARMUP_COEFF,
  KID_WARMUP_APPLY,
  KID_WARMUP_RESIDENT,
  KID_WARMUP_TRAIL,
  KID_FILL,
  KID_COPY,
  KID_COUNT
};
const char* const kKernelNames[KID_COUNT] = {
    "momentum_z_sumsq", "compress_resident", "chunk_scale",     "sign_pack_error", "compress_deferred", "server_unpack_avg",
    "server_scale",     "server_sign_pack", "server_resident", "ratios_pass",     "ratios_finalize",
    "decompress_apply", "ratios_apply_resident", "ratios_apply_hist", "ratios_apply_hist_lds", "ratios_apply_small", "warmup_small", "variance_dense", "ratios_big_hist", "ratios_trail", "momentum_dense", "error_dense", "momentum_scale", "warmup_moments",   "warmup_coeff",    "warmup_apply",
    "warmup_resident",  "warmup_trail", "fill",            "copy"};

// Single-launch form of a list whose tiles all fit on the device at once (k_ratios_apply_small,
// k_warmup_small).
struct SmallPlan {
  int u = 0;                            // spans per tile; 0: not used
  int tpc = 0, n_tiles = 0, max_seg = 0;
  bool empty_layers = false;
  size_t lds_bytes = 0;
  SmallTile* d_tiles = nullptr;
  int* d_seg_layer = nullptr;
  int* d_layer_seg0 = nullptr;
  bool two_levels = false;                  // (k_warmup_small) of arrivals
  unsigned long long* d_slots = nullptr;    // [segments] (k_ratios_apply_small), or (k_warmup_small)
  double* d_partial = nullptr;          // [2 * segments]
  unsigned long long* d_counter = nullptr;
  unsigned long long* d_flag = nullptr;
};

struct ProfRec {
  int kid;
  hipEvent_t e0, e1;
};

// Split of the work between a kernel with a per-layer barrier and the plain kernels.  The barrier
// kernel takes "listed" tiles: the TILE_LB tiles that lie wholly inside one layer, for every layer
// whose such tiles all fit on the device at once (80 % of that kernel's workgroup slots).  The
// plain kernels take every other 1024-element tile that holds parameters ("rest" tiles: layers
// that are too large, the spans where layers meet, small tensors), and finish the layers that
// have no listed tile.  (Listing only the last tiles of a layer that is too large was measured:
// a run of layers that each fill the device to the limit stalls at every barrier, and the kernel
// fell from 5.8 to 3.5 TB/s on a GPT-1.3B-shaped list.)
struct LayerSplit {
  bool on = false;          // at least one tile is listed
  int n_fused_tiles = 0;    // listed TILE_LB tiles
  int n_rest_tiles = 0;     // TILE_MAIN tiles outside them that hold parameters
  int64_t n_layers = 0;     // layers with listed tiles
  int64_t n_params = 0;     // parameters in listed tiles
  int* d_fused_tiles = nullptr;
  int* d_n_listed = nullptr;               // [L] listed tiles of each layer
  int* d_list_begin = nullptr;             // [L] index in d_fused_tiles of the layer's first listed tile
  int* d_seg_first = nullptr;              // [L] first / one past the last segment (TILE_MAIN tiling) that the
  int* d_seg_end = nullptr;                //     layer's listed tiles cover
  float* d_listed_max = nullptr;           // [n_fused_tiles] partial results of the listed tiles
  double* d_listed_sums = nullptr;         // [2*n_fused_tiles]
  bool in_lds = false;      // form of k_ratios_apply_hist
  int tile = 0;             // elements per listed tile
  int tpc = 0;              // such tiles per chunk
  int* d_rest_tiles = nullptr;
  // The layers that are too large for the barrier kernel: their TILE_LB tiles ("big" tiles) take the
  // ratio pass with the variance in deferred form (ob_lamb_ratios_apply_hist only)
  bool big_on = false;                     // there are such tiles (and no wait has expired)
  int n_big_tiles = 0;
  int64_t n_big_params = 0;
  int* d_big_tiles = nullptr;
  // k_warmup_trail over them: its workgroups in order, and the end of each launch's share
  int one_level = ARRIVE_ONE_LEVEL;        // arrivals of a layer that are counted in one level
  bool trail_wait = false;
  unsigned int* d_items = nullptr;
  int n_items = 0;
  std::vector<int64_t> item_end;
  int* d_big_n = nullptr;                  // [L] big tiles of each layer
  int* d_big_begin = nullptr;              // [L] position of the first
  int* d_big_seg_first = nullptr;          // [L] first / one past the last segment that they cover
  int* d_big_seg_end = nullptr;
  int* d_count0 = nullptr;                 // [L] first counter
  unsigned int* d_count = nullptr;         // [counters] lines
  double* d_sub_sums = nullptr;            // [2 * counters]
  double* d_part_sums = nullptr;           // [2 * parts]
  bool hist_each_step = false;             // ob_lamb_ratios_apply takes ob_lamb_ratios_apply_hist's kernels
  // k_ratios_trail over them, the same way
  bool ratios_trail = false, trail_each_step = false;   // (ratios_trail_each_step)
  bool trail_pays[2] = {false, false};     // ratios_trail_pays, without and with a 16-bit copy
  float* d_sub_max = nullptr;              // [counters]
  float* d_tile_max = nullptr;             // [big tiles]
  unsigned long long* d_trail_flag = nullptr;   // [L]
  unsigned char* d_has_tiles = nullptr;    // [L] 1 for layers with listed or big tiles
  // k_ratios_apply_hist with the plain ratio pass in its launch (LayerSync), which counts arrivals of its own
  bool rest_in_launch = false;
  int n_alone = 0;
  int* d_alone = nullptr;
  int* d_arr0 = nullptr;
  int* d_skip_first = nullptr;
  int* d_skip_end = nullptr;
  int64_t n_arrivals = 0;
  unsigned long long* d_counter_rest = nullptr;
  unsigned long long* d_sub_rest = nullptr;
  unsigned long long* d_flag_rest = nullptr;
  int64_t n_events = 0;                    // 0: the update of the rest tiles is a launch of its own
  unsigned int* d_events = nullptr;
  unsigned long long* d_launches = nullptr;
  unsigned int* d_tail_launches = nullptr; // [rest tiles]
  int n_rest_ratio_tiles = 0;              // TILE_MAIN tiles outside the listed and the big tiles
  int* d_rest_ratio_tiles = nullptr;
  int n_cov_tiles = 0;                     // TILE_MAIN tiles inside the listed or the big tiles
  int* d_cov_tiles = nullptr;
  unsigned char* d_has_listed = nullptr;   // [L] 1 for layers that the barrier kernel finishes
  unsigned long long* d_counter = nullptr; // [L * CTR_STRIDE] (generation << 32) | arrivals
  unsigned long long* d_sub = nullptr;     // [group_lines(n_fused_tiles, L) * CTR_STRIDE] group counters
  unsigned long long* d_flag = nullptr;    // [L] (generation << 32) | payload
};

}  // namespace

struct ob_lamb_ctx {
  // configuration
  int64_t L = 0, N = 0, n_pad = 0, n_c = 0;
  int32_t W = 1, server_chunk = 0;
  float beta1, beta2, beta3, eta, c_min, c_max, r_min, r_max, r_thr, wd;
  float omb1, omb2, omb3, one_m_thr, one_p_thr, invW;
  // tiling
  int tpc = 0;        // TILE_MAIN tiles per chunk
  int n_tiles = 0;    // W * tpc
  int tpc_srv = 0;    // TILE_SRV tiles of the server chunk
  int u_srv = 1;      // spans per tile of the server kernel without a barrier
  int n_srv = 0;      // such tiles of the server chunk
  int n_segs = 0;     // (tile, layer) segments
  // device memory
  int device = -1;
  int64_t* d_off = nullptr;       // [L+2]
  int* d_first_layer = nullptr;   // [n_tiles]
  int* d_tile_seg0 = nullptr;     // [n_tiles+1]
  int* d_seg_layer = nullptr;     // [n_segs]
  int* d_layer_seg0 = nullptr;    // [L+1]
  double* d_partials = nullptr;   // [n_tiles]
  double* d_partials_srv = nullptr;  // [tpc_srv]
  double* d_seg_sums = nullptr;   // [2*n_segs]
  double* d_sigma = nullptr;      // [L] per-layer RMS (momentum-scale generation)
  float* d_seg_max = nullptr;     // [n_segs] per-segment max(v_frozen/v_fresh)
  // (chunk, layer) pairs and the per-step values of the variance in deferred form (VTerms)
  int n_pairs = 0;
  int* d_pair_base = nullptr;     // [W+1]
  int* d_pair_lfirst = nullptr;   // [W]
  int* d_pair_c = nullptr;        // [n_pairs]
  int* d_pair_l = nullptr;        // [n_pairs]
  float* d_vterms = nullptr;      // [(VF_MAX_OLD+1) * n_pairs * 2]
  // single-pass worker compression (k_compress_resident)
  bool resident = false;          // selected at create when the device can hold 2 chunks of tiles
  int tpc_res = 0, n_tiles_res = 0;
  int* d_first_layer_res = nullptr;        // [n_tiles_res]
  double* d_partials_res = nullptr;        // [n_tiles_res]
  unsigned long long* d_counter = nullptr; // [W * CTR_STRIDE] (generation << 32) | arrivals
  unsigned long long* d_sub = nullptr;     // [W * groups(tpc_res) * CTR_STRIDE] group counters
  unsigned long long* d_flag = nullptr;    // [W] (generation << 32) | scale bits
  unsigned int* d_errflag = nullptr;       // [1] raised when a bounded wait expired
  // single-pass server kernel (k_server_resident): selected at create when all of its workgroups
  // fit on the device at once
  int u_srv_res = 0;                           // its tile size in 1024-element spans; 0: not used
  int tpc_srv_res = 0;                         // such tiles of the server chunk
  double* d_partials_srv_res = nullptr;        // [tpc_srv_res]
  unsigned long long* d_counter_srv = nullptr; // [CTR_STRIDE]
  unsigned long long* d_sub_srv = nullptr;     // [groups(tpc_srv_res) * CTR_STRIDE]
  unsigned long long* d_flag_srv = nullptr;    // [1]
  int spin_limit = OB_SPIN_LIMIT_DEFAULT;
  // kernels with a per-layer barrier (k_ratios_apply_resident, k_warmup_resident): their common
  // tiling (TILE_LB; the segment arrays are those of the TILE_MAIN tiling) and, for each, the split
  // of the work between it and the plain kernels
  LayerSplit sp_apply;                     // ob_lamb_ratios_apply
  LayerSplit sp_warm;                      // ob_lamb_warmup_step
  SmallPlan sm_apply, sm_warm;             // the same calls on lists small enough for one launch
  bool sum_lds = false;                    // worker_sum_lds
  unsigned int* d_ticket = nullptr;        // chunk_ticket: counters of the worker's chunks (NULL: not used)
  unsigned int* d_ticket_srv = nullptr;    // ... of the served chunk
  double* d_ticket_part = nullptr;
  double* d_ticket_part_srv = nullptr;
  void* d_mem = nullptr;                   // the allocation that holds all of the arrays above (Workspace)
  size_t device_bytes = 0;                 // its size
  // diagnostics
  bool profile = false;
  std::vector<ProfRec> prof;
  std::string hip_err;
};

namespace {

bool hip_ok(ob_lamb_ctx* ctx, hipError_t e, const char* what) {
  if (e == hipSuccess) return true;
  if (ctx) ctx->hip_err = std::string(what) + ": " + hipGetErrorString(e);
  return false;
}

inline bool misaligned(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

struct Launch {
  ob_lamb_ctx* ctx;
  hipStream_t stream;
  bool ok = true;
  Launch(ob_lamb_ctx* c, void* s) : ctx(c), stream(reinterpret_cast<hipStream_t>(s)) {}
  // A timing record for the coming launch (profile mode).  record_start: also record its first
  // event on the stream now (device copies); kernels hand both events to the launch instead, which
  // stamps them with the kernel's own start and end on the device.
  bool begin(int kid, bool record_start) {
    if (!ctx->profile || !ok) return false;
    ProfRec r;
    r.kid = kid;
    ok = hip_ok(ctx, hipEventCreate(&r.e0), "hipEventCreate") &&
         hip_ok(ctx, hipEventCreate(&r.e1), "hipEventCreate") &&
         (!record_start || hip_ok(ctx, hipEventRecord(r.e0, stream), "hipEventRecord"));
    if (ok) ctx->prof.push_back(r);
    return ok;
  }
  void end(const char* name, bool record_stop) {
    if (!ok) return;
    ok = hip_ok(ctx, hipGetLastError(), name);
    if (ok && ctx->profile && record_stop)
      ok = hip_ok(ctx, hipEventRecord(ctx->prof.back().e1, stream), "hipEventRecord");
  }
};

#define OB_LAUNCH_S(la, kid, kernel, grid, block, lds_bytes, ...)                 \
  do {                                                                            \
    if ((la).ok && (grid) > 0) {                                                  \
      if ((la).begin(kid, false))                                                 \
        hipExtLaunchKernelGGL(kernel, dim3((unsigned)(grid)), dim3(block), lds_bytes, (la).stream, \
                              (la).ctx->prof.back().e0, (la).ctx->prof.back().e1, 0, __VA_ARGS__); \
      else if ((la).ok)                                                           \
        hipLaunchKernelGGL(kernel, dim3((unsigned)(grid)), dim3(block), lds_bytes, (la).stream, __VA_ARGS__); \
      (la).end(kKernelNames[kid], false);                                         \
    }                                                                             \
  } while (0)
#define OB_LAUNCH_B(la, kid, kernel, grid, block, ...) OB_LAUNCH_S(la, kid, kernel, grid, block, 0, __VA_ARGS__)
#define OB_LAUNCH(la, kid, kernel, grid, ...) OB_LAUNCH_B(la, kid, kernel, grid, BLOCK, __VA_ARGS__)

// The device memory of a context is ONE allocation, so that what ob_lamb_create costs does not grow with the
// number of tables a configuration needs: upload() and alloc_zero() note what goes where, commit() allocates, sets
// the pointers, copies the small tables together and the large ones from where they are.  Every array starts at a
// multiple of 256 bytes.  (A context of four 512x512 tensors, some 60 arrays: 490 us with an allocation each, 69.)
class Workspace {
 public:
  template <class T>
  void upload(T** dst, std::vector<T> src) {
    auto keep = std::make_shared<std::vector<T>>(std::move(src));
    const size_t bytes = keep->size() * sizeof(T);
    (bytes < SMALL ? small_ : large_).push_back({reinterpret_cast<void**>(dst), keep->data(), bytes, keep});
  }
  template <class T>
  void alloc_zero(T** dst, size_t count) {
    zeroed_.push_back({reinterpret_cast<void**>(dst), nullptr, count * sizeof(T), nullptr});
  }
  bool commit(ob_lamb_ctx* ctx) {
    std::vector<unsigned char> head(size_of(small_));
    const size_t zero_at = head.size() + size_of(large_), total = zero_at + size_of(zeroed_);
    if (!hip_ok(ctx, hipMalloc(&ctx->d_mem, total), "hipMalloc")) return false;
    ctx->device_bytes = total;
    unsigned char* const base = static_cast<unsigned char*>(ctx->d_mem);
    size_t at = 0;
    for (const Array& a : small_) {
      if (a.bytes) std::memcpy(head.data() + at, a.src, a.bytes);
      *a.dst = base + at;
      at += room(a.bytes);
    }
    bool ok = hip_ok(ctx, hipMemcpy(base, head.data(), head.size(), hipMemcpyHostToDevice), "hipMemcpy");
    for (const Array& a : large_) {
      ok = ok && hip_ok(ctx, hipMemcpy(base + at, a.src, a.bytes, hipMemcpyHostToDevice), "hipMemcpy");
      *a.dst = base + at;
      at += room(a.bytes);
    }
    for (const Array& a : zeroed_) {
      *a.dst = base + at;
      at += room(a.bytes);
    }
    return ok && hip_ok(ctx, hipMemset(base + zero_at, 0, total - zero_at), "hipMemset");
  }

 private:
  struct Array {
    void** dst;
    const void* src;
    size_t bytes;
    std::shared_ptr<void> keep;   // what src points into
  };
  static constexpr size_t SMALL = 65536;
  static size_t room(size_t bytes) { return (std::max<size_t>(bytes, 1) + 255) / 256 * 256; }
  static size_t size_of(const std::vector<Array>& v) {
    size_t n = 0;
    for (const Array& a : v) n += room(a.bytes);
    return n;
  }
  std::vector<Array> small_, large_, zeroed_;
};

ob_status check_common(const ob_lamb_ctx* ctx, const ob_lamb_state* st) {
  if (!ctx || !st) return OB_ERR_NULL;
  // the context's tables live on the device it was created on
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev != ctx->device) return OB_ERR_ARG;
  return OB_OK;
}

#define REQUIRE_PTR(p)                    \
  do {                                    \
    if ((p) == nullptr) return OB_ERR_NULL; \
    if (misaligned(p)) return OB_ERR_ALIGN; \
  } while (0)

// ---- small helpers for the entry points -------------------------------------------------------

LayerTab layer_tab(const ob_lamb_ctx* ctx, const ob_lamb_state* st, const int* first_layer) {
  LayerTab lt;
  lt.mom_scale = st->mom_scale;
  lt.off = ctx->d_off;
  lt.first_layer = first_layer;
  lt.L = (int)ctx->L;
  return lt;
}

// Calls f(std::bool_constant<a>, std::bool_constant<b>) so that kernels can take a and b as
// template arguments.
template <class F>
void dispatch2(bool a, bool b, F f) {
  if (a) {
    if (b) f(std::true_type{}, std::true_type{});
    else f(std::true_type{}, std::false_type{});
  } else {
    if (b) f(std::false_type{}, std::true_type{});
    else f(std::false_type{}, std::false_type{});
  }
}

// Calls f(std::bool_constant<a>).
template <class F>
void dispatch1(bool a, F f) {
  if (a) f(std::true_type{});
  else f(std::false_type{});
}

// Gradient argument of the _lp entry points -> kernel argument; *lp: 16-bit source.
ob_status grad_source(const void* grad, int dtype, float scale, GradSrc* gs, bool* lp) {
  if (!grad) return OB_ERR_NULL;
  if (misaligned(grad)) return OB_ERR_ALIGN;
  if (dtype != OB_F32 && dtype != OB_F16 && dtype != OB_BF16) return OB_ERR_ARG;
  if (dtype == OB_F32 && scale != 1.0f) return OB_ERR_ARG;
  if (!std::isfinite(scale)) return OB_ERR_ARG;
  gs->p = grad;
  gs->scale = scale;
  gs->bf16 = (dtype == OB_BF16) ? 1 : 0;
  *lp = (dtype != OB_F32);
  return OB_OK;
}

// 16-bit parameter copy of the _lp entry points (NULL: none).
struct XLp {
  void* p = nullptr;
  int bf16 = 0;
};
ob_status x_lp_target(void* x_lp, int dtype, XLp* out) {
  out->p = nullptr;
  out->bf16 = 0;
  if (!x_lp) return OB_OK;
  if (dtype != OB_F16 && dtype != OB_BF16) return OB_ERR_ARG;
  if (misaligned(x_lp)) return OB_ERR_ALIGN;
  out->p = x_lp;
  out->bf16 = (dtype == OB_BF16) ? 1 : 0;
  return OB_OK;
}

// The momentum source of a call: dense st->m if given, else the 1-bit form.
ob_status momentum_source(const ob_lamb_state* st, bool* packed, PackedMom* pm) {
  pm->bits = nullptr;
  pm->scales = nullptr;
  if (st->m) {
    if (misaligned(st->m)) return OB_ERR_ALIGN;
    *packed = false;
    return OB_OK;
  }
  if (!st->m_packed || !st->m_scales) return OB_ERR_NULL;
  if (misaligned(st->m_packed)) return OB_ERR_ALIGN;
  *packed = true;
  pm->bits = st->m_packed;
  pm->scales = st->m_scales;
  return OB_OK;
}

// Plans and uploads one LayerSplit.
void build_split(ob_lamb_ctx* ctx, Workspace* ws, const Tiling& tl, int tile_lb, const Tiling& tm,
                 const std::vector<int64_t>& h_off, int64_t max_tiles, const BigRule& rule, bool trail, int cus, LayerSplit* sp,
                 std::vector<unsigned char>* lagging) {
  const int64_t L = ctx->L;
  SplitPlan pl;
  plan_split(tl, tile_lb, tm, h_off, ctx->n_c, L, max_tiles, rule, &pl);
  sp->tile = tile_lb;
  sp->tpc = (int)tl.tpc;
  sp->n_layers = pl.n_layers;
  sp->n_params = pl.n_params;
  sp->on = !pl.fused_tiles.empty();
  sp->n_fused_tiles = (int)pl.fused_tiles.size();
  sp->n_rest_tiles = (int)pl.rest_tiles.size();
  std::vector<int> cov;
  for (int64_t t = 0; t < tm.n_tiles; ++t)
    if (pl.covered[(size_t)t] || pl.covered_big[(size_t)t]) cov.push_back((int)t);
  sp->n_cov_tiles = (int)cov.size();
  sp->n_big_tiles = (int)pl.big_tiles.size();
  sp->big_on = sp->n_big_tiles > 0;
  sp->n_big_params = pl.n_big_params;
  sp->n_rest_ratio_tiles = (int)pl.rest_ratio_tiles.size();
  lagging->assign((size_t)tm.n_tiles, 0);
  for (int t : cov) (*lagging)[(size_t)t] = 1;
  sp->one_level = arrivals_one_level(sp->n_fused_tiles, cus);
  sp->trail_wait = max_tiles > 0;
  // (where both are possible, four steps, us, rest_in_launch / k_ratios_trail: 3880 large and 560 listed tiles 904 / 894, 3800 and 1150
  // 960 / 955, 2500 and 2030 903 / 910; the line: three times the listed tiles and 12 tiles a CU)
  const bool rest = !trail && rest_in_launch(sp->n_rest_ratio_tiles, sp->n_fused_tiles, sp->n_big_tiles, cus, sp->n_layers);
  sp->ratios_trail = !trail && sp->trail_wait && ratios_trail(pl.big_n, cus) &&
                     (!rest || (sp->n_big_tiles >= 3 * sp->n_fused_tiles && sp->n_big_tiles >= 12 * cus));
  for (int copy = 0; copy < 2; ++copy) sp->trail_pays[copy] = ratios_trail_pays(pl.big_n, copy != 0);
  sp->rest_in_launch = rest && !sp->ratios_trail;
  sp->trail_each_step = sp->big_on && ratios_trail_each_step(pl.big_n);
  if ((trail && sp->big_on) || sp->ratios_trail) {
    static_assert(TILE_WU == 8 * SPAN && TILE_LB == 8 * SPAN, "tiles of k_warmup_trail and k_ratios_trail");
    const int parts = trail ? TRAIL_PARTS : 1;   // of a tile
    std::vector<int> n = pl.big_n, begin = pl.big_begin;   // in parts
    for (int& q : n) q *= parts;
    for (int& q : begin) q *= parts;
    std::vector<unsigned int> items;
    if (trail) trail_items(n, begin, sp->trail_wait ? trail_lag(cus) : 0, TRAIL_GROUP, &items, &sp->item_end);
    else ratios_trail_items(n, begin, cus, &items);
    sp->n_items = (int)items.size();
    ws->upload(&sp->d_items, std::move(items));
    std::vector<int> count0((size_t)L, 0);
    std::vector<unsigned char> has_tiles = pl.has_listed;
    int counters = 0;
    for (int64_t l = 0; l < L; ++l) {
      count0[(size_t)l] = counters;
      if (n[(size_t)l] == 0) continue;
      has_tiles[(size_t)l] = 1;
      counters += 1 + (n[(size_t)l] + TICKET_SUB - 1) / TICKET_SUB;
    }
    ws->upload(&sp->d_count0, std::move(count0));
    ws->upload(&sp->d_has_tiles, std::move(has_tiles));
    ws->upload(&sp->d_big_n, std::move(pl.big_n));
    ws->upload(&sp->d_big_begin, std::move(pl.big_begin));
    ws->upload(&sp->d_big_seg_first, std::move(pl.big_seg_first));
    ws->upload(&sp->d_big_seg_end, std::move(pl.big_seg_end));
    ws->alloc_zero(&sp->d_count, (size_t)counters * 2 * CTR_STRIDE);
    if (trail) {
      ws->alloc_zero(&sp->d_sub_sums, 2 * (size_t)counters);
      ws->alloc_zero(&sp->d_part_sums, 2 * (size_t)TRAIL_PARTS * (size_t)sp->n_big_tiles);
    } else {
      ws->alloc_zero(&sp->d_sub_max, (size_t)counters);
      ws->alloc_zero(&sp->d_tile_max, (size_t)sp->n_big_tiles);
    }
    ws->alloc_zero(&sp->d_trail_flag, (size_t)L);
  }
  if (sp->rest_in_launch) {
    ArrivalPlan ap;
    plan_arrivals(pl, tm, L, &ap);
    sp->n_arrivals = ap.n_arrivals;
    sp->n_alone = (int)ap.alone.size();
    if (!sp->big_on && sp->n_rest_ratio_tiles > 0) {
      sp->n_events = coefficient_events(pl, tm, L, ap);
      ws->alloc_zero(&sp->d_events, 2 * CTR_STRIDE);
      ws->alloc_zero(&sp->d_launches, CTR_STRIDE);
      ws->alloc_zero(&sp->d_tail_launches, (size_t)sp->n_rest_ratio_tiles);
    }
    ws->upload(&sp->d_alone, std::move(ap.alone));
    ws->upload(&sp->d_arr0, std::move(ap.arr0));
    ws->upload(&sp->d_skip_first, std::move(ap.skip_first));
    ws->upload(&sp->d_skip_end, std::move(ap.skip_end));
    ws->alloc_zero(&sp->d_counter_rest, (size_t)L * CTR_STRIDE);
    ws->alloc_zero(&sp->d_sub_rest, group_lines(sp->n_arrivals, L) * CTR_STRIDE);
    ws->alloc_zero(&sp->d_flag_rest, (size_t)L);
  }
  ws->upload(&sp->d_cov_tiles, std::move(cov));
  ws->upload(&sp->d_big_tiles, std::move(pl.big_tiles));
  ws->upload(&sp->d_rest_ratio_tiles, std::move(pl.rest_ratio_tiles));
  ws->upload(&sp->d_fused_tiles, std::move(pl.fused_tiles));
  ws->upload(&sp->d_n_listed, std::move(pl.n_listed));
  ws->upload(&sp->d_list_begin, std::move(pl.list_begin));
  ws->upload(&sp->d_seg_first, std::move(pl.seg_first));
  ws->upload(&sp->d_seg_end, std::move(pl.seg_end));
  ws->upload(&sp->d_rest_tiles, std::move(pl.rest_tiles));
  ws->upload(&sp->d_has_listed, std::move(pl.has_listed));
  ws->alloc_zero(&sp->d_listed_max, (size_t)sp->n_fused_tiles);
  ws->alloc_zero(&sp->d_listed_sums, 2 * (size_t)sp->n_fused_tiles);
  ws->alloc_zero(&sp->d_counter, (size_t)L * CTR_STRIDE);
  ws->alloc_zero(&sp->d_sub, group_lines(sp->n_fused_tiles, L) * CTR_STRIDE);
  ws->alloc_zero(&sp->d_flag, (size_t)L);
}

// Chooses and uploads a SmallPlan: small_choice among the U whose tiles take at most 80 % of the device's workgroup slots
// (slots(U, dynamic LDS bytes)).  vals, tables: 4-byte words of LDS per element and per segment of a tile that
// meets several layers; by_slots: the barriers are those of slots; split: the barrier kernel of the larger lists.
template <class F>
bool build_small(ob_lamb_ctx* ctx, Workspace* ws, SmallTilings* tilings, const std::vector<int64_t>& h_off,
                 const std::vector<unsigned char>& lagging, const LayerSplit& split, int vals, int tables, bool by_slots, int cus,
                 F slots, SmallPlan* sp) {
  static_assert(TILE_MAIN == SPAN, "the TILE_MAIN tiling is that of U = 1");
  bool fits[3] = {false, false, false};
  size_t lds_bytes[3] = {0, 0, 0};
  for (int i = 0; i < 3; ++i) {
    const SmallShape& s = tilings->sh[i];
    if (s.n_tiles == 0) continue;
    lds_bytes[i] = 4 * ((size_t)vals * (SPAN << i) + (size_t)tables * (size_t)s.max_seg);
    int64_t n_slots = 0;
    if (!slots(1 << i, lds_bytes[i], &n_slots)) return false;
    fits[i] = 5 * (s.n_tiles + 8) <= 4 * n_slots;
  }
  int choice = small_choice(tilings->sh, fits, by_slots, cus);
  if (choice >= 0 && split.on && split.n_rest_tiles == 0 && ((int64_t)tilings->sh[choice].max_arrivals << choice) > SMALL_MAX_SPANS)
    choice = -1;
  const int best = choice < 0 ? 0 : 1 << choice;
  const SmallShape sh = choice < 0 ? SmallShape() : tilings->sh[choice];
  if (best) sp->lds_bytes = lds_bytes[choice];
  const Tiling* tp = best ? tilings->get(best, ctx->n_c, ctx->W, ctx->L, h_off) : nullptr;
  if (tp) {
    const Tiling& t = *tp;
    std::vector<SmallTile> tiles;
    small_tiles(t, best, tilings->tm, h_off, ctx->n_c, ctx->L, lagging, &tiles);
    sp->tpc = (int)sh.tpc;
    sp->n_tiles = (int)sh.n_tiles;
    sp->max_seg = sh.max_seg;
    for (int64_t l = 0; l < ctx->L; ++l)
      if (t.layer_seg0[(size_t)l + 1] == t.layer_seg0[(size_t)l]) sp->empty_layers = true;
    ws->upload(&sp->d_tiles, std::move(tiles));
    ws->upload(&sp->d_seg_layer, t.seg_layer);
    ws->upload(&sp->d_layer_seg0, t.layer_seg0);
    if (by_slots) {
      ws->alloc_zero(&sp->d_slots, t.seg_layer.size());
    } else {
      ws->alloc_zero(&sp->d_partial, 2 * t.seg_layer.size());
      sp->two_levels = sh.max_arrivals > SMALL_ONE_LEVEL;
      const size_t groups = sp->two_levels ? group_lines((int64_t)t.seg_layer.size(), ctx->L) : 0;
      ws->alloc_zero(&sp->d_counter, ((size_t)ctx->L + groups) * CTR_STRIDE);
      ws->alloc_zero(&sp->d_flag, (size_t)ctx->L * CTR_STRIDE);
    }
    sp->u = best;
  }
  return true;
}

SmallTab small_tab(const ob_lamb_ctx* ctx, const SmallPlan& sp) {
  SmallTab t;
  t.tiles = sp.d_tiles; t.n_tiles = sp.n_tiles; t.tpc = sp.tpc; t.max_seg = sp.max_seg; t.n_c = ctx->n_c;
  t.seg_layer = sp.d_seg_layer; t.layer_seg0 = sp.d_layer_seg0;
  t.partial = sp.d_slots ? (void*)sp.d_slots : (void*)sp.d_partial;
  t.counter = sp.d_counter; t.flag = sp.d_flag;
  t.errflag = ctx->d_errflag; t.spin_limit = ctx->spin_limit;
  return t;
}

// Calls f(integral_constant<int, u>) for u in {1, 2, 4}.
template <class F>
void dispatch_u(int u, F f) {
  switch (u) {
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    default: f(std::integral_constant<int, 4>{}); break;
  }
}

// Which chunks get their scale from the kernel that forms the partials (chunk_ticket) instead of a launch of
// k_chunk_scale.  That launch costs 2.5 us and a gap; the ticket costs every workgroup a wait for its stores and
// a returning atomic before it retires, and the last ones of up to 64 tiles a second one where a chunk has more
// than 64 (TICKET_SUB).  n_tiles: the worker's 1024-element tiles; a round: 8 workgroups per CU.  A step, us, with
// a launch / with the ticket in the worker's call (256 CUs):
//   chunks of at most 64 tiles: 1024 tiles 26.4 / 22.6, 2048 28.8 / 27.7, 4096 41.2 / 41.0, 8192 61.8 / 61.0, 16384 110.2 / 110.3
//   more:  640 tiles 27.1 / 23.3, 1536 26.7 / 23.9, 2560 31.6 / 31.2, 3072 32.8 / 33.2, 6144 50.3 / 50.1, 8192 59.0 / 59.4,
//          14336 93.2 / 94.0, 24576 137.2 / 140.8, 40960 220.1 / 227.1; chunks of 512 39.7 / 40.2, of 1376 75.1 / 74.4
// and in the server's, whose grid is the one chunk:
//   at most 64 tiles: of 1024 26.4 / 22.8, of 4096 41.2 / 41.3, of 8192 61.8 / 61.3, of 16384 110.2 / 108.7
//   more:  of 640 27.1 / 23.4, of 2560 31.6 / 32.0, of 6144 50.3 / 50.7, of 8192 59.0 / 59.3, of 24576 137.2 / 139.4, of 40960 220.1 /
//          221.8; but chunks of 1376 75.1 / 74.0 (eight workers), of 2048 102.9 / 101.7, which the line leaves with a launch
// (Steps with the host in them; lists of less than 1000 tiles are bound by it.)
bool two_level_ticket(int tpc, int n_tiles, int cus) { return tpc <= 256 && n_tiles <= 3 * 8 * cus; }
bool worker_ticket(int tpc, int n_tiles, int cus) {
  return (tpc <= TICKET_SUB && n_tiles <= 5 * 8 * cus) || two_level_ticket(tpc, n_tiles, cus);
}
bool server_ticket(int tpc, int n_tiles, int cus) { return tpc <= TICKET_SUB || two_level_ticket(tpc, n_tiles, cus); }

ChunkTicket chunk_ticket_of(unsigned int* count, double* part, int n_chunks, int tpc, float* scales, float* own_scale,
                            int own_chunk) {
  ChunkTicket tk;
  tk.count = count; tk.sub_part = part; tk.n_chunks = n_chunks; tk.spc = (tpc + TICKET_SUB - 1) / TICKET_SUB;
  tk.scales = scales; tk.own_scale = own_scale; tk.own_chunk = own_chunk;
  return tk;
}

ListedTiles listed_tiles(const ob_lamb_ctx* ctx, const LayerSplit& sp) {
  ListedTiles lt;
  lt.tile_list = sp.d_fused_tiles; lt.list_begin = sp.d_list_begin; lt.n_listed = sp.d_n_listed;
  lt.seg_first = sp.d_seg_first; lt.seg_end = sp.d_seg_end; lt.layer_seg0 = ctx->d_layer_seg0;
  lt.n_c = ctx->n_c; lt.tpc = sp.tpc; lt.tpc_span = ctx->tpc;
  lt.one_level = sp.one_level;
  return lt;
}

// ... of the layers that are too large for the barrier kernel
ListedTiles big_tiles(const ob_lamb_ctx* ctx, const LayerSplit& sp) {
  ListedTiles lt = listed_tiles(ctx, sp);
  lt.tile_list = sp.d_big_tiles; lt.list_begin = sp.d_big_begin; lt.n_listed = sp.d_big_n;
  lt.seg_first = sp.d_big_seg_first; lt.seg_end = sp.d_big_seg_end;
  return lt;
}

// Which form of k_ratios_apply_hist a list takes: with registers only OB_LB_MINW (5) workgroups fit on a CU, with
// LDS LH_WG_LDS (6), and each is the better one by how many rounds of the device's workgroups its listed tiles
// make.  Whole steps on 256 CUs, us, registers / LDS, lists of equal square tensors and of BERT shape (whose word
// embedding is too large to be listed: what counts is the kernel's tiles, not the parameters):
//   one round only with LDS (1281 to 1536 tiles): 1345 94.0 / 89.7, 1440 82.8 / 77.9, 1536 86.6 / 81.0
//   below and between, where the way through LDS costs more than a sixth workgroup gives: 864 54.8 / 56.8,
//     1027 68.2 / 69.5, 1608 184.9 / 187.3, 1913 109.2 / 113.9, 2056 110.3 / 111.6, 2304 113.4 / 115.8, 2516 244.4 / 244.2
//   two full rounds with registers (2560 tiles) to six with LDS (9216): 2560 128.3 / 122.6, 2789 142.3 / 138.3,
//     3072 148.3 / 140.5, 4896 221.2 / 209.0, 7776 330.6 / 318.5, 8928 381.7 / 362.8, 9216 393.2 / 386.2; the least
//     gain in 2800x2800 tensors (957 tiles each): 2869 156.7 / 156.5, 3827 199.2 / 200.2, 8605 416.8 / 418.2
//   beyond, where more tiles in flight make the arrays' reads slower: 9561 460.6 / 468.3, 9760 432.0 / 443.0,
//     10489 579.4 / 586.2, 13386 636.3 / 670.7
constexpr int LH_LDS_MIN_ROUNDS = 2, LH_LDS_MAX_ROUNDS = 6;
bool lh_in_lds(int64_t n_tiles, int cus) {
  const int64_t r = (int64_t)OB_LB_MINW * cus, l = (int64_t)LH_WG_LDS * cus;
  return (n_tiles > r && n_tiles <= l) || (n_tiles >= LH_LDS_MIN_ROUNDS * r && n_tiles <= LH_LDS_MAX_ROUNDS * l);
}

// Whether ob_lamb_ratios_apply, which rewrites the variance at every step, takes ob_lamb_ratios_apply_hist's kernels with no history: the
// same bytes, in fewer launches or in the form of the kernel that the list's rounds favour.  A step, us, k_ratios_apply_resident and the plain
// kernels around it / these (256 CUs):
//   rest tiles' passes in the launch: 4.2 M 50.4 / 41.5, 11 M 95.3 / 81.4, 15 M 117 / 110, 30 M 190.7 / 182, 49 M with a 16-bit copy 315.5 / 298.5
//   v_frozen in LDS: 21 M 135.2 / 134.4, 32 M 201 / 192, 42 M 252.3 / 247, 63 M 378.6 / 367
//   neither: 4.2 M without rest tiles 39.8 / 40.5, 260 M 1422.4 / 1423.8, 215 M with a 16-bit copy 1254 / 1262, 314 M 1785.6 / 1790.5
//   k_ratios_trail: 1.3e9 in layers of which the largest is a twelfth 7370 / 7240, 300 M with one of more than a third 1523.6 / 1528.5
//   k_ratios_big_hist: 110 M 626.5 / 637.5, 336 M 1818 / 1827.5
// (Lists of less than a tile a CU come here only where a configuration asks for the larger lists' launches.)
bool hist_each_step(const LayerSplit& sp, int cus) {
  if (!sp.on || sp.n_fused_tiles < cus) return false;
  if (sp.big_on) return sp.ratios_trail && sp.trail_each_step;
  return sp.in_lds || (sp.rest_in_launch && sp.n_rest_ratio_tiles > 0);
}

// Largest number of one layer's tiles that a barrier kernel with `per_cu` resident workgroups per
// CU may hold: 80 % of the device's slots, or the configuration's fused_max_tiles if that is lower
// (cap; 0 = none).
int64_t split_max_tiles(int per_cu, int cus, int32_t cap) {
  int64_t max_tiles = (4 * (int64_t)per_cu * cus) / 5 - OB_SPLIT_MARGIN;
  if (cap > 0 && cap < max_tiles) max_tiles = cap;
  return max_tiles < 0 ? 0 : max_tiles;
}

RatioArgs ratio_args(const ob_lamb_ctx* ctx, const ob_lamb_state* st, const uint32_t* packed_all,
                     const float* server_scales, const PackedMom& pm) {
  RatioArgs ra;
  ra.packed = packed_all; ra.sscales = server_scales; ra.m = st->m; ra.pm = pm;
  ra.v_fresh = st->v_fresh; ra.v_frozen = st->v_frozen;
  ra.beta1 = ctx->beta1; ra.omb1 = ctx->omb1; ra.beta2 = ctx->beta2; ra.omb2 = ctx->omb2;
  ra.r_prev = st->r_prev; ra.one_m_thr = ctx->one_m_thr; ra.r_min = ctx->r_min;
  return ra;
}

// Launches of the plain ratio pass and finalize kernels.  tiles: the 1024-element tiles to cover
// (NULL: all, in order), n_launch_tiles of them; layers with done_elsewhere[l] != 0 (NULL: none) are
// left to be finished by the kernel with the per-layer barrier.
void launch_ratios(Launch& la, ob_lamb_ctx* ctx, const ob_lamb_state* st, const uint32_t* packed_all,
                   const float* server_scales, bool packed_m, const PackedMom& pm, const int* tiles,
                   int n_launch_tiles, const unsigned char* done_elsewhere, bool finalize) {
  const RatioArgs ra = ratio_args(ctx, st, packed_all, server_scales, pm);
  const LayerTab lt = layer_tab(ctx, st, ctx->d_first_layer);
  dispatch2(st->mom_scale != nullptr, packed_m, [&](auto hk, auto pk) {
    dispatch1(keeps_second_reads(ctx->N, ctx->W), [&](auto kp) {
      OB_LAUNCH(la, KID_RATIOS_PASS, (k_ratios_pass<U_MAIN, decltype(hk)::value, decltype(pk)::value, decltype(kp)::value>),
                n_launch_tiles, ra, ctx->d_seg_max, ctx->n_c, ctx->tpc, lt, ctx->d_tile_seg0, ctx->d_seg_layer, tiles);
    });
  });
  if (finalize)
    OB_LAUNCH_B(la, KID_RATIOS_FINALIZE, k_ratios_finalize, (int)ctx->L, FBLOCK, ctx->d_seg_max,
                ctx->d_layer_seg0, st->c_avg, st->r_prev, st->coeff_c, ctx->one_m_thr, ctx->one_p_thr,
                ctx->r_min, ctx->r_max, done_elsewhere);
}

ApplyArgs apply_args(const ob_lamb_ctx* ctx, const ob_lamb_state* st, const uint32_t* packed_all,
                     const float* server_scales, float lr, const XLp& xl) {
  ApplyArgs aa;
  aa.packed = packed_all; aa.sscales = server_scales; aa.v_frozen = st->v_frozen; aa.x = st->x;
  aa.m = st->m; aa.coeff_c = st->coeff_c; aa.lr = lr; aa.eta = ctx->eta;
  aa.x_lp = xl.p; aa.x_lp_bf16 = xl.bf16;
  return aa;
}

void launch_apply(Launch& la, ob_lamb_ctx* ctx, const ob_lamb_state* st, const uint32_t* packed_all,
                  const float* server_scales, float lr, const int* tiles, int n_launch_tiles, const XLp& xl) {
  const ApplyArgs aa = apply_args(ctx, st, packed_all, server_scales, lr, xl);
  const LayerTab lt = layer_tab(ctx, st, ctx->d_first_layer);
  dispatch2(st->mom_scale != nullptr, st->m != nullptr, [&](auto hk, auto wm) {
    dispatch1(xl.p != nullptr, [&](auto lx) {
      OB_LAUNCH(la, KID_APPLY,
                (k_decompress_apply<U_MAIN, decltype(hk)::value, decltype(wm)::value, decltype(lx)::value>),
                n_launch_tiles, aa, ctx->n_c, ctx->tpc, lt, tiles);
    });
  });
}

void launch_ratios_apply_small(Launch& la, ob_lamb_ctx* ctx, const ob_lamb_state* st, const RatioArgs& ra,
                               const VfHist& vh, const ApplyArgs& aa) {
  const SmallPlan& sm = ctx->sm_apply;
  RatioClip rc;
  rc.c_avg = st->c_avg; rc.r_prev = st->r_prev; rc.coeff_c = st->coeff_c;
  rc.one_m_thr = ctx->one_m_thr; rc.one_p_thr = ctx->one_p_thr; rc.r_min = ctx->r_min; rc.r_max = ctx->r_max;
  const LayerTab lt = layer_tab(ctx, st, ctx->d_first_layer);
  dispatch_u(sm.u, [&](auto u) {
    dispatch2(st->mom_scale != nullptr, aa.x_lp != nullptr, [&](auto hk, auto lx) {
      OB_LAUNCH_S(la, KID_RATIOS_APPLY_SMALL,
                  (k_ratios_apply_small<decltype(u)::value, decltype(hk)::value, decltype(lx)::value>),
                  sm.n_tiles + (sm.empty_layers ? 1 : 0), BLOCK, sm.lds_bytes, ra, vh, aa, small_tab(ctx, sm), rc, lt);
    });
  });
}

// commit of the 1-bit momentum (see ob_lamb_decompress_apply)
void commit_packed_momentum(Launch& la, ob_lamb_ctx* ctx, const ob_lamb_state* st,
                                   const uint32_t* packed_all, const float* server_scales) {
  if (!(st->m_packed && st->m_packed != packed_all)) return;
  la.begin(KID_COPY, true);
  if (la.ok)
    la.ok = hip_ok(ctx, hipMemcpyAsync(st->m_packed, packed_all, (size_t)ctx->n_pad / 8,
                                       hipMemcpyDeviceToDevice, la.stream), "hipMemcpyAsync") &&
            hip_ok(ctx, hipMemcpyAsync(st->m_scales, server_scales, (size_t)ctx->W * sizeof(float),
                                       hipMemcpyDeviceToDevice, la.stream), "hipMemcpyAsync");
  la.end("copy", true);
}

ob_status check_ratios_args(const ob_lamb_ctx* ctx, const ob_lamb_state* st, const uint32_t* packed_all,
                                   const float* server_scales) {
  if (ob_status s = check_common(ctx, st)) return s;
  REQUIRE_PTR(packed_all); REQUIRE_PTR(st->v_fresh); REQUIRE_PTR(st->v_frozen);
  if (!server_scales || !st->c_avg || !st->r_prev || !st->coeff_c) return OB_ERR_NULL;
  return OB_OK;
}

ob_status check_apply_args(const ob_lamb_ctx* ctx, const ob_lamb_state* st, const uint32_t* packed_all,
                                  const float* server_scales, float lr) {
  if (ob_status s = check_common(ctx, st)) return s;
  REQUIRE_PTR(packed_all); REQUIRE_PTR(st->x); REQUIRE_PTR(st->v_frozen);
  if (!server_scales || !st->coeff_c) return OB_ERR_NULL;
  if (!std::isfinite(lr)) return OB_ERR_ARG;
  if (st->m && misaligned(st->m)) return OB_ERR_ALIGN;
  if (!st->m && !st->m_packed) return OB_ERR_NULL;  // the momentum has to be committed somewhere
  if (st->m_packed && !st->m_scales) return OB_ERR_NULL;
  if (st->m_packed && misaligned(st->m_packed)) return OB_ERR_ALIGN;
  return OB_OK;
}

}  // namespace

extern "C" {

int64_t ob_lamb_padded_len_for(int64_t n, int32_t W) {
  if (n < 0 || W < 1) return 0;
  const int64_t q = 256 * (int64_t)W;
  const int64_t r = ((n + q - 1) / q) * q;
  return r > 0 ? r : q;
}

const char* ob_lamb_status_string(ob_status s) {
  switch (s) {
    case OB_OK: return "ok";
    case OB_ERR_NULL: return "required pointer is NULL";
    case OB_ERR_ARG: return "invalid argument";
    case OB_ERR_ALIGN: return "device pointer not 16-byte aligned";
    case OB_ERR_STATE: return "invalid state";
    case OB_ERR_HIP: return "HIP runtime error";
    case OB_ERR_SIZE: return "size exceeds the capacity of the static scratch";
  }
  return "unknown status";
}

const char* ob_lamb_last_hip_error(const ob_lamb_ctx* ctx) { return ctx ? ctx->hip_err.c_str() : ""; }

static ob_status create_ctx(const ob_lamb_config* cfg, ob_lamb_ctx** out);

ob_status ob_lamb_create(const ob_lamb_config* cfg, ob_lamb_ctx** out) {
  // the host tables are std::vectors: a failed allocation must not leave the C ABI as an exception
  try {
    return create_ctx(cfg, out);
  } catch (const std::bad_alloc&) {
    if (out) *out = nullptr;
    return OB_ERR_ARG;
  }
}

static ob_status check_config(const ob_lamb_config* cfg) {
  if (!cfg || !cfg->layer_offsets) return OB_ERR_NULL;
  const int64_t L = cfg->num_layers;
  if (L < 1 || L > (int64_t)1 << 24 || cfg->num_workers < 1 || cfg->num_workers > 65536) return OB_ERR_ARG;
  if (cfg->server_chunk < 0 || cfg->server_chunk >= cfg->num_workers) return OB_ERR_ARG;
  if (cfg->layer_offsets[0] != 0) return OB_ERR_ARG;
  for (int64_t l = 0; l < L; ++l)
    if (cfg->layer_offsets[l + 1] < cfg->layer_offsets[l]) return OB_ERR_ARG;
  const int64_t N = cfg->layer_offsets[L];
  if (N < 1 || N > ((int64_t)1 << 40)) return OB_ERR_ARG;
  const float fl[] = {cfg->beta1, cfg->beta2, cfg->beta3, cfg->eta, cfg->c_min, cfg->c_max,
                      cfg->r_min, cfg->r_max, cfg->r_threshold, cfg->weight_decay};
  for (float f : fl)
    if (!std::isfinite(f)) return OB_ERR_ARG;
  if (cfg->c_min > cfg->c_max || cfg->r_min > cfg->r_max) return OB_ERR_ARG;
  if ((cfg->flags & ~OB_CFG_NO_BARRIERS) != 0u || cfg->fused_max_tiles < 0 || cfg->spin_limit < OB_SPIN_NONE)
    return OB_ERR_ARG;
  return OB_OK;
}

// Offsets with the sentinel the per-element paths rely on.
static std::vector<int64_t> host_offsets(const ob_lamb_config* cfg) {
  const int64_t L = cfg->num_layers;
  std::vector<int64_t> h_off((size_t)L + 2);
  for (int64_t l = 0; l <= L; ++l) h_off[(size_t)l] = cfg->layer_offsets[l];
  h_off[(size_t)L + 1] = std::numeric_limits<int64_t>::max();
  return h_off;
}

ob_status ob_lamb_plan_split(const ob_lamb_config* cfg, int64_t max_tiles, uint8_t* span_owner,
                             int32_t* layer_listed) {
  if (ob_status s = check_config(cfg)) return s;
  if (!span_owner || !layer_listed) return OB_ERR_NULL;
  if (max_tiles < 0) return OB_ERR_ARG;
  try {
    const int64_t L = cfg->num_layers, W = cfg->num_workers;
    const int64_t n_c = ob_lamb_padded_len_for(cfg->layer_offsets[L], cfg->num_workers) / W;
    const std::vector<int64_t> h_off = host_offsets(cfg);
    Tiling tm, tl;
    if (!build_tiling(TILE_MAIN, n_c, W, L, h_off, &tm) || !build_tiling(TILE_LB, n_c, W, L, h_off, &tl))
      return OB_ERR_ARG;
    SplitPlan pl;
    plan_split(tl, TILE_LB, tm, h_off, n_c, L, max_tiles, BigRule(), &pl);
    for (int64_t t = 0; t < tm.n_tiles; ++t) span_owner[t] = pl.covered[(size_t)t] ? 2 : 0;
    for (int t : pl.rest_tiles) span_owner[t] = 1;
    for (int64_t l = 0; l < L; ++l) layer_listed[l] = pl.n_listed[(size_t)l];
    return OB_OK;
  } catch (const std::bad_alloc&) {
    return OB_ERR_ARG;
  }
}

ob_status ob_lamb_plan_big_tiles(const ob_lamb_config* cfg, int64_t max_tiles, uint8_t* span_big) {
  if (ob_status s = check_config(cfg)) return s;
  if (!span_big) return OB_ERR_NULL;
  if (max_tiles < 0) return OB_ERR_ARG;
  try {
    const int64_t L = cfg->num_layers, W = cfg->num_workers;
    const int64_t n_c = ob_lamb_padded_len_for(cfg->layer_offsets[L], cfg->num_workers) / W;
    const std::vector<int64_t> h_off = host_offsets(cfg);
    Tiling tm, tl;
    if (!build_tiling(TILE_MAIN, n_c, W, L, h_off, &tm) || !build_tiling(TILE_LB, n_c, W, L, h_off, &tl))
      return OB_ERR_ARG;
    SplitPlan pl;
    plan_split(tl, TILE_LB, tm, h_off, n_c, L, max_tiles, BigRule(), &pl);
    for (int64_t t = 0; t < tm.n_tiles; ++t) span_big[t] = pl.covered_big[(size_t)t] ? 1 : 0;
    return OB_OK;
  } catch (const std::bad_alloc&) {
    return OB_ERR_ARG;
  }
}

namespace { ob_status static_scratch(double** out); }

static ob_status create_ctx(const ob_lamb_config* cfg, ob_lamb_ctx** out) {
  if (out) *out = nullptr;
  if (!out) return OB_ERR_NULL;
  if (ob_status s = check_config(cfg)) return s;
  {
    // set-up time is also when this device's copy of the static scratch array (used by
    // ob_lamb_server_reduce_static, which must not do anything but launch) is looked up
    double* unused = nullptr;
    if (ob_status s = static_scratch(&unused)) return s;
  }
  const int64_t L = cfg->num_layers;
  const int64_t N = cfg->layer_offsets[L];

  ob_lamb_ctx* ctx = new (std::nothrow) ob_lamb_ctx();
  if (!ctx) return OB_ERR_ARG;
  struct Guard {   // frees the context and what it holds on every path that does not hand it over
    ob_lamb_ctx* c;
    ~Guard() { ob_lamb_destroy(c); }
  } guard{ctx};
  ctx->L = L;
  ctx->N = N;
  ctx->W = cfg->num_workers;
  ctx->server_chunk = cfg->server_chunk;
  ctx->n_pad = ob_lamb_padded_len_for(N, ctx->W);
  ctx->n_c = ctx->n_pad / ctx->W;
  ctx->beta1 = cfg->beta1; ctx->beta2 = cfg->beta2; ctx->beta3 = cfg->beta3;
  ctx->eta = cfg->eta; ctx->c_min = cfg->c_min; ctx->c_max = cfg->c_max;
  ctx->r_min = cfg->r_min; ctx->r_max = cfg->r_max; ctx->r_thr = cfg->r_threshold;
  ctx->wd = cfg->weight_decay;
  ctx->omb1 = 1.0f - ctx->beta1;
  ctx->omb2 = 1.0f - ctx->beta2;
  ctx->omb3 = 1.0f - ctx->beta3;
  ctx->one_m_thr = 1.0f - ctx->r_thr;
  ctx->one_p_thr = 1.0f + ctx->r_thr;
  ctx->invW = 1.0f / (float)ctx->W;

  const int64_t tpc_srv = (ctx->n_c + TILE_SRV - 1) / TILE_SRV;
  if (tpc_srv > 0x7fffffff) return OB_ERR_ARG;
  ctx->tpc_srv = (int)tpc_srv;

  const std::vector<int64_t> h_off = host_offsets(cfg);
  Tiling tm, tl, tw;
  if (!build_tiling(TILE_MAIN, ctx->n_c, ctx->W, L, h_off, &tm) ||
      !build_tiling(TILE_LB, ctx->n_c, ctx->W, L, h_off, &tl) ||
      !build_tiling(TILE_WU, ctx->n_c, ctx->W, L, h_off, &tw))
    return OB_ERR_ARG;
  const int64_t n_tiles = tm.n_tiles;
  ctx->tpc = (int)tm.tpc;
  ctx->n_tiles = (int)tm.n_tiles;
  ctx->n_segs = (int)tm.seg_layer.size();

  // single-pass worker compression: its own (larger) tiles and the layer of each tile's start
  const int64_t tpc_res = (ctx->n_c + TILE_RES - 1) / TILE_RES;
  ctx->tpc_res = (int)tpc_res;
  ctx->n_tiles_res = (int)(tpc_res * ctx->W);
  std::vector<int> first_res((size_t)ctx->n_tiles_res);
  for (int64_t t = 0; t < ctx->n_tiles_res; ++t) {
    const int64_t tile0 = (t / tpc_res) * ctx->n_c + (t % tpc_res) * TILE_RES;
    int64_t lo = 0, hi = L + 1;
    while (hi - lo > 1) {
      const int64_t mid = (lo + hi) / 2;
      if (h_off[(size_t)mid] <= tile0) lo = mid; else hi = mid;
    }
    first_res[(size_t)t] = (int)lo;
  }

  Workspace ws;
  bool ok = hip_ok(ctx, hipGetDevice(&ctx->device), "hipGetDevice");
  if (ok) {
    // The single-pass kernel needs a whole chunk's workgroups on the device at once (see the
    // kernel's comment); it is used only when they fill at most 80 % of the device's workgroup
    // slots (it still beats two passes at 61 % on MI355X), else the two-pass kernels run.
    int per_cu = 0, cus = 0;
    ok = hip_ok(ctx, hipOccupancyMaxActiveBlocksPerMultiprocessor(
                         &per_cu, k_compress_resident<U_RES, G_RES, true, false>, BLOCK, 0),
                "hipOccupancyMaxActiveBlocksPerMultiprocessor") &&
         hip_ok(ctx, hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device),
                "hipDeviceGetAttribute");
    // every instantiation is built for at least OB_RES_MINW workgroups per CU (its launch bounds); count
    // no more than that, whatever this one reaches
    const int64_t slots = (int64_t)std::min(per_cu, OB_RES_MINW) * cus;
    // a lower bound of the device-side waits (tests of the expiry path: with OB_SPIN_NONE every wait
    // gives up without polling, all kernels still run to their end)
    if (cfg->spin_limit == OB_SPIN_NONE) ctx->spin_limit = 0;
    else if (cfg->spin_limit > 0 && cfg->spin_limit < ctx->spin_limit) ctx->spin_limit = cfg->spin_limit;
    ctx->u_srv = server_spans(ctx->W, ctx->tpc_srv, cus);
    ctx->sum_lds = worker_sum_lds(ctx->n_tiles, cus);
    ctx->n_srv = (ctx->tpc_srv + ctx->u_srv - 1) / ctx->u_srv;
    const bool two_pass = (cfg->flags & OB_CFG_TWO_PASS_COMPRESS) != 0;
    ctx->resident = ok && !two_pass && 5 * (tpc_res + 8) <= 4 * slots;
    // the single-pass server kernel: same rule for the one chunk it covers
    int per_cu_s[3] = {0, 0, 0};
    ok = ok &&
         hip_ok(ctx, hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu_s[0], k_server_resident<U_SRV_RES[0]>, BLOCK, 0),
                "hipOccupancyMaxActiveBlocksPerMultiprocessor") &&
         hip_ok(ctx, hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu_s[1], k_server_resident<U_SRV_RES[1]>, BLOCK, 0),
                "hipOccupancyMaxActiveBlocksPerMultiprocessor") &&
         hip_ok(ctx, hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu_s[2], k_server_resident<U_SRV_RES[2]>, BLOCK, 0),
                "hipOccupancyMaxActiveBlocksPerMultiprocessor");
    // the tile table of the chunk's partials is sized for the smallest tile
    ctx->tpc_srv_res = (int)((ctx->n_c + SPAN - 1) / SPAN);
    for (int i = 0; ok && i < 3 && ctx->u_srv_res == 0 && !two_pass; ++i) {
      const int64_t tiles = (ctx->n_c + (int64_t)SPAN * U_SRV_RES[i] - 1) / ((int64_t)SPAN * U_SRV_RES[i]);
      if (5 * (tiles + 8) <= 4 * (int64_t)per_cu_s[i] * cus) ctx->u_srv_res = U_SRV_RES[i];
    }
  }
  // the two kernels with a per-layer barrier: which layers each of them takes.  The slot count is
  // the kernel's launch bound (every instantiation reaches it), whatever the one queried reaches.
  if (ok) {
    int per_cu_a = 0, per_cu_w = 0, cus = 0;
    ok = hip_ok(ctx, hipOccupancyMaxActiveBlocksPerMultiprocessor(
                         &per_cu_a, k_ratios_apply_resident<U_LB, true>, BLOCK, 0),
                "hipOccupancyMaxActiveBlocksPerMultiprocessor") &&
         hip_ok(ctx, hipOccupancyMaxActiveBlocksPerMultiprocessor(
                         &per_cu_w, k_warmup_resident<U_WU, G_WU, 0, false>, BLOCK, 0),
                "hipOccupancyMaxActiveBlocksPerMultiprocessor") &&
         hip_ok(ctx, hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device),
                "hipDeviceGetAttribute");
    int per_cu_h = 0;   // the same tiles go through the kernel with the variance in deferred form
    ok = ok && hip_ok(ctx, hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu_h, k_ratios_apply_hist<true, false, 0, true>, BLOCK, 0),
                      "hipOccupancyMaxActiveBlocksPerMultiprocessor");
    per_cu_a = std::min(per_cu_a, per_cu_h);
    ok = ok && hip_ok(ctx, hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu_h, k_ratios_apply_hist<true, false, S_LH, true>, BLOCK, 0),
                      "hipOccupancyMaxActiveBlocksPerMultiprocessor");
    per_cu_a = std::min(per_cu_a, per_cu_h);
    const int64_t max_a = (cfg->flags & OB_CFG_NO_FUSED_APPLY)
                              ? 0 : split_max_tiles(std::min(per_cu_a, OB_LB_MINW), cus, cfg->fused_max_tiles);
    const int64_t max_w = (cfg->flags & OB_CFG_TWO_PASS_WARMUP)
                              ? 0 : split_max_tiles(std::min(per_cu_w, OB_WU_MINW), cus, cfg->fused_max_tiles);
    std::vector<unsigned char> lagging, unused;
    build_split(ctx, &ws, tl, TILE_LB, tm, h_off, max_a, BigRule(), false, cus, &ctx->sp_apply, &lagging);
    build_split(ctx, &ws, tw, TILE_WU, tm, h_off, max_w, trail_rule(max_w > 0, cfg->fused_max_tiles, cus), true, cus, &ctx->sp_warm,
                &unused);
    ctx->sp_apply.in_lds = lh_in_lds(ctx->sp_apply.n_fused_tiles, cus);
    ctx->sp_apply.hist_each_step = hist_each_step(ctx->sp_apply, cus);
    // one launch instead of three or four where the whole list fits on the device at once (unless the
    // configuration lowers what the barrier kernels may take)
    auto slots_of = [&](auto kernel, size_t bytes, int min_per_cu, int64_t* out) {
      int per_cu = 0;
      if (!hip_ok(ctx, hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, BLOCK, bytes),
                  "hipOccupancyMaxActiveBlocksPerMultiprocessor"))
        return false;
      *out = (int64_t)std::min(per_cu, min_per_cu) * cus;   // (every instantiation reaches its launch bound)
      return true;
    };
    SmallTilings tilings(tm, ctx->n_c, ctx->W, L, h_off);
    if (ok && cfg->fused_max_tiles == 0 && !(cfg->flags & OB_CFG_NO_FUSED_APPLY))
      ok = build_small(ctx, &ws, &tilings, h_off, lagging, ctx->sp_apply, 1, 4, true, cus, [&](int U, size_t bytes, int64_t* n) {
        bool r = false;
        dispatch_u(U, [&](auto u) {
          constexpr int UU = decltype(u)::value;
          r = slots_of(k_ratios_apply_small<UU, true, true>, bytes, small_min_wg(UU), n);
        });
        return r;
      }, &ctx->sm_apply);
    if (ok && cfg->fused_max_tiles == 0 && !(cfg->flags & OB_CFG_TWO_PASS_WARMUP))
      ok = build_small(ctx, &ws, &tilings, h_off, std::vector<unsigned char>((size_t)tm.n_tiles, 0), ctx->sp_warm,
                       2, 3, false, cus, [&](int U, size_t bytes, int64_t* n) {
        bool r = false;
        dispatch_u(U, [&](auto u) {
          constexpr int UU = decltype(u)::value;
          r = slots_of(k_warmup_small<UU, 1, true, true>, bytes, small_min_wg(UU), n);
        });
        return r;
      }, &ctx->sm_warm);
    // chunk_ticket: counters (128-byte lines) and the first-level sums
    static_assert(TILE_SRV == TILE_MAIN, "the served chunk has the tiles of the worker's chunks");
    const size_t spc = (size_t)((ctx->tpc + TICKET_SUB - 1) / TICKET_SUB), line = 2 * CTR_STRIDE;
    if (worker_ticket(ctx->tpc, ctx->n_tiles, cus)) {
      ws.alloc_zero(&ctx->d_ticket, (size_t)ctx->W * (1 + spc) * line);
      ws.alloc_zero(&ctx->d_ticket_part, (size_t)ctx->W * spc);
    }
    if (ctx->u_srv > 1 || server_ticket(ctx->tpc, ctx->n_tiles, cus)) {
      ws.alloc_zero(&ctx->d_ticket_srv, (1 + spc) * line);
      ws.alloc_zero(&ctx->d_ticket_part_srv, spc);
    }
  }
  ws.upload(&ctx->d_first_layer_res, std::move(first_res));
  ws.upload(&ctx->d_off, h_off);
  ws.upload(&ctx->d_first_layer, std::move(tm.first));
  ws.upload(&ctx->d_tile_seg0, std::move(tm.tile_seg0));
  ws.upload(&ctx->d_seg_layer, std::move(tm.seg_layer));
  ws.upload(&ctx->d_layer_seg0, std::move(tm.layer_seg0));
  ws.alloc_zero(&ctx->d_partials_res, (size_t)ctx->n_tiles_res);
  ws.alloc_zero(&ctx->d_counter, (size_t)ctx->W * CTR_STRIDE);
  ws.alloc_zero(&ctx->d_sub, (size_t)ctx->W * arrival_groups(ctx->tpc_res) * CTR_STRIDE);
  ws.alloc_zero(&ctx->d_flag, (size_t)ctx->W);
  ws.alloc_zero(&ctx->d_errflag, 1);
  ws.alloc_zero(&ctx->d_partials_srv_res, (size_t)ctx->tpc_srv_res);
  ws.alloc_zero(&ctx->d_counter_srv, (size_t)CTR_STRIDE);
  ws.alloc_zero(&ctx->d_sub_srv, arrival_groups(ctx->tpc_srv_res) * CTR_STRIDE);
  ws.alloc_zero(&ctx->d_flag_srv, 1);
  ws.alloc_zero(&ctx->d_partials, (size_t)n_tiles);
  ws.alloc_zero(&ctx->d_partials_srv, (size_t)tpc_srv);
  ws.alloc_zero(&ctx->d_seg_sums, 2 * (size_t)ctx->n_segs);
  ws.alloc_zero(&ctx->d_sigma, (size_t)L);
  ws.alloc_zero(&ctx->d_seg_max, (size_t)ctx->n_segs);
  if (ok && !ctx->sp_apply.rest_in_launch) {
    // the layers that meet each chunk (empty layers in between included; a chunk that lies in the
    // padding has none)
    std::vector<int> pair_base((size_t)ctx->W + 1, 0), pair_lfirst((size_t)ctx->W, 0), pair_c, pair_l;
    int64_t l = 0;
    for (int64_t c = 0; c < ctx->W; ++c) {
      const int64_t c0 = c * ctx->n_c, c1 = std::min((c + 1) * ctx->n_c, N);
      pair_base[(size_t)c] = (int)pair_c.size();
      if (c0 < N) {
        while (h_off[(size_t)l + 1] <= c0) ++l;      // the layer that holds element c0
        pair_lfirst[(size_t)c] = (int)l;
        for (int64_t q = l; q < L && h_off[(size_t)q] < c1; ++q) {
          pair_c.push_back((int)c);
          pair_l.push_back((int)q);
        }
      }
    }
    pair_base[(size_t)ctx->W] = (int)pair_c.size();
    ctx->n_pairs = (int)pair_c.size();
    ws.upload(&ctx->d_pair_base, std::move(pair_base));
    ws.upload(&ctx->d_pair_lfirst, std::move(pair_lfirst));
    ws.upload(&ctx->d_pair_c, std::move(pair_c));
    ws.upload(&ctx->d_pair_l, std::move(pair_l));
    ws.alloc_zero(&ctx->d_vterms, (size_t)(VF_MAX_OLD + 1) * (size_t)ctx->n_pairs * 2);
  }
  ok = ok && ws.commit(ctx) && hip_ok(ctx, hipDeviceSynchronize(), "hipDeviceSynchronize");
  if (!ok) return OB_ERR_HIP;
  guard.c = nullptr;
  *out = ctx;
  return OB_OK;
}

void ob_lamb_destroy(ob_lamb_ctx* ctx) {
  if (!ctx) return;
  for (auto& r : ctx->prof) {
    (void)hipEventDestroy(r.e0);
    (void)hipEventDestroy(r.e1);
  }
  if (ctx->d_mem) (void)hipFree(ctx->d_mem);
  delete ctx;
}

int64_t ob_lamb_num_params(const ob_lamb_ctx* ctx) { return ctx ? ctx->N : 0; }
int64_t ob_lamb_padded_len(const ob_lamb_ctx* ctx) { return ctx ? ctx->n_pad : 0; }
int64_t ob_lamb_chunk_len(const ob_lamb_ctx* ctx) { return ctx ? ctx->n_c : 0; }
size_t ob_lamb_workspace_bytes(const ob_lamb_ctx* ctx) { return ctx ? ctx->device_bytes : 0; }

ob_status ob_lamb_warmup_step_lp(ob_lamb_ctx* ctx, const ob_lamb_state* st, const void* grad,
                                 ob_dtype grad_dtype, float grad_scale, float lr, void* x_lp,
                                 ob_dtype x_dtype, void* hip_stream) {
  if (ob_status s = check_common(ctx, st)) return s;
  GradSrc gs;
  bool lpg = false;
  if (ob_status s = grad_source(grad, grad_dtype, grad_scale, &gs, &lpg)) return s;
  XLp xl;
  if (ob_status s = x_lp_target(x_lp, x_dtype, &xl)) return s;
  REQUIRE_PTR(st->x); REQUIRE_PTR(st->m); REQUIRE_PTR(st->v_fresh);
  if (!st->c_avg || !st->coeff_c) return OB_ERR_NULL;
  if (!std::isfinite(lr)) return OB_ERR_ARG;
  Launch la(ctx, hip_stream);
  const LayerTab lt = layer_tab(ctx, st, ctx->d_first_layer);
  auto moments = [&](const int* tiles, int n_launch_tiles) {
    dispatch1(lpg, [&](auto lg) {
      OB_LAUNCH(la, KID_WARMUP_MOMENTS, (k_warmup_moments<U_MAIN, decltype(lg)::value ? 1 : 0>), n_launch_tiles,
                gs, st->m, st->v_fresh, st->x, ctx->d_seg_sums, ctx->n_c, ctx->tpc, ctx->beta1, ctx->omb1,
                ctx->beta2, ctx->omb2, ctx->eta, ctx->wd, lt, ctx->d_tile_seg0, ctx->d_seg_layer, tiles);
    });
  };
  auto coeff = [&](const unsigned char* done_elsewhere, unsigned long long* clear_flag) {
    OB_LAUNCH_B(la, KID_WARMUP_COEFF, k_warmup_coeff, (int)ctx->L, FBLOCK, ctx->d_seg_sums, ctx->d_layer_seg0,
                st->coeff_c, st->c_avg, ctx->c_min, ctx->c_max, ctx->beta3, ctx->omb3, done_elsewhere, clear_flag);
  };
  auto apply = [&](const int* tiles, int n_launch_tiles) {
    dispatch1(xl.p != nullptr, [&](auto lx) {
      OB_LAUNCH(la, KID_WARMUP_APPLY, (k_warmup_apply<U_MAIN, decltype(lx)::value>), n_launch_tiles, st->m,
                st->v_fresh, st->x, st->coeff_c, ctx->n_c, ctx->tpc, lr, ctx->eta, ctx->wd, lt, xl.p, xl.bf16,
                tiles);
    });
  };
  WarmClip wc;
  wc.coeff_c = st->coeff_c; wc.c_avg = st->c_avg; wc.c_min = ctx->c_min; wc.c_max = ctx->c_max;
  wc.beta3 = ctx->beta3; wc.omb3 = ctx->omb3;
  if (ctx->sm_warm.u) {   // one launch
    const SmallPlan& sm = ctx->sm_warm;
    dispatch_u(sm.u, [&](auto u) {
      dispatch2(lpg, xl.p != nullptr, [&](auto lg, auto lx) {
        dispatch1(sm.two_levels, [&](auto two) {
          OB_LAUNCH_S(la, KID_WARMUP_SMALL,
                      (k_warmup_small<decltype(u)::value, decltype(lg)::value ? 1 : 0, decltype(lx)::value, decltype(two)::value>),
                      sm.n_tiles + (sm.empty_layers ? 1 : 0), BLOCK, sm.lds_bytes, gs, st->m, st->v_fresh, st->x,
                      small_tab(ctx, sm), wc, ctx->beta1, ctx->omb1, ctx->beta2, ctx->omb2, ctx->eta, ctx->wd, lr, lt,
                      xl.p, xl.bf16);
        });
      });
    });
    return la.ok ? OB_OK : OB_ERR_HIP;
  }
  LayerSplit& sp = ctx->sp_warm;
  if (!sp.on && !sp.big_on) {   // two passes over everything
    moments(nullptr, ctx->n_tiles);
    coeff(nullptr, nullptr);
    apply(nullptr, ctx->n_tiles);
    return la.ok ? OB_OK : OB_ERR_HIP;
  }
  // 1. moments and partial sums of everything outside the tiles of the next two kernels; the layers without such
  //    tiles get their c here (an empty layer too), the sums of the others wait in seg_sums
  const int* rest = sp.big_on ? sp.d_rest_ratio_tiles : sp.d_rest_tiles;
  const int n_rest = sp.big_on ? sp.n_rest_ratio_tiles : sp.n_rest_tiles;
  moments(rest, n_rest);
  if (sp.n_layers < ctx->L) coeff(sp.big_on ? sp.d_has_tiles : sp.d_has_listed, sp.big_on ? sp.d_trail_flag : nullptr);
  // 2. the layers that are too large for the kernel with the per-layer barrier
  if (sp.big_on) {
    TrailTab tt;
    tt.lt = big_tiles(ctx, sp);
    tt.count0 = sp.d_count0; tt.count = sp.d_count; tt.sub_sums = sp.d_sub_sums; tt.part_sums = sp.d_part_sums;
    tt.flag = sp.d_trail_flag; tt.seg_sums = ctx->d_seg_sums;
    tt.errflag = ctx->d_errflag; tt.spin_limit = ctx->spin_limit; tt.wait = sp.trail_wait ? 1 : 0;
    int64_t from = 0;
    for (int64_t end : sp.item_end) {
      tt.items = sp.d_items + from;
      dispatch2(lpg, xl.p != nullptr, [&](auto lg, auto lx) {
        OB_LAUNCH(la, KID_WARMUP_TRAIL, (k_warmup_trail<decltype(lg)::value ? 1 : 0, decltype(lx)::value>), (int)(end - from),
                  gs, st->m, st->v_fresh, st->x, tt, wc, ctx->beta1, ctx->omb1, ctx->beta2, ctx->omb2, ctx->eta, ctx->wd,
                  lr, lt, xl.p, xl.bf16);
      });
      from = end;
    }
  }
  // 3. the listed tiles: moments, layer barrier, update
  WarmSync ws;
  ws.seg_sums = ctx->d_seg_sums; ws.listed_sums = sp.d_listed_sums; ws.lt = listed_tiles(ctx, sp);
  ws.counter = sp.d_counter; ws.sub = sp.d_sub; ws.flag = sp.d_flag; ws.errflag = ctx->d_errflag;
  ws.spin_limit = ctx->spin_limit;
  ws.coeff_c = st->coeff_c; ws.c_avg = st->c_avg;
  ws.c_min = ctx->c_min; ws.c_max = ctx->c_max; ws.beta3 = ctx->beta3; ws.omb3 = ctx->omb3;
  if (sp.on) dispatch2(lpg, xl.p != nullptr, [&](auto lg, auto lx) {
    OB_LAUNCH(la, KID_WARMUP_RESIDENT,
              (k_warmup_resident<U_WU, G_WU, decltype(lg)::value ? 1 : 0, decltype(lx)::value>), sp.n_fused_tiles,
              gs, st->m, st->v_fresh, st->x, ws, ctx->beta1, ctx->omb1, ctx->beta2, ctx->omb2, ctx->eta, ctx->wd,
              lr, lt, xl.p, xl.bf16);
  });
  // 4. update of everything else, with the coefficients of steps 1 to 3
  apply(rest, n_rest);
  return la.ok ? OB_OK : OB_ERR_HIP;
}

ob_status ob_lamb_warmup_step(ob_lamb_ctx* ctx, const ob_lamb_state* st, const float* grad, float lr,
                              void* hip_stream) {
  return ob_lamb_warmup_step_lp(ctx, st, grad, OB_F32, 1.0f, lr, nullptr, OB_F32, hip_stream);
}

ob_status ob_lamb_freeze(ob_lamb_ctx* ctx, const ob_lamb_state* st, void* hip_stream) {
  if (ob_status s = check_common(ctx, st)) return s;
  REQUIRE_PTR(st->v_fresh); REQUIRE_PTR(st->v_frozen);
  if (!st->r_prev) return OB_ERR_NULL;
  Launch la(ctx, hip_stream);
  la.begin(KID_COPY, true);
  if (la.ok)
    la.ok = hip_ok(ctx, hipMemcpyAsync(st->v_frozen, st->v_fresh, (size_t)ctx->n_pad * sizeof(float),
                                       hipMemcpyDeviceToDevice, la.stream), "hipMemcpyAsync");
  la.end("copy", true);
  OB_LAUNCH(la, KID_FILL, k_fill, (int)((ctx->L + BLOCK - 1) / BLOCK), st->r_prev, ctx->L, 1.0f);
  return la.ok ? OB_OK : OB_ERR_HIP;
}

ob_status ob_lamb_compress_local_lp(ob_lamb_ctx* ctx, const ob_lamb_state* st, const void* grad,
                                    ob_dtype grad_dtype, float grad_scale, uint32_t* packed_out,
                                    float* scales_out, void* hip_stream) {
  if (ob_status s = check_common(ctx, st)) return s;
  GradSrc gs;
  bool lpg = false;
  if (ob_status s = grad_source(grad, grad_dtype, grad_scale, &gs, &lpg)) return s;
  REQUIRE_PTR(st->err_worker); REQUIRE_PTR(packed_out);
  if (!scales_out) return OB_ERR_NULL;
  bool packed_m = false;
  PackedMom pm;
  if (ob_status s = momentum_source(st, &packed_m, &pm)) return s;
  if (packed_m && st->m_packed == packed_out) return OB_ERR_ARG;  // would be overwritten while read
  if ((st->own_packed_in == nullptr) != (st->own_scale_in == nullptr)) return OB_ERR_NULL;
  if (st->own_packed_in && misaligned(st->own_packed_in)) return OB_ERR_ALIGN;
  OwnCopy oc;
  oc.packed = st->own_packed_in; oc.scale = st->own_scale_in; oc.chunk = ctx->server_chunk;
  Launch la(ctx, hip_stream);
  PackedErr pe;
  pe.bits = st->err_packed; pe.scales = st->err_scales;
  if ((st->err_packed == nullptr) != (st->err_scales == nullptr)) return OB_ERR_NULL;
  if (st->err_packed) {
    // deferred error: the whole call is one streaming pass plus the scales -- no barrier, no second pass
    if (misaligned(st->err_packed)) return OB_ERR_ALIGN;
    if (packed_m && st->m_packed == st->err_packed) return OB_ERR_ARG;
    const LayerTab lt = layer_tab(ctx, st, ctx->d_first_layer);
    const ChunkTicket tk = chunk_ticket_of(ctx->d_ticket, ctx->d_ticket_part, ctx->W, ctx->tpc, scales_out, oc.scale, oc.chunk);
    if (ctx->sum_lds && lpg && packed_m && !st->mom_scale && !tk.count)
      OB_LAUNCH(la, KID_COMPRESS_DEFERRED, (k_momentum_z_sumsq<U_MAIN, false, true, 1, true, false, true>), ctx->n_tiles, gs, st->m,
                pm, st->err_worker, ctx->d_partials, ctx->n_c, ctx->tpc, ctx->beta1, ctx->omb1, lt, pe, packed_out, oc, tk);
    else
      dispatch2(st->mom_scale != nullptr, packed_m, [&](auto hk, auto pk) {
        dispatch2(lpg, tk.count != nullptr, [&](auto lg, auto ti) {
          OB_LAUNCH(la, KID_COMPRESS_DEFERRED,
                    (k_momentum_z_sumsq<U_MAIN, decltype(hk)::value, decltype(pk)::value,
                                        decltype(lg)::value ? 1 : 0, true, decltype(ti)::value>),
                    ctx->n_tiles, gs, st->m, pm, st->err_worker, ctx->d_partials, ctx->n_c, ctx->tpc,
                    ctx->beta1, ctx->omb1, lt, pe, packed_out, oc, tk);
        });
      });
    if (!tk.count)
      OB_LAUNCH_B(la, KID_CHUNK_SCALE, k_chunk_scale, ctx->W, FBLOCK, ctx->d_partials, ctx->tpc, ctx->n_c, scales_out,
                  oc.scale, oc.chunk);
    return la.ok ? OB_OK : OB_ERR_HIP;
  }
  if (ctx->resident) {
    ChunkSync cs;
    cs.partials = ctx->d_partials_res;
    cs.counter = ctx->d_counter;
    cs.sub = ctx->d_sub;
    cs.flag = ctx->d_flag;
    cs.errflag = ctx->d_errflag;
    cs.spin_limit = ctx->spin_limit;
    const LayerTab lt = layer_tab(ctx, st, ctx->d_first_layer_res);
    dispatch2(st->mom_scale != nullptr, packed_m, [&](auto hk, auto pk) {
      dispatch2(lpg, !packed_m && keeps_second_reads(ctx->N, ctx->W), [&](auto lg, auto kp) {
        OB_LAUNCH(la, KID_COMPRESS_RESIDENT,
                  (k_compress_resident<U_RES, G_RES, decltype(hk)::value, decltype(pk)::value, OB_RES_MINW,
                                       decltype(lg)::value ? 1 : 0, decltype(kp)::value && !decltype(pk)::value>),
                  ctx->n_tiles_res, gs, st->m, pm, st->err_worker, packed_out, scales_out, cs, ctx->n_c,
                  ctx->tpc_res, ctx->beta1, ctx->omb1, lt, oc);
      });
    });
    return la.ok ? OB_OK : OB_ERR_HIP;
  }
  const LayerTab lt = layer_tab(ctx, st, ctx->d_first_layer);
  dispatch2(st->mom_scale != nullptr, packed_m, [&](auto hk, auto pk) {
    dispatch1(lpg, [&](auto lg) {
      OB_LAUNCH(la, KID_MOMENTUM_Z,
                (k_momentum_z_sumsq<U_MAIN, decltype(hk)::value, decltype(pk)::value, decltype(lg)::value ? 1 : 0>),
                ctx->n_tiles, gs, st->m, pm, st->err_worker, ctx->d_partials, ctx->n_c, ctx->tpc,
                ctx->beta1, ctx->omb1, lt, pe, packed_out, oc, ChunkTicket{});
    });
  });
  OB_LAUNCH_B(la, KID_CHUNK_SCALE, k_chunk_scale, ctx->W, FBLOCK, ctx->d_partials, ctx->tpc, ctx->n_c, scales_out,
              (float*)nullptr, 0);
  OB_LAUNCH(la, KID_SIGN_PACK, (k_sign_pack_error<U_MAIN>), ctx->n_tiles, st->err_worker, packed_out,
            scales_out, ctx->n_c, ctx->tpc);
  if (oc.packed) {   // the two-pass form copies the rank's own chunk afterwards
    const int64_t wpc = ctx->n_c / 32;
    la.begin(KID_COPY, true);
    if (la.ok)
      la.ok = hip_ok(ctx, hipMemcpyAsync(oc.packed, packed_out + (int64_t)oc.chunk * wpc, (size_t)wpc * 4,
                                         hipMemcpyDeviceToDevice, la.stream), "hipMemcpyAsync") &&
              hip_ok(ctx, hipMemcpyAsync(oc.scale, scales_out + oc.chunk, sizeof(float),
                                         hipMemcpyDeviceToDevice, la.stream), "hipMemcpyAsync");
    la.end("copy", true);
  }
  return la.ok ? OB_OK : OB_ERR_HIP;
}

ob_status ob_lamb_compress_local(ob_lamb_ctx* ctx, const ob_lamb_state* st, const float* grad,
                                 uint32_t* packed_out, float* scales_out, void* hip_stream) {
  return ob_lamb_compress_local_lp(ctx, st, grad, OB_F32, 1.0f, packed_out, scales_out, hip_stream);
}

ob_status ob_lamb_server_reduce(ob_lamb_ctx* ctx, const ob_lamb_state* st, const uint32_t* packed_in,
                                const float* scales_in, uint32_t* packed_out, float* scale_out,
                                void* hip_stream) {
  if (ob_status s = check_common(ctx, st)) return s;
  REQUIRE_PTR(packed_in); REQUIRE_PTR(packed_out); REQUIRE_PTR(st->err_server);
  if (!scales_in || !scale_out) return OB_ERR_NULL;
  // the kernels address packed_in with 32-bit byte offsets
  if ((int64_t)ctx->W * (ctx->n_c / 8) >= ((int64_t)1 << 31)) return OB_ERR_SIZE;
  Launch la(ctx, hip_stream);
  if ((st->srv_err_packed == nullptr) != (st->srv_err_scale == nullptr)) return OB_ERR_NULL;
  if (st->srv_err_packed) {
    // deferred server error: one pass over the chunk plus its scale -- no barrier, no second pass
    if (misaligned(st->srv_err_packed)) return OB_ERR_ALIGN;
    if (st->srv_err_packed == packed_out) return OB_ERR_ARG;
    const ChunkTicket tk = chunk_ticket_of(ctx->d_ticket_srv, ctx->d_ticket_part_srv, 1, ctx->n_srv, scale_out,
                                           st->srv_err_scale, 0);
    dispatch1(tk.count != nullptr, [&](auto ti) {
      dispatch_u(ctx->u_srv, [&](auto u) {
        OB_LAUNCH(la, KID_SERVER_AVG, (k_server_unpack_avg<decltype(u)::value, true, decltype(ti)::value>), ctx->n_srv, packed_in,
                  scales_in, st->err_server, ctx->d_partials_srv, ctx->n_c, (int)ctx->W, ctx->invW, st->srv_err_packed,
                  st->srv_err_scale, packed_out, tk);
      });
    });
    if (!tk.count)
      OB_LAUNCH_B(la, KID_SERVER_SCALE, k_chunk_scale, 1, FBLOCK, ctx->d_partials_srv, ctx->n_srv, ctx->n_c, scale_out,
                st->srv_err_scale, 0);
    return la.ok ? OB_OK : OB_ERR_HIP;
  }
  if (ctx->u_srv_res) {
    ChunkSync cs;
    cs.partials = ctx->d_partials_srv_res;
    cs.counter = ctx->d_counter_srv;
    cs.sub = ctx->d_sub_srv;
    cs.flag = ctx->d_flag_srv;
    cs.errflag = ctx->d_errflag;
    cs.spin_limit = ctx->spin_limit;
    const int64_t tile = (int64_t)SPAN * ctx->u_srv_res;
    const int tiles = (int)((ctx->n_c + tile - 1) / tile);
    auto launch = [&](auto u) {
      OB_LAUNCH(la, KID_SERVER_RESIDENT, (k_server_resident<decltype(u)::value>), tiles, packed_in, scales_in,
                st->err_server, packed_out, scale_out, cs, ctx->n_c, (int)ctx->W, ctx->invW);
    };
    switch (ctx->u_srv_res) {
      case 1: launch(std::integral_constant<int, 1>{}); break;
      case 2: launch(std::integral_constant<int, 2>{}); break;
      default: launch(std::integral_constant<int, 4>{}); break;
    }
    return la.ok ? OB_OK : OB_ERR_HIP;
  }
  dispatch_u(ctx->u_srv, [&](auto u) {
    OB_LAUNCH(la, KID_SERVER_AVG, (k_server_unpack_avg<decltype(u)::value>), ctx->n_srv, packed_in, scales_in,
              st->err_server, ctx->d_partials_srv, ctx->n_c, (int)ctx->W, ctx->invW, (uint32_t*)nullptr,
              (const float*)nullptr, (uint32_t*)nullptr, ChunkTicket{});
  });
  OB_LAUNCH_B(la, KID_SERVER_SCALE, k_chunk_scale, 1, FBLOCK, ctx->d_partials_srv, ctx->n_srv, ctx->n_c, scale_out,
              (float*)nullptr, 0);
  OB_LAUNCH(la, KID_SERVER_PACK, (k_sign_pack_error<U_SRV>), ctx->tpc_srv, st->err_server, packed_out,
            scale_out, ctx->n_c, ctx->tpc_srv);
  return la.ok ? OB_OK : OB_ERR_HIP;
}

ob_status ob_lamb_layer_ratios(ob_lamb_ctx* ctx, const ob_lamb_state* st, const uint32_t* packed_all,
                               const float* server_scales, void* hip_stream) {
  if (ob_status s = check_ratios_args(ctx, st, packed_all, server_scales)) return s;
  bool packed_m = false;
  PackedMom pm;
  if (ob_status s = momentum_source(st, &packed_m, &pm)) return s;
  Launch la(ctx, hip_stream);
  launch_ratios(la, ctx, st, packed_all, server_scales, packed_m, pm, nullptr, ctx->n_tiles, nullptr, true);
  return la.ok ? OB_OK : OB_ERR_HIP;
}

ob_status ob_lamb_decompress_apply_lp(ob_lamb_ctx* ctx, const ob_lamb_state* st, const uint32_t* packed_all,
                                      const float* server_scales, float lr, void* x_lp, ob_dtype x_dtype,
                                      void* hip_stream) {
  if (ob_status s = check_apply_args(ctx, st, packed_all, server_scales, lr)) return s;
  XLp xl;
  if (ob_status s = x_lp_target(x_lp, x_dtype, &xl)) return s;
  Launch la(ctx, hip_stream);
  launch_apply(la, ctx, st, packed_all, server_scales, lr, nullptr, ctx->n_tiles, xl);
  commit_packed_momentum(la, ctx, st, packed_all, server_scales);
  return la.ok ? OB_OK : OB_ERR_HIP;
}

ob_status ob_lamb_decompress_apply(ob_lamb_ctx* ctx, const ob_lamb_state* st, const uint32_t* packed_all,
                                   const float* server_scales, float lr, void* hip_stream) {
  return ob_lamb_decompress_apply_lp(ctx, st, packed_all, server_scales, lr, nullptr, OB_F32, hip_stream);
}

ob_status ob_lamb_ratios_apply_lp(ob_lamb_ctx* ctx, const ob_lamb_state* st, const uint32_t* packed_all,
                                  const float* server_scales, float lr, void* x_lp, ob_dtype x_dtype,
                                  void* hip_stream) {
  if (ob_status s = check_ratios_args(ctx, st, packed_all, server_scales)) return s;
  XLp xl;
  if (ob_status s = x_lp_target(x_lp, x_dtype, &xl)) return s;
  REQUIRE_PTR(st->x);
  if (!std::isfinite(lr)) return OB_ERR_ARG;
  bool packed_m = false;
  PackedMom pm;
  pm.bits = nullptr;
  pm.scales = nullptr;
  // momentum source: dense st->m if given (then it is also where the new momentum is written),
  // else the 1-bit form of the previous step (then nothing is written: the new momentum is
  // packed_all/server_scales themselves)
  if (ob_status s = momentum_source(st, &packed_m, &pm)) return s;
  if (packed_m && st->m_packed == packed_all) return OB_ERR_ARG;
  Launch la(ctx, hip_stream);
  if (ctx->sm_apply.u && packed_m) {   // one launch
    VfHist vh{};
    vh.write_v = 1;
    launch_ratios_apply_small(la, ctx, st, ratio_args(ctx, st, packed_all, server_scales, pm), vh,
                              apply_args(ctx, st, packed_all, server_scales, lr, xl));
    return la.ok ? OB_OK : OB_ERR_HIP;
  }
  LayerSplit& sp = ctx->sp_apply;
  if (packed_m && sp.on && sp.hist_each_step)
    return ob_lamb_ratios_apply_hist_lp(ctx, st, packed_all, server_scales, lr, nullptr, x_lp, x_dtype, hip_stream);
  if (!sp.on || !packed_m) {
    // no tile qualifies, or the momentum is a dense array (the barrier kernel reads and commits the 1-bit
    // form only): the two plain kernels
    launch_ratios(la, ctx, st, packed_all, server_scales, packed_m, pm, nullptr, ctx->n_tiles, nullptr, true);
    launch_apply(la, ctx, st, packed_all, server_scales, lr, nullptr, ctx->n_tiles, xl);
    return la.ok ? OB_OK : OB_ERR_HIP;
  }
  const RatioArgs ra = ratio_args(ctx, st, packed_all, server_scales, pm);
  const ApplyArgs aa = apply_args(ctx, st, packed_all, server_scales, lr, xl);
  const bool hk = st->mom_scale != nullptr;  // (here the momentum is in 1-bit form and st->m is NULL)
  const LayerTab lt = layer_tab(ctx, st, ctx->d_first_layer);
  // 1. ratio pass over everything outside the listed tiles; its segment maxima wait in seg_max: of
  //    the layers with listed tiles for the layer barrier, of the others (the ratio of an empty layer,
  //    0, still goes through the clips) for the leading workgroups of the same launch
  const int n_lead = (sp.n_layers < ctx->L) ? (int)ctx->L : 0;   // (finished by the barrier kernel's leading workgroups)
  launch_ratios(la, ctx, st, packed_all, server_scales, packed_m, pm, sp.d_rest_tiles, sp.n_rest_tiles,
                sp.d_has_listed, false);
  // 2. the listed tiles: ratio pass, layer barrier, update
  LayerSync ls{};
  ls.seg_max = ctx->d_seg_max; ls.listed_max = sp.d_listed_max; ls.lt = listed_tiles(ctx, sp);
  ls.counter = sp.d_counter; ls.sub = sp.d_sub; ls.flag = sp.d_flag; ls.errflag = ctx->d_errflag;
  ls.spin_limit = ctx->spin_limit;
  ls.c_avg = st->c_avg; ls.r_prev = st->r_prev; ls.coeff_c = st->coeff_c;
  ls.one_m_thr = ctx->one_m_thr; ls.one_p_thr = ctx->one_p_thr; ls.r_min = ctx->r_min; ls.r_max = ctx->r_max;
  ls.n_lead = n_lead;
  dispatch2(hk, xl.p != nullptr, [&](auto k_, auto lx) {
    OB_LAUNCH(la, KID_RATIOS_APPLY_RESIDENT,
              (k_ratios_apply_resident<U_LB, decltype(k_)::value, decltype(lx)::value>), sp.n_fused_tiles + n_lead,
              ra, aa, ls, lt);
  });
  // 3. update of everything outside the listed tiles, with the coefficients of steps 1 and 2
  launch_apply(la, ctx, st, packed_all, server_scales, lr, sp.d_rest_tiles, sp.n_rest_tiles, xl);
  return la.ok ? OB_OK : OB_ERR_HIP;
}

ob_status ob_lamb_ratios_apply(ob_lamb_ctx* ctx, const ob_lamb_state* st, const uint32_t* packed_all,
                               const float* server_scales, float lr, void* hip_stream) {
  return ob_lamb_ratios_apply_lp(ctx, st, packed_all, server_scales, lr, nullptr, OB_F32, hip_stream);
}

}  // extern "C"

namespace {
// The caller's history -> the kernels' (validated; h == NULL: none, write).
ob_status vf_history(const ob_lamb_vf_history* h, VfHist* out) {
  static_assert(OB_VF_MAX_OLD == VF_MAX_OLD, "header and kernels disagree");
  out->n_old = 0;
  out->write_v = 1;
  for (int i = 0; i < VF_MAX_OLD; ++i) {
    out->bits[i] = nullptr;
    out->scales[i] = nullptr;
  }
  if (!h) return OB_OK;
  if (h->n_old < 0 || h->n_old > OB_VF_MAX_OLD) return OB_ERR_ARG;
  for (int i = 0; i < h->n_old; ++i) {
    if (!h->bits[i] || !h->scales[i]) return OB_ERR_NULL;
    if (misaligned(h->bits[i])) return OB_ERR_ALIGN;
    out->bits[i] = h->bits[i];
    out->scales[i] = h->scales[i];
  }
  out->n_old = h->n_old;
  out->write_v = h->write_v ? 1 : 0;
  return OB_OK;
}

VTerms vterms(const ob_lamb_ctx* ctx) {
  VTerms vt;
  vt.t = ctx->d_vterms; vt.pair_base = ctx->d_pair_base; vt.pair_lfirst = ctx->d_pair_lfirst;
  vt.pair_c = ctx->d_pair_c; vt.pair_l = ctx->d_pair_l; vt.n_pairs = ctx->n_pairs;
  return vt;
}

}  // namespace

extern "C" {

ob_status ob_lamb_ratios_apply_hist_lp(ob_lamb_ctx* ctx, const ob_lamb_state* st, const uint32_t* packed_all,
                                       const float* server_scales, float lr, const ob_lamb_vf_history* h,
                                       void* x_lp, ob_dtype x_dtype, void* hip_stream) {
  if (ob_status s = check_ratios_args(ctx, st, packed_all, server_scales)) return s;
  XLp xl;
  if (ob_status s = x_lp_target(x_lp, x_dtype, &xl)) return s;
  REQUIRE_PTR(st->x);
  if (!std::isfinite(lr)) return OB_ERR_ARG;
  bool packed_m = false;
  PackedMom pm;
  if (ob_status s = momentum_source(st, &packed_m, &pm)) return s;
  if (!packed_m || st->m_packed == packed_all) return OB_ERR_ARG;   // the history is one of 1-bit momenta
  VfHist vh;
  if (ob_status s = vf_history(h, &vh)) return s;
  Launch la(ctx, hip_stream);
  if (ctx->sm_apply.u) {   // one launch
    launch_ratios_apply_small(la, ctx, st, ratio_args(ctx, st, packed_all, server_scales, pm), vh,
                              apply_args(ctx, st, packed_all, server_scales, lr, xl));
    return la.ok ? OB_OK : OB_ERR_HIP;
  }
  LayerSplit& sp = ctx->sp_apply;
  if (!sp.on && !sp.big_on) {
    // no tile works from the history: the whole array is kept up to date
    launch_ratios(la, ctx, st, packed_all, server_scales, packed_m, pm, nullptr, ctx->n_tiles, nullptr, true);
    launch_apply(la, ctx, st, packed_all, server_scales, lr, nullptr, ctx->n_tiles, xl);
    return la.ok ? OB_OK : OB_ERR_HIP;
  }
  const RatioArgs ra = ratio_args(ctx, st, packed_all, server_scales, pm);
  const ApplyArgs aa = apply_args(ctx, st, packed_all, server_scales, lr, xl);
  const LayerTab lt = layer_tab(ctx, st, ctx->d_first_layer);
  // the three stages of ob_lamb_ratios_apply; the kernel with the per-layer barrier and the ratio
  // pass of the layers that are too large for it work from the history (outside their tiles the plain
  // ratio pass keeps the array up to date at every step: on 1024-element tiles that pass is bound by
  // its launch shape, not by the bytes it moves).  Without the barrier kernel (OB_CFG_NO_FUSED_APPLY)
  // every layer with enough whole tiles counts as too large: no wait anywhere, and still no rewrite
  // of the array at every step.
  // launch 1, where the barrier kernel's launch does not do it: the two values of every (chunk, layer) pair and step of
  // the history (leading workgroups) and the plain ratio pass outside the tiles that work from the history
  const bool hk = st->mom_scale != nullptr;
  const bool rest_in_launch = sp.on && sp.rest_in_launch;
  const bool trail = sp.ratios_trail && (!h || sp.trail_pays[xl.p ? 1 : 0]);   // (no h: the array is written at every step)
  const VTerms vt = vterms(ctx);   // (vt.t = NULL where the ratio pass runs in the barrier kernel's launch)
  if (!rest_in_launch) {
    const int n_flags = trail ? (int)ctx->L : 0;
    const int n_lead_vt = (std::max(ctx->n_pairs, n_flags) + BLOCK - 1) / BLOCK;
    dispatch1(hk, [&](auto k_) {
      OB_LAUNCH(la, KID_RATIOS_PASS, (k_ratios_pass_vterms<U_MAIN, decltype(k_)::value>),
                sp.n_rest_ratio_tiles + n_lead_vt, ra, ctx->d_seg_max, ctx->n_c, ctx->tpc, lt, ctx->d_tile_seg0,
                ctx->d_seg_layer, sp.d_rest_ratio_tiles, vh, vt, ctx->d_vterms, n_lead_vt, sp.d_trail_flag, n_flags);
    });
  }
  // launch 2: the layers that are too large for the barrier kernel: ratio pass from the history and update, or the ratio pass alone
  if (trail) {
    RatioTrailTab tt;
    tt.items = sp.d_items;
    tt.lt = big_tiles(ctx, sp);
    tt.count0 = sp.d_count0; tt.count = sp.d_count; tt.sub_max = sp.d_sub_max; tt.tile_max = sp.d_tile_max;
    tt.flag = sp.d_trail_flag; tt.seg_max = ctx->d_seg_max; tt.errflag = ctx->d_errflag; tt.spin_limit = ctx->spin_limit;
    tt.c_avg = st->c_avg; tt.r_prev = st->r_prev; tt.coeff_c = st->coeff_c;
    tt.one_m_thr = ctx->one_m_thr; tt.one_p_thr = ctx->one_p_thr; tt.r_min = ctx->r_min; tt.r_max = ctx->r_max;
    dispatch2(hk, xl.p != nullptr, [&](auto k_, auto lx) {
      OB_LAUNCH(la, KID_RATIOS_TRAIL, (k_ratios_trail<decltype(k_)::value, decltype(lx)::value>), sp.n_items, ra, vh, vt,
                aa, tt, lt);
    });
  } else if (sp.big_on)
    dispatch1(hk, [&](auto k_) {
      OB_LAUNCH(la, KID_RATIOS_BIG_HIST, (k_ratios_big_hist<decltype(k_)::value>), sp.n_big_tiles, ra, vh, vt, ctx->d_seg_max,
                sp.d_big_tiles, ctx->n_c, sp.tpc, ctx->tpc, lt, ctx->d_tile_seg0);
    });
  if (!sp.on) {
    OB_LAUNCH_B(la, KID_RATIOS_FINALIZE, k_ratios_finalize, (int)ctx->L, FBLOCK, ctx->d_seg_max,
                ctx->d_layer_seg0, st->c_avg, st->r_prev, st->coeff_c, ctx->one_m_thr, ctx->one_p_thr,
                ctx->r_min, ctx->r_max, (const unsigned char*)(trail ? sp.d_has_tiles : nullptr));
    if (trail) launch_apply(la, ctx, st, packed_all, server_scales, lr, sp.d_rest_ratio_tiles, sp.n_rest_ratio_tiles, xl);
    else launch_apply(la, ctx, st, packed_all, server_scales, lr, nullptr, ctx->n_tiles, xl);
    return la.ok ? OB_OK : OB_ERR_HIP;
  }
  // launch 3: the barrier kernel; its leading workgroups run launch 1's pass (its last ones then the update of the same tiles, where there
  // are no large ones beside them) or finish the layers without listed tiles
  // (lines 18-20 from the segment maxima that launches 1 and 2 left), the others the listed tiles
  LayerSync ls{};
  ls.seg_max = ctx->d_seg_max; ls.listed_max = sp.d_listed_max; ls.lt = listed_tiles(ctx, sp);
  ls.counter = sp.d_counter; ls.sub = sp.d_sub; ls.flag = sp.d_flag; ls.errflag = ctx->d_errflag;
  ls.spin_limit = ctx->spin_limit;
  ls.c_avg = st->c_avg; ls.r_prev = st->r_prev; ls.coeff_c = st->coeff_c;
  ls.one_m_thr = ctx->one_m_thr; ls.one_p_thr = ctx->one_p_thr; ls.r_min = ctx->r_min; ls.r_max = ctx->r_max;
  ls.n_lead = (sp.n_layers < ctx->L) ? (int)ctx->L : 0;
  if (trail) ls.done = sp.d_has_tiles;
  if (rest_in_launch) {
    ls.n_alone = sp.n_alone; ls.n_lead = sp.n_alone + sp.n_rest_ratio_tiles;
    ls.rest_tiles = sp.d_rest_ratio_tiles; ls.alone = sp.d_alone; ls.arr0 = sp.d_arr0;
    ls.skip_first = sp.d_skip_first; ls.skip_end = sp.d_skip_end;
    ls.tile_seg0 = ctx->d_tile_seg0; ls.seg_layer = ctx->d_seg_layer;
    ls.counter = sp.d_counter_rest; ls.sub = sp.d_sub_rest; ls.flag = sp.d_flag_rest;
    ls.n_tiles = sp.n_fused_tiles; ls.n_events = (unsigned int)sp.n_events; ls.events = sp.d_events; ls.launches = sp.d_launches;
    ls.tail_launches = sp.d_tail_launches;
  }
  dispatch2(hk, xl.p != nullptr, [&](auto k_, auto lx) {
    dispatch2(sp.in_lds, rest_in_launch, [&](auto in_lds, auto rest) {
      OB_LAUNCH(la, sp.in_lds ? KID_RATIOS_APPLY_HIST_LDS : KID_RATIOS_APPLY_HIST,
                (k_ratios_apply_hist<decltype(k_)::value, decltype(lx)::value, decltype(in_lds)::value ? S_LH : 0,
                                     decltype(rest)::value>),
                sp.n_fused_tiles + ls.n_lead + (ls.n_events ? sp.n_rest_ratio_tiles : 0), ra, vh, vt, aa, ls, lt);
    });
  });
  if (ls.n_events) return la.ok ? OB_OK : OB_ERR_HIP;   // (the rest tiles are updated in that launch)
  if (trail) launch_apply(la, ctx, st, packed_all, server_scales, lr, sp.d_rest_ratio_tiles, sp.n_rest_ratio_tiles, xl);
  else launch_apply(la, ctx, st, packed_all, server_scales, lr, sp.d_rest_tiles, sp.n_rest_tiles, xl);
  return la.ok ? OB_OK : OB_ERR_HIP;
}

ob_status ob_lamb_ratios_apply_hist(ob_lamb_ctx* ctx, const ob_lamb_state* st, const uint32_t* packed_all,
                                    const float* server_scales, float lr, const ob_lamb_vf_history* h,
                                    void* hip_stream) {
  return ob_lamb_ratios_apply_hist_lp(ctx, st, packed_all, server_scales, lr, h, nullptr, OB_F32, hip_stream);
}

ob_status ob_lamb_variance_dense(ob_lamb_ctx* ctx, const ob_lamb_state* st, const uint32_t* packed_all,
                                 const float* server_scales, const ob_lamb_vf_history* h, float* v_out,
                                 void* hip_stream) {
  if (ob_status s = check_common(ctx, st)) return s;
  REQUIRE_PTR(packed_all); REQUIRE_PTR(st->v_fresh); REQUIRE_PTR(st->v_frozen); REQUIRE_PTR(v_out);
  if (!server_scales) return OB_ERR_NULL;
  bool packed_m = false;
  PackedMom pm;
  if (ob_status s = momentum_source(st, &packed_m, &pm)) return s;
  if (!packed_m || st->m_packed == packed_all) return OB_ERR_ARG;
  VfHist vh;
  if (ob_status s = vf_history(h, &vh)) return s;
  vh.write_v = (v_out == st->v_fresh) ? 1 : 0;   // in place: through the array's own pointer
  Launch la(ctx, hip_stream);
  if (!vh.write_v) {   // everything outside the listed tiles is up to date in the array itself
    la.begin(KID_COPY, true);
    if (la.ok)
      la.ok = hip_ok(ctx, hipMemcpyAsync(v_out, st->v_fresh, (size_t)ctx->n_pad * sizeof(float),
                                         hipMemcpyDeviceToDevice, la.stream), "hipMemcpyAsync");
    la.end("copy", true);
  }
  LayerSplit& sp = ctx->sp_apply;
  if ((sp.on || sp.big_on) && sp.n_cov_tiles > 0) {
    const RatioArgs ra = ratio_args(ctx, st, packed_all, server_scales, pm);
    const LayerTab lt = layer_tab(ctx, st, ctx->d_first_layer);
    dispatch1(st->mom_scale != nullptr, [&](auto k_) {
      OB_LAUNCH(la, KID_VARIANCE_DENSE, (k_variance_dense<decltype(k_)::value>), sp.n_cov_tiles, ra, vh,
                vh.write_v ? (float*)nullptr : v_out, ctx->n_c, ctx->tpc, lt, sp.d_cov_tiles);
    });
  }
  return la.ok ? OB_OK : OB_ERR_HIP;
}

ob_status ob_lamb_momentum_dense(ob_lamb_ctx* ctx, const ob_lamb_state* st, float* m_out, void* hip_stream) {
  if (ob_status s = check_common(ctx, st)) return s;
  REQUIRE_PTR(m_out); REQUIRE_PTR(st->m_packed);
  if (!st->m_scales) return OB_ERR_NULL;
  PackedMom pm;
  pm.bits = st->m_packed;
  pm.scales = st->m_scales;
  Launch la(ctx, hip_stream);
  const LayerTab lt = layer_tab(ctx, st, ctx->d_first_layer);
  if (st->mom_scale)
    OB_LAUNCH(la, KID_MOMENTUM_DENSE, (k_momentum_dense<U_MAIN, true>), ctx->n_tiles, pm, m_out, ctx->n_c,
              ctx->tpc, lt);
  else
    OB_LAUNCH(la, KID_MOMENTUM_DENSE, (k_momentum_dense<U_MAIN, false>), ctx->n_tiles, pm, m_out, ctx->n_c,
              ctx->tpc, lt);
  return la.ok ? OB_OK : OB_ERR_HIP;
}

ob_status ob_lamb_error_dense(ob_lamb_ctx* ctx, const ob_lamb_state* st, float* err_out, void* hip_stream) {
  if (ob_status s = check_common(ctx, st)) return s;
  REQUIRE_PTR(err_out); REQUIRE_PTR(st->err_worker); REQUIRE_PTR(st->err_packed);
  if (!st->err_scales) return OB_ERR_NULL;
  PackedErr pe;
  pe.bits = st->err_packed; pe.scales = st->err_scales;
  Launch la(ctx, hip_stream);
  OB_LAUNCH(la, KID_ERROR_DENSE, k_error_dense, ctx->n_tiles, st->err_worker, pe, err_out, ctx->n_c, ctx->tpc);
  return la.ok ? OB_OK : OB_ERR_HIP;
}

ob_status ob_lamb_server_error_dense(ob_lamb_ctx* ctx, const ob_lamb_state* st, float* err_out,
                                     void* hip_stream) {
  if (ob_status s = check_common(ctx, st)) return s;
  REQUIRE_PTR(err_out); REQUIRE_PTR(st->err_server); REQUIRE_PTR(st->srv_err_packed);
  if (!st->srv_err_scale) return OB_ERR_NULL;
  PackedErr pe;
  pe.bits = st->srv_err_packed; pe.scales = st->srv_err_scale;
  Launch la(ctx, hip_stream);
  // the served chunk as a one-chunk buffer
  OB_LAUNCH(la, KID_ERROR_DENSE, k_error_dense, ctx->tpc_srv, st->err_server, pe, err_out, ctx->n_c,
            ctx->tpc_srv);
  return la.ok ? OB_OK : OB_ERR_HIP;
}

ob_status ob_lamb_momentum_scale(ob_lamb_ctx* ctx, const ob_lamb_state* st, void* hip_stream) {
  if (ob_status s = check_common(ctx, st)) return s;
  REQUIRE_PTR(st->m);
  if (!st->mom_scale) return OB_ERR_NULL;
  Launch la(ctx, hip_stream);
  const LayerTab lt = layer_tab(ctx, st, ctx->d_first_layer);
  constexpr int R = 8;   // tiles per workgroup
  static_assert(U_MAIN == 1, "the segment tables are those of the 1024-element tiling");
  OB_LAUNCH(la, KID_MOMENTUM_SCALE, (k_momentum_sumsq<R>), (ctx->n_tiles + R - 1) / R, st->m, ctx->d_seg_sums,
            ctx->n_c, ctx->tpc, ctx->n_tiles, lt, ctx->d_tile_seg0, ctx->d_seg_layer);
  OB_LAUNCH_B(la, KID_MOMENTUM_SCALE, k_layer_rms, (int)ctx->L, FBLOCK, ctx->d_seg_sums, ctx->d_layer_seg0,
              ctx->d_off, ctx->d_sigma);
  OB_LAUNCH_B(la, KID_MOMENTUM_SCALE, k_momentum_scale, 1, FBLOCK, ctx->d_sigma, ctx->d_off, (int)ctx->L,
              st->mom_scale);
  return la.ok ? OB_OK : OB_ERR_HIP;
}

ob_status ob_lamb_check_device_status(ob_lamb_ctx* ctx, void* hip_stream) {
  if (!ctx) return OB_ERR_NULL;
  hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
  unsigned int f = 0;
  if (!hip_ok(ctx, hipStreamSynchronize(stream), "hipStreamSynchronize") ||
      !hip_ok(ctx, hipMemcpy(&f, ctx->d_errflag, sizeof(f), hipMemcpyDeviceToHost), "hipMemcpy"))
    return OB_ERR_HIP;
  if (f == 0) return OB_OK;
  // a bounded wait expired: the step that raised it produced undefined outputs.  Re-arm the
  // synchronisation state and fall back to the two-pass kernels for the rest of this context.
  ctx->resident = false;
  ctx->u_srv_res = 0;
  const size_t line = sizeof(unsigned long long) * CTR_STRIDE;
  (void)hipMemset(ctx->d_counter_srv, 0, line);
  (void)hipMemset(ctx->d_sub_srv, 0, line * arrival_groups(ctx->tpc_srv_res));
  (void)hipMemset(ctx->d_flag_srv, 0, sizeof(unsigned long long));
  for (LayerSplit* sp : {&ctx->sp_apply, &ctx->sp_warm}) {
    sp->on = false;
    sp->big_on = sp->ratios_trail = false;   // (after an expiry every call takes the plain kernels)
    (void)hipMemset(sp->d_counter, 0, line * (size_t)ctx->L);
    (void)hipMemset(sp->d_sub, 0, line * group_lines(sp->n_fused_tiles, ctx->L));
    (void)hipMemset(sp->d_flag, 0, sizeof(unsigned long long) * (size_t)ctx->L);
  }
  ctx->sm_apply.u = 0;
  ctx->sm_warm.u = 0;
  (void)hipMemset(ctx->d_counter, 0, line * (size_t)ctx->W);
  (void)hipMemset(ctx->d_sub, 0, line * (size_t)ctx->W * arrival_groups(ctx->tpc_res));
  (void)hipMemset(ctx->d_flag, 0, sizeof(unsigned long long) * (size_t)ctx->W);
  (void)hipMemset(ctx->d_errflag, 0, sizeof(unsigned int));
  (void)hipDeviceSynchronize();
  return OB_ERR_STATE;
}

int64_t ob_lamb_fused_layers(const ob_lamb_ctx* ctx) { return (ctx && ctx->sp_apply.on) ? ctx->sp_apply.n_layers : 0; }
int64_t ob_lamb_fused_params(const ob_lamb_ctx* ctx) { return (ctx && ctx->sp_apply.on) ? ctx->sp_apply.n_params : 0; }
int64_t ob_lamb_big_tile_params(const ob_lamb_ctx* ctx) { return (ctx && ctx->sp_apply.big_on) ? ctx->sp_apply.n_big_params : 0; }
int64_t ob_lamb_warmup_fused_layers(const ob_lamb_ctx* ctx) { return (ctx && ctx->sp_warm.on) ? ctx->sp_warm.n_layers : 0; }
int64_t ob_lamb_warmup_fused_params(const ob_lamb_ctx* ctx) { return (ctx && ctx->sp_warm.on) ? ctx->sp_warm.n_params : 0; }

int32_t ob_lamb_uses_single_pass(const ob_lamb_ctx* ctx) { return (ctx && ctx->resident) ? 1 : 0; }
int32_t ob_lamb_server_single_pass(const ob_lamb_ctx* ctx) { return ctx ? ctx->u_srv_res : 0; }

ob_status ob_lamb_profile_enable(ob_lamb_ctx* ctx, int on) {
  if (!ctx) return OB_ERR_NULL;
  ctx->profile = (on != 0);
  return OB_OK;
}

int32_t ob_lamb_profile_read(ob_lamb_ctx* ctx, int32_t cap, const char** names, double* total_ms,
                             int64_t* launches) {
  if (!ctx) return 0;
  double ms[KID_COUNT] = {0};
  int64_t cnt[KID_COUNT] = {0};
  for (auto& r : ctx->prof) {
    float t = 0.0f;
    if (hipEventSynchronize(r.e1) == hipSuccess && hipEventElapsedTime(&t, r.e0, r.e1) == hipSuccess) {
      ms[r.kid] += t;
      cnt[r.kid] += 1;
    }
    (void)hipEventDestroy(r.e0);
    (void)hipEventDestroy(r.e1);
  }
  ctx->prof.clear();
  int32_t n = 0;
  for (int k = 0; k < KID_COUNT; ++k) {
    if (!cnt[k]) continue;
    if (n < cap) {
      if (names) names[n] = kKernelNames[k];
      if (total_ms) total_ms[n] = ms[k];
      if (launches) launches[n] = cnt[k];
    }
    ++n;
  }
  return n;
}

}  // extern "C"

// ---- Algorithm 1 line 10 for callers that cannot allocate -------------------------------------
// ob_lamb_server_reduce needs a context, whose creation allocates the partial sums that its
// kernels pass from the averaging pass to the scale.  This variant keeps them in a fixed array in
// the library's own device image instead: no context, no allocation of any kind.
namespace {
constexpr int64_t STATIC_MAX_CHUNK = (int64_t)1 << 25;                 // elements of the served chunk
constexpr int64_t STATIC_MAX_TILES = STATIC_MAX_CHUNK / TILE_SRV;      // 32768 partial sums = 256 KiB
}
// One copy per GPU the library runs on, alive until the process ends.  In host code this name is
// only a handle for hipGetSymbolAddress, never a device address.
static __device__ __align__(256) double scratch[STATIC_MAX_TILES];

namespace {
constexpr int STATIC_MAX_DEVICES = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[STATIC_MAX_DEVICES] = {};   // per device: the address of ITS copy of `scratch`

// Device address of the current device's scratch array (looked up once per device).
ob_status static_scratch(double** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return OB_ERR_HIP;
  if (dev < 0 || dev >= STATIC_MAX_DEVICES) return OB_ERR_ARG;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return OB_ERR_HIP;
    g_scratch_ptr[dev] = static_cast<double*>(p);
  }
  *out = g_scratch_ptr[dev];
  return OB_OK;
}
}  // namespace

extern "C" {

int64_t ob_lamb_static_max_chunk_len(void) { return STATIC_MAX_CHUNK; }

ob_status ob_lamb_diag_copy(const float* src, float* dst, int64_t n, void* hip_stream) {
  if (n < 0 || n > ((int64_t)1 << 40)) return OB_ERR_ARG;
  REQUIRE_PTR(src); REQUIRE_PTR(dst);
  if (n == 0) return OB_OK;
  const int64_t tiles = (n + SPAN - 1) / SPAN;
  if (tiles > 0x7fffffff) return OB_ERR_ARG;
  hipLaunchKernelGGL(k_diag_copy, dim3((unsigned)tiles), dim3(BLOCK), 0, reinterpret_cast<hipStream_t>(hip_stream),
                     src, dst, n);
  return hipGetLastError() == hipSuccess ? OB_OK : OB_ERR_HIP;
}

ob_status ob_lamb_server_reduce_static(int32_t num_workers, int64_t chunk_len, const uint32_t* packed_in,
                                       const float* scales_in, float* err_server, uint32_t* packed_out,
                                       float* scale_out, void* hip_stream) {
  if (num_workers < 1 || num_workers > 65536 || chunk_len < 256 || chunk_len % 256 != 0) return OB_ERR_ARG;
  if (chunk_len > STATIC_MAX_CHUNK) return OB_ERR_SIZE;
  if ((int64_t)num_workers * (chunk_len / 8) >= ((int64_t)1 << 31)) return OB_ERR_SIZE;   // 32-bit offsets into packed_in
  REQUIRE_PTR(packed_in); REQUIRE_PTR(packed_out); REQUIRE_PTR(err_server);
  if (!scales_in || !scale_out) return OB_ERR_NULL;
  double* partials = nullptr;
  if (ob_status s = static_scratch(&partials)) return s;
  hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
  const int tiles = (int)((chunk_len + TILE_SRV - 1) / TILE_SRV);   // <= STATIC_MAX_TILES
  const float invW = 1.0f / (float)num_workers;
  // the three kernels of ob_lamb_server_reduce's barrier-free form; every partial that the second
  // reads has been written by the first, so the array's previous contents do not matter
  hipLaunchKernelGGL((k_server_unpack_avg<U_SRV>), dim3((unsigned)tiles), dim3(BLOCK), 0, stream, packed_in,
                     scales_in, err_server, partials, chunk_len, (int)num_workers, invW, (uint32_t*)nullptr,
                     (const float*)nullptr, (uint32_t*)nullptr, ChunkTicket{});
  hipLaunchKernelGGL(k_chunk_scale, dim3(1), dim3(FBLOCK), 0, stream, partials, tiles, chunk_len, scale_out,
                     (float*)nullptr, 0);
  hipLaunchKernelGGL((k_sign_pack_error<U_SRV>), dim3((unsigned)tiles), dim3(BLOCK), 0, stream, err_server,
                     packed_out, scale_out, chunk_len, tiles);
  return hipGetLastError() == hipSuccess ? OB_OK : OB_ERR_HIP;
}

}  // extern "C"
