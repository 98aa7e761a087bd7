// Device code of libonebitlamb (gfx950): every kernel of the compression-stage step of 1-bit LAMB
// (arXiv 2104.06069, Algorithm 1) and of the LAMB warmup step (eq. (1)).  Included by
// onebitlamb.hip only.
//
// Arithmetic contract: IEEE binary32, one rounding per operation (the build passes
// -ffp-contract=off; hipcc's default divide and sqrt are correctly rounded), evaluated in the
// operation order written below; the sum-of-squares reductions accumulate in binary64 in a fixed
// order.  Never build with -ffast-math.
//
// Layout of the work.  The padded flat buffer is W chunks of n_c elements (n_c % 256 == 0).
// Every N-sized kernel runs on "tiles": tile (c, b) is elements [c*n_c + b*TILE, +TILE) clipped
// to the chunk, so a tile never crosses a chunk boundary and its length is a multiple of 256.
// A workgroup of 256 threads owns one tile; thread t touches elements tile0 + u*1024 + 4*t + k
// (u < U, k < 4) with 128-bit accesses, i.e. each wavefront-wide access covers 256 consecutive
// elements = 8 consecutive 32-bit words of a packed sign stream.
//
// Layers (tensors) are arbitrary, unaligned ranges of the flat buffer.  A host-built table gives
// the layer of each tile's first element (L = padding); a tile that lies inside one layer takes a
// vectorised path with per-tile scalars, a tile that meets a layer boundary or the end of the
// parameters takes a per-element path that walks the offset table.
//
// The momentum m_{t-1} has two sources: a dense fp32 array, or (template flag PACKED_M) the 1-bit
// form it has had since line 13 of the previous step: m[i] = (bit ? +s_c : -s_c) / k_l for
// i < N and 0 in the padding, where s_c is the previous step's server scale of chunk c.  Both give
// the same bits: the dense array holds exactly those values.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "ob_plan.h"

namespace obk {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int FBLOCK = 1024;     // threads per workgroup of the small per-layer / per-chunk finalize kernels
#define OB_AGENT __HIP_MEMORY_SCOPE_AGENT
#ifndef OB_POLL_SLEEP
#define OB_POLL_SLEEP 16  // s_sleep argument (units of 64 clocks) between two polls of a barrier flag
#endif

// Every N-sized array is read once and written once per kernel: 128-bit nontemporal (streaming)
// accesses, which measure ~10 % faster than plain ones on MI355X for these patterns.
__device__ __forceinline__ v4f ld4(const float* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const v4f*>(p));
}
__device__ __forceinline__ void st4(float* p, v4f v) {
  __builtin_nontemporal_store(v, reinterpret_cast<v4f*>(p));
}

// What the next kernel of the step reads again is loaded without the nontemporal hint: k_compress_resident's dense momentum,
// which k_ratios_pass reads, and that kernel's v_frozen, which k_decompress_apply does (keeps_second_reads says for which lists).
// Where they cover the whole buffer, k_ratios_pass goes from its end to its start (tile_from_end), so that the 256 MB
// memory-side cache still holds what it and the kernel after it read first, and the L2s, tile by tile, what fits them.
// Measured (4 bytes per element each, of the 53 that a step moves), us a step, everything nontemporal and from the start /
// v_frozen kept, k_decompress_apply from the end / both kept, k_ratios_pass from the end: 110 M parameters 902 / 884 / 865,
// 42 M 357 / 346 / 331, 80 M 649 / 630 / 611, 8 M 86.4 / 86.4 / 84.3, 336 M 2679 / - / 2661; from the end with each tile on another XCD /
// on its own: 42 M 319.5 / 319.4, 21 M 167.5 / 165.4, 11 M 103.0 / 100.4, 4.2 M 57.8 / 56.8, 2.1 M 43.9 / 42.7, 1 M 36.9 / 36.2.
__device__ __forceinline__ v4f ld4_keep(const float* p) { return *reinterpret_cast<const v4f*>(p); }
// Which of the two is a template argument (for a value of the launch: the cache policy of the buffer builtins): the
// compiler merges two loads of one address under a condition into one without the hint.
template <bool KEEP>
__device__ __forceinline__ v4f ld4_keep_if(const float* p) {
  if constexpr (KEEP) return ld4_keep(p);
  else return ld4(p);
}

// 16 bytes per lane from p straight into LDS: lane i's to dst[i], dst the same for the whole
// wavefront, all of whose lanes take part.  The data is there after lds_loads_done() of the same wavefront.
__device__ __forceinline__ void lds_load16(const float* p, v4f* dst) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)p,
                                   (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}
__device__ __forceinline__ void lds_loads_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// 16-bit storage of the mixed-precision variant (the paper trains in FP16, Section 6): a gradient
// may arrive as IEEE binary16 or bfloat16 and a 16-bit copy of the parameters may be written; all
// arithmetic stays binary32.  GT / LPX are template flags so that the fp32-only instantiations
// keep their code.
typedef unsigned short v4h __attribute__((ext_vector_type(4)));

struct GradSrc {
  const void* __restrict__ p;   // float (GT == 0) or 16-bit patterns (GT == 1)
  float scale;                  // g = value * scale (GT == 1 only; the inverse loss scale)
  int bf16;                     // GT == 1: 0 = binary16, 1 = bfloat16
};

__device__ __forceinline__ float lp_to_float(unsigned short h, int bf16) {
  if (bf16) return __uint_as_float((unsigned int)h << 16);
  return (float)__builtin_bit_cast(_Float16, h);   // exact
}

// binary32 -> nearest 16-bit value, ties to even; NaN -> the format's canonical quiet NaN
__device__ __forceinline__ unsigned short float_to_lp(float x, int bf16) {
  if (bf16) {
    const unsigned int u = __float_as_uint(x);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)0x7fc0;
    return (unsigned short)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
  }
  if (x != x) return (unsigned short)0x7e00;
  return __builtin_bit_cast(unsigned short, (_Float16)x);   // hardware convert, round to nearest even
}

// The thread's 4 gradient values at flat index i (a multiple of 4): the load, and the values from what it
// brought.  (Apart, so that a kernel can request everything before it converts anything: the conversion
// branches on the format, and no load moves across that branch.)
template <int GT>
__device__ __forceinline__ typename std::conditional<GT == 0, v4f, v4h>::type grad_request(const GradSrc& gs, int64_t i) {
  if constexpr (GT == 0) return ld4(reinterpret_cast<const float*>(gs.p) + i);
  else return __builtin_nontemporal_load(reinterpret_cast<const v4h*>(reinterpret_cast<const unsigned short*>(gs.p) + i));
}
__device__ __forceinline__ v4f grad_value(const GradSrc&, v4f g) { return g; }
__device__ __forceinline__ v4f grad_value(const GradSrc& gs, v4h h) {
  v4f r;
#pragma unroll
  for (int k = 0; k < 4; ++k) r[k] = lp_to_float(h[k], gs.bf16) * gs.scale;
  return r;
}
template <int GT>
__device__ __forceinline__ v4f load_grad(const GradSrc& gs, int64_t i) { return grad_value(gs, grad_request<GT>(gs, i)); }

// (i0: uniform.)
__device__ __forceinline__ void st4_lp(void* __restrict__ base, int64_t i0, int o, v4f v, int bf16) {
  v4h h;
#pragma unroll
  for (int k = 0; k < 4; ++k) h[k] = float_to_lp(v[k], bf16);
  __builtin_nontemporal_store(h, reinterpret_cast<v4h*>(reinterpret_cast<unsigned short*>(base) + i0 + o));
}

// Reductions over a wavefront, valid in lane 0: the lanes' halves, rows of 16 and parts of a row meet by register moves
// (whole wavefronts only).  Through LDS (ds_bpermute) each of the six steps is a round trip of some 130 clocks, twice that for a
// double, at the end of every tile's chain.  A step, us, LDS / moves: four 512x512 tensors 23.4 / 22.3, 336 M parameters with bf16 gradient
// and copy 1775 / 1737, fp32 1707 / 1696; a LAMB step of 3 M 27.0 / 26.5.
template <int STEP>   // lane i's value of lane i + 32 >> STEP, for the lanes that lane 0's result is made of
__device__ __forceinline__ unsigned int lane_down(unsigned int v) {
  if constexpr (STEP == 0) return __builtin_amdgcn_permlane32_swap(v, v, false, false)[1];
  else if constexpr (STEP == 1) return __builtin_amdgcn_permlane16_swap(v, v, false, false)[1];
  else return __builtin_amdgcn_update_dpp(0u, v, 0x100 + (32 >> STEP) /* row_shl */, 0xf, 0xf, true);
}
template <int STEP>
__device__ __forceinline__ float lane_down(float v) { return __uint_as_float(lane_down<STEP>(__float_as_uint(v))); }
template <int STEP>
__device__ __forceinline__ double lane_down(double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const unsigned long long r = (unsigned long long)lane_down<STEP>((unsigned int)b) |
                               (unsigned long long)lane_down<STEP>((unsigned int)(b >> 32)) << 32;
  return __builtin_bit_cast(double, r);
}
template <class T, class F>
__device__ __forceinline__ T wave_reduce(T v, F f) {
  v = f(v, lane_down<0>(v));
  v = f(v, lane_down<1>(v));
  v = f(v, lane_down<2>(v));
  v = f(v, lane_down<3>(v));
  v = f(v, lane_down<4>(v));
  return f(v, lane_down<5>(v));
}
__device__ __forceinline__ double wave_sum(double v) { return wave_reduce(v, [](double a, double b) { return a + b; }); }
// of non-NaN values
__device__ __forceinline__ float wave_max(float v) { return wave_reduce(v, [](float a, float b) { return (b > a) ? b : a; }); }

// Sum of one double per thread over a workgroup of NT threads, in a fixed order; result valid in
// thread 0.  lds: [NT / WAVE] doubles.
template <int NT = BLOCK, bool THROUGH_LDS = false>
__device__ __forceinline__ double block_sum(double v, double* lds) {
  if constexpr (THROUGH_LDS) {
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) v += __shfl_down(v, o, WAVE);
  } else {
    v = wave_sum(v);
  }
  const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
  __syncthreads();  // protects lds against the previous use
  if (lane == 0) lds[wv] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0) {
#pragma unroll
    for (int i = 0; i < NT / WAVE; ++i) r += lds[i];
  }
  return r;
}

// Max of one non-NaN, non-negative float per thread over a workgroup of NT threads; valid in
// thread 0.  lds: [NT / WAVE] floats.
template <int NT = BLOCK>
__device__ __forceinline__ float block_max(float v, float* lds) {
  v = wave_max(v);
  const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
  __syncthreads();
  if (lane == 0) lds[wv] = v;
  __syncthreads();
  float r = 0.0f;
  if (threadIdx.x == 0) {
#pragma unroll
    for (int i = 0; i < NT / WAVE; ++i) r = (lds[i] > r) ? lds[i] : r;
  }
  return r;
}

// off has L+2 entries, off[L+1] = INT64_MAX, so the walk stops at L (= padding) at the latest.
__device__ __forceinline__ int walk_layer(int l, int64_t i, const int64_t* __restrict__ off) {
  while (i >= off[l + 1]) ++l;
  return l;
}

// Sign nibble of the lane's 4 elements -> the 32-bit word of its 8-lane group (in every lane of
// the group).  Element 4*lane + k of the 256-element span is bit 4*(lane%8) + k of word lane/8.
// THROUGH_LDS (here and in block_sum): by ds_bpermute, as k_compress_resident does, whose 16 spans a tile leave a barrier together.  A step of the plain
// form on the same buffers, us, register moves / LDS: 214 M elements 1703 / 1687, 100 M 786 / 781, 54 M 419 / 412, 34 M 265 / 261, 18 M 146.3 /
// 145.6, 4.4 M 55.8 / 54.9; with a bf16 gradient 54 M 393 / 394, 18 M 138.2 / 138.9, 4.4 M 54.0 / 54.8; either one alone changes nothing.  Occupancy (5
// workgroups) and spills (none) are alike; what differs is how closely the 16 spans' stores follow each other.  k_server_resident, of 1 to 4 spans and with
// the same barrier, keeps the moves: its call 8.7 / 9.1 (8 workers, 1.4 M elements), 17.1 / 17.5 (64, 1.7 M), 37.1 / 37.5 (256, 1.3 M).
template <bool THROUGH_LDS = false>
__device__ __forceinline__ unsigned int gather_word(unsigned int nibble) {
  unsigned int v = nibble << (4 * (threadIdx.x & 7));
  if constexpr (THROUGH_LDS) {
    v |= __shfl_xor(v, 1, WAVE);
    v |= __shfl_xor(v, 2, WAVE);
    v |= __shfl_xor(v, 4, WAVE);
    return v;
  }
  v |= __builtin_amdgcn_update_dpp(0u, v, 0xb1 /* quad_perm 1 0 3 2 */, 0xf, 0xf, true);
  v |= __builtin_amdgcn_update_dpp(0u, v, 0x4e /* quad_perm 2 3 0 1 */, 0xf, 0xf, true);
  v |= __builtin_amdgcn_update_dpp(0u, v, 0x141 /* row_half_mirror */, 0xf, 0xf, true);
  return v;
}

// The lane's sign nibble from a packed stream: the bits of elements span0 + 4*threadIdx.x + k,
// span0 uniform and a multiple of 1024.
__device__ __forceinline__ unsigned int load_nibble(const uint32_t* __restrict__ packed, int64_t span0) {
  return (packed + (span0 >> 5))[threadIdx.x >> 3] >> (4 * (threadIdx.x & 7));  // bits 0..3 are the lane's
}

struct TilePos {
  int t;          // tile index (chunk-major)
  int c;          // chunk
  int64_t tile0;  // first element
  int len;        // elements in the tile (multiple of 256)
};

// Tile t of the tiling with TILE elements per tile and tpc tiles per chunk.
template <int TILE>
__device__ __forceinline__ TilePos tile_pos(int64_t n_c, int tpc, int t) {
  TilePos p;
  p.t = t;
  p.c = t / tpc;
  const int b = t - p.c * tpc;
  const int64_t in_chunk = (int64_t)b * TILE;
  p.tile0 = (int64_t)p.c * n_c + in_chunk;
  const int64_t rest = n_c - in_chunk;
  p.len = rest < TILE ? (int)rest : TILE;
  return p;
}

// Per-layer tables (device pointers) shared by the layer-aware kernels.
struct LayerTab {
  const float* __restrict__ mom_scale;   // [L] k_l of Appendix A.5.2 (only read when HAS_K)
  const int64_t* __restrict__ off;       // [L+2]
  const int* __restrict__ first_layer;   // [tiles of the launching kernel's tile size]
  int L;
};

// The layer-wise N-sized kernels take an optional tile list: the launch then covers tile
// tile_list[blockIdx.x] instead of tile blockIdx.x (the tiles outside the ones a kernel with a
// per-layer barrier handles).
__device__ __forceinline__ int listed_tile(const int* __restrict__ tile_list) {
  return tile_list ? tile_list[blockIdx.x] : (int)blockIdx.x;
}

// Momentum source in 1-bit form (only read when PACKED_M).
struct PackedMom {
  const uint32_t* __restrict__ bits;     // [N_pad/32]
  const float* __restrict__ scales;      // [W]
};

// Second destination of the worker's chunk `chunk` (see ob_lamb_state.own_packed_in); packed == NULL: none.
struct OwnCopy {
  uint32_t* packed;   // [n_c/32]
  float* scale;       // [1]
  int chunk;
};

// The worker error in deferred form (only read when DEFER): err holds z of the previous step, and
// delta = z - C[z] is formed on the fly from the previous step's own sign words and chunk scales,
// delta[i] = err[i] - (bit_i ? s_c : -s_c) -- the very subtraction of Algorithm 1 line 7, one step
// late.  With all scales 0 the array is the error itself (x - (+-0) = x).
struct PackedErr {
  const uint32_t* bits;     // [N_pad/32] this worker's own previous output (may be packed_out itself)
  const float* scales;      // [W]        ... and its scales (may be scales_out itself)
};

__device__ __forceinline__ v4f deferred_error(v4f e, unsigned int nib, float s) {
  v4f r;
#pragma unroll
  for (int k = 0; k < 4; ++k) r[k] = e[k] - (((nib >> k) & 1u) ? s : -s);
  return r;
}

// ---------------------------------------------------------------------------------------------
// z = k_l * (beta1*m + (1-beta1)*g) + err       (Algorithm 1 lines 6-7, Appendix A.5.2)
// Per-tile constants and the per-access evaluation, shared by the two-pass and single-pass kernels.
// ---------------------------------------------------------------------------------------------
template <bool HAS_K, bool PACKED_M>
struct ZTile {
  bool uniform;  // one set of constants serves the whole tile
  bool pad;      // the whole tile lies in the padding
  int l0;        // layer of the tile's first element (HAS_K)
  float kt;      // k of the tile's layer (uniform tiles)
  float bm;      // beta1 * |m| (PACKED_M; for HAS_K only on uniform tiles)
  float s_prev;  // previous server scale of the chunk (PACKED_M)
  int64_t N;
  // layer cursor of the per-element path (HAS_K, tile meets a layer boundary)
  int cur_l;
  int64_t cur_end;
  float cur_k, cur_b;
  bool cur_real;

  __device__ __forceinline__ void init(const LayerTab& lt, const PackedMom& pm, const TilePos& p,
                                       float beta1) {
    uniform = true; pad = false; l0 = 0; kt = 1.0f; bm = 0.0f; s_prev = 0.0f; N = 0;
    cur_l = 0; cur_end = 0; cur_k = 1.0f; cur_b = 0.0f; cur_real = false;
    if (PACKED_M) s_prev = pm.scales[p.c];
    if (HAS_K) {
      // k differs from layer to layer: the tile must lie inside one layer (or in the padding)
      l0 = lt.first_layer[p.t];
      uniform = (p.tile0 + p.len <= lt.off[l0 + 1]);
      pad = (l0 >= lt.L);
      if (uniform && !pad) {
        kt = lt.mom_scale[l0];
        if (PACKED_M) bm = beta1 * (s_prev / kt);
      }
      if (!uniform) {  // l0 < L here: a tile that starts in the padding is uniform
        cur_l = l0;
        cur_end = lt.off[l0 + 1];
        cur_real = true;
        cur_k = lt.mom_scale[l0];
        if (PACKED_M) cur_b = beta1 * (s_prev / cur_k);
      }
    } else if (PACKED_M) {
      // only the end of the parameters matters: the 1-bit momentum is 0 in the padding
      N = lt.off[lt.L];
      pad = (p.tile0 >= N);
      uniform = pad || (p.tile0 + p.len <= N);
      bm = beta1 * s_prev;
    }
  }

  // G, E: gradient and carried error; M: dense momentum (ignored when PACKED_M); nib: the sign
  // bits of the packed momentum (ignored otherwise); i0: flat index of the first element.
  // Calls must come in increasing i0 for one thread (the per-element path keeps a cursor).
  // KNOWN_UNIFORM: the caller has tested `uniform` itself (a copy of its loop without the other
  // paths in it).
  template <bool KNOWN_UNIFORM = false>
  __device__ __forceinline__ v4f z(const LayerTab& lt, float beta1, float omb1, v4f G, v4f M,
                                   unsigned int nib, v4f E, int64_t i0) {
    v4f r;
    if (KNOWN_UNIFORM || uniform) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float bmk;
        if (PACKED_M) bmk = pad ? 0.0f : (((nib >> k) & 1u) ? bm : -bm);
        else bmk = beta1 * M[k];
        const float mloc = bmk + omb1 * G[k];
        r[k] = HAS_K ? kt * mloc + E[k] : mloc + E[k];
      }
    } else if (HAS_K) {
      // A thread's elements come in increasing order over the whole tile, so the layer cursor
      // only moves forward and its constants are re-formed only when a boundary is crossed.
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int64_t i = i0 + k;
        if (i >= cur_end) {
          do {
            ++cur_l;
            cur_end = lt.off[cur_l + 1];
          } while (i >= cur_end);
          cur_real = (cur_l < lt.L);
          cur_k = cur_real ? lt.mom_scale[cur_l] : 1.0f;
          if (PACKED_M) cur_b = beta1 * (s_prev / cur_k);
        }
        float bmk;
        if (PACKED_M) bmk = cur_real ? (((nib >> k) & 1u) ? cur_b : -cur_b) : 0.0f;
        else bmk = beta1 * M[k];
        const float mloc = bmk + omb1 * G[k];
        r[k] = cur_k * mloc + E[k];
      }
    } else {  // PACKED_M without k: the tile straddles the end of the parameters
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float bmk = (i0 + k < N) ? (((nib >> k) & 1u) ? bm : -bm) : 0.0f;
        r[k] = (bmk + omb1 * G[k]) + E[k];
      }
    }
    return r;
  }
};

// ---------------------------------------------------------------------------------------------
// The chunk's scale without a launch of its own: the last workgroup of the chunk to finish sums the
// partials.  Arrivals are counted in two levels, TICKET_SUB tiles each (atomics on one cache line are
// served one at a time); whoever completes a counter sets it back, so nothing changes from call to call.
// Only the first wavefront takes part, after the workgroup's stores: nothing waits for anything.
// ---------------------------------------------------------------------------------------------
struct ChunkTicket {
  unsigned int* count;     // lines of CTR_STRIDE 8-byte words: [chunks] second level, [chunks * spc] first level
  double* sub_part;        // [chunks * spc]
  int n_chunks, spc;       // first-level counters per chunk
  float* scales;           // [chunks]
  float* own_scale;        // also receives the scale of chunk own_chunk (NULL: none)
  int own_chunk;
};
__device__ __forceinline__ bool ticket_arrive(unsigned int* counter, unsigned int n, double* payload, double s) {
  int last = 0;
  if ((threadIdx.x & (WAVE - 1)) == 0) {
    __hip_atomic_store(payload, s, __ATOMIC_RELAXED, OB_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the payload is there before the arrival
    last = (__hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, OB_AGENT) + 1u == n);
    if (last) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, OB_AGENT);
  }
  return __builtin_amdgcn_readfirstlane(last) != 0;
}
// s: the tile's partial (lane 0); first wavefront only
__device__ __forceinline__ void chunk_ticket(const ChunkTicket& tk, double* partials, const TilePos& p, int tpc,
                                             int64_t n_c, double s) {
  constexpr int LINE = 2 * CTR_STRIDE;
  const int lane = threadIdx.x & (WAVE - 1);
  const int b = p.t - p.c * tpc, sub = b / TICKET_SUB, first = sub * TICKET_SUB;
  const int n = (tpc - first < TICKET_SUB) ? tpc - first : TICKET_SUB;
  const int64_t si = (int64_t)p.c * tk.spc + sub;
  if (!ticket_arrive(tk.count + (tk.n_chunks + si) * LINE, (unsigned int)n, &partials[p.t], s)) return;
  double q = (lane < n) ? __hip_atomic_load(&partials[(int64_t)p.c * tpc + first + lane], __ATOMIC_RELAXED, OB_AGENT) : 0.0;
  q = wave_sum(q);
  if (tk.spc > 1) {
    if (!ticket_arrive(tk.count + (int64_t)p.c * LINE, (unsigned int)tk.spc, &tk.sub_part[si], q)) return;
    q = 0.0;
    for (int j = lane; j < tk.spc; j += WAVE)
      q += __hip_atomic_load(&tk.sub_part[(int64_t)p.c * tk.spc + j], __ATOMIC_RELAXED, OB_AGENT);
    q = wave_sum(q);
  }
  if (lane == 0) {
    const float sc = (float)sqrt(q / (double)n_c);
    tk.scales[p.c] = sc;
    if (tk.own_scale && p.c == tk.own_chunk) *tk.own_scale = sc;
  }
}

// ---------------------------------------------------------------------------------------------
// K1  z written over err, and the tile's sum of z^2 in fp64: the first of the two passes of the
// worker compression (k_sign_pack_error is the second), or, with DEFER, all of it.
// ---------------------------------------------------------------------------------------------
// DEFER: the whole of lines 6-7 in this one pass, with no wait for the chunk's scale: the carried
// error arrives in deferred form (PackedErr), z is written over it AS the next deferred error, and
// the sign words of z are packed and written here as well (they do not depend on the scale); the
// scale itself follows from the tile partials, in k_chunk_scale or (TICKET) in the last workgroup of
// the chunk to finish.  packed_out / pe.bits may be the same buffer: a word is read and rewritten by
// the same 8 lanes, in program order.
// SUM_LDS (and the sign words): worker_sum_lds in the host code.
template <int U, bool HAS_K, bool PACKED_M, int GT = 0, bool DEFER = false, bool TICKET = false, bool SUM_LDS = false>
__global__ __launch_bounds__(BLOCK) void k_momentum_z_sumsq(
    GradSrc g, const float* __restrict__ m, PackedMom pm,
    float* __restrict__ err, double* __restrict__ partials, int64_t n_c, int tpc, float beta1,
    float omb1, LayerTab lt, PackedErr pe, uint32_t* packed_out, OwnCopy oc, ChunkTicket tk) {
  constexpr int TILE = SPAN * U;
  __shared__ double lds[BLOCK / WAVE];
  const TilePos p = tile_pos<TILE>(n_c, tpc, (int)blockIdx.x);
  const int o0 = threadIdx.x * 4;
  const float se = DEFER ? pe.scales[p.c] : 0.0f;
  v4f G[U], M[U], E[U];
  unsigned int NB[U], EB[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    M[u] = 0.0f; NB[u] = 0u; EB[u] = 0u;
    if (o < p.len) {
      G[u] = load_grad<GT>(g, p.tile0 + o);
      if (PACKED_M) NB[u] = load_nibble(pm.bits, p.tile0 + u * SPAN);
      else M[u] = ld4(m + p.tile0 + o);
      if (DEFER) EB[u] = load_nibble(pe.bits, p.tile0 + u * SPAN);
      E[u] = ld4(err + p.tile0 + o);
    }
  }
  ZTile<HAS_K, PACKED_M> zt;
  zt.init(lt, pm, p, beta1);
  uint32_t* own = (DEFER && oc.packed && p.c == oc.chunk) ? oc.packed : nullptr;   // uniform
  const int64_t own_tile0 = (p.tile0 - (int64_t)p.c * n_c) >> 5;
  double acc = 0.0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    if (o < p.len) {   // uniform over the wavefront (len is a multiple of 256), as the shuffles below require
      if (DEFER) E[u] = deferred_error(E[u], EB[u], se);
      const v4f z = zt.z(lt, beta1, omb1, G[u], M[u], NB[u], E[u], p.tile0 + o);
      st4(err + p.tile0 + o, z);
      unsigned int nib = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        acc += (double)z[k] * (double)z[k];
        if (DEFER) nib |= ((z[k] >= 0.0f) ? 1u : 0u) << k;
      }
      if (DEFER) {
        const unsigned int word = gather_word<SUM_LDS>(nib);
        if ((threadIdx.x & 7) == 0) {
          const int64_t span0 = p.tile0 + u * SPAN;
          (packed_out + (span0 >> 5))[threadIdx.x >> 3] = word;
          if (own) (own + own_tile0 + u * (SPAN / 32))[threadIdx.x >> 3] = word;
        }
      }
    }
  }
  const double s = block_sum<BLOCK, SUM_LDS>(acc, lds);
  if (TICKET) {
    if (threadIdx.x < WAVE) chunk_ticket(tk, partials, p, tpc, n_c, s);
  } else if (threadIdx.x == 0) {
    partials[p.t] = s;
  }
}

// scale[c] = sqrt(sum of the chunk's tile partials / n_c), summed in a fixed order.
// own_scale (may be NULL): also receives the scale of chunk own_chunk.
__global__ __launch_bounds__(FBLOCK) void k_chunk_scale(const double* __restrict__ partials, int tpc,
                                                        int64_t n_c, float* __restrict__ scales,
                                                        float* __restrict__ own_scale, int own_chunk) {
  __shared__ double lds[FBLOCK / WAVE];
  const int c = blockIdx.x;
  double a = 0.0;
  for (int j = threadIdx.x; j < tpc; j += FBLOCK) a += partials[(int64_t)c * tpc + j];
  const double S = block_sum<FBLOCK>(a, lds);
  if (threadIdx.x == 0) {
    const float sc = (float)sqrt(S / (double)n_c);
    scales[c] = sc;
    if (own_scale && c == own_chunk) *own_scale = sc;
  }
}

// Dense view of a worker error held in deferred form: out[i] = err[i] - (bit_i ? s_c : -s_c) over the
// whole padded buffer (out may be err itself).
__global__ __launch_bounds__(BLOCK) void k_error_dense(const float* __restrict__ err, PackedErr pe,
                                                       float* __restrict__ out, int64_t n_c, int tpc) {
  const TilePos p = tile_pos<SPAN>(n_c, tpc, (int)blockIdx.x);
  const int o = threadIdx.x * 4;
  if (o >= p.len) return;
  const float se = pe.scales[p.c];
  const unsigned int nb = load_nibble(pe.bits, p.tile0);
  st4(out + p.tile0 + o, deferred_error(ld4(err + p.tile0 + o), nb, se));
}

// Sign, pack and error update of one 128-bit access held in registers (Algorithm 1 line 7/10).
// span0: flat index of the first element of the workgroup-wide access (uniform, multiple of 1024);
// the thread's elements are span0 + 4*threadIdx.x + k.
// own: if not NULL, the words are also written there at word index own_word0 + (thread's word) (the
// copy of this rank's own chunk in its server's input).
template <bool THROUGH_LDS = false>   // (gather_word)
__device__ __forceinline__ void sign_pack_store(v4f z, float s, float* __restrict__ err,
                                                uint32_t* __restrict__ packed, int64_t span0,
                                                uint32_t* __restrict__ own = nullptr, int64_t own_word0 = 0) {
  unsigned int nib = 0;
  v4f e;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const bool b = (z[k] >= 0.0f);
    nib |= (b ? 1u : 0u) << k;
    e[k] = z[k] - (b ? s : -s);
  }
  st4(err + span0 + threadIdx.x * 4, e);
  const unsigned int word = gather_word<THROUGH_LDS>(nib);
  if ((threadIdx.x & 7) == 0) {
    (packed + (span0 >> 5))[threadIdx.x >> 3] = word;
    if (own) (own + own_word0)[threadIdx.x >> 3] = word;
  }
}

// ---------------------------------------------------------------------------------------------
// K2 (two-pass path)  bits = (z >= 0), packed; err <- z - (+-scale)
// ---------------------------------------------------------------------------------------------
template <int U>
__global__ __launch_bounds__(BLOCK) void k_sign_pack_error(float* __restrict__ err,
                                                           uint32_t* __restrict__ packed,
                                                           const float* __restrict__ scales,
                                                           int64_t n_c, int tpc) {
  constexpr int TILE = SPAN * U;
  const TilePos p = tile_pos<TILE>(n_c, tpc, (int)blockIdx.x);
  const float s = scales[p.c];
  const int o0 = threadIdx.x * 4;
  v4f Z[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    if (o < p.len) Z[u] = ld4(err + p.tile0 + o);
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    // uniform over the wavefront (len is a multiple of 256), as the shuffles inside require
    if (o < p.len) sign_pack_store(Z[u], s, err, packed, p.tile0 + u * SPAN);
  }
}

// ---------------------------------------------------------------------------------------------
// Per-chunk arrival barrier of the single-pass kernels.
//
// Each workgroup of a chunk publishes one fp64 partial and arrives; the last one to arrive sums
// the chunk's partials in a fixed order, turns the sum into the scale and publishes it; the others
// wait for it.  Returns the chunk's scale to every thread.
//
// Progress: workgroups are dispatched in index order and a chunk's tiles are consecutive indices,
// so the oldest unfinished chunk always has all of its tiles resident or dispatchable provided the
// device can hold one chunk's workgroups at once; the host selects these kernels only when a
// chunk's workgroups take at most 80 % of the device's slots.
// Every wait is bounded by spin_limit polls: on expiry the workgroup raises
// *errflag, uses whatever it last read and goes on to exit, and all later waits end at once.
//
// Synchronisation uses relaxed agent-scope atomics whose payload travels in the atomic itself
// (partials: one double each; flag[c]: generation in the high word, scale bits in the low word),
// so no cache write-back/invalidate is needed; the store of the partial is complete (an explicit s_waitcnt)
// before the arrival counter is incremented.
//
// The barrier carries its own launch numbering, so a launch needs nothing from the host that
// changes from call to call (a captured launch can be replayed): counter[c] holds the generation
// in its high word and the arrivals of the running launch in its low word.  An arriving workgroup
// learns both from its fetch-add; the last one publishes the result under generation + 1 and then
// adds 2^32 - tpc to the counter (arrivals back to 0, generation + 1); the others wait for a flag
// of generation + 1.  All of it wraps harmlessly.
// ---------------------------------------------------------------------------------------------
struct ChunkSync {
  double* partials;             // [tiles of the launching kernel]
  unsigned long long* counter;  // [chunks * CTR_STRIDE] (generation << 32) | arrivals
  unsigned long long* sub;      // [chunks * groups(tiles of a chunk) * CTR_STRIDE] group counters
  unsigned long long* flag;     // [chunks] (generation << 32) | bits of the scale
  unsigned int* errflag;        // [1]
  int spin_limit;
};

// Between a workgroup's publication of its payload (write-through atomic stores) and its arrival:
// the stores have been acknowledged before the arrival is issued, so whoever sees the arrival
// finds the payload.  (A release fence of workgroup scope emits no wait here, and one of agent
// scope would also write back the L2's dirty lines, i.e. the kernel's own streaming stores.)
__device__ __forceinline__ void payload_before_arrival() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// One arrival at `counter` of a barrier with n participants: returns ((generation + 1) << 32) |
// (1 if this was the last arrival).
__device__ __forceinline__ unsigned long long barrier_arrive(unsigned long long* counter, int n) {
  const unsigned long long prev = __hip_atomic_fetch_add(counter, 1ull, __ATOMIC_RELAXED, OB_AGENT);
  const unsigned int want = (unsigned int)(prev >> 32) + 1u;
  const bool last = ((unsigned int)prev + 1u == (unsigned int)n);
  return ((unsigned long long)want << 32) | (last ? 1ull : 0ull);
}

// Whoever completes a counter re-arms it: the next generation, no arrivals.
__device__ __forceinline__ void barrier_rearm(unsigned long long* counter, int n) {
  (void)__hip_atomic_fetch_add(counter, (1ull << 32) - (unsigned long long)n, __ATOMIC_RELAXED, OB_AGENT);
}

// The same for arrival j of n, counted in two levels where there are more than one_level of them: atomics on one
// cache line are served one after the other, and the tiles of a layer arrive close together.  The last of each ARRIVE_SUB
// neighbours arrives at `top` for all of them (every payload of the group was in memory before its arrival).
// sub: the barrier's group counters, CTR_STRIDE words apart; they advance with `top`, one generation a launch.
// Measured, us, one level / two, a step and a LAMB step: one tensor of 384 tiles 44.2 / 41.9, 25.3 / 23.6; of 512 44.3 / 42.2,
// 28.6 / 25.8; of 957 67.1 / 64.4, 54.2 / 51.7; two of 512 64.1 / 61.1, 45.6 / 42.2; 954 among small ones 90.0 / 86.4; twelve of
// 957 565 / 559, 514 / 514.  Up to 256 the second round trip costs what the queue does: one of 256 35.2 / 35.1, four 67.6 / 66.5,
// twelve 149 / 149; and up to 512 in lists of many rounds of the device, whose tiles arrive spread out: 96 of 128 and 48 of 512
// 1728 / 1738 (arrivals_one_level in the host code).  Groups of 16 or 64: the same.
// In the chunk barriers (k_compress_resident, k_server_resident), a step of two tensors in plain form, elements among workers: 0.5 M among
// one 38.9 / 34.3, 1.5 M among one 56.1 / 41.0, 4 M among four 64.7 / 54.8, 8 M among eight 86.0 / 76.1, among one 102.4 / 99.2, 16 M and
// more the same.
__device__ __forceinline__ int top_arrivals(int n, int one_level) { return n > one_level ? (n + ARRIVE_SUB - 1) / ARRIVE_SUB : n; }
__device__ __forceinline__ unsigned long long barrier_arrive(unsigned long long* top, unsigned long long* sub, int j, int n,
                                                             int one_level = ARRIVE_ONE_LEVEL) {
  if (n > one_level) {
    const int g = j / ARRIVE_SUB, rest = n - g * ARRIVE_SUB;
    const int m = rest < ARRIVE_SUB ? rest : ARRIVE_SUB;
    unsigned long long* c = sub + (int64_t)g * CTR_STRIDE;
    const unsigned long long r = barrier_arrive(c, m);
    if ((r & 1ull) == 0ull) return r;
    barrier_rearm(c, m);
  }
  return barrier_arrive(top, top_arrivals(n, one_level));
}

// The publication by the last of n arrivals: flag <- (want << 32) | payload, then the counter is re-armed.
__device__ __forceinline__ unsigned long long barrier_publish(unsigned long long* flag,
                                                              unsigned long long* top, int n,
                                                              unsigned int want, unsigned int payload,
                                                              int one_level = ARRIVE_ONE_LEVEL) {
  const unsigned long long f = ((unsigned long long)want << 32) | (unsigned long long)payload;
  __hip_atomic_store(flag, f, __ATOMIC_RELAXED, OB_AGENT);
  barrier_rearm(top, top_arrivals(n, one_level));
  return f;
}

// Bounded wait (thread 0 of a workgroup) for a flag of generation `want`: at most spin_limit polls
// (0: none, the wait expires at once whatever the flag holds); returns the flag word last read (0
// if none was).  On expiry *errflag is raised; once it is raised every wait ends within 64 polls.
// The first 64 polls are SLEEP * 64 clocks apart, the others OB_POLL_SLEEP * 64: how long spin_limit
// polls take does not depend on the kernel.
template <int SLEEP = OB_POLL_SLEEP>
__device__ __forceinline__ unsigned long long barrier_wait(const unsigned long long* flag,
                                                           unsigned int want, unsigned int* errflag,
                                                           int spin_limit) {
  unsigned long long f = 0ull;
  for (int it = 0;; ++it) {
    if (it >= spin_limit) {
      atomicOr(errflag, 1u);
      break;
    }
    f = __hip_atomic_load(flag, __ATOMIC_RELAXED, OB_AGENT);
    if ((unsigned int)(f >> 32) == want) break;
    if ((it & 63) == 63 && __hip_atomic_load(errflag, __ATOMIC_RELAXED, OB_AGENT) != 0u) break;
    if (SLEEP != OB_POLL_SLEEP && it < 64) __builtin_amdgcn_s_sleep(SLEEP);
    else __builtin_amdgcn_s_sleep(OB_POLL_SLEEP);
  }
  return f;
}

template <bool THROUGH_LDS = false>   // (block_sum)
__device__ __forceinline__ float chunk_barrier_scale(const ChunkSync& cs, int tile, int c, int tpc,
                                                     int64_t n_c, double part, double* lds,
                                                     unsigned long long* bc,
                                                     float* __restrict__ scale_out) {
  unsigned long long* counter = &cs.counter[(int64_t)c * CTR_STRIDE];
  if (threadIdx.x == 0) {
    __hip_atomic_store(&cs.partials[tile], part, __ATOMIC_RELAXED, OB_AGENT);
    payload_before_arrival();
    const int groups = (tpc + ARRIVE_SUB - 1) / ARRIVE_SUB;
    *bc = barrier_arrive(counter, cs.sub + (int64_t)c * groups * CTR_STRIDE, tile - c * tpc, tpc);
  }
  __syncthreads();
  const bool last = ((*bc & 1ull) != 0ull);
  const unsigned int want = (unsigned int)(*bc >> 32);
  __syncthreads();
  if (last) {
    // four loads in flight per thread: every waiter of the chunk is waiting for this sum (the
    // partials are >= +0, so the zeros that stand in for missing ones change nothing)
    double a = 0.0;
    const double* part_c = cs.partials + (int64_t)c * tpc;
    for (int j = threadIdx.x; j < tpc; j += 4 * BLOCK) {
      double v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        v[q] = (j + q * BLOCK < tpc) ? __hip_atomic_load(&part_c[j + q * BLOCK], __ATOMIC_RELAXED, OB_AGENT) : 0.0;
#pragma unroll
      for (int q = 0; q < 4; ++q) a += v[q];
    }
    const double S = block_sum<BLOCK, THROUGH_LDS>(a, lds);
    if (threadIdx.x == 0) {
      const float sc = (float)sqrt(S / (double)n_c);
      scale_out[c] = sc;
      *bc = barrier_publish(&cs.flag[c], counter, tpc, want, __float_as_uint(sc));
    }
  } else if (threadIdx.x == 0) {
    *bc = barrier_wait(&cs.flag[c], want, cs.errflag, cs.spin_limit);
  }
  __syncthreads();
  return __uint_as_float((unsigned int)(*bc & 0xffffffffull));
}

// ---------------------------------------------------------------------------------------------
// K1+K2 in one pass: Algorithm 1 lines 6-7 with each input read once.  A workgroup computes z for
// its tile (U*4 registers per thread), goes through the chunk barrier, then signs, packs and writes
// the error from registers.  z never goes to memory.  Loads are issued G accesses at a time to
// bound the staging registers.
// ---------------------------------------------------------------------------------------------
template <int U, int G, bool HAS_K, bool PACKED_M, int MINW = 4, int GT = 0, bool KEEP = false>
__global__ __launch_bounds__(BLOCK, MINW) void k_compress_resident(
    GradSrc g, const float* __restrict__ m, PackedMom pm,
    float* __restrict__ err, uint32_t* __restrict__ packed, float* __restrict__ scales,
    ChunkSync cs, int64_t n_c, int tpc, float beta1, float omb1, LayerTab lt, OwnCopy oc) {
  constexpr int TILE = SPAN * U;
  __shared__ double lds[BLOCK / WAVE];
  __shared__ unsigned long long bc;
  const TilePos p = tile_pos<TILE>(n_c, tpc, (int)blockIdx.x);
  const int o0 = threadIdx.x * 4;
  ZTile<HAS_K, PACKED_M> zt;
  zt.init(lt, pm, p, beta1);
  v4f Z[U];
  double acc = 0.0;
  // (Issuing the next group's loads before evaluating the current one, or a branch-free path for
  // full tiles, measured no faster: the kernel is bound by the barrier, not by load latency.)
  auto stream = [&](auto known_uniform) {
#pragma unroll
    for (int u0 = 0; u0 < U; u0 += G) {
      v4f Gr[G], M[G], E[G];
      unsigned int NB[G];
#pragma unroll
      for (int j = 0; j < G; ++j) {
        const int o = (u0 + j) * SPAN + o0;
        M[j] = 0.0f; NB[j] = 0u;
        if (o < p.len) {
          Gr[j] = load_grad<GT>(g, p.tile0 + o);
          if (PACKED_M) NB[j] = load_nibble(pm.bits, p.tile0 + (u0 + j) * SPAN);
          else M[j] = ld4_keep_if<KEEP>(m + p.tile0 + o);
          E[j] = ld4(err + p.tile0 + o);
        }
      }
#pragma unroll
      for (int j = 0; j < G; ++j) {
        const int o = (u0 + j) * SPAN + o0;
        if (o < p.len) {
          const v4f z = zt.template z<decltype(known_uniform)::value>(lt, beta1, omb1, Gr[j], M[j], NB[j],
                                                                      E[j], p.tile0 + o);
          Z[u0 + j] = z;
#pragma unroll
          for (int k = 0; k < 4; ++k) acc += (double)z[k] * (double)z[k];
        }
      }
    }
  };
  // With k, a tile inside one layer runs a copy of the loop that holds nothing of the per-element
  // path: every tile of a chunk waits for the chunk's slowest one, and with the layer cursor of
  // that path in the same loop all tiles ran 9 % slower.
  if (HAS_K && zt.uniform) stream(std::true_type{});
  else stream(std::false_type{});
  const double part = block_sum<BLOCK, true>(acc, lds);
  const float s = chunk_barrier_scale<true>(cs, p.t, p.c, tpc, n_c, part, lds, &bc, scales);
  uint32_t* own = (oc.packed && p.c == oc.chunk) ? oc.packed : nullptr;   // uniform
  const int64_t own_tile0 = (p.tile0 - (int64_t)p.c * n_c) >> 5;           // the tile's first word within its chunk
  if (own && p.t == p.c * tpc && threadIdx.x == 0) *oc.scale = s;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    if (o < p.len) sign_pack_store<true>(Z[u], s, err, packed, p.tile0 + u * SPAN, own, own_tile0 + u * (SPAN / 32));
  }
}

// ---------------------------------------------------------------------------------------------
// K3  server: zb = (sum_w +-s_w, sequentially) * (1/W) + err_server   (Algorithm 1 line 10)
// Workers strictly in order 0..W-1 (the fp32 sum is order dependent).  The W additions per element
// are the whole cost (the inputs are one bit per element and worker), so the loop is written for
// the vector ALU: three instructions per element and worker -- shift the worker's word so that the
// element's bit is bit 0, add that bit, moved to bit 31, to the bit pattern of -s (the carry out of
// bit 31 is dropped: bit 1 gives +s, bit 0 leaves -s; one v_lshl_add_u32), add to the accumulator --
// with no compare/select through a lane mask.  The scales come from LDS (staged SRV_STAGE at a
// time), the sign words of the next G workers are requested before those of the current G are
// consumed, and nothing inside the loop branches on the tile's shape: a wavefront whose elements lie
// beyond the tile's end skips the loop.
// ---------------------------------------------------------------------------------------------
constexpr int SRV_STAGE = 1024;   // scales held in LDS at a time
// The sign words are fetched with buffer loads: the wavefront-uniform part of the address (worker
// block, span of the tile) travels in a scalar register, the thread's part in one 32-bit register,
// so no vector instruction is spent on addresses.  Every address is inside [packed_in, packed_in +
// W*n_c/32) by construction (the descriptor's range check does not see the scalar part, so it is
// not relied on).  Offsets are 32-bit: the host admits W*n_c/8 < 2^31 bytes.
constexpr int OB_BUFFER_RSRC_WORD3 = 0x00020000;   // raw 32-bit data format word of gfx9-family descriptors

template <int U>
__device__ __forceinline__ void server_average(const uint32_t* __restrict__ packed_in,
                                               const float* __restrict__ scales_in, int64_t n_c,
                                               int W, const TilePos& p, float (&acc)[U][4],
                                               unsigned int* lds_negs /* [SRV_STAGE] */) {
  constexpr int G = (U >= 8) ? 1 : 8 / U;   // workers whose sign words are in flight together
  const int o0 = threadIdx.x * 4;
  const bool active = (o0 < p.len);   // uniform over a wavefront: len is a multiple of 256
  const int wpc_bytes = (int)(n_c >> 3);   // bytes per worker block
  // descriptor of the tile's column of packed_in: from the tile's first word to the end of the array
  const int64_t col0 = p.tile0 >> 5;
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint32_t*>(packed_in + col0), 0, (int)(((int64_t)W * (n_c >> 5) - col0) * 4), OB_BUFFER_RSRC_WORD3);
  // byte offset of the thread's word of span 0 in a worker's block; span u lies 128 bytes further.
  // The spans a partial tile lacks (only the chunk's last tile has any; uniform over the workgroup)
  // read span 0 again and their sums are never used: the words that follow the tile would lie in
  // the next worker's block and, for the last worker, beyond the end of the array.
  const int voff0 = 4 * (int)(threadIdx.x >> 3);
  int uoff[U];
#pragma unroll
  for (int u = 0; u < U; ++u) uoff[u] = (u * SPAN < p.len) ? 128 * u : 0;
  unsigned int shk[4];                // position of the thread's k-th bit in its word
#pragma unroll
  for (int k = 0; k < 4; ++k) shk[k] = 4u * (threadIdx.x & 7) + (unsigned)k;
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int k = 0; k < 4; ++k) acc[u][k] = 0.0f;
  auto add_worker = [&](const unsigned int (&word)[U], unsigned int negs) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const unsigned int t = ((word[u] >> shk[k]) << 31) + negs;   // bit ? +s : -s
        acc[u][k] = acc[u][k] + __uint_as_float(t);
      }
  };
  auto load_worker = [&](unsigned int (&word)[U], int w) {
    const int soff = w * wpc_bytes;   // uniform
#pragma unroll
    for (int u = 0; u < U; ++u)
      word[u] = (unsigned int)__builtin_amdgcn_raw_buffer_load_b32(rsrc, voff0, soff + uoff[u], 0);
  };
  for (int wb = 0; wb < W; wb += SRV_STAGE) {
    const int nb = (W - wb < SRV_STAGE) ? W - wb : SRV_STAGE;
    __syncthreads();
    for (int i = threadIdx.x; i < nb; i += BLOCK) lds_negs[i] = __float_as_uint(scales_in[wb + i]) ^ 0x80000000u;
    __syncthreads();
    if (!active) continue;
    const int full = nb - nb % G;
    unsigned int cur[G][U], nxt[G][U];
    if (full > 0) {
#pragma unroll
      for (int j = 0; j < G; ++j) load_worker(cur[j], wb + j);
    }
    for (int j0 = 0; j0 < full; j0 += G) {
      if (j0 + G < full) {
#pragma unroll
        for (int j = 0; j < G; ++j) load_worker(nxt[j], wb + j0 + G + j);
      }
#pragma unroll
      for (int j = 0; j < G; ++j) add_worker(cur[j], lds_negs[j0 + j]);
#pragma unroll
      for (int j = 0; j < G; ++j)
#pragma unroll
        for (int u = 0; u < U; ++u) cur[j][u] = nxt[j][u];
    }
    for (int j = full; j < nb; ++j) {   // the last nb % G workers
      unsigned int word[U];
      load_worker(word, wb + j);
      add_worker(word, lds_negs[j]);
    }
  }
}

// two-pass form: zb written over err_server, tile partial of sum zb^2.
// DEFER: the server error in deferred form (as for the worker, see PackedErr; here one chunk, one
// scale): err_s holds zb of the previous call, the carried error is err_s - C[zb] with the server's
// own previous output `keep` (read and rewritten in place), and the sign words of the new zb are
// written here, to packed_out and to `keep`; no second pass over the chunk is needed.
template <int U, bool DEFER = false, bool TICKET = false>
__global__ __launch_bounds__(BLOCK) void k_server_unpack_avg(
    const uint32_t* __restrict__ packed_in, const float* __restrict__ scales_in,
    float* __restrict__ err_s, double* __restrict__ partials, int64_t n_c, int W, float invW,
    uint32_t* keep, const float* keep_scale, uint32_t* packed_out, ChunkTicket tk) {
  constexpr int TILE = SPAN * U;
  __shared__ double lds[BLOCK / WAVE];
  __shared__ unsigned int lds_negs[SRV_STAGE];
  const TilePos p = tile_pos<TILE>(n_c, (int)gridDim.x, (int)blockIdx.x);  // one chunk: c == 0
  const int o0 = threadIdx.x * 4;
  const float se = DEFER ? keep_scale[0] : 0.0f;
  float acc[U][4];
  server_average<U>(packed_in, scales_in, n_c, W, p, acc, lds_negs);
  double sq = 0.0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    if (o < p.len) {   // uniform over the wavefront, as the shuffles below require
      v4f e = ld4(err_s + p.tile0 + o);   // (requested before the sum over the workers: 28 instead of 22 us at 6.9M elements)
      if (DEFER) e = deferred_error(e, load_nibble(keep, p.tile0 + u * SPAN), se);
      v4f z;
      unsigned int nib = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        z[k] = acc[u][k] * invW + e[k];
        sq += (double)z[k] * (double)z[k];
        if (DEFER) nib |= ((z[k] >= 0.0f) ? 1u : 0u) << k;
      }
      st4(err_s + p.tile0 + o, z);
      if (DEFER) {
        const unsigned int word = gather_word(nib);
        if ((threadIdx.x & 7) == 0) {
          const int64_t w0 = (p.tile0 + u * SPAN) >> 5;
          (packed_out + w0)[threadIdx.x >> 3] = word;
          (keep + w0)[threadIdx.x >> 3] = word;
        }
      }
    }
  }
  const double s = block_sum(sq, lds);
  if (TICKET) {
    if (threadIdx.x < WAVE) chunk_ticket(tk, partials, p, (int)gridDim.x, n_c, s);
  } else if (threadIdx.x == 0) {
    partials[p.t] = s;
  }
}

// K3+K4 in one pass: Algorithm 1 line 10 on the served chunk with zb kept in registers across the
// chunk barrier above (one chunk: c = 0, its own counter, flag and partials), instead of three
// launches and a round trip of zb through err_server.  The host selects it only when all of its
// workgroups fit on the device at once.
// Workgroups per CU the kernel is built for: 8 (at most 64 registers) for the smaller tiles; the
// 4096-element tile needs a few more registers than that and takes 7 rather than spill in its loop.
template <int U>
__global__ __launch_bounds__(BLOCK, (U >= 4 ? 7 : 8)) void k_server_resident(
    const uint32_t* __restrict__ packed_in, const float* __restrict__ scales_in,
    float* __restrict__ err_s, uint32_t* __restrict__ packed_out, float* __restrict__ scale_out,
    ChunkSync cs, int64_t n_c, int W, float invW) {
  constexpr int TILE = SPAN * U;
  __shared__ double lds[BLOCK / WAVE];
  __shared__ unsigned long long bc;
  __shared__ unsigned int lds_negs[SRV_STAGE];
  const TilePos p = tile_pos<TILE>(n_c, (int)gridDim.x, (int)blockIdx.x);  // one chunk: c == 0
  const int o0 = threadIdx.x * 4;
  float acc[U][4];
  server_average<U>(packed_in, scales_in, n_c, W, p, acc, lds_negs);
  v4f Z[U];
  double sq = 0.0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    Z[u] = 0.0f;
    if (o < p.len) {
      const v4f e = ld4(err_s + p.tile0 + o);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        Z[u][k] = acc[u][k] * invW + e[k];
        sq += (double)Z[u][k] * (double)Z[u][k];
      }
    }
  }
  const double part = block_sum(sq, lds);
  const float s = chunk_barrier_scale(cs, p.t, 0, (int)gridDim.x, n_c, part, lds, &bc, scale_out);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    if (o < p.len) sign_pack_store(Z[u], s, err_s, packed_out, p.tile0 + u * SPAN);
  }
}

// ---------------------------------------------------------------------------------------------
// K5  per layer: global momentum, reconstructed gradient, fresh variance, max(v_frozen/v_fresh)
//     (Algorithm 1 lines 13, 15-17).  One maximum per (tile, layer) segment, no atomics.
// With the previous momentum in 1-bit form the reconstructed gradient takes only two magnitudes
// per tile, (s' - beta1 s)/(1-beta1) and (s' + beta1 s)/(1-beta1), whose squares are hoisted.
// The tile's registers and the two evaluation paths are shared with the fused ratio+update kernel.
// ---------------------------------------------------------------------------------------------
// bit ? a : b on the bit patterns, with the bit taken from position `pos` of `word` (two vector
// instructions: a signed one-bit field extract gives the all-ones / all-zeros mask)
__device__ __forceinline__ float select_by_bit(unsigned int word, int pos, float a, float b) {
  const unsigned int m = (unsigned int)__builtin_amdgcn_sbfe((int)word, (unsigned int)pos, 1u);
  float r;
  asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(r) : "v"(m), "v"(a), "v"(b));   // (in C the compiler makes three of it: and, compare, select)
  return r;
}

// The largest quotient n/d (each correctly rounded; NaN not taken) of a tile, of which only what exceeds `bound` matters: a
// wavefront's largest so far, or what the clips of lines 18-19 raise every smaller ratio to.  A division is a dozen instructions,
// one of them at quarter rate; whether n/d can exceed the bound is one fma, whose sign is that of n - bound*d: negative means
// n/d < bound for d > 0 (a rounded quotient is then at most the bound), and where it is not, or a d has its sign bit set, the
// quotients are formed.  Underflow of the fma gives a zero, which counts as not negative.  What may pass unformed besides: an infinite d, whose
// quotient is 0 or NaN; a NaN n or d, whose product fmaxf ignores and whose quotient is a NaN, not taken; with the bound at 0, n = anything over
// d = inf (the fma a NaN), the same 0 or NaN; with the bound at infinity everything, as nothing exceeds it.
// Measured with UpdateTerm and select_by_bit's two instructions, four steps, us, before / after: 11 M parameters 327 / 322, 336 M fp32 6785 /
// 6748, bf16 6946 / 6876 (the vector work of k_ratios_apply_hist, counted over four launches of a period 71 instructions an element, then 53, next
// to memory at 88 % of a copy's rate).
struct MaxQuotient {
  float bound;   // uniform over the wavefront
  float r;       // the lane's
  // lo: what line 18 raises a ratio to at least; r_min: line 19
  __device__ __forceinline__ void start(float lo, float r_min) {
    const float b = fmaxf(fmaxf(lo, r_min), 0.0f);
    bound = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(b)));
    r = 0.0f;
  }
  // all lanes of the wavefront; later: more follows
  __device__ __forceinline__ void add(const v4f& n, const v4f& d, bool later) {
    const float t = fmaxf(fmaxf(fmaf(-bound, d[0], n[0]), fmaf(-bound, d[1], n[1])),
                          fmaxf(fmaf(-bound, d[2], n[2]), fmaf(-bound, d[3], n[3])));
    const unsigned int sign = __float_as_uint(d[0]) | __float_as_uint(d[1]) | __float_as_uint(d[2]) | __float_as_uint(d[3]);
    if (__ballot(!(t < 0.0f) || (int)sign < 0) == 0ull) return;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float q = n[k] / d[k];
      if (q > r) r = q;
    }
    if (later) bound = fmaxf(bound, __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(wave_max(r)))));
  }
};

// n/(sqrt(v)+eta) as sqrtf and operator/ give it, without what those do for operands at the ends of the number range: the correctly
// rounded square root and quotient for v at most 2^60 and not negative, |n| zero or within [2^-80, 2^40], eta within [2^-22 = 2.4e-7, 2^20];
// values of v below 2^-96 count as that (their root is then less than half a unit of eta's last place, which is 2^-45 or more).  With a
// smaller eta every wavefront pays the check and takes the long form: a step, us, eta = 1e-6 / 1e-8, on the same buffers: 11 M parameters 77.0 / 78.9,
// 336 M 1702 / 1709, 1.3e9 6702 / 6800; a LAMB step of 3 M 22.5 / 23.2, of 336 M 1687 / 1690.
// The root: Newton's step on v_rsq_f32's estimate, equal to sqrtf for every one of the 1.3e9 values of [2^-96, 2^60] (compared one by one
// on the device; the tests have every mantissa of two binades and 1.7e7 values over all of them).  The quotient: two residuals after
// one step on v_rcp_f32's (Markstein), which is operator/'s own sequence between its scalings; no residual is subnormal in these ranges.
constexpr float SHORT_V_LOW = 0x1p-96f, SHORT_V_TOP = 0x1p60f, SHORT_N_LOW = 0x1p-80f, SHORT_N_TOP = 0x1p40f, SHORT_ETA_LOW = 0x1p-22f, SHORT_ETA_TOP = 0x1p20f;
constexpr unsigned int SHORT_V_TOP_BITS = __builtin_bit_cast(unsigned int, SHORT_V_TOP), SHORT_N_LOW_BITS = __builtin_bit_cast(unsigned int, SHORT_N_LOW);
__device__ __forceinline__ float short_denominator(float v, float eta) {   // sqrtf(v) + eta
  const float z = fmaxf(v, SHORT_V_LOW), y = __builtin_amdgcn_rsqf(z), g = z * y;
  return fmaf(fmaf(-g, g, z), 0.5f * y, g) + eta;
}
__device__ __forceinline__ float short_quotient(float n, float d) {   // n / d; a zero without its sign where n is -0
  const float r0 = __builtin_amdgcn_rcpf(d), r = fmaf(fmaf(-d, r0, 1.0f), r0, r0);
  const float q0 = n * r, q1 = fmaf(fmaf(-d, q0, n), r, q0);
  return fmaf(fmaf(-d, q1, n), r, q1);
}

// m_t/(sqrt(v_frozen)+eta) of line 21 with m_t = +-sp.
struct UpdateTerm {
  float sp, eta;
  unsigned int top;   // the lane's largest bit pattern of v_frozen
  __device__ __forceinline__ void start(float sp_, float eta_) { sp = sp_; eta = eta_; top = 0u; }
  __device__ __forceinline__ void see(const v4f& v) {
#pragma unroll
    for (int k = 0; k < 4; ++k) top = __float_as_uint(v[k]) > top ? __float_as_uint(v[k]) : top;
  }
  __device__ __forceinline__ bool in_range() const {   // uniform; all lanes of the wavefront
    const float a = fabsf(sp);
    const bool ok = (a == 0.0f || (a >= SHORT_N_LOW && a <= SHORT_N_TOP)) && eta >= SHORT_ETA_LOW && eta <= SHORT_ETA_TOP && top <= SHORT_V_TOP_BITS;
    return __ballot(!ok) == 0ull;
  }
  // v: four values of v_frozen, replaced by their terms; bits pos .. pos + 3 of word: the signs of m_t
  __device__ __forceinline__ void terms(v4f& v, unsigned int word, int pos, bool in_range) const {
    if (in_range) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float q = short_quotient(sp, short_denominator(v[k], eta));
        v[k] = __uint_as_float(__float_as_uint(q) ^ (~(word << (31 - pos - k)) & 0x80000000u));
      }
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float mt = ((word >> (pos + k)) & 1u) ? sp : -sp;
        v[k] = mt / (sqrtf(v[k]) + eta);
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float q = v[k];
      asm volatile("" : "+v"(q));   // evaluated here, not sunk below a wait that follows
      v[k] = q;
    }
  }
};

struct RatioArgs {
  const uint32_t* __restrict__ packed;   // [N_pad/32] the W recompressed chunks
  const float* __restrict__ sscales;     // [W] their scales
  const float* __restrict__ m;           // dense previous momentum (unless PACKED_M)
  PackedMom pm;                          // 1-bit previous momentum (PACKED_M)
  float* __restrict__ v_fresh;
  const float* __restrict__ v_frozen;
  float beta1, omb1, beta2, omb2;
  const float* __restrict__ r_prev;      // [L], and the bounds of lines 18-19 (k_ratios_big_hist, whose launch changes no ratio)
  float one_m_thr, r_min;
};

template <int U, bool HAS_K, bool PACKED_M>
struct RatioTile {
  unsigned int NB[U], OB[U];
  v4f M[U], VF[U], VZ[U];

  template <bool KEEP_V_FROZEN = false>
  __device__ __forceinline__ void load(const RatioArgs& ra, const TilePos& p) {
    const int o0 = threadIdx.x * 4;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int o = u * SPAN + o0;
      M[u] = 0.0f; OB[u] = 0u; NB[u] = 0u; VF[u] = 0.0f; VZ[u] = 0.0f;
      if (o < p.len) {
        NB[u] = load_nibble(ra.packed, p.tile0 + u * SPAN);
        if (PACKED_M) OB[u] = load_nibble(ra.pm.bits, p.tile0 + u * SPAN);
        else M[u] = ld4(ra.m + (p.tile0 + u * SPAN) + o0);
        VF[u] = ld4(ra.v_fresh + (p.tile0 + u * SPAN) + o0);
        VZ[u] = ld4_keep_if<KEEP_V_FROZEN>(ra.v_frozen + (p.tile0 + u * SPAN) + o0);
      }
    }
  }

  // Tile inside layer l0: updates v_fresh, returns the thread's max of v_frozen/v_fresh.
  // VZ keeps v_frozen.  DEFER: the new v_fresh stays in VF for store_v_fresh() instead of being
  // stored at once (a barrier arrival that follows then does not wait for these stores).
  // ss, s_prev: new and previous server scale of the chunk; kt: k of the layer (1 without HAS_K).
  // lo, r_min (DEFER): of MaxQuotient, which the others do without (one span, and bound by memory).
  template <bool DEFER = false>
  __device__ __forceinline__ float uniform_pass(const RatioArgs& ra, const TilePos& p, float ss,
                                                float s_prev, float kt, float lo = 0.0f, float r_min = 0.0f) {
    const int o0 = threadIdx.x * 4;
    const float sp = HAS_K ? ss / kt : ss;
    float t_same = 0.0f, t_diff = 0.0f;
    if (PACKED_M) {
      const float bm = ra.beta1 * (HAS_K ? s_prev / kt : s_prev);
      const float g_same = (sp - bm) / ra.omb1;     // new and old momentum of equal sign
      const float g_diff = (sp - (-bm)) / ra.omb1;  // of opposite sign
      t_same = ra.omb2 * (g_same * g_same);
      t_diff = ra.omb2 * (g_diff * g_diff);
    }
    float r = 0.0f;
    MaxQuotient mq;
    if (DEFER) mq.start(lo, r_min);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int o = u * SPAN + o0;
      if (o < p.len) {
        v4f vf;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          float t;
          if (PACKED_M) {
            t = select_by_bit(NB[u] ^ OB[u], k, t_diff, t_same);
          } else {
            const float mt = ((NB[u] >> k) & 1u) ? sp : -sp;
            const float gr = (mt - ra.beta1 * M[u][k]) / ra.omb1;
            t = ra.omb2 * (gr * gr);
          }
          vf[k] = ra.beta2 * VF[u][k] + t;
          if (!DEFER) {
            const float q = VZ[u][k] / vf[k];
            if (q > r) r = q;
          }
        }
        if (DEFER) {
          mq.add(VZ[u], vf, u + 1 < U);
          VF[u] = vf;
        } else {
          st4(ra.v_fresh + (p.tile0 + u * SPAN) + o0, vf);
        }
      }
    }
    return DEFER ? mq.r : r;
  }

  __device__ __forceinline__ void store_v_fresh(const RatioArgs& ra, const TilePos& p) const {
    const int o0 = threadIdx.x * 4;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int o = u * SPAN + o0;
      if (o < p.len) st4(ra.v_fresh + (p.tile0 + u * SPAN) + o0, VF[u]);
    }
  }

  // Tile that meets a layer boundary or the end of the parameters: element by element, leaving
  // the padding alone.  VZ is overwritten by the quotients (0 in the padding).
  __device__ __forceinline__ void element_pass(const RatioArgs& ra, const LayerTab& lt,
                                               const TilePos& p, int l0, float ss, float s_prev) {
    const int o0 = threadIdx.x * 4;
    const int64_t N = lt.off[lt.L];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int o = u * SPAN + o0;
      if (o < p.len) {
        int l = l0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int64_t i = p.tile0 + o + k;
          float q = 0.0f;
          if (i < N) {
            l = walk_layer(l, i, lt.off);
            const float kk = HAS_K ? lt.mom_scale[l] : 1.0f;
            const float sp = HAS_K ? ss / kk : ss;
            const float mt = ((NB[u] >> k) & 1u) ? sp : -sp;
            float bmk;
            if (PACKED_M) {
              const float b = ra.beta1 * (HAS_K ? s_prev / kk : s_prev);
              bmk = ((OB[u] >> k) & 1u) ? b : -b;
            } else {
              bmk = ra.beta1 * M[u][k];
            }
            const float gr = (mt - bmk) / ra.omb1;
            const float vf = ra.beta2 * VF[u][k] + ra.omb2 * (gr * gr);
            ra.v_fresh[i] = vf;
            q = VZ[u][k] / vf;
          }
          VZ[u][k] = q;
        }
      }
    }
  }

  // After element_pass: the thread's max of the quotients of elements in [a, b).
  __device__ __forceinline__ float segment_max(const TilePos& p, int64_t a, int64_t b) const {
    const int o0 = threadIdx.x * 4;
    float r = 0.0f;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int o = u * SPAN + o0;
      if (o < p.len) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int64_t i = p.tile0 + o + k;
          if (i >= a && i < b && VZ[u][k] > r) r = VZ[u][k];
        }
      }
    }
    return r;
  }
};

// The ratio pass of one tile (a workgroup; lds: [BLOCK / WAVE]).  SAME_LAUNCH: the maxima are read by other
// workgroups of the launch.  KEEP: v_frozen by ld4_keep.
template <int U, bool HAS_K, bool PACKED_M, bool KEEP, bool SAME_LAUNCH = false>
__device__ __forceinline__ void ratios_pass_tile(const RatioArgs& ra, float* __restrict__ seg_max,
                                                 int64_t n_c, int tpc, const LayerTab& lt,
                                                 const int* __restrict__ tile_seg0,
                                                 const int* __restrict__ seg_layer, int tile, float* lds) {
  constexpr int TILE = SPAN * U;
  const TilePos p = tile_pos<TILE>(n_c, tpc, tile);
  const int l0 = lt.first_layer[p.t];
  if (l0 >= lt.L) return;  // tile lies in the padding (it has no segment)
  // every scalar the tile needs is requested before the streaming loads, so that nothing is
  // looked up after they return (these workgroups are short: latency counts)
  const float ss = ra.sscales[p.c];
  const float s_prev = PACKED_M ? ra.pm.scales[p.c] : 0.0f;
  const float kt = HAS_K ? lt.mom_scale[l0] : 1.0f;
  const int64_t l0_end = lt.off[l0 + 1];
  const int s0 = tile_seg0[p.t];
  RatioTile<U, HAS_K, PACKED_M> rt;
  rt.template load<KEEP>(ra, p);
  auto store = [&](int s, float r) {
    if (SAME_LAUNCH) __hip_atomic_store(&seg_max[s], r, __ATOMIC_RELAXED, OB_AGENT);
    else seg_max[s] = r;
  };
  const bool uniform = (p.tile0 + p.len <= l0_end);
  if (uniform) {
    float r = rt.uniform_pass(ra, p, ss, s_prev, kt);
    r = block_max(r, lds);
    if (threadIdx.x == 0) store(s0, r);
  } else {
    rt.element_pass(ra, lt, p, l0, ss, s_prev);
    const int s1 = tile_seg0[p.t + 1];
    for (int s = s0; s < s1; ++s) {
      const int l = seg_layer[s];
      float r = rt.segment_max(p, lt.off[l], lt.off[l + 1]);
      r = block_max(r, lds);
      if (threadIdx.x == 0) store(s, r);
    }
  }
}

template <int U, bool HAS_K, bool PACKED_M, bool KEEP>
__global__ __launch_bounds__(BLOCK) void k_ratios_pass(RatioArgs ra, float* __restrict__ seg_max,
                                                       int64_t n_c, int tpc, LayerTab lt,
                                                       const int* __restrict__ tile_seg0,
                                                       const int* __restrict__ seg_layer,
                                                       const int* __restrict__ tile_list) {
  __shared__ float lds[BLOCK / WAVE];
  const int tile = tile_list ? tile_list[blockIdx.x] : tile_from_end(blockIdx.x, gridDim.x);   // (ld4_keep)
  ratios_pass_tile<U, HAS_K, PACKED_M, KEEP>(ra, seg_max, n_c, tpc, lt, tile_seg0, seg_layer, tile, lds);
}

// Algorithm 1 lines 18-19 for one layer given the raw ratio.  rp: r_prev[l].
__device__ __forceinline__ float ratio_clip(float r, float rp, float one_m_thr, float one_p_thr, float r_min, float r_max) {
  const float lo = one_m_thr * rp, hi = one_p_thr * rp;
  r = (r > lo) ? r : lo;
  r = (r < hi) ? r : hi;
  r = (r > r_min) ? r : r_min;
  r = (r < r_max) ? r : r_max;
  return r;
}
// ... lines 18-20 (thread 0 of a workgroup).
// rp, ca: r_prev[l] and c_avg[l], read by the caller (early, where their latency hides).
__device__ __forceinline__ float ratio_clip_commit(float r, int l, float rp, float ca,
                                                   float* __restrict__ r_prev,
                                                   float* __restrict__ coeff_c, float one_m_thr,
                                                   float one_p_thr, float r_min, float r_max) {
  r = ratio_clip(r, rp, one_m_thr, one_p_thr, r_min, r_max);
  r_prev[l] = r;
  const float c = r * ca;
  coeff_c[l] = c;
  return c;
}

// K6  per layer: max over the layer's segments (0 for an empty layer), then lines 18-20.
// One workgroup of NT threads per layer; lds: [NT / WAVE].
template <int NT>
__device__ __forceinline__ void ratios_finalize_layer(int l, const float* __restrict__ seg_max,
                                                      const int* __restrict__ layer_seg0,
                                                      const float* __restrict__ c_avg,
                                                      float* __restrict__ r_prev, float* __restrict__ coeff_c,
                                                      float one_m_thr, float one_p_thr, float r_min,
                                                      float r_max, float* lds) {
  const int s0 = layer_seg0[l], s1 = layer_seg0[l + 1];
  const float rp = r_prev[l], ca = c_avg[l];
  float r = 0.0f;
  // four loads in flight per thread: a tensor too large for the kernel with the per-layer barrier
  // has tens of thousands of segments, and this one workgroup walks them alone (the maxima are
  // >= +0 or NaN, so the zeros that stand in for missing ones change nothing)
  for (int s = s0 + threadIdx.x; s < s1; s += 4 * NT) {
    float q[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) q[u] = (s + u * NT < s1) ? seg_max[s + u * NT] : 0.0f;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (q[u] > r) r = q[u];
  }
  r = block_max<NT>(r, lds);
  if (threadIdx.x == 0)
    (void)ratio_clip_commit(r, l, rp, ca, r_prev, coeff_c, one_m_thr, one_p_thr, r_min, r_max);
}

__global__ __launch_bounds__(FBLOCK) void k_ratios_finalize(const float* __restrict__ seg_max,
                                                            const int* __restrict__ layer_seg0,
                                                            const float* __restrict__ c_avg,
                                                            float* __restrict__ r_prev,
                                                            float* __restrict__ coeff_c,
                                                            float one_m_thr, float one_p_thr,
                                                            float r_min, float r_max,
                                                            const unsigned char* __restrict__ done_elsewhere) {
  __shared__ float lds[FBLOCK / WAVE];
  const int l = blockIdx.x;
  if (done_elsewhere && done_elsewhere[l]) return;  // the kernel with the per-layer barrier finishes it
  ratios_finalize_layer<FBLOCK>(l, seg_max, layer_seg0, c_avg, r_prev, coeff_c, one_m_thr, one_p_thr, r_min, r_max,
                                lds);
}

// ---------------------------------------------------------------------------------------------
// K7  x <- x - (lr*c_l) * m_t/(sqrt(v_frozen)+eta);  m <- m_t (when WRITE_M)
//     (Algorithm 1 lines 13, 21)
// ---------------------------------------------------------------------------------------------
struct ApplyArgs {
  const uint32_t* __restrict__ packed;
  const float* __restrict__ sscales;
  const float* __restrict__ v_frozen;
  float* __restrict__ x;
  float* __restrict__ m;              // written when WRITE_M
  const float* __restrict__ coeff_c;
  float lr, eta;
  void* __restrict__ x_lp;            // 16-bit copy of the updated x (LPX)
  int x_lp_bf16;
};

// Tile inside layer l0 with coefficient c: update from registers.
template <int U, bool HAS_K, bool WRITE_M, bool LPX = false>
__device__ __forceinline__ void apply_uniform(const ApplyArgs& aa, const TilePos& p, float ss,
                                              float kt, float c, const unsigned int (&NB)[U],
                                              const v4f (&VZ)[U], const v4f (&X)[U]) {
  const int o0 = threadIdx.x * 4;
  const float sp = HAS_K ? ss / kt : ss;
  const float a = aa.lr * c;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    if (o < p.len) {
      v4f xn, mn;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float mt = ((NB[u] >> k) & 1u) ? sp : -sp;
        const float uu = mt / (sqrtf(VZ[u][k]) + aa.eta);
        xn[k] = X[u][k] - a * uu;
        mn[k] = mt;
      }
      st4(aa.x + p.tile0 + o, xn);
      if (LPX) st4_lp(aa.x_lp, p.tile0 + u * SPAN, o0, xn, aa.x_lp_bf16);
      if (WRITE_M) st4(aa.m + p.tile0 + o, mn);
    }
  }
}

// Tile that meets a layer boundary: element by element, coefficients read from coeff_c.
template <int U, bool HAS_K, bool WRITE_M, bool LPX = false>
__device__ __forceinline__ void apply_elements(const ApplyArgs& aa, const LayerTab& lt,
                                               const TilePos& p, int l0, float ss,
                                               const unsigned int (&NB)[U], const v4f (&VZ)[U],
                                               const v4f (&X)[U]) {
  const int o0 = threadIdx.x * 4;
  const int64_t N = lt.off[lt.L];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    if (o < p.len) {
      int l = l0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int64_t i = p.tile0 + o + k;
        if (i < N) {
          l = walk_layer(l, i, lt.off);
          const float sp = HAS_K ? ss / lt.mom_scale[l] : ss;
          const float a = aa.lr * aa.coeff_c[l];
          const float mt = ((NB[u] >> k) & 1u) ? sp : -sp;
          const float uu = mt / (sqrtf(VZ[u][k]) + aa.eta);
          const float xn = X[u][k] - a * uu;
          aa.x[i] = xn;
          if (LPX) reinterpret_cast<unsigned short*>(aa.x_lp)[i] = float_to_lp(xn, aa.x_lp_bf16);
          if (WRITE_M) aa.m[i] = mt;
        }
      }
    }
  }
}

template <int U, bool HAS_K, bool WRITE_M, bool LPX = false>
__global__ __launch_bounds__(BLOCK) void k_decompress_apply(ApplyArgs aa, int64_t n_c, int tpc,
                                                            LayerTab lt,
                                                            const int* __restrict__ tile_list) {
  constexpr int TILE = SPAN * U;
  const TilePos p = tile_pos<TILE>(n_c, tpc, listed_tile(tile_list));
  const int l0 = lt.first_layer[p.t];
  if (l0 >= lt.L) return;
  // scalars first (see k_ratios_pass), then the streaming loads
  const float ss = aa.sscales[p.c];
  const float kt = HAS_K ? lt.mom_scale[l0] : 1.0f;
  const float c0 = aa.coeff_c[l0];
  const int64_t l0_end = lt.off[l0 + 1];
  const int o0 = threadIdx.x * 4;
  unsigned int NB[U];
  v4f X[U], VZ[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    NB[u] = 0u; X[u] = 0.0f; VZ[u] = 0.0f;
    if (o < p.len) {
      NB[u] = load_nibble(aa.packed, p.tile0 + u * SPAN);
      VZ[u] = ld4(aa.v_frozen + p.tile0 + o);
      X[u] = ld4(aa.x + p.tile0 + o);
    }
  }
  const bool uniform = (p.tile0 + p.len <= l0_end);
  if (uniform) apply_uniform<U, HAS_K, WRITE_M, LPX>(aa, p, ss, kt, c0, NB, VZ, X);
  else apply_elements<U, HAS_K, WRITE_M, LPX>(aa, lt, p, l0, ss, NB, VZ, X);
}

// ---------------------------------------------------------------------------------------------
// K5+K6+K7 in one pass: Algorithm 1 lines 13-21 with v_frozen and the sign words read once.
// A workgroup runs the ratio pass on its tile of U 1024-element spans, keeps v_frozen and the signs
// in registers, arrives at its layer's barrier, and while the layer completes writes v_fresh,
// fetches x and forms m_t/(sqrt(v_frozen)+eta) in place of v_frozen; once the layer's coefficient
// c_t is published only a multiply and a subtract per element are left before x is stored.
//
// The kernel covers "listed" tiles: the tiles that lie inside ONE layer, for every layer whose such
// tiles all fit on the device at once (80 % of its workgroup slots).  Everything else -- layers
// that are too large, the spans where layers meet, small tensors -- goes through the plain kernels
// on 1024-element tiles: the ratio pass before this kernel (the maxima of those segments wait in
// seg_max) and the update after it.
//
// Per-layer barrier: like the per-chunk one above (same self-numbering counter and flag words),
// but the payload of a tile is its fp32 maximum of v_frozen/v_fresh (order-independent); the last
// of the layer's listed tiles to arrive reduces ALL of the layer's maxima, applies the two clips
// (lines 18-19), commits r_prev and coeff_c and publishes c_t in flag[l].  The dispatch-order
// argument of the chunk barrier applies per layer; all waits are bounded (errflag).
// ---------------------------------------------------------------------------------------------
// What the last arriver of a layer needs to find the layer's partial results: the listed tiles
// publish into an array of their own, indexed like the launch (tile_list position = blockIdx), and
// the plain kernels' segments of the layer lie before the first and after the last listed tile
// (the listed tiles of a layer are contiguous in position): [layer_seg0[l], seg_first[l]) and
// [seg_end[l], layer_seg0[l+1]) of the 1024-element tiling's segment array.
struct ListedTiles {
  const int* tile_list;         // listed tiles, by position (the launch's blockIdx -> tile)
  const int* list_begin;        // [L] index in tile_list of the layer's first listed tile
  const int* n_listed;          // [L] listed tiles of the layer
  const int* seg_first;         // [L] first segment owned by the layer's listed tiles
  const int* seg_end;           // [L] one past the last segment owned by them
  const int* layer_seg0;        // [L+1] segments of each layer
  int64_t n_c;
  int tpc, tpc_span;            // tiles of this kernel / spans per chunk
  int one_level;                // arrivals of a layer that are counted in one level (barrier_arrive)
};

// The ranges of one layer, read by every workgroup at its start (uniform, next to its other
// scalars) so that the one that turns out to arrive last has them at hand.
struct LayerParts {
  int nl, lb;                 // listed tiles: tile_list[lb .. lb+nl)
  int a, s_first, s_end, b;   // plain segments: [a, s_first) and [s_end, b)
};
__device__ __forceinline__ LayerParts layer_parts(const ListedTiles& lt, int l) {
  LayerParts q;
  q.nl = lt.n_listed[l]; q.lb = lt.list_begin[l];
  q.a = lt.layer_seg0[l]; q.s_first = lt.seg_first[l]; q.s_end = lt.seg_end[l]; q.b = lt.layer_seg0[l + 1];
  return q;
}

// The last arriver's walk over a layer's partial results, strided over the workgroup's threads:
// comb(load(i)) for every listed tile of the layer (i = its position in tile_list), four loads in
// flight per thread (every waiter of the layer is waiting for this; `zero` stands in for missing
// ones and must leave comb's result unchanged), then plain(j) for every plain-kernel segment j.
template <class T, class FL, class FC, class FP>
__device__ __forceinline__ void for_layer_parts(const LayerParts& q, T zero, FL load, FC comb, FP plain) {
  for (int j = threadIdx.x; j < q.nl; j += 4 * BLOCK) {
    T v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = (j + u * BLOCK < q.nl) ? load(q.lb + j + u * BLOCK) : zero;
#pragma unroll
    for (int u = 0; u < 4; ++u) comb(v[u]);
  }
  for (int j = q.a + threadIdx.x; j < q.s_first; j += BLOCK) plain(j);
  for (int j = q.s_end + threadIdx.x; j < q.b; j += BLOCK) plain(j);
}

struct LayerSync {
  float* seg_max;               // [segments of the 1024-element tiling] maxima left by the plain ratio pass
  float* listed_max;            // [listed tiles] maxima of this launch's tiles
  ListedTiles lt;
  unsigned long long* counter;  // [L * CTR_STRIDE] (generation << 32) | arrivals
  unsigned long long* sub;      // group counters (group_line)
  unsigned long long* flag;     // [L] (generation << 32) | bits of c_t
  unsigned int* errflag;
  int spin_limit;
  const float* c_avg;
  float* r_prev;
  float* coeff_c;
  float one_m_thr, one_p_thr, r_min, r_max;
  int n_lead;                   // leading workgroups of the launch: without REST one per layer, that
                                // finish the layers without listed tiles (0: a kernel of its own has done that)
  const unsigned char* done;    // [L] 1 for those of them that an earlier launch has finished (NULL: none)
  // k_ratios_apply_hist with the plain ratio pass in its launch (REST): the leading workgroups
  // finish the n_alone layers that have no arrivals and run the pass of the rest_tiles, whose segments arrive too
  const int* rest_tiles;
  const int* alone;
  int n_alone;
  const int* arr0;              // [L] arrivals of the layers before
  const int* skip_first;        // [L] first / one past the last of the layer's segments that no rest tile forms
  const int* skip_end;
  const int* tile_seg0;
  const int* seg_layer;
  // ... and the update of the rest tiles in its last workgroups (n_events = 0: a launch of its own)
  int n_tiles;                  // workgroups before them
  unsigned int n_events;        // after which every c_t is there (coefficient_events)
  unsigned int* events;
  unsigned long long* launches; // 2^32 * launches whose c_t were all there
  unsigned int* tail_launches;  // [rest tiles] launches that the tile's update has been through
};

// One of those events (thread 0; its c_t have been stored at agent scope): the last one of the launch lets the updates go.
__device__ __forceinline__ void coefficient_event(const LayerSync& ls) {
  payload_before_arrival();
  if (__hip_atomic_fetch_add(ls.events, 1u, __ATOMIC_RELAXED, OB_AGENT) + 1u != ls.n_events) return;
  __hip_atomic_store(ls.events, 0u, __ATOMIC_RELAXED, OB_AGENT);
  const unsigned long long n = __hip_atomic_load(ls.launches, __ATOMIC_RELAXED, OB_AGENT);   // (nobody else writes it)
  __hip_atomic_store(ls.launches, n + (1ull << 32), __ATOMIC_RELAXED, OB_AGENT);
}
__device__ __forceinline__ void store_coeff(float* coeff_c, int l, float c) {
  __hip_atomic_store(&coeff_c[l], c, __ATOMIC_RELAXED, OB_AGENT);
}

// All of layer l's maxima, the two clips (lines 18-19), and the publication of c_t (a layer that is one segment of a rest
// tile has no barrier): by the whole workgroup that arrived last of n.
template <bool REST = false>
__device__ __forceinline__ void layer_finish(const LayerSync& ls, int l, const LayerParts& lp, float rp, float ca, int n,
                                             unsigned int want, float* lds) {
  float q = 0.0f;
  // four loads in flight per thread: every waiter of the layer is waiting for this, and a layer that is too large to be
  // listed has tens of thousands of segments (the maxima are >= +0, so that missing ones as 0 change nothing)
  auto range = [&](const float* v, int j0, int j1) {
    for (int j = j0 + (int)threadIdx.x; j < j1; j += 4 * BLOCK) {
      float t[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        t[u] = (j + u * BLOCK < j1) ? __hip_atomic_load(&v[j + u * BLOCK], __ATOMIC_RELAXED, OB_AGENT) : 0.0f;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (t[u] > q) q = t[u];
    }
  };
  range(ls.listed_max, lp.lb, lp.lb + lp.nl);
  range(ls.seg_max, lp.a, lp.s_first);
  range(ls.seg_max, lp.s_end, lp.b);
  q = block_max(q, lds);
  if (threadIdx.x == 0) {
    const float c = ratio_clip_commit(q, l, rp, ca, ls.r_prev, ls.coeff_c, ls.one_m_thr,
                                      ls.one_p_thr, ls.r_min, ls.r_max);
    if (n > 1 || lp.nl > 0)
      (void)barrier_publish(&ls.flag[l], &ls.counter[(int64_t)l * CTR_STRIDE], n, want, __float_as_uint(c), ls.lt.one_level);
    if (REST && ls.n_events) {
      store_coeff(ls.coeff_c, l, c);
      coefficient_event(ls);
    }
  }
}

// Publishes the maximum r of the workgroup's listed tile (of layer l; bid: its position in
// tile_list) and arrives; if this was the layer's last arrival, finishes the layer.  All threads call; r is valid
// in thread 0.  lp, rp, ca: the layer's ranges, r_prev[l] and c_avg[l], read at the start of the kernel; first, n: the
// layer's first arrival in the numbering of all, and how many it has.
template <bool REST = false>
__device__ __forceinline__ void layer_arrive(const LayerSync& ls, int bid, int l, const LayerParts& lp, int first, int n,
                                             float rp, float ca, float r, float* lds, unsigned long long* bc) {
  if (threadIdx.x == 0) {
    __hip_atomic_store(&ls.listed_max[bid], r, __ATOMIC_RELAXED, OB_AGENT);
    payload_before_arrival();
    *bc = barrier_arrive(&ls.counter[(int64_t)l * CTR_STRIDE], ls.sub + group_line(first, l), bid - lp.lb, n, ls.lt.one_level);
  }
  __syncthreads();
  const bool last = ((*bc & 1ull) != 0ull);
  const unsigned int want = (unsigned int)(*bc >> 32);
  __syncthreads();
  if (last) layer_finish<REST>(ls, l, lp, rp, ca, n, want, lds);
  // every thread leaves with the generation to wait for in *bc's high word (the last arriver too)
}

// A rest tile's half of the barriers (whole workgroup, after its ratio pass with SAME_LAUNCH): its first and last
// segments arrive at their layers, those in between, layers of their own, are finished here.
__device__ __forceinline__ void rest_arrive(const LayerSync& ls, int tile, float* lds, unsigned long long* bc /* [2] */) {
  const int s0 = ls.tile_seg0[tile], s1 = ls.tile_seg0[tile + 1], n_end = (s1 - s0 > 1) ? 2 : 1;
  auto arrivals = [&](const LayerParts& lp, int l, int* a, int* e) {
    *a = ls.skip_first[l];
    *e = ls.skip_end[l];
    return layer_arrivals(lp.nl, lp.a, *a, *e, lp.b);
  };
  if (threadIdx.x == 0) payload_before_arrival();   // (thread 0 has stored the maxima)
  __syncthreads();
  const int e = threadIdx.x / WAVE;
  if (e < n_end && (threadIdx.x & (WAVE - 1)) == 0) {
    const int sg = e ? s1 - 1 : s0, l = ls.seg_layer[sg];
    const LayerParts lp = layer_parts(ls.lt, l);
    int a, b;
    const int n = arrivals(lp, l, &a, &b);
    const int j = rest_arrival(sg, lp.nl, lp.a, a, b);
    bc[e] = (n == 1) ? 1ull : barrier_arrive(&ls.counter[(int64_t)l * CTR_STRIDE], ls.sub + group_line(ls.arr0[l], l), j, n, ls.lt.one_level);
  }
  __syncthreads();
  for (int sg = s0 + 1 + (int)threadIdx.x; sg < s1 - 1; sg += BLOCK) {
    const int l = ls.seg_layer[sg];
    const float r = __hip_atomic_load(&ls.seg_max[sg], __ATOMIC_RELAXED, OB_AGENT);
    const float c = ratio_clip_commit(r, l, ls.r_prev[l], ls.c_avg[l], ls.r_prev, ls.coeff_c, ls.one_m_thr, ls.one_p_thr, ls.r_min,
                                      ls.r_max);
    store_coeff(ls.coeff_c, l, c);
  }
  if (ls.n_events && s1 - s0 > 2) {   // uniform
    payload_before_arrival();
    __syncthreads();
    if (threadIdx.x == 0) coefficient_event(ls);
  }
  for (int q = 0; q < n_end; ++q) {   // uniform
    if ((bc[q] & 1ull) == 0ull) continue;
    const int l = ls.seg_layer[q ? s1 - 1 : s0];
    const LayerParts lp = layer_parts(ls.lt, l);
    int a, b;
    const int n = arrivals(lp, l, &a, &b);
    layer_finish<true>(ls, l, lp, ls.r_prev[l], ls.c_avg[l], n, (unsigned int)(bc[q] >> 32), lds);
  }
}

// The update of rest tile number i (whole workgroup), in the launch that forms its layers' c_t: everything is loaded and, in a tile inside one layer,
// m_t/(sqrt(v_frozen)+eta) formed before the wait.  The tile's own count of launches says which one this is.
template <bool HAS_K, bool LPX>
__device__ __forceinline__ void rest_update(const ApplyArgs& aa, const LayerSync& ls, const LayerTab& lt, int i) {
  const TilePos p = tile_pos<SPAN>(ls.lt.n_c, ls.lt.tpc_span, ls.rest_tiles[i]);
  const int l0 = lt.first_layer[p.t];
  const unsigned int want = ls.tail_launches[i] + 1u;
  const float ss = aa.sscales[p.c];
  const float kt = HAS_K ? lt.mom_scale[l0] : 1.0f;
  const bool uniform = (p.tile0 + p.len <= lt.off[l0 + 1]);
  const int o = threadIdx.x * 4;
  unsigned int nib = 0u;
  v4f X, VZ;
  X = 0.0f; VZ = 0.0f;
  if (o < p.len) {
    nib = load_nibble(aa.packed, p.tile0);
    VZ = ld4(aa.v_frozen + p.tile0 + o);
    X = ld4(aa.x + p.tile0 + o);
  }
  if (uniform) {
    UpdateTerm ut;
    ut.start(HAS_K ? ss / kt : ss, aa.eta);
    ut.see(VZ);
    ut.terms(VZ, nib, 0, ut.in_range());
  }
  if (threadIdx.x == 0) {
    (void)barrier_wait(ls.launches, want, ls.errflag, ls.spin_limit);
    ls.tail_launches[i] = want;
  }
  __syncthreads();
  if (o >= p.len) return;
  auto coeff = [&](int l) { return __hip_atomic_load(&ls.coeff_c[l], __ATOMIC_RELAXED, OB_AGENT); };   // past this XCD's caches
  if (uniform) {
    const float a = aa.lr * coeff(l0);
    v4f xn;
#pragma unroll
    for (int k = 0; k < 4; ++k) xn[k] = X[k] - a * VZ[k];
    st4(aa.x + p.tile0 + o, xn);
    if (LPX) st4_lp(aa.x_lp, p.tile0, o, xn, aa.x_lp_bf16);
    return;
  }
  const int64_t N = lt.off[lt.L];
  int l = l0, cur = -1;
  float sp = 0.0f, a = 0.0f;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int64_t j = p.tile0 + o + k;
    if (j < N) {
      l = walk_layer(l, j, lt.off);
      if (l != cur) {
        cur = l;
        sp = HAS_K ? ss / lt.mom_scale[l] : ss;
        a = aa.lr * coeff(l);
      }
      const float mt = ((nib >> k) & 1u) ? sp : -sp;
      const float xn = X[k] - a * (mt / (sqrtf(VZ[k]) + aa.eta));
      aa.x[j] = xn;
      if (LPX) reinterpret_cast<unsigned short*>(aa.x_lp)[j] = float_to_lp(xn, aa.x_lp_bf16);
    }
  }
}

// Waits (bounded) until layer l's coefficient of this launch is published; returns it to all
// threads.  *bc still holds what layer_arrive left there.
__device__ __forceinline__ float layer_wait(const LayerSync& ls, int l, unsigned long long* bc) {
  __syncthreads();
  if (threadIdx.x == 0) *bc = barrier_wait(&ls.flag[l], (unsigned int)(*bc >> 32), ls.errflag, ls.spin_limit);
  __syncthreads();
  return __uint_as_float((unsigned int)(*bc & 0xffffffffull));
}

// A leading workgroup of a barrier kernel's launch (blockIdx.x < ls.n_lead, one per layer): lines 18-20 for
// layer blockIdx.x if it has no listed tile -- its segment maxima were left by earlier kernels and nothing
// in this launch reads what is written here -- in the shadow of this launch instead of in a launch of its own.
__device__ __forceinline__ void lead_finalize(const LayerSync& ls, float* lds) {
  const int l = (int)blockIdx.x;
  if (ls.lt.n_listed[l] == 0 && !(ls.done && ls.done[l]))
    ratios_finalize_layer<BLOCK>(l, ls.seg_max, ls.lt.layer_seg0, ls.c_avg, ls.r_prev, ls.coeff_c, ls.one_m_thr,
                                 ls.one_p_thr, ls.r_min, ls.r_max, lds);
}

// Instantiated for the momentum in 1-bit form only: with a dense momentum the extra array the
// tile must hold costs more (spills or occupancy) than the second read of v_frozen saves, so the
// host then takes the two-kernel path.  5 workgroups per CU (<= 96 VGPRs at U = 8) measured best:
// 4 leaves too few workgroup slots next to the ones waiting at a barrier, 6 and more spill.
#ifndef OB_LB_MINW
#define OB_LB_MINW 5
#endif
template <int U, bool HAS_K, bool LPX = false>
__global__ __launch_bounds__(BLOCK, OB_LB_MINW) void k_ratios_apply_resident(
    RatioArgs ra, ApplyArgs aa, LayerSync ls, LayerTab lt) {
  // lt.first_layer: of the 1024-element tiling
  constexpr int TILE = SPAN * U;
  __shared__ float lds[BLOCK / WAVE];
  __shared__ unsigned long long bc;
  const int bid = (int)blockIdx.x - ls.n_lead;   // position in tile_list
  if (bid < 0) {
    lead_finalize(ls, lds);
    return;
  }
  const int64_t n_c = ls.lt.n_c;
  const int tpc = ls.lt.tpc;
  const TilePos p = tile_pos<TILE>(n_c, tpc, ls.lt.tile_list[bid]);
  const int sp0 = p.c * ls.lt.tpc_span + (p.t - p.c * tpc) * U;  // the tile's first span
  const int l0 = lt.first_layer[sp0];  // the layer the tile lies in
  const float ss = ra.sscales[p.c];
  const float s_prev = ra.pm.scales[p.c];
  const float kt = HAS_K ? lt.mom_scale[l0] : 1.0f;
  const LayerParts lp = layer_parts(ls.lt, l0);
  const float rp = ls.r_prev[l0], ca = ls.c_avg[l0];
  const int o0 = threadIdx.x * 4;
  RatioTile<U, HAS_K, true> rt;
  rt.load(ra, p);
  float r = rt.template uniform_pass<true>(ra, p, ss, s_prev, kt, ls.one_m_thr * rp, ls.r_min);
  r = block_max(r, lds);
  layer_arrive(ls, bid, l0, lp, lp.lb, lp.nl, rp, ca, r, lds, &bc);   // before the stores of v_fresh: nothing to wait for
  rt.store_v_fresh(ra, p);
  v4f X[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {  // x is fetched while the layer completes
    const int o = u * SPAN + o0;
    X[u] = 0.0f;
    if (o < p.len) X[u] = ld4(aa.x + (p.tile0 + u * SPAN) + o0);
  }
  // m_t/(sqrt(v_frozen)+eta) does not depend on the layer's coefficient: it is formed now, in place
  // of v_frozen, so that the square root and the division run while the layer completes instead
  // of after it (the same operations on the same operands as apply_uniform's)
  UpdateTerm ut;
  ut.start(HAS_K ? ss / kt : ss, aa.eta);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    if (o < p.len) ut.see(rt.VZ[u]);
  }
  const bool in_range = ut.in_range();   // uniform
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    if (o < p.len) ut.terms(rt.VZ[u], rt.NB[u], 0, in_range);
  }
  const float c = layer_wait(ls, l0, &bc);
  const float a = aa.lr * c;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    if (o < p.len) {
      v4f xn;
#pragma unroll
      for (int k = 0; k < 4; ++k) xn[k] = X[u][k] - a * rt.VZ[u][k];
      st4(aa.x + (p.tile0 + u * SPAN) + o0, xn);
      if (LPX) st4_lp(aa.x_lp, p.tile0 + u * SPAN, o0, xn, aa.x_lp_bf16);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// The fresh variance in deferred form (Algorithm 1 line 16 evaluated every step, stored every few).
//
// With the momentum in 1-bit form the reconstructed gradient of line 15 takes two magnitudes per
// (chunk, layer) and step, chosen per element by whether the momentum's sign bit flipped.  So the
// variance after a more steps follows from the variance array as last written ("base") and the
// sign words and scales of the a+1 momenta since then, by the very operations line 16 would have
// performed step by step (v <- beta2*v + t, t one of the two values of that step): the ratio of
// line 17 needs the up-to-date variance of every element in registers, but the array need not be
// rewritten each time.  A step then reads the base (4 bytes per element, as before) plus one bit
// per element and older step, and writes nothing; every few steps the caller asks for the array to
// be brought up to date (write_v) and the history starts anew.
//
// Planes, newest first: 0 = the new momentum (RatioArgs.packed / sscales), 1 = the previous one
// (RatioArgs.pm), 2 + i = VfHist.bits[i] / scales[i] for i < n_old (so bits[0] is the momentum
// before the previous one).  The base is the variance as of plane n_old + 1.
// ---------------------------------------------------------------------------------------------
constexpr int VF_MAX_OLD = 7;
struct VfHist {
  int n_old;                            // 0..VF_MAX_OLD
  int write_v;                          // store the up-to-date variance
  const uint32_t* bits[VF_MAX_OLD];     // [N_pad/32] each
  const float* scales[VF_MAX_OLD];      // [W] each
};

// The two values omb2*g^2 of one step (the operations of RatioTile::uniform_pass, in its order).
// s_new, s_old: the chunk's scale of the step's momentum and of the one before.
template <bool HAS_K>
__device__ __forceinline__ void variance_terms(const RatioArgs& ra, float s_new, float s_old, float kt,
                                               float* t_same, float* t_diff) {
  const float sp = HAS_K ? s_new / kt : s_new;
  const float bm = ra.beta1 * (HAS_K ? s_old / kt : s_old);
  const float g_same = (sp - bm) / ra.omb1;     // new and old momentum of equal sign
  const float g_diff = (sp - (-bm)) / ra.omb1;  // of opposite sign
  *t_same = ra.omb2 * (g_same * g_same);
  *t_diff = ra.omb2 * (g_diff * g_diff);
}

// scale of plane q (newest first) for chunk c; q is a compile-time constant where it is called
__device__ __forceinline__ float plane_scale(const RatioArgs& ra, const VfHist& h, int q, int c) {
  return q == 0 ? ra.sscales[c] : (q == 1 ? ra.pm.scales[c] : h.scales[q - 2][c]);
}
__device__ __forceinline__ const uint32_t* plane_bits(const RatioArgs& ra, const VfHist& h, int q) {
  return q == 0 ? ra.packed : (q == 1 ? ra.pm.bits : h.bits[q - 2]);
}

// The two values of every step are the same for all elements of a (chunk, layer) pair.  In long lists they are formed
// once per call for every pair and step, by leading workgroups of the plain ratio pass's launch, and fetched from there.
// Pairs: the layers that meet chunk c, in layer order, are pairs pair_base[c] .. pair_base[c+1]-1;
// the pair of (c, l) is pair_base[c] + l - pair_lfirst[c].
struct VTerms {
  const float* __restrict__ t;   // [VF_MAX_OLD + 1 steps][n_pairs][2]: t_same, t_diff; step s (1 = newest) at s - 1
  const int* pair_base;       // [W + 1]
  const int* pair_lfirst;     // [W]
  const int* pair_c;          // [n_pairs]
  const int* pair_l;          // [n_pairs]
  int n_pairs;
};
__device__ __forceinline__ int pair_of(const VTerms& vt, int c, int l) { return vt.pair_base[c] + l - vt.pair_lfirst[c]; }

template <bool HAS_K>
__device__ __forceinline__ void variance_terms_of_pair(const RatioArgs& ra, const VfHist& h, const VTerms& vt,
                                                       const float* __restrict__ mom_scale,
                                                       float* __restrict__ out /* = vt.t */, int pr) {
  if (pr >= vt.n_pairs) return;
  const int c = vt.pair_c[pr], l = vt.pair_l[pr];
  const float kt = HAS_K ? mom_scale[l] : 1.0f;
  const int a = h.n_old + 1;
#pragma unroll
  for (int s = 1; s <= VF_MAX_OLD + 1; ++s) {
    if (s <= a) {
      float t_same, t_diff;
      variance_terms<HAS_K>(ra, plane_scale(ra, h, s - 1, c), plane_scale(ra, h, s, c), kt, &t_same, &t_diff);
      float* o = out + ((int64_t)(s - 1) * vt.n_pairs + pr) * 2;
      o[0] = t_same;
      o[1] = t_diff;
    }
  }
}

// The two values of every step for a tile, from where the walk reads them.  StepTable: the table of the launch before.  StepTerms: formed
// by the wavefront's lanes, those of step s in lane s - 1 of each group of 8, once for all steps, while its loads are in flight,
// which makes that launch unnecessary; over 37000 tiles it costs more (6910 / 6970 us for four steps).
// k_ratios_apply_hist is a kernel each: with both in one it spilled 20 to 49 scalar registers and vector ones beside a 16-bit copy (four steps, us,
// both / one each: 40 tensors of 1 M 922 / 910, 110 M and a bf16 copy 2445 / 2417, 336 M and larger within 0.1 %).
// (A stride of 64 bits here makes k_ratios_apply_hist spill 13 to 27 vector registers at OB_LB_MINW workgroups per CU.)
struct StepTable {
  const float* tt;
  int n_pairs;
  __device__ __forceinline__ void find(const VTerms& vt, int c, int l) {
    tt = vt.t + (int64_t)pair_of(vt, c, l) * 2;
    n_pairs = vt.n_pairs;
  }
  __device__ __forceinline__ float t_same(int s) const { return tt[(int64_t)(s - 1) * n_pairs * 2]; }
  __device__ __forceinline__ float t_diff(int s) const { return tt[(int64_t)(s - 1) * n_pairs * 2 + 1]; }
};
struct StepTerms {
  float same, diff;
  template <bool HAS_K>
  __device__ __forceinline__ void form(const RatioArgs& ra, const VfHist& h, int c, float kt) {
    const int s = (int)(threadIdx.x & 7) + 1;
    float s_new = 0.0f, s_old = 0.0f;
#pragma unroll
    for (int q = 0; q < VF_MAX_OLD + 2; ++q)
      if (q <= h.n_old + 1) {   // uniform
        const float v = plane_scale(ra, h, q, c);
        if (q == s - 1) s_new = v;
        if (q == s) s_old = v;
      }
    variance_terms<HAS_K>(ra, s_new, s_old, kt, &same, &diff);
  }
  // From the table, or formed where the launch before has not (vt.t = NULL): k_ratios_big_hist, which keeps its registers with both.
  // StepTable's loads from within the
  // walk cost it 0.4 us of 10 (316 tiles; in long lists up to 1 %); with only the table's half of this it spills 24 registers (4 to 9 % of a step).
  template <bool HAS_K>
  __device__ __forceinline__ void get(const VTerms& vt, const RatioArgs& ra, const VfHist& h, int c, int l, float kt) {
    if (vt.t) {   // uniform
      const int s = (int)(threadIdx.x & 7) < h.n_old + 1 ? (int)(threadIdx.x & 7) : h.n_old;
      const float2 t = reinterpret_cast<const float2*>(vt.t)[(int64_t)s * vt.n_pairs + pair_of(vt, c, l)];
      same = t.x;
      diff = t.y;
    } else {
      form<HAS_K>(ra, h, c, kt);
    }
  }
  // of step s, uniform
  __device__ __forceinline__ float t_same(int s) const { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(same), s - 1)); }
  __device__ __forceinline__ float t_diff(int s) const { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(diff), s - 1)); }
};

// The terms and the plain ratio pass (momentum in 1-bit form, tile list) in one launch: the first n_lead
// workgroups form the terms and clear flags, the others run the plain ratio pass of tile_list[blockIdx.x - n_lead].
// Neither reads what the other writes; both are over before the kernels that use the terms start.
template <int U, bool HAS_K>
__global__ __launch_bounds__(BLOCK) void k_ratios_pass_vterms(RatioArgs ra, float* __restrict__ seg_max,
                                                              int64_t n_c, int tpc, LayerTab lt,
                                                              const int* __restrict__ tile_seg0,
                                                              const int* __restrict__ seg_layer,
                                                              const int* __restrict__ tile_list, VfHist h,
                                                              VTerms vt, float* __restrict__ vt_out, int n_lead,
                                                              unsigned long long* __restrict__ clear_flag, int n_flags) {
  __shared__ float lds[BLOCK / WAVE];
  const int bid = (int)blockIdx.x - n_lead;
  if (bid < 0) {
    const int f = (int)(blockIdx.x * BLOCK + threadIdx.x);
    if (f < n_flags) clear_flag[f] = 0ull;   // (k_ratios_trail's, of the call before)
    variance_terms_of_pair<HAS_K>(ra, h, vt, lt.mom_scale, vt_out, (int)(blockIdx.x * BLOCK + threadIdx.x));
    return;
  }
  ratios_pass_tile<U, HAS_K, true, true>(ra, seg_max, n_c, tpc, lt, tile_seg0, seg_layer, tile_list[bid], lds);
}

// Dense view of a variance held in deferred form, over the 1024-element tiles inside the tiles of
// the two kernels below (each lies inside one layer): the up-to-date variance goes to the base
// array itself if h.write_v, else to vf_dense (another array, which leaves the base as it is).
template <bool HAS_K>
__global__ __launch_bounds__(BLOCK) void k_variance_dense(RatioArgs ra, VfHist h, float* __restrict__ vf_dense, int64_t n_c, int tpc,
                                                          LayerTab lt, const int* __restrict__ tile_list) {
  const TilePos p = tile_pos<SPAN>(n_c, tpc, tile_list[blockIdx.x]);
  const int l0 = lt.first_layer[p.t];
  if (l0 >= lt.L || p.tile0 + p.len > lt.off[l0 + 1]) return;   // (not a tile of those kernels: nothing lags there)
  const int a = h.n_old + 1;   // steps to apply
  StepTerms st;
  st.form<HAS_K>(ra, h, p.c, HAS_K ? lt.mom_scale[l0] : 1.0f);
  const int o = threadIdx.x * 4;
  if (o >= p.len) return;   // all lanes of a wavefront or none
  float* vf_out = h.write_v ? ra.v_fresh : vf_dense;   // uniform
  unsigned int NBq[VF_MAX_OLD + 2];   // the lane's nibble of every plane, newest first
#pragma unroll
  for (int q = 0; q < VF_MAX_OLD + 2; ++q) {
    NBq[q] = 0u;
    if (q <= a) NBq[q] = load_nibble(plane_bits(ra, h, q), p.tile0);
  }
  v4f V = ld4(ra.v_fresh + p.tile0 + o);
#pragma unroll
  for (int s = VF_MAX_OLD + 1; s >= 1; --s) {
    if (s <= a) {   // uniform: the step from plane s to plane s-1
      const float t_same = st.t_same(s), t_diff = st.t_diff(s);
      const unsigned int flip = NBq[s] ^ NBq[s - 1];
#pragma unroll
      for (int k = 0; k < 4; ++k) V[k] = ra.beta2 * V[k] + select_by_bit(flip, k, t_diff, t_same);
    }
  }
  st4(vf_out + p.tile0 + o, V);
}

// The ratio pass with the variance in deferred form on 8192-element tiles that lie inside one layer,
// for the layers that are too large for the kernel with the per-layer barrier (their update still
// runs as the plain kernel).  On such tiles the pass moves bytes at the streaming rate, so reading
// the stale array and the momenta's sign words instead of rewriting the array pays; on 1024-element
// tiles it does not.  Same loads, exchange and
// walk through the steps as k_ratios_apply_hist.  The tile's maximum goes to the segment of its
// first 1024-element span, 0 to the segments of its other spans (k_ratios_finalize takes the
// maximum over all of a layer's segments).
// The lane's word of a plane: span lane/8, word lane%8 of the wavefront's 8 words (256 elements) of that span, as an index
// into the plane; and the lane's own nibbles of the 8 spans, packed into one register, from the words that the lanes hold.
__device__ __forceinline__ int64_t lane_word(const TilePos& p, bool* have) {
  const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
  const int e0 = (lane >> 3) * SPAN + wv * (WAVE * 4) + (lane & 7) * 32;
  *have = (e0 < p.len);   // len is a multiple of 256: a wavefront's part of a span is all there or all missing
  return (p.tile0 + e0) >> 5;
}
__device__ __forceinline__ unsigned int lane_nibbles(unsigned int word) {
  const int lane = threadIdx.x & (WAVE - 1), src = lane >> 3;   // src + 8*u: the lane that holds this lane's word of span u
  const unsigned int sh = 4u * (lane & 7);
  unsigned int packed = 0u;
#pragma unroll
  for (int u = 0; u < 8; ++u) packed |= ((__shfl(word, 8 * u + src, WAVE) >> sh) & 15u) << (4 * u);
  return packed;
}

template <bool HAS_K>
__global__ __launch_bounds__(BLOCK, OB_LB_MINW) void k_ratios_big_hist(RatioArgs ra, VfHist h, VTerms vt, float* __restrict__ seg_max,
                                                           const int* __restrict__ big_tiles, int64_t n_c,
                                                           int tpc_big, int tpc_span, LayerTab lt,
                                                           const int* __restrict__ tile_seg0) {
  constexpr int U = 8;
  __shared__ float lds[BLOCK / WAVE];
  const TilePos p = tile_pos<SPAN * U>(n_c, tpc_big, big_tiles[blockIdx.x]);
  const int sp0 = p.c * tpc_span + (p.t - p.c * tpc_big) * U;  // the tile's first span
  const int l0 = lt.first_layer[sp0];  // the layer the tile lies in (lt.first_layer: of the 1024-element tiling)
  const float rp = ra.r_prev[l0];
  const int a = h.n_old + 1;   // steps to apply
  const int o0 = threadIdx.x * 4;
  bool have_word;
  const int64_t wi = lane_word(p, &have_word);
  unsigned int Wq[VF_MAX_OLD + 2];
#pragma unroll
  for (int q = 0; q < VF_MAX_OLD + 2; ++q) {
    Wq[q] = 0u;
    if (q <= a && have_word) Wq[q] = plane_bits(ra, h, q)[wi];
  }
  v4f V[U], VZ[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    V[u] = 0.0f; VZ[u] = 0.0f;
    if (o < p.len) {
      V[u] = ld4(ra.v_fresh + p.tile0 + o);
      VZ[u] = ld4(ra.v_frozen + p.tile0 + o);
    }
  }
  StepTerms st;
  st.get<HAS_K>(vt, ra, h, p.c, l0, HAS_K ? lt.mom_scale[l0] : 1.0f);
#pragma unroll
  for (int s = VF_MAX_OLD + 1; s >= 1; --s)
    if (s <= a) Wq[s] ^= Wq[s - 1];
#pragma unroll
  for (int q = 1; q < VF_MAX_OLD + 2; ++q)   // (plane 0 itself is not needed here: only the flips)
    if (q <= a) Wq[q] = lane_nibbles(Wq[q]);   // uniform
#pragma unroll
  for (int s = VF_MAX_OLD + 1; s >= 1; --s) {
    if (s <= a) {   // uniform: the step from plane s to plane s-1
      const float t_same = st.t_same(s), t_diff = st.t_diff(s);
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < 4; ++k) V[u][k] = ra.beta2 * V[u][k] + select_by_bit(Wq[s], 4 * u + k, t_diff, t_same);
    }
  }
  MaxQuotient mq;
  mq.start(ra.one_m_thr * rp, ra.r_min);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    if (o < p.len) {
      mq.add(VZ[u], V[u], u + 1 < U);
      if (h.write_v) st4(ra.v_fresh + p.tile0 + o, V[u]);
    }
  }
  const float r = block_max(mq.r, lds);
  const int nspan = (p.len + SPAN - 1) / SPAN;
  if (threadIdx.x < nspan) seg_max[tile_seg0[sp0 + threadIdx.x]] = (threadIdx.x == 0) ? r : 0.0f;
}

// The same pass, and the update of the same layers, as two kinds of workgroups of one launch: a layer's update follows its
// ratio pass closely enough to find v_frozen in the 256 MB memory-side cache, and the two take turns, so that the device
// reads and writes alike at any time.
// `items` lists the workgroups in the order of dispatch: the tiles in position order for the ratio pass, and from
// some way after a layer's last tile on parts of its tiles for the update (ratios_trail_items in the host code, which says
// when this is taken and what it gives).  The last ratio workgroup of a layer
// to finish takes the maximum over all of the layer (arrivals counted in two levels, as in chunk_ticket), finishes lines 18-20
// and publishes c_t in flag[l], which an earlier launch of the call has cleared.  An update workgroup requests v_frozen, x and
// the signs, none of which a ratio workgroup writes, forms m_t/(sqrt(v_frozen)+eta) and then waits for that flag, which by then
// is normally there.  Ratio workgroups wait for nothing and an update workgroup only for ones dispatched before it: progress needs
// in-order dispatch, not co-residency; the wait is bounded (errflag).
// Bound by HBM and the memory-side cache together: 21.6 bytes per element are asked for (four-step average), 4.1 of them a second time.  1.21e9 elements
// in layers of 12.6, 16.8 and 103 M: 3.64 ms a step, 7.2 TB/s of what is asked for, 5.8 without the second reads; 4.04 in two kernels; with v_frozen not kept 4.4.
// (The ratio pass stands in both kernels: as a function of its own it makes each of them spill 306 vector registers.)
struct RatioTrailTab {
  const unsigned int* items;    // flags above | tile's position in lt.tile_list
  ListedTiles lt;               // the tiles of these layers (positions as for the barrier kernel)
  const int* count0;            // [L] the layer's first counter: second level, then the first-level ones
  unsigned int* count;          // lines of CTR_STRIDE 8-byte words
  float* sub_max;               // [counters] of the first-level groups
  float* tile_max;              // [tiles]
  unsigned long long* flag;     // [L] 2^32 | bits of c_t once known
  const float* seg_max;         // maxima left by the plain ratio pass
  unsigned int* errflag;
  int spin_limit;
  const float* c_avg;
  float* r_prev;
  float* coeff_c;
  float one_m_thr, one_p_thr, r_min, r_max;
};
// First wavefront of a ratio workgroup; pos: the tile's position, r: its maximum (lane 0).  rp, ca: r_prev[l] and c_avg[l].
__device__ __forceinline__ void ratios_trail_finish(const RatioTrailTab& tt, int pos, int l, const LayerParts& lp, int64_t c0,
                                                    float rp, float ca, float r) {
  constexpr int LINE = 2 * CTR_STRIDE;
  const int lane = threadIdx.x & (WAVE - 1);
  auto arrive = [&](unsigned int* counter, unsigned int n, float* payload, float v) {
    int last = 0;
    if (lane == 0) {
      __hip_atomic_store(payload, v, __ATOMIC_RELAXED, OB_AGENT);
      payload_before_arrival();
      last = (__hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, OB_AGENT) + 1u == n);
      if (last) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, OB_AGENT);
    }
    return __builtin_amdgcn_readfirstlane(last) != 0;
  };
  const int sub = (pos - lp.lb) / TICKET_SUB, first = sub * TICKET_SUB;
  const int n = (lp.nl - first < TICKET_SUB) ? lp.nl - first : TICKET_SUB;
  const int n_sub = (lp.nl + TICKET_SUB - 1) / TICKET_SUB;
  const int64_t cs = c0 + 1 + sub;
  if (!arrive(tt.count + cs * LINE, (unsigned int)n, &tt.tile_max[pos], r)) return;
  float q = 0.0f;
  if (lane < n) q = __hip_atomic_load(&tt.tile_max[lp.lb + first + lane], __ATOMIC_RELAXED, OB_AGENT);
  q = wave_max(q);
  if (!arrive(tt.count + c0 * LINE, (unsigned int)n_sub, &tt.sub_max[cs], q)) return;
  q = 0.0f;
  const float* sub_max = tt.sub_max + c0 + 1;
  for (int s = lane; s < n_sub; s += 4 * WAVE) {   // four in flight (the maxima are >= +0: missing ones as 0 change nothing)
    float v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      v[j] = (s + j * WAVE < n_sub) ? __hip_atomic_load(&sub_max[s + j * WAVE], __ATOMIC_RELAXED, OB_AGENT) : 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (v[j] > q) q = v[j];
  }
  for (int s = lp.a + lane; s < lp.s_first; s += WAVE)    // written by an earlier kernel
    if (tt.seg_max[s] > q) q = tt.seg_max[s];
  for (int s = lp.s_end + lane; s < lp.b; s += WAVE)
    if (tt.seg_max[s] > q) q = tt.seg_max[s];
  q = wave_max(q);
  if (lane == 0) {
    const float c = ratio_clip_commit(q, l, rp, ca, tt.r_prev, tt.coeff_c, tt.one_m_thr, tt.one_p_thr, tt.r_min, tt.r_max);
    __hip_atomic_store(&tt.flag[l], (1ull << 32) | (unsigned long long)__float_as_uint(c), __ATOMIC_RELAXED, OB_AGENT);
  }
}

template <bool HAS_K, bool LPX>
__global__ __launch_bounds__(BLOCK, OB_LB_MINW) void k_ratios_trail(RatioArgs ra, VfHist h, VTerms vt, ApplyArgs aa,
                                                                    RatioTrailTab tt, LayerTab lt) {
  constexpr int U = 8;
  __shared__ float lds[BLOCK / WAVE];
  __shared__ float c_of_layer;
  const unsigned int item = tt.items[blockIdx.x];
  const int pos = (int)(item & (RATIOS_TRAIL_PART - 1u)), part = (int)((item & ~TRAIL_UPDATE) / RATIOS_TRAIL_PART);
  const TilePos p = tile_pos<SPAN * U>(tt.lt.n_c, tt.lt.tpc, tt.lt.tile_list[pos]);
  const int sp0 = p.c * tt.lt.tpc_span + (p.t - p.c * tt.lt.tpc) * U;  // the tile's first span
  const int l0 = lt.first_layer[sp0];  // the layer the tile lies in (lt.first_layer: of the 1024-element tiling)
  if (item & TRAIL_UPDATE) {
    constexpr int U = RATIOS_TRAIL_U;
    TilePos q = p;
    const int in_tile = part * (U * SPAN);
    q.tile0 += in_tile;
    q.len -= in_tile;            // (a short tile may lack its last parts: <= 0)
    if (q.len <= 0) return;
    const float ss = aa.sscales[q.c];
    const float kt = HAS_K ? lt.mom_scale[l0] : 1.0f;
    const int o0 = threadIdx.x * 4;
    unsigned int NB[U];
    v4f VZ[U], X[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int o = u * SPAN + o0;
      NB[u] = 0u; VZ[u] = 0.0f; X[u] = 0.0f;
      if (o < q.len) {
        NB[u] = load_nibble(aa.packed, q.tile0 + u * SPAN);
        VZ[u] = ld4(aa.v_frozen + (q.tile0 + u * SPAN) + o0);
        X[u] = ld4(aa.x + (q.tile0 + u * SPAN) + o0);
      }
    }
    UpdateTerm ut;
    ut.start(HAS_K ? ss / kt : ss, aa.eta);
#pragma unroll
    for (int u = 0; u < U; ++u) ut.see(VZ[u]);   // (zeros where there is nothing)
    const bool in_range = ut.in_range();   // uniform
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int o = u * SPAN + o0;
      if (o < q.len) ut.terms(VZ[u], NB[u], 0, in_range);
    }
    if (threadIdx.x == 0)
      c_of_layer = __uint_as_float((unsigned int)(barrier_wait(&tt.flag[l0], 1u, tt.errflag, tt.spin_limit) & 0xffffffffull));
    __syncthreads();
    const float al = aa.lr * c_of_layer;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int o = u * SPAN + o0;
      if (o < q.len) {
        v4f xn;
#pragma unroll
        for (int k = 0; k < 4; ++k) xn[k] = X[u][k] - al * VZ[u][k];
        st4(aa.x + (q.tile0 + u * SPAN) + o0, xn);
        if (LPX) st4_lp(aa.x_lp, q.tile0 + u * SPAN, o0, xn, aa.x_lp_bf16);
      }
    }
    return;
  }
  const LayerParts lp = layer_parts(tt.lt, l0);
  const int64_t c0 = tt.count0[l0];
  const float rp = tt.r_prev[l0], ca = tt.c_avg[l0];
  const int a = h.n_old + 1;   // steps to apply
  const int o0 = threadIdx.x * 4;
  bool have_word;
  const int64_t wi = lane_word(p, &have_word);
  unsigned int Wq[VF_MAX_OLD + 2];
#pragma unroll
  for (int q = 0; q < VF_MAX_OLD + 2; ++q) {
    Wq[q] = 0u;
    if (q <= a && have_word) Wq[q] = plane_bits(ra, h, q)[wi];
  }
  v4f V[U], VZ[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    V[u] = 0.0f; VZ[u] = 0.0f;
    if (o < p.len) {
      V[u] = ld4(ra.v_fresh + (p.tile0 + u * SPAN) + o0);
      VZ[u] = ld4_keep(ra.v_frozen + (p.tile0 + u * SPAN) + o0);
    }
  }
  StepTerms st;
  st.get<HAS_K>(vt, ra, h, p.c, l0, HAS_K ? lt.mom_scale[l0] : 1.0f);
#pragma unroll
  for (int s = VF_MAX_OLD + 1; s >= 1; --s)
    if (s <= a) Wq[s] ^= Wq[s - 1];
#pragma unroll
  for (int q = 1; q < VF_MAX_OLD + 2; ++q)   // (plane 0 itself is not needed here: only the flips)
    if (q <= a) Wq[q] = lane_nibbles(Wq[q]);   // uniform
#pragma unroll
  for (int s = VF_MAX_OLD + 1; s >= 1; --s) {
    if (s <= a) {   // uniform: the step from plane s to plane s-1
      const float t_same = st.t_same(s), t_diff = st.t_diff(s);
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < 4; ++k) V[u][k] = ra.beta2 * V[u][k] + select_by_bit(Wq[s], 4 * u + k, t_diff, t_same);
    }
  }
  MaxQuotient mq;
  mq.start(ra.one_m_thr * rp, ra.r_min);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    if (o < p.len) {
      mq.add(VZ[u], V[u], u + 1 < U);
      if (h.write_v) st4(ra.v_fresh + (p.tile0 + u * SPAN) + o0, V[u]);
    }
  }
  const float r = block_max(mq.r, lds);
  if (threadIdx.x < WAVE) ratios_trail_finish(tt, pos, l0, lp, c0, rp, ca, r);
}

// k_ratios_apply_resident with the variance in deferred form.  A wavefront's part of a tile is 64
// words of every plane (8 spans x 8 words): each lane fetches ONE word of each plane and the lanes
// then pass each other the words they need; what a lane keeps of a plane is its 8 nibbles packed
// into one register.
//
// S > 0: v_frozen of S spans goes straight into LDS, and m/(sqrt(v_frozen)+eta) later in its place, 24 KB for
// 6 spans: 72 to 79 registers instead of 96, so that 6 workgroups fit on a CU instead of 5.  Which form a
// list takes: lh_in_lds in the host code.
//
// Here and in k_ratios_big_hist spans are addressed as tile0 + (span and lane): a scalar base and a 32-bit offset for every access.  As (tile0 + span) + lane,
// which k_ratios_trail has (880 M elements in four layers 3412 / 3487 us the other way), they become 64-bit vector addresses, an addition with carry
// or two before each load, which a list of few rounds waits for.  This kernel, us, so / as in k_ratios_trail: 4.3 M elements 21.8 / 22.8, 8.2 M 33.3 / 34.6, 11 M 40.5 /
// 42.1, 42 M 93.1 / 95.2, 110 M 247.3 / 247.6, 336 M 887 / 883; the call on 61 drawn lists of 3 to 60 M
// 1.9 % shorter on average (0.938 to 1.026 of the time; above 1 four that rewrite the variance at every step), above 60 M the same.
constexpr int LH_WG_LDS = 6;   // workgroups per CU with S > 0
template <bool HAS_K, bool LPX, int S, bool REST>
__global__ __launch_bounds__(BLOCK, S > 0 ? LH_WG_LDS : OB_LB_MINW) void k_ratios_apply_hist(
    RatioArgs ra, VfHist h, VTerms vt, ApplyArgs aa, LayerSync ls, LayerTab lt) {
  constexpr int U = 8;
  constexpr int TILE = SPAN * U;
  __shared__ float lds[BLOCK / WAVE];
  __shared__ unsigned long long bc;
  __shared__ v4f zs[S > 0 ? S * BLOCK : 1];
  const int bid = (int)blockIdx.x - ls.n_lead;   // position in tile_list
  if (bid < 0) {
    if constexpr (REST) {
      __shared__ unsigned long long bc_rest[2];
      const int lead = (int)blockIdx.x - ls.n_alone;
      if (lead < 0) {   // (uniform)
        const int l = ls.alone[blockIdx.x];
        ratios_finalize_layer<BLOCK>(l, ls.seg_max, ls.lt.layer_seg0, ls.c_avg, ls.r_prev, ls.coeff_c,
                                     ls.one_m_thr, ls.one_p_thr, ls.r_min, ls.r_max, lds);
        if (ls.n_events && threadIdx.x == 0) {
          store_coeff(ls.coeff_c, l, ls.coeff_c[l]);   // (this thread's own)
          coefficient_event(ls);
        }
      } else {
        const int tile = ls.rest_tiles[lead];
        ratios_pass_tile<1, HAS_K, true, true, true>(ra, ls.seg_max, ls.lt.n_c, ls.lt.tpc_span, lt, ls.tile_seg0, ls.seg_layer,
                                                     tile, lds);
        rest_arrive(ls, tile, lds, bc_rest);
      }
    } else {
      lead_finalize(ls, lds);
    }
    return;
  }
  if constexpr (REST) {
    if (bid >= ls.n_tiles) {   // (uniform)
      rest_update<HAS_K, LPX>(aa, ls, lt, bid - ls.n_tiles);
      return;
    }
  }
  const int tpc = ls.lt.tpc;
  const TilePos p = tile_pos<TILE>(ls.lt.n_c, tpc, ls.lt.tile_list[bid]);
  const int sp0 = p.c * ls.lt.tpc_span + (p.t - p.c * tpc) * U;  // the tile's first span
  const int l0 = lt.first_layer[sp0];  // the layer the tile lies in (lt.first_layer: of the 1024-element tiling)
  const float kt = HAS_K ? lt.mom_scale[l0] : 1.0f;
  const float ss = ra.sscales[p.c];
  const LayerParts lp = layer_parts(ls.lt, l0);
  const float rp = ls.r_prev[l0], ca = ls.c_avg[l0];
  const int first = REST ? ls.arr0[l0] : lp.lb;
  typename std::conditional<REST, StepTerms, StepTable>::type st;
  if constexpr (!REST) st.find(vt, p.c, l0);
  const int a = h.n_old + 1;   // steps to apply
  const int o0 = threadIdx.x * 4;
  bool have_word;
  const int64_t wi = lane_word(p, &have_word);
  unsigned int Wq[VF_MAX_OLD + 2];
#pragma unroll
  for (int q = 0; q < VF_MAX_OLD + 2; ++q) {
    Wq[q] = 0u;
    if (q <= a && have_word) Wq[q] = plane_bits(ra, h, q)[wi];
  }
  v4f V[U], VZ[U];   // (VZ[0 .. S): unused)
  const int wv_u = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    V[u] = 0.0f; VZ[u] = 0.0f;
    if (o < p.len) {   // all lanes of a wavefront or none
      V[u] = ld4(ra.v_fresh + p.tile0 + o);
      if (u < S) lds_load16(ra.v_frozen + p.tile0 + o, &zs[u * BLOCK + wv_u * WAVE]);
      else VZ[u] = ld4(ra.v_frozen + p.tile0 + o);
    }
  }
  if constexpr (REST) st.template form<HAS_K>(ra, h, p.c, kt);
  // flips between consecutive planes, formed on the words as loaded; plane 0 stays (line 21 needs it)
#pragma unroll
  for (int s = VF_MAX_OLD + 1; s >= 1; --s)
    if (s <= a) Wq[s] ^= Wq[s - 1];
  // the lanes' own nibbles of every span, 8 to a register
#pragma unroll
  for (int q = 0; q < VF_MAX_OLD + 2; ++q)
    if (q <= a) Wq[q] = lane_nibbles(Wq[q]);   // uniform
#pragma unroll
  for (int s = VF_MAX_OLD + 1; s >= 1; --s) {
    if (s <= a) {   // uniform: the step from plane s to plane s-1
      const float t_same = st.t_same(s), t_diff = st.t_diff(s);
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < 4; ++k) V[u][k] = ra.beta2 * V[u][k] + select_by_bit(Wq[s], 4 * u + k, t_diff, t_same);
    }
  }
  MaxQuotient mq;
  mq.start(ls.one_m_thr * rp, ls.r_min);
  UpdateTerm ut;
  ut.start(HAS_K ? ss / kt : ss, aa.eta);
  if (S > 0) lds_loads_done();
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    if (o < p.len) {
      const v4f vz = (u < S) ? zs[u * BLOCK + threadIdx.x] : VZ[u];
      mq.add(vz, V[u], u + 1 < U);
      ut.see(vz);
    }
  }
  const float r = block_max(mq.r, lds);
  // before any store: nothing to wait for
  layer_arrive<REST>(ls, bid, l0, lp, first, REST ? layer_arrivals(lp.nl, lp.a, lp.s_first, lp.s_end, lp.b) : lp.nl, rp, ca, r,
               lds, &bc);
  if (h.write_v) {   // uniform
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int o = u * SPAN + o0;
      if (o < p.len) st4(ra.v_fresh + p.tile0 + o, V[u]);
    }
  }
  v4f X[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {  // x is fetched while the layer completes
    const int o = u * SPAN + o0;
    X[u] = 0.0f;
    if (o < p.len) X[u] = ld4(aa.x + p.tile0 + o);
  }
  // m_t/(sqrt(v_frozen)+eta), formed in place of v_frozen while the layer completes (the same
  // operations on the same operands as apply_uniform's)
  const bool in_range = ut.in_range();   // uniform
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    if (o < p.len) {
      v4f z = (u < S) ? zs[u * BLOCK + threadIdx.x] : VZ[u];
      ut.terms(z, Wq[0], 4 * u, in_range);
      if (u < S) zs[u * BLOCK + threadIdx.x] = z;
      else VZ[u] = z;
    }
  }
  const float c = layer_wait(ls, l0, &bc);
  const float al = aa.lr * c;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    if (o < p.len) {
      const v4f z = (u < S) ? zs[u * BLOCK + threadIdx.x] : VZ[u];
      v4f xn;
#pragma unroll
      for (int k = 0; k < 4; ++k) xn[k] = X[u][k] - al * z[k];
      st4(aa.x + p.tile0 + o, xn);
      if (LPX) st4_lp(aa.x_lp, p.tile0 + u * SPAN, o0, xn, aa.x_lp_bf16);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Small lists: Algorithm 1 lines 13-21 of the whole buffer in one launch.
//
// Where all 1024*U-element tiles of the buffer fit on the device at once, the three launches of the
// split above cost more than the work: every launch is a chain of dependent look-ups, loads and
// reductions of a few microseconds whatever it moves.  Here every tile, whatever layers it meets, is one
// workgroup that runs the ratio pass, takes part in the barriers of its layers and then the update, with
// x, v_frozen and the signs in registers.  U is 1, 2 or 4: small tiles keep a workgroup's own chain of
// look-ups and divisions short, large ones the number of workgroups small (small_cost in the host code).
//
// In a tile that meets several layers, what depends on the layer alone is formed once per segment (with momentum
// scaling, by each element: 24 tensors of 300x300 28.5 instead of 20.5 us) and each lane looks its segments up once.
//
// A layer wholly inside a tile needs no barrier; only the first and the last segment of a tile can belong
// to a layer that goes on elsewhere.  Barriers without counters (slots, below); bounded waits and co-residency rule (80 % of
// the workgroup slots) as for the other barriers.  The spans that k_ratios_apply_hist would handle
// from the variance's history ("lagging") do so here too, so that what the v_fresh array holds between two
// calls does not depend on the kernel; their two values per step are formed by each thread.
// Measured: four 512x512 tensors 8.8 us with slots, 9.7 with counted arrivals (k_ratios_apply_resident 12.6); 46 tensors of 2
// to 64000 elements 9.4, 10.4 (26 us in three launches, and the gaps between them).
// ---------------------------------------------------------------------------------------------
// workgroups per CU that the kernels are built for (their registers at each U)
constexpr int small_min_wg(int u) { return u == 1 ? 8 : (u == 2 ? 5 : 4); }
// k_warmup_small's arrivals counted in one level up to SMALL_ONE_LEVEL (a LAMB step, us, in one level / two: 200 arrivals 10.0 / 8.8, 256
// 12.2 / 10.3, 313 12.0 / 9.9, 392 13.3 / 10.4, 400 11.9 / 8.6, 588 19.5 / 16.5; 128 10.8 / 10.4 and 124 10.6 / 10.6).  A kernel of its own
// for lists without longer layers: carrying both forms costs it 0.2 to 0.5 us of 11 to 17.
template <bool TWO_LEVELS>
constexpr int small_one_level() { return TWO_LEVELS ? SMALL_ONE_LEVEL : 0x7fffffff; }
constexpr int SMALL_POLL_SLEEP = 2;   // (the whole launch lasts some 10 us: at first a poll every 128 clocks)
struct SmallTab {
  const SmallTile* tiles;
  int n_tiles, tpc, max_seg;
  int64_t n_c;
  const int* seg_layer;         // [segments]
  const int* layer_seg0;        // [L+1]
  void* partial;                // k_ratios_apply_small: [segments] slots; k_warmup_small: [2 * segments] double sums
  unsigned long long* counter;  // k_warmup_small: [L * CTR_STRIDE], then the group counters (group_line)
  unsigned long long* flag;     // k_warmup_small: [L * CTR_STRIDE]
  unsigned int* errflag;
  int spin_limit;
};
struct RatioClip {
  const float* c_avg;
  float* r_prev;
  float* coeff_c;
  float one_m_thr, one_p_thr, r_min, r_max;
};

// Segment tables of a tile that meets several layers, in LDS: where each segment ends (relative to the
// tile) and its layer; values of the segment; then the segment's coefficient.
struct SmallSegs {
  int* end;
  int* layer;
  float* coeff;    // (k_ratios_apply_small: first the variance's term of an unchanged sign)
  float* val;      // (k_ratios_apply_small only: the term of a changed sign, then |m_t|)
  __device__ __forceinline__ void load(const SmallTab& sm, const SmallTile& ti, const TilePos& p,
                                       const int64_t* __restrict__ off) {
    for (int s = threadIdx.x; s < ti.nseg; s += BLOCK) {
      const int l = sm.seg_layer[ti.seg0 + s];
      const int64_t e = off[l + 1] - p.tile0;
      layer[s] = l;
      end[s] = e < p.len ? (int)e : p.len;
    }
  }
  // segment of the element at `o` (nseg: padding)
  __device__ __forceinline__ int find(int nseg, int o) const {
    int lo = 0, hi = nseg;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (end[mid] > o) hi = mid; else lo = mid + 1;
    }
    return lo;
  }
  // where segment s ends (padding: never)
  __device__ __forceinline__ int end_of(int nseg, int s) const { return s < nseg ? end[s] : 0x7fffffff; }
};

// First half of the barriers of a tile: thread 0 arrives for its first segment, thread WAVE for its last
// one (if that is another).  store(e): publishes the segment's partial result.  bc[e] = (generation << 32) |
// (1: the layer's last arrival) | (2: the layer is this segment alone, no barrier).
template <bool TWO_LEVELS, class F>
__device__ __forceinline__ void small_arrive(const SmallTab& sm, int L, const SmallTile& ti, int n_end, const int (&s0_end)[2],
                                             unsigned long long* bc, F store) {
  const int e = threadIdx.x / WAVE;
  if (e < n_end && (threadIdx.x & (WAVE - 1)) == 0) {
    const int n = e ? ti.n_last : ti.n_first, l = e ? ti.l_last : ti.l0;
    if (n == 1) {
      bc[e] = 2ull;
    } else {
      store(e);
      payload_before_arrival();
      unsigned long long* top = &sm.counter[(int64_t)l * CTR_STRIDE];
      if constexpr (TWO_LEVELS) {
        const int s0 = e ? s0_end[1] : s0_end[0], s = ti.seg0 + (e ? ti.nseg - 1 : 0);
        bc[e] = barrier_arrive(top, sm.counter + (int64_t)L * CTR_STRIDE + group_line(s0, l), s - s0, n, SMALL_ONE_LEVEL);
      } else {
        bc[e] = barrier_arrive(top, n);
      }
    }
  }
  __syncthreads();
}

// The barrier of a layer in k_ratios_apply_small: every workgroup publishes its segment's partial result in a slot of its
// own, together with the number of the launch, and every workgroup reads all slots of the layer until each holds that
// number, so that only a store and a load lie between the last partial result and its readers.  (Arrivals counted at an
// atomic, whose last one reads the results and publishes the coefficient, are five such trips, and with the two fp64
// sums of k_warmup_small, four words a slot, those cost less: 10.6 us instead of 12.6 for four tensors of 262144.)  A step, us,
// counted / slots: four of 262144 23.9 / 22.3, two of 1 M 36.4 / 32.1, one of 1.6 M
// (391 segments) 30.2 / 29.5, of 2.9 M (706) 37.6 / 37.3; 24 of 65536 27.0 / 27.4.  The number is one more
// than what the slot held: nothing that changes from call to call comes from the host.  What a workgroup has read of r_prev and c_avg it has
// before it publishes; the layer's first segment's workgroup writes them, once all have published.
__device__ __forceinline__ unsigned long long slot_load(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, OB_AGENT);
}
__device__ __forceinline__ void slot_store(unsigned long long* p, unsigned int want, unsigned int payload) {
  __hip_atomic_store(p, ((unsigned long long)want << 32) | payload, __ATOMIC_RELAXED, OB_AGENT);
}
// The thread's slots of the n at p, each when it holds generation `want`: take(payload).  Waits are bounded as in barrier_wait.
template <class F>
__device__ __forceinline__ void slots_wait(const SmallTab& sm, const unsigned long long* p, int n, unsigned int want, F take) {
  int it = 0;
  for (int i = threadIdx.x; i < n; i += BLOCK) {
    unsigned long long v = slot_load(p + i);
    while (sm.spin_limit == 0 || (unsigned int)(v >> 32) != want) {
      if (it >= sm.spin_limit) {
        atomicOr(sm.errflag, 1u);
        break;
      }
      if ((it & 63) == 63 && __hip_atomic_load(sm.errflag, __ATOMIC_RELAXED, OB_AGENT) != 0u) break;
      if (it < 64) __builtin_amdgcn_s_sleep(SMALL_POLL_SLEEP);
      else __builtin_amdgcn_s_sleep(OB_POLL_SLEEP);
      ++it;
      v = slot_load(p + i);
    }
    take((unsigned int)v);
  }
}

template <int U, bool HAS_K, bool LPX>
__global__ __launch_bounds__(BLOCK, small_min_wg(U)) void k_ratios_apply_small(
    RatioArgs ra, VfHist h, ApplyArgs aa, SmallTab sm, RatioClip rc, LayerTab lt) {
  constexpr int TILE = SPAN * U;
  extern __shared__ int dyn_lds[];
  __shared__ float lds[BLOCK / WAVE];
  __shared__ float c_end[2];
  if ((int)blockIdx.x == sm.n_tiles) {   // the layers without elements go through the clips too
    for (int l = threadIdx.x; l < lt.L; l += BLOCK)
      if (sm.layer_seg0[l + 1] == sm.layer_seg0[l])
        (void)ratio_clip_commit(0.0f, l, rc.r_prev[l], rc.c_avg[l], rc.r_prev, rc.coeff_c, rc.one_m_thr, rc.one_p_thr,
                                rc.r_min, rc.r_max);
    return;
  }
  const SmallTile ti = sm.tiles[blockIdx.x];
  if (ti.nseg == 0) return;
  TilePos p;
  p.t = (int)blockIdx.x;
  p.c = ti.chunk_kind >> 2;
  const int64_t in_chunk = (int64_t)(p.t - p.c * sm.tpc) * TILE;
  p.tile0 = (int64_t)p.c * sm.n_c + in_chunk;
  p.len = (sm.n_c - in_chunk < TILE) ? (int)(sm.n_c - in_chunk) : TILE;
  const bool inside = (ti.chunk_kind & 1) != 0, lagging = (ti.chunk_kind & 2) != 0;
  const int a = lagging ? h.n_old + 1 : 1;       // steps to apply (uniform)
  const int o0 = threadIdx.x * 4;
  unsigned int NB[VF_MAX_OLD + 2][U];            // the lane's nibble of every plane, newest first
  v4f V[U], VZ[U], X[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    V[u] = 0.0f; VZ[u] = 0.0f; X[u] = 0.0f;
#pragma unroll
    for (int q = 0; q < VF_MAX_OLD + 2; ++q) {
      NB[q][u] = 0u;
      if (q <= a && o < p.len) NB[q][u] = load_nibble(plane_bits(ra, h, q), p.tile0 + u * SPAN);
    }
    if (o < p.len) {
      V[u] = ld4(ra.v_fresh + p.tile0 + o);
      VZ[u] = ld4(ra.v_frozen + p.tile0 + o);
      X[u] = ld4(aa.x + p.tile0 + o);
    }
  }
  const float ss = ra.sscales[p.c];
  float* const vals = reinterpret_cast<float*>(dyn_lds);      // [TILE] quotients (tiles that meet several layers)
  SmallSegs sg;
  sg.end = dyn_lds + TILE; sg.layer = sg.end + sm.max_seg;
  sg.coeff = reinterpret_cast<float*>(sg.layer + sm.max_seg);
  sg.val = sg.coeff + sm.max_seg;
  int s_of[U];                                   // segment of the lane's first element of each span
  const int last_seg = ti.nseg - 1;
  const int n_end = ti.nseg > 1 ? 2 : 1;
  const int l_end[2] = {ti.l0, ti.l_last};
  float r_end[2] = {0.0f, 0.0f};                 // maxima of the first and the last segment (thread 0)
  // what finishing a layer takes, requested with everything else
  const float rp_end[2] = {rc.r_prev[ti.l0], rc.r_prev[ti.l_last]}, ca_end[2] = {rc.c_avg[ti.l0], rc.c_avg[ti.l_last]};
  const int s0_end[2] = {sm.layer_seg0[ti.l0], sm.layer_seg0[ti.l_last]}, n_of[2] = {ti.n_first, ti.n_last};
  const int s_end[2] = {ti.seg0, ti.seg0 + last_seg};
  unsigned long long* const slots = static_cast<unsigned long long*>(sm.partial);
  const unsigned int want[2] = {(unsigned int)(slot_load(&slots[s_end[0]]) >> 32) + 1u,
                                (unsigned int)(slot_load(&slots[s_end[1]]) >> 32) + 1u};
  if (inside) {
    const float kt = HAS_K ? lt.mom_scale[ti.l0] : 1.0f;
#pragma unroll
    for (int s = VF_MAX_OLD + 1; s >= 1; --s) {
      if (s <= a) {
        float t_same, t_diff;
        variance_terms<HAS_K>(ra, plane_scale(ra, h, s - 1, p.c), plane_scale(ra, h, s, p.c), kt, &t_same, &t_diff);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int k = 0; k < 4; ++k)
            V[u][k] = ra.beta2 * V[u][k] + select_by_bit(NB[s][u] ^ NB[s - 1][u], k, t_diff, t_same);
      }
    }
    float r = 0.0f;
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float q = VZ[u][k] / V[u][k];      // (0/0 beyond the tile's end: NaN, not taken)
        if (q > r) r = q;
      }
    r_end[0] = block_max(r, lds);
  } else {
    sg.load(sm, ti, p, lt.off);
    const float s_prev = ra.pm.scales[p.c];
    float t_same, t_diff;
    variance_terms<false>(ra, ss, s_prev, 1.0f, &t_same, &t_diff);
    if (HAS_K)   // (each thread's own entries of `layer`)
      for (int s = threadIdx.x; s < ti.nseg; s += BLOCK)
        variance_terms<true>(ra, ss, s_prev, lt.mom_scale[sg.layer[s]], &sg.coeff[s], &sg.val[s]);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int o = u * SPAN + o0;
      s_of[u] = 0;
      if (o < p.len) {
        int s = sg.find(ti.nseg, o), e = sg.end_of(ti.nseg, s);
        s_of[u] = s;
        if (HAS_K && s < ti.nseg) { t_same = sg.coeff[s]; t_diff = sg.val[s]; }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (o + k >= e) {
            do e = sg.end_of(ti.nseg, ++s); while (o + k >= e);
            if (HAS_K && s < ti.nseg) { t_same = sg.coeff[s]; t_diff = sg.val[s]; }
          }
          float q = 0.0f;
          if (s < ti.nseg) {
            V[u][k] = ra.beta2 * V[u][k] + ((((NB[0][u] ^ NB[1][u]) >> k) & 1u) ? t_diff : t_same);
            q = VZ[u][k] / V[u][k];
          }
          vals[o + k] = q;
        }
      }
    }
    __syncthreads();
    if (HAS_K)
      for (int s = threadIdx.x; s < ti.nseg; s += BLOCK) sg.val[s] = ss / lt.mom_scale[sg.layer[s]];
    // a wavefront per segment; the layers that lie inside the tile are finished here
    const int lane = threadIdx.x & (WAVE - 1);
    for (int s = threadIdx.x / WAVE; s < ti.nseg; s += BLOCK / WAVE) {
      float r = 0.0f;
      for (int o = (s ? sg.end[s - 1] : 0) + lane; o < sg.end[s]; o += WAVE)
        if (vals[o] > r) r = vals[o];
      r = wave_max(r);
      if (lane == 0) sg.coeff[s] = r;
    }
    __syncthreads();
    r_end[0] = sg.coeff[0];
    r_end[1] = sg.coeff[last_seg];
  }
  if (threadIdx.x == 0) {
#pragma unroll
    for (int e = 0; e < 2; ++e)
      if (e < n_end && n_of[e] > 1) {
        asm volatile("" ::"v"(rp_end[e]), "v"(ca_end[e]) : "memory");   // both are there before the slot says so
        slot_store(&slots[s_end[e]], want[e], __float_as_uint(r_end[e]));
      }
  }
  if (!inside) {   // the layers in between lie inside the tile
    __syncthreads();
    for (int s = 1 + (int)threadIdx.x; s < last_seg; s += BLOCK) {
      const int l = sg.layer[s];
      sg.coeff[s] = ratio_clip_commit(sg.coeff[s], l, rc.r_prev[l], rc.c_avg[l], rc.r_prev, rc.coeff_c, rc.one_m_thr,
                                      rc.one_p_thr, rc.r_min, rc.r_max);
    }
  }
  // while the layers complete: the variance is stored, m_t/(sqrt(v_frozen)+eta) formed in place of v_frozen
  if (inside) {
    const float sp = HAS_K ? ss / lt.mom_scale[ti.l0] : ss;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int o = u * SPAN + o0;
      if (o < p.len) {
        if (!lagging || h.write_v) st4(ra.v_fresh + p.tile0 + o, V[u]);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float mt = ((NB[0][u] >> k) & 1u) ? sp : -sp;
          float uu = mt / (sqrtf(VZ[u][k]) + aa.eta);
          asm volatile("" : "+v"(uu));   // evaluated here, not sunk below the wait
          VZ[u][k] = uu;
        }
      }
    }
  } else {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int o = u * SPAN + o0;
      if (o < p.len) {
        int s = s_of[u], e = sg.end_of(ti.nseg, s);
        float sp = (HAS_K && s < ti.nseg) ? sg.val[s] : ss;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (o + k >= e) {
            do e = sg.end_of(ti.nseg, ++s); while (o + k >= e);
            if (HAS_K && s < ti.nseg) sp = sg.val[s];
          }
          if (s < ti.nseg) {
            ra.v_fresh[p.tile0 + o + k] = V[u][k];
            const float mt = ((NB[0][u] >> k) & 1u) ? sp : -sp;
            float uu = mt / (sqrtf(VZ[u][k]) + aa.eta);
            asm volatile("" : "+v"(uu));
            VZ[u][k] = uu;
          }
        }
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    if (e >= n_end) break;   // (uniform)
    float q = r_end[e];
    if (n_of[e] > 1) {
      q = 0.0f;
      slots_wait(sm, slots + s0_end[e], n_of[e], want[e], [&](unsigned int w) {
        const float v = __uint_as_float(w);
        if (v > q) q = v;
      });
      q = block_max(q, lds);
    }
    if (threadIdx.x == 0) {
      const float r = ratio_clip(q, rp_end[e], rc.one_m_thr, rc.one_p_thr, rc.r_min, rc.r_max), c = r * ca_end[e];
      if (s_end[e] == s0_end[e]) {
        rc.r_prev[l_end[e]] = r;
        rc.coeff_c[l_end[e]] = c;
      }
      c_end[e] = c;
    }
  }
  __syncthreads();
  if (inside) {
    const float al = aa.lr * c_end[0];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int o = u * SPAN + o0;
      if (o < p.len) {
        v4f xn;
#pragma unroll
        for (int k = 0; k < 4; ++k) xn[k] = X[u][k] - al * VZ[u][k];
        st4(aa.x + p.tile0 + o, xn);
        if (LPX) st4_lp(aa.x_lp, p.tile0 + u * SPAN, o0, xn, aa.x_lp_bf16);
      }
    }
  } else {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int o = u * SPAN + o0;
      if (o < p.len) {
        int s = s_of[u], e = sg.end_of(ti.nseg, s);
        auto coeff = [&](int q) { return aa.lr * (q == 0 ? c_end[0] : q == last_seg ? c_end[1] : sg.coeff[q]); };
        float al = s < ti.nseg ? coeff(s) : 0.0f;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (o + k >= e) {
            do e = sg.end_of(ti.nseg, ++s); while (o + k >= e);
            if (s < ti.nseg) al = coeff(s);
          }
          if (s < ti.nseg) {
            const float xn = X[u][k] - al * VZ[u][k];
            aa.x[p.tile0 + o + k] = xn;
            if (LPX) reinterpret_cast<unsigned short*>(aa.x_lp)[p.tile0 + o + k] = float_to_lp(xn, aa.x_lp_bf16);
          }
        }
      }
    }
  }
}

// Dense view of a momentum held in 1-bit form: m[i] = (bit ? s_c : -s_c)/k_l for i < N (the
// padding of m is left untouched).
template <int U, bool HAS_K>
__global__ __launch_bounds__(BLOCK) void k_momentum_dense(PackedMom pm, float* __restrict__ m,
                                                          int64_t n_c, int tpc, LayerTab lt) {
  constexpr int TILE = SPAN * U;
  const TilePos p = tile_pos<TILE>(n_c, tpc, (int)blockIdx.x);
  const int l0 = lt.first_layer[p.t];
  const int L = lt.L;
  if (l0 >= L) return;
  const int o0 = threadIdx.x * 4;
  const float ss = pm.scales[p.c];
  const bool uniform = (p.tile0 + p.len <= lt.off[l0 + 1]);
  const int64_t N = lt.off[L];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    if (o < p.len) {
      const unsigned int nb = load_nibble(pm.bits, p.tile0 + u * SPAN);
      if (uniform) {
        const float sp = HAS_K ? ss / lt.mom_scale[l0] : ss;
        v4f mn;
#pragma unroll
        for (int k = 0; k < 4; ++k) mn[k] = ((nb >> k) & 1u) ? sp : -sp;
        st4(m + p.tile0 + o, mn);
      } else {
        int l = l0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int64_t i = p.tile0 + o + k;
          if (i < N) {
            l = walk_layer(l, i, lt.off);
            const float sp = HAS_K ? ss / lt.mom_scale[l] : ss;
            m[i] = ((nb >> k) & 1u) ? sp : -sp;
          }
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// K8  LAMB warmup step, eq. (1)
//   a: m, v update; per (tile, layer) segment the fp64 sums of x^2 and u^2
//   b: per layer: c = clip(||x||/||u||), c_avg moving average (Algorithm 1 line 2)
//   c: x <- x - (lr*c) u, with u recomputed from the stored m, v (same operations, same value)
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ float lamb_u(float mn, float vn, float x, float eta, float wd) {
  float u = mn / (sqrtf(vn) + eta);
  if (wd != 0.0f) u = u + wd * x;
  return u;
}

// lamb_u of four elements, by all lanes of a wavefront: the shorter root and quotient where every lane's operands lie in their range
// (here the numerator, m, differs from element to element; its sign is put back at the end, as a residual of zero loses that of -0).  A LAMB step, us, lamb_u / this: 3 M parameters in one launch 24.9 / 23.45, 11 M 76.2 / 75.8, 110 M with a 16-bit
// copy 589.3 / 588.6, 336 M 1678.6 / 1679.9, which memory bounds.
__device__ __forceinline__ v4f lamb_u4(const v4f& m, const v4f& v, const v4f& x, float eta, float wd) {
  unsigned int top = 0u, low = 0xffffffffu;
  float big = 0.0f;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const unsigned int vb = __float_as_uint(v[k]), mb = 2u * __float_as_uint(m[k]) - 1u;   // (zero: the largest)
    top = vb > top ? vb : top;
    low = mb < low ? mb : low;
    big = fmaxf(big, fabsf(m[k]));   // (a NaN stays one in either form)
  }
  const bool ok = top <= SHORT_V_TOP_BITS && low >= 2u * SHORT_N_LOW_BITS - 1u && big <= SHORT_N_TOP && eta >= SHORT_ETA_LOW && eta <= SHORT_ETA_TOP;
  v4f u;
  if (__ballot(!ok) == 0ull) {
#pragma unroll
    for (int k = 0; k < 4; ++k) u[k] = __builtin_copysignf(short_quotient(fabsf(m[k]), short_denominator(v[k], eta)), m[k]);
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) u[k] = m[k] / (sqrtf(v[k]) + eta);
  }
  if (wd != 0.0f) {   // uniform
#pragma unroll
    for (int k = 0; k < 4; ++k) u[k] = u[k] + wd * x[k];
  }
  return u;
}

template <int U, int GT = 0>
__global__ __launch_bounds__(BLOCK) void k_warmup_moments(
    GradSrc g, float* __restrict__ m, float* __restrict__ v,
    const float* __restrict__ x, double* __restrict__ seg_sums /* [2*n_segs] */, int64_t n_c,
    int tpc, float beta1, float omb1, float beta2, float omb2, float eta, float wd, LayerTab lt,
    const int* __restrict__ tile_seg0, const int* __restrict__ seg_layer,
    const int* __restrict__ tile_list) {
  constexpr int TILE = SPAN * U;
  __shared__ double lds[BLOCK / WAVE];
  const TilePos p = tile_pos<TILE>(n_c, tpc, listed_tile(tile_list));
  const int l0 = lt.first_layer[p.t];
  const int L = lt.L;
  if (l0 >= L) return;
  const int o0 = threadIdx.x * 4;
  const bool uniform = (p.tile0 + p.len <= lt.off[l0 + 1]);
  v4f G[U], M[U], V[U], X[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    G[u] = 0.0f; M[u] = 0.0f; V[u] = 0.0f; X[u] = 0.0f;
    if (o < p.len) {
      G[u] = load_grad<GT>(g, p.tile0 + o);
      M[u] = ld4(m + p.tile0 + o);
      V[u] = ld4(v + p.tile0 + o);
      X[u] = ld4(x + p.tile0 + o);
    }
  }
  // new moments (kept in M, V)
#pragma unroll
  for (int u = 0; u < U; ++u) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      M[u][k] = beta1 * M[u][k] + omb1 * G[u][k];
      V[u][k] = beta2 * V[u][k] + omb2 * (G[u][k] * G[u][k]);
    }
  }
  const int s0 = tile_seg0[p.t];
  if (uniform) {
    double sx = 0.0, su = 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int o = u * SPAN + o0;
      if (o < p.len) {
        st4(m + p.tile0 + o, M[u]);
        st4(v + p.tile0 + o, V[u]);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float uu = lamb_u(M[u][k], V[u][k], X[u][k], eta, wd);
          sx += (double)X[u][k] * (double)X[u][k];
          su += (double)uu * (double)uu;
        }
      }
    }
    sx = block_sum(sx, lds);
    su = block_sum(su, lds);
    if (threadIdx.x == 0) {
      seg_sums[2 * (int64_t)s0] = sx;
      seg_sums[2 * (int64_t)s0 + 1] = su;
    }
  } else {
    const int64_t N = lt.off[L];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int o = u * SPAN + o0;
      if (o < p.len) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int64_t i = p.tile0 + o + k;
          if (i < N) {
            m[i] = M[u][k];
            v[i] = V[u][k];
          }
        }
      }
    }
    const int s1 = tile_seg0[p.t + 1];
    for (int s = s0; s < s1; ++s) {
      const int l = seg_layer[s];
      const int64_t a = lt.off[l], b = lt.off[l + 1];
      double sx = 0.0, su = 0.0;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int o = u * SPAN + o0;
        if (o < p.len) {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int64_t i = p.tile0 + o + k;
            if (i >= a && i < b) {
              const float uu = lamb_u(M[u][k], V[u][k], X[u][k], eta, wd);
              sx += (double)X[u][k] * (double)X[u][k];
              su += (double)uu * (double)uu;
            }
          }
        }
      }
      sx = block_sum(sx, lds);
      su = block_sum(su, lds);
      if (threadIdx.x == 0) {
        seg_sums[2 * (int64_t)s] = sx;
        seg_sums[2 * (int64_t)s + 1] = su;
      }
    }
  }
}

// eq. (1)'s coefficient of one layer from its sums of x^2 and u^2, and Algorithm 1 line 2
// (thread 0 of a workgroup).
// ca: c_avg[l], read by the caller (early, where its latency hides).
__device__ __forceinline__ float warmup_coeff_commit(double sx, double su, int l, float ca,
                                                     float* __restrict__ coeff_c,
                                                     float* __restrict__ c_avg, float c_min,
                                                     float c_max, float beta3, float omb3) {
  const float nx = (float)sqrt(sx), nu = (float)sqrt(su);
  float c = nx / nu;
  c = (c > c_min) ? c : c_min;
  c = (c < c_max) ? c : c_max;
  coeff_c[l] = c;
  c_avg[l] = beta3 * ca + omb3 * c;
  return c;
}

struct WarmClip {
  float* coeff_c;
  float* c_avg;
  float c_min, c_max, beta3, omb3;
};

__global__ __launch_bounds__(FBLOCK) void k_warmup_coeff(const double* __restrict__ seg_sums,
                                                         const int* __restrict__ layer_seg0,
                                                         float* __restrict__ coeff_c,
                                                         float* __restrict__ c_avg, float c_min,
                                                         float c_max, float beta3, float omb3,
                                                         const unsigned char* __restrict__ done_elsewhere,
                                                         unsigned long long* __restrict__ clear_flag) {
  __shared__ double lds[FBLOCK / WAVE];
  const int l = blockIdx.x;
  if (clear_flag && threadIdx.x == 0) clear_flag[l] = 0ull;   // (of k_warmup_trail, which runs after this kernel)
  if (done_elsewhere && done_elsewhere[l]) return;  // the kernel with the per-layer barrier finishes it
  const int s0 = layer_seg0[l], s1 = layer_seg0[l + 1];
  const float ca = c_avg[l];
  double sx = 0.0, su = 0.0;
  for (int s = s0 + threadIdx.x; s < s1; s += 4 * FBLOCK) {   // four pairs in flight per thread
    double vx[4], vu[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool in = (s + u * FBLOCK < s1);
      vx[u] = in ? seg_sums[2 * (int64_t)(s + u * FBLOCK)] : 0.0;
      vu[u] = in ? seg_sums[2 * (int64_t)(s + u * FBLOCK) + 1] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) { sx += vx[u]; su += vu[u]; }
  }
  sx = block_sum<FBLOCK>(sx, lds);
  su = block_sum<FBLOCK>(su, lds);
  if (threadIdx.x == 0) (void)warmup_coeff_commit(sx, su, l, ca, coeff_c, c_avg, c_min, c_max, beta3, omb3);
}

template <int U, bool LPX = false>
__global__ __launch_bounds__(BLOCK) void k_warmup_apply(
    const float* __restrict__ m, const float* __restrict__ v, float* __restrict__ x,
    const float* __restrict__ coeff_c, int64_t n_c, int tpc, float lr, float eta, float wd,
    LayerTab lt, void* __restrict__ x_lp, int x_lp_bf16, const int* __restrict__ tile_list) {
  constexpr int TILE = SPAN * U;
  const TilePos p = tile_pos<TILE>(n_c, tpc, listed_tile(tile_list));
  const int l0 = lt.first_layer[p.t];
  const int L = lt.L;
  if (l0 >= L) return;
  const int o0 = threadIdx.x * 4;
  const bool uniform = (p.tile0 + p.len <= lt.off[l0 + 1]);
  v4f M[U], V[U], X[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    if (o < p.len) {
      M[u] = ld4(m + p.tile0 + o);
      V[u] = ld4(v + p.tile0 + o);
      X[u] = ld4(x + p.tile0 + o);
    }
  }
  if (uniform) {
    const float a = lr * coeff_c[l0];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int o = u * SPAN + o0;
      if (o < p.len) {
        v4f xn;
#pragma unroll
        for (int k = 0; k < 4; ++k)
          xn[k] = X[u][k] - a * lamb_u(M[u][k], V[u][k], X[u][k], eta, wd);
        st4(x + p.tile0 + o, xn);
        if (LPX) st4_lp(x_lp, p.tile0 + u * SPAN, o0, xn, x_lp_bf16);
      }
    }
  } else {
    const int64_t N = lt.off[L];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int o = u * SPAN + o0;
      if (o < p.len) {
        int l = l0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int64_t i = p.tile0 + o + k;
          if (i < N) {
            l = walk_layer(l, i, lt.off);
            const float a = lr * coeff_c[l];
            const float xn = X[u][k] - a * lamb_u(M[u][k], V[u][k], X[u][k], eta, wd);
            x[i] = xn;
            if (LPX) reinterpret_cast<unsigned short*>(x_lp)[i] = float_to_lp(xn, x_lp_bf16);
          }
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// K8 a+b+c in one pass: eq. (1) with g, m, v and x read once.  A workgroup updates the moments of
// its tile, writes them, keeps u and x in registers and LDS, publishes the tile's fp64 sums of x^2 and u^2
// and arrives at its layer's barrier; the last of the layer's listed tiles to arrive sums ALL of
// the layer's segment sums in a fixed order, forms c, commits coeff_c and c_avg (Algorithm 1 line
// 2) and publishes c; the others wait for it and then update x from registers.  Same split of the
// work as for k_ratios_apply_resident (listed tiles here; everything else through
// k_warmup_moments before, whose sums wait in seg_sums, and k_warmup_apply after), same
// synchronisation and bounded waits.
// ---------------------------------------------------------------------------------------------
struct WarmSync {
  const double* seg_sums;       // [2 * segments of the 1024-element tiling] sums left by k_warmup_moments
  double* listed_sums;          // [2 * listed tiles] sums of this launch's tiles
  ListedTiles lt;
  unsigned long long* counter;  // [L * CTR_STRIDE] (generation << 32) | arrivals
  unsigned long long* sub;      // group counters (group_line)
  unsigned long long* flag;     // [L] (generation << 32) | bits of c
  unsigned int* errflag;
  int spin_limit;
  float* coeff_c;
  float* c_avg;
  float c_min, c_max, beta3, omb3;
};

// Bound by HBM and, between a layer's arrival and its coefficient, by the workgroups that wait with their tile
// in hand: what fits on the device at once limits both the layers that the kernel takes and what streams
// while others wait.  With u and x of all 8 spans in registers 4 workgroups fit on a CU (a layer of at most
// 811 tiles); with x of OB_WU_LDS spans in LDS (24 KB a workgroup) and loads one span at a time there are 6
// (1220 tiles), and a handful of registers spilled.  Measured, fp32 gradient: twelve 2800x2800 tensors, which
// took two passes before (40 bytes per element instead of 28), 620 -> 526 us; ten 3100x3100 639 -> 537 us;
// one layer of 7.8 M elements among small ones (11 M in all) 88.1 -> 81.5 us; twenty 2048x2048, taken by both
// forms, 408 -> 397 us; the 336 M BERT list 1734 -> 1723 us.  5 workgroups of 6 spans in LDS: 1743 us there;
// 6 workgroups with loads two spans at a time spill 16 registers: 1757 us.
#ifndef OB_WU_MINW
#define OB_WU_MINW 6
#endif
#ifndef OB_WU_LDS
#define OB_WU_LDS 6
#endif
template <int U, int G, int GT, bool LPX>
__global__ __launch_bounds__(BLOCK, OB_WU_MINW) void k_warmup_resident(
    GradSrc g, float* __restrict__ m, float* __restrict__ v, float* __restrict__ x, WarmSync ws,
    float beta1, float omb1, float beta2, float omb2, float eta, float wd, float lr, LayerTab lt,
    void* __restrict__ x_lp, int x_lp_bf16) {
  constexpr int TILE = SPAN * U;
  __shared__ double lds[BLOCK / WAVE];
  __shared__ unsigned long long bc;
  constexpr int S = OB_WU_LDS;   // spans whose x waits in LDS (each thread reads back its own values)
  __shared__ v4f xs[S > 0 ? S * BLOCK : 1];
  const int tpc = ws.lt.tpc;
  const TilePos p = tile_pos<TILE>(ws.lt.n_c, tpc, ws.lt.tile_list[blockIdx.x]);
  const int sp0 = p.c * ws.lt.tpc_span + (p.t - p.c * tpc) * U;  // the tile's first span (1024-element tiling)
  const int l0 = lt.first_layer[sp0];   // the layer the tile lies in
  const LayerParts lp = layer_parts(ws.lt, l0);
  const float ca = ws.c_avg[l0];
  const int o0 = threadIdx.x * 4;
  v4f UU[U], X[U];
  v4f Ml[G], Vl[G];   // m and v of the last group: stored after the arrival, which then waits for no store
  double sx = 0.0, su = 0.0;
#pragma unroll
  for (int u0 = 0; u0 < U; u0 += G) {
    v4f Gr[G], M[G], V[G];
#pragma unroll
    for (int j = 0; j < G; ++j) {
      const int o = (u0 + j) * SPAN + o0;
      X[u0 + j] = 0.0f; UU[u0 + j] = 0.0f;
      if (o < p.len) {
        Gr[j] = load_grad<GT>(g, p.tile0 + o);
        M[j] = ld4(m + (p.tile0 + (u0 + j) * SPAN) + o0);
        V[j] = ld4(v + (p.tile0 + (u0 + j) * SPAN) + o0);
        X[u0 + j] = ld4(x + (p.tile0 + (u0 + j) * SPAN) + o0);
      }
    }
#pragma unroll
    for (int j = 0; j < G; ++j) {
      const int o = (u0 + j) * SPAN + o0;
      if (o < p.len) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          M[j][k] = beta1 * M[j][k] + omb1 * Gr[j][k];
          V[j][k] = beta2 * V[j][k] + omb2 * (Gr[j][k] * Gr[j][k]);
        }
        if (u0 + G < U) {
          st4(m + (p.tile0 + (u0 + j) * SPAN) + o0, M[j]);
          st4(v + (p.tile0 + (u0 + j) * SPAN) + o0, V[j]);
        } else {
          Ml[j] = M[j];
          Vl[j] = V[j];
        }
        UU[u0 + j] = lamb_u4(M[j], V[j], X[u0 + j], eta, wd);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          sx += (double)X[u0 + j][k] * (double)X[u0 + j][k];
          su += (double)UU[u0 + j][k] * (double)UU[u0 + j][k];
        }
        if (u0 + j < S) xs[(u0 + j) * BLOCK + threadIdx.x] = X[u0 + j];
      }
    }
  }
  sx = block_sum(sx, lds);
  su = block_sum(su, lds);
  // arrive: publish the tile's sums, then count; the last arriver finishes the layer
  unsigned long long* counter = &ws.counter[(int64_t)l0 * CTR_STRIDE];
  if (threadIdx.x == 0) {
    __hip_atomic_store(&ws.listed_sums[2 * (int64_t)blockIdx.x], sx, __ATOMIC_RELAXED, OB_AGENT);
    __hip_atomic_store(&ws.listed_sums[2 * (int64_t)blockIdx.x + 1], su, __ATOMIC_RELAXED, OB_AGENT);
    payload_before_arrival();
    bc = barrier_arrive(counter, ws.sub + group_line(lp.lb, l0), (int)blockIdx.x - lp.lb, lp.nl, ws.lt.one_level);
  }
  __syncthreads();
  const bool last = ((bc & 1ull) != 0ull);
  const unsigned int want = (unsigned int)(bc >> 32);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < G; ++j) {
    const int o = (U - G + j) * SPAN + o0;
    if (o < p.len) {
      st4(m + (p.tile0 + (U - G + j) * SPAN) + o0, Ml[j]);
      st4(v + (p.tile0 + (U - G + j) * SPAN) + o0, Vl[j]);
    }
  }
  float c;
  if (last) {
    double tx = 0.0, tu = 0.0;
    struct Sums { double x, u; };
    for_layer_parts(
        lp, Sums{0.0, 0.0},   // the sums are >= +0: adding these zeros changes nothing
        [&](int i) {
          Sums v;
          v.x = __hip_atomic_load(&ws.listed_sums[2 * (int64_t)i], __ATOMIC_RELAXED, OB_AGENT);
          v.u = __hip_atomic_load(&ws.listed_sums[2 * (int64_t)i + 1], __ATOMIC_RELAXED, OB_AGENT);
          return v;
        },
        [&](const Sums& v) { tx += v.x; tu += v.u; },
        [&](int j) {   // written by an earlier kernel
          tx += ws.seg_sums[2 * (int64_t)j];
          tu += ws.seg_sums[2 * (int64_t)j + 1];
        });
    tx = block_sum(tx, lds);
    tu = block_sum(tu, lds);
    if (threadIdx.x == 0) {
      const float cc = warmup_coeff_commit(tx, tu, l0, ca, ws.coeff_c, ws.c_avg, ws.c_min, ws.c_max,
                                           ws.beta3, ws.omb3);
      bc = barrier_publish(&ws.flag[l0], counter, lp.nl, want, __float_as_uint(cc), ws.lt.one_level);
    }
  } else if (threadIdx.x == 0) {
    bc = barrier_wait(&ws.flag[l0], want, ws.errflag, ws.spin_limit);
  }
  __syncthreads();
  c = __uint_as_float((unsigned int)(bc & 0xffffffffull));
  const float a = lr * c;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    if (o < p.len) {
      const v4f xo = (u < S) ? xs[u * BLOCK + threadIdx.x] : X[u];
      v4f xn;
#pragma unroll
      for (int k = 0; k < 4; ++k) xn[k] = xo[k] - a * UU[u][k];
      st4(x + (p.tile0 + u * SPAN) + o0, xn);
      if (LPX) st4_lp(x_lp, p.tile0 + u * SPAN, o0, xn, x_lp_bf16);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// K8 a+b+c for the layers that are too large for k_warmup_resident: moments (a) and update (c) as two kinds
// of workgroups of one launch, on parts of the 8192-element tiles that lie inside one layer.  Nothing is held
// on chip in between; the update's reads of m, v and x (12 of 40 bytes per element) come from the
// memory-side cache instead of HBM: a layer's update follows its moments as closely as its coefficient allows,
// the moments' stores of what is updated next and their load of x do not bypass that cache, and everything else does.
//
// `items` lists the workgroups in the order of dispatch: the parts in position order for the moments, and a
// layer's parts for the update `lag` parts after its last one (trail_items in the host code).  The last moments
// workgroup of a layer to finish adds up the sums (arrivals counted in two levels, as in chunk_ticket) and
// publishes c in flag[l].  An update workgroup requests x, which no moments workgroup writes, then waits for that
// flag, which by then is normally there, and only then loads m and v and forms u.  Moments workgroups wait for
// nothing and an update workgroup only for ones dispatched before it, so progress needs in-order dispatch, not
// co-residency.  Without `wait` the launch ends between a layer's two passes instead.
//
// The two passes of a part may run on different XCDs, whose L2 caches do not see each other's lines: the
// moments store m and v through to memory (agent scope) and wait for the acknowledgements before they arrive,
// and the update must load them after it has seen the flag, which those arrivals lead to, and past its own caches: a load
// before the flag finds values of the step before.
// ---------------------------------------------------------------------------------------------
constexpr int CACHE_NT = 2, CACHE_AGENT = 16;     // cache policy bits of the buffer builtins (nt, sc1)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t part_rsrc(const float* p, int bytes) {   // p uniform
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, bytes, OB_BUFFER_RSRC_WORD3);
}
template <int POLICY>
__device__ __forceinline__ v4f buf_ld4(__amdgpu_buffer_rsrc_t r, int byte) {
  return __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(r, byte, 0, POLICY));
}
template <int POLICY>
__device__ __forceinline__ void buf_st4(__amdgpu_buffer_rsrc_t r, int byte, v4f v) {
  typedef unsigned int v4u __attribute__((ext_vector_type(4)));
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, v), r, byte, 0, POLICY);
}
struct TrailTab {
  const unsigned int* items;    // of this launch: flags above | tile's position in lt.tile_list * TRAIL_PARTS + part
  ListedTiles lt;               // the tiles of these layers (positions as for the barrier kernels)
  const int* count0;            // [L] the layer's first counter: second level, then the first-level ones
  unsigned int* count;          // lines of CTR_STRIDE 8-byte words
  double* sub_sums;             // [2 * counters] of the first-level groups
  double* part_sums;            // [2 * parts]
  unsigned long long* flag;     // [L] 2^32 | bits of c once known; cleared by an earlier launch of the call
  const double* seg_sums;       // [2 * segments] sums left by k_warmup_moments
  unsigned int* errflag;
  int spin_limit;
  int wait;                     // an update waits for flag[l] (else: coeff_c[l] is there)
};

// First wavefront of a moments workgroup; part: its number, sx, su: its sums (lane 0).
__device__ __forceinline__ bool trail_arrive(unsigned int* counter, unsigned int n, double* payload, double sx, double su) {
  int last = 0;
  if ((threadIdx.x & (WAVE - 1)) == 0) {
    __hip_atomic_store(payload, sx, __ATOMIC_RELAXED, OB_AGENT);
    __hip_atomic_store(payload + 1, su, __ATOMIC_RELAXED, OB_AGENT);
    payload_before_arrival();
    last = (__hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, OB_AGENT) + 1u == n);
    if (last) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, OB_AGENT);
  }
  return __builtin_amdgcn_readfirstlane(last) != 0;
}
// l, lp, c0, ca: the layer, its ranges, first counter and c_avg (read early, where their latency hides).
__device__ __forceinline__ void trail_finish(const TrailTab& tt, const WarmClip& wc, int part, int l, const LayerParts& lp,
                                             int64_t c0, float ca, double sx, double su) {
  constexpr int LINE = 2 * CTR_STRIDE;
  const int lane = threadIdx.x & (WAVE - 1);
  const int n_parts = lp.nl * TRAIL_PARTS, part0 = lp.lb * TRAIL_PARTS;
  const int sub = (part - part0) / TICKET_SUB, first = sub * TICKET_SUB;
  const int n = (n_parts - first < TICKET_SUB) ? n_parts - first : TICKET_SUB;
  const int n_sub = (n_parts + TICKET_SUB - 1) / TICKET_SUB;
  const int64_t cs = c0 + 1 + sub;
  if (!trail_arrive(tt.count + cs * LINE, (unsigned int)n, &tt.part_sums[2 * (int64_t)part], sx, su)) return;
  double tx = 0.0, tu = 0.0;
  if (lane < n) {
    tx = __hip_atomic_load(&tt.part_sums[2 * ((int64_t)part0 + first + lane)], __ATOMIC_RELAXED, OB_AGENT);
    tu = __hip_atomic_load(&tt.part_sums[2 * ((int64_t)part0 + first + lane) + 1], __ATOMIC_RELAXED, OB_AGENT);
  }
  tx = wave_sum(tx);
  tu = wave_sum(tu);
  if (!trail_arrive(tt.count + c0 * LINE, (unsigned int)n_sub, &tt.sub_sums[2 * cs], tx, tu)) return;
  const double* sub_sums = tt.sub_sums + 2 * (c0 + 1);
  tx = 0.0; tu = 0.0;
  for (int s = lane; s < n_sub; s += 4 * WAVE) {   // four pairs in flight (the sums are >= +0: adding zeros changes nothing)
    double vx[4], vu[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const bool in = (s + q * WAVE < n_sub);
      vx[q] = in ? __hip_atomic_load(&sub_sums[2 * (s + q * WAVE)], __ATOMIC_RELAXED, OB_AGENT) : 0.0;
      vu[q] = in ? __hip_atomic_load(&sub_sums[2 * (s + q * WAVE) + 1], __ATOMIC_RELAXED, OB_AGENT) : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) { tx += vx[q]; tu += vu[q]; }
  }
  auto plain = [&](int s) {   // written by an earlier kernel
    tx += tt.seg_sums[2 * (int64_t)s];
    tu += tt.seg_sums[2 * (int64_t)s + 1];
  };
  for (int s = lp.a + lane; s < lp.s_first; s += WAVE) plain(s);
  for (int s = lp.s_end + lane; s < lp.b; s += WAVE) plain(s);
  tx = wave_sum(tx);
  tu = wave_sum(tu);
  if (lane == 0) {
    const float c = warmup_coeff_commit(tx, tu, l, ca, wc.coeff_c, wc.c_avg, wc.c_min, wc.c_max, wc.beta3, wc.omb3);
    __hip_atomic_store(&tt.flag[l], (1ull << 32) | (unsigned long long)__float_as_uint(c), __ATOMIC_RELAXED, OB_AGENT);
  }
}

// Bound by HBM and the memory-side cache together (28 bytes per element from one, 12 from the other).  Measured: 1.21e9
// elements in layers of 12.6, 16.8 and 103 M, bf16: 6870 us, in two passes 8000 to 8300 (4350-4740 + 3470-3590); with nothing
// kept 7250.  Parts of 1024, 2048 and 4096 elements: 6860, 6870, 6940.  The same pattern of accesses without
// arithmetic: 6660.
// x is kept in every part, m and v in those with TRAIL_KEEP.  x kept in those only: 1.3e9 elements 7352 us instead of 7346, lists with
// an embedding of 31 M bf16 483.0 instead of 478.5, of 61 M fp32 612.6 instead of 607.6.
template <int GT, bool LPX>
__global__ __launch_bounds__(BLOCK, 8) void k_warmup_trail(
    GradSrc g, float* __restrict__ m, float* __restrict__ v, float* __restrict__ x, TrailTab tt, WarmClip wc,
    float beta1, float omb1, float beta2, float omb2, float eta, float wd, float lr, LayerTab lt,
    void* __restrict__ x_lp, int x_lp_bf16) {
  constexpr int U = TRAIL_U;
  __shared__ double lds[BLOCK / WAVE];
  __shared__ float c_of_layer;
  const unsigned int item = tt.items[blockIdx.x];
  const int part = (int)(item & (TRAIL_KEEP - 1u));
  TilePos p = tile_pos<8 * SPAN>(tt.lt.n_c, tt.lt.tpc, tt.lt.tile_list[part / TRAIL_PARTS]);
  const int sp0 = p.c * tt.lt.tpc_span + (p.t - p.c * tt.lt.tpc) * 8;  // the tile's first span
  const int in_tile = (part % TRAIL_PARTS) * (U * SPAN);
  p.tile0 += in_tile;
  p.len -= in_tile;            // (a short tile may lack its last parts: <= 0)
  if (p.len > U * SPAN) p.len = U * SPAN;
  const int o0 = threadIdx.x * 4;
  v4f M[U], V[U], X[U];
#pragma unroll
  for (int u = 0; u < U; ++u) { M[u] = 0.0f; V[u] = 0.0f; X[u] = 0.0f; }
  const __amdgpu_buffer_rsrc_t rm = part_rsrc(m + p.tile0, U * SPAN * 4), rv = part_rsrc(v + p.tile0, U * SPAN * 4);
  const int l0 = lt.first_layer[sp0];   // the layer the tile lies in (lt.first_layer: of the 1024-element tiling)
  if (item & TRAIL_UPDATE) {
    if (p.len <= 0) return;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int o = u * SPAN + o0;
      if (o < p.len) X[u] = ld4(x + p.tile0 + o);
    }
    if (threadIdx.x == 0)
      c_of_layer = tt.wait ? __uint_as_float((unsigned int)(barrier_wait(&tt.flag[l0], 1u, tt.errflag, tt.spin_limit) & 0xffffffffull))
                           : wc.coeff_c[l0];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int o = u * SPAN + o0;
      if (o < p.len) {
        M[u] = buf_ld4<CACHE_AGENT | CACHE_NT>(rm, 4 * o);
        V[u] = buf_ld4<CACHE_AGENT | CACHE_NT>(rv, 4 * o);
      }
    }
    const float a = lr * c_of_layer;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int o = u * SPAN + o0;
      if (o < p.len) {
        const v4f uu = lamb_u4(M[u], V[u], X[u], eta, wd);
        v4f xn;
#pragma unroll
        for (int k = 0; k < 4; ++k) xn[k] = X[u][k] - a * uu[k];
        st4(x + p.tile0 + o, xn);
        if (LPX) st4_lp(x_lp, p.tile0 + u * SPAN, o0, xn, x_lp_bf16);
      }
    }
    return;
  }
  const bool keep = (item & TRAIL_KEEP) != 0;   // uniform
  const LayerParts lp = layer_parts(tt.lt, l0);
  const int64_t count0 = tt.count0[l0];
  const float ca = wc.c_avg[l0];
  decltype(grad_request<GT>(g, 0)) GR[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    if (o < p.len) {
      GR[u] = grad_request<GT>(g, p.tile0 + o);
      M[u] = ld4(m + p.tile0 + o);
      V[u] = ld4(v + p.tile0 + o);
      X[u] = ld4_keep(x + p.tile0 + o);
    }
  }
  double sx = 0.0, su = 0.0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    if (o < p.len) {
      const v4f G = grad_value(g, GR[u]);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        M[u][k] = beta1 * M[u][k] + omb1 * G[k];
        V[u][k] = beta2 * V[u][k] + omb2 * (G[k] * G[k]);
      }
      if (keep) {
        buf_st4<CACHE_AGENT>(rm, 4 * o, M[u]);
        buf_st4<CACHE_AGENT>(rv, 4 * o, V[u]);
      } else {
        buf_st4<CACHE_AGENT | CACHE_NT>(rm, 4 * o, M[u]);
        buf_st4<CACHE_AGENT | CACHE_NT>(rv, 4 * o, V[u]);
      }
      const v4f uu = lamb_u4(M[u], V[u], X[u], eta, wd);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        sx += (double)X[u][k] * (double)X[u][k];
        su += (double)uu[k] * (double)uu[k];
      }
    }
  }
  payload_before_arrival();   // (every wavefront's stores, before the barriers inside)
  sx = block_sum(sx, lds);
  su = block_sum(su, lds);
  if (threadIdx.x < WAVE) trail_finish(tt, wc, part, l0, lp, count0, ca, sx, su);
}

// ---------------------------------------------------------------------------------------------
// Small lists: eq. (1) of the whole buffer in one launch (see k_ratios_apply_small: same tiles, segments
// and barriers, with the fp64 sums of x^2 and u^2 in place of the maxima).
// Measured: 3.04 M parameters, binary16 gradient: 26 us (37 us in four launches).
// ---------------------------------------------------------------------------------------------
template <int U, int GT, bool LPX, bool TWO_LEVELS>
__global__ __launch_bounds__(BLOCK, small_min_wg(U)) void k_warmup_small(
    GradSrc g, float* __restrict__ m, float* __restrict__ v, float* __restrict__ x, SmallTab sm, WarmClip wc,
    float beta1, float omb1, float beta2, float omb2, float eta, float wd, float lr, LayerTab lt,
    void* __restrict__ x_lp, int x_lp_bf16) {
  constexpr int TILE = SPAN * U;
  extern __shared__ int dyn_lds[];
  __shared__ double lds[BLOCK / WAVE];
  __shared__ double end_sum[2][2];
  __shared__ unsigned long long bc[2];
  __shared__ float c_end[2];
  if ((int)blockIdx.x == sm.n_tiles) {   // the layers without elements
    for (int l = threadIdx.x; l < lt.L; l += BLOCK)
      if (sm.layer_seg0[l + 1] == sm.layer_seg0[l])
        (void)warmup_coeff_commit(0.0, 0.0, l, wc.c_avg[l], wc.coeff_c, wc.c_avg, wc.c_min, wc.c_max, wc.beta3, wc.omb3);
    return;
  }
  const SmallTile ti = sm.tiles[blockIdx.x];
  if (ti.nseg == 0) return;
  TilePos p;
  p.t = (int)blockIdx.x;
  p.c = ti.chunk_kind >> 2;
  const int64_t in_chunk = (int64_t)(p.t - p.c * sm.tpc) * TILE;
  p.tile0 = (int64_t)p.c * sm.n_c + in_chunk;
  p.len = (sm.n_c - in_chunk < TILE) ? (int)(sm.n_c - in_chunk) : TILE;
  const bool inside = (ti.chunk_kind & 1) != 0;
  const int o0 = threadIdx.x * 4;
  v4f G[U], M[U], V[U], X[U], UU[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    G[u] = 0.0f; M[u] = 0.0f; V[u] = 0.0f; X[u] = 0.0f;
    if (o < p.len) {
      G[u] = load_grad<GT>(g, p.tile0 + o);
      M[u] = ld4(m + p.tile0 + o);
      V[u] = ld4(v + p.tile0 + o);
      X[u] = ld4(x + p.tile0 + o);
    }
  }
  float* const val_x = reinterpret_cast<float*>(dyn_lds);     // [TILE] (tiles that meet several layers)
  float* const val_u = val_x + TILE;                          // [TILE]
  SmallSegs sg;
  sg.end = dyn_lds + 2 * TILE; sg.layer = sg.end + sm.max_seg;
  sg.coeff = reinterpret_cast<float*>(sg.layer + sm.max_seg);
  if (!inside) sg.load(sm, ti, p, lt.off);
  // what the last arriver of a layer needs, requested with everything else
  const float ca_end[2] = {wc.c_avg[ti.l0], wc.c_avg[ti.l_last]};
  const int s0_end[2] = {sm.layer_seg0[ti.l0], sm.layer_seg0[ti.l_last]};
  double sx = 0.0, su = 0.0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    UU[u] = 0.0f;
    if (o < p.len) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        M[u][k] = beta1 * M[u][k] + omb1 * G[u][k];
        V[u][k] = beta2 * V[u][k] + omb2 * (G[u][k] * G[u][k]);
      }
      UU[u] = lamb_u4(M[u], V[u], X[u], eta, wd);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (inside) {
          sx += (double)X[u][k] * (double)X[u][k];
          su += (double)UU[u][k] * (double)UU[u][k];
        } else {
          val_x[o + k] = X[u][k];
          val_u[o + k] = UU[u][k];
        }
      }
    }
  }
  const int last_seg = ti.nseg - 1;
  const int n_end = ti.nseg > 1 ? 2 : 1;
  const int l_end[2] = {ti.l0, ti.l_last};
  if (inside) {
    sx = block_sum(sx, lds);
    su = block_sum(su, lds);
    if (threadIdx.x == 0) {
      end_sum[0][0] = sx;
      end_sum[0][1] = su;
    }
  } else {
    __syncthreads();
    const int lane = threadIdx.x & (WAVE - 1);
    for (int s = threadIdx.x / WAVE; s < ti.nseg; s += BLOCK / WAVE) {   // a wavefront per segment
      double tx = 0.0, tu = 0.0;
      for (int o = (s ? sg.end[s - 1] : 0) + lane; o < sg.end[s]; o += WAVE) {
        tx += (double)val_x[o] * (double)val_x[o];
        tu += (double)val_u[o] * (double)val_u[o];
      }
      tx = wave_sum(tx);
      tu = wave_sum(tu);
      if (lane == 0) {
        if (s == 0 || s == last_seg) {
          const int e = (s == 0) ? 0 : 1;
          end_sum[e][0] = tx;
          end_sum[e][1] = tu;
        } else {   // the layer lies inside the tile
          const int l = sg.layer[s];
          sg.coeff[s] = warmup_coeff_commit(tx, tu, l, wc.c_avg[l], wc.coeff_c, wc.c_avg, wc.c_min, wc.c_max,
                                            wc.beta3, wc.omb3);
        }
      }
    }
  }
  __syncthreads();
  double* const partial = static_cast<double*>(sm.partial);
  small_arrive<TWO_LEVELS>(sm, lt.L, ti, n_end, s0_end, bc, [&](int e) {
    double* q = partial + 2 * (int64_t)(ti.seg0 + (e ? last_seg : 0));
    __hip_atomic_store(q, end_sum[e][0], __ATOMIC_RELAXED, OB_AGENT);
    __hip_atomic_store(q + 1, end_sum[e][1], __ATOMIC_RELAXED, OB_AGENT);
  });
  for (int e = 0; e < n_end; ++e) {   // (uniform)
    if ((bc[e] & 3ull) == 0ull) continue;
    const int l = l_end[e], s0 = s0_end[e], s1 = s0 + (e ? ti.n_last : ti.n_first);
    double tx = end_sum[e][0], tu = end_sum[e][1];
    if (bc[e] & 1ull) {
      tx = 0.0; tu = 0.0;
      for (int s = s0 + threadIdx.x; s < s1; s += BLOCK) {
        tx += __hip_atomic_load(&partial[2 * (int64_t)s], __ATOMIC_RELAXED, OB_AGENT);
        tu += __hip_atomic_load(&partial[2 * (int64_t)s + 1], __ATOMIC_RELAXED, OB_AGENT);
      }
      tx = block_sum(tx, lds);
      tu = block_sum(tu, lds);
    }
    if (threadIdx.x == 0) {
      const float c = warmup_coeff_commit(tx, tu, l, ca_end[e], wc.coeff_c, wc.c_avg, wc.c_min, wc.c_max, wc.beta3,
                                          wc.omb3);
      c_end[e] = c;
      if (bc[e] & 1ull)
        (void)barrier_publish(&sm.flag[(int64_t)l * CTR_STRIDE], &sm.counter[(int64_t)l * CTR_STRIDE], s1 - s0,
                              (unsigned int)(bc[e] >> 32), __float_as_uint(c), small_one_level<TWO_LEVELS>());
    }
  }
  // while the layers complete: the moments are stored
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    if (o < p.len) {
      if (inside) {
        st4(m + p.tile0 + o, M[u]);
        st4(v + p.tile0 + o, V[u]);
      } else {
        const int end = sg.end[last_seg];
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (o + k < end) {
            m[p.tile0 + o + k] = M[u][k];
            v[p.tile0 + o + k] = V[u][k];
          }
      }
    }
  }
  {
    const int e = threadIdx.x / WAVE;
    if (e < n_end && (threadIdx.x & (WAVE - 1)) == 0 && (bc[e] & 2ull) == 0ull) {
      const unsigned long long f = barrier_wait<SMALL_POLL_SLEEP>(&sm.flag[(int64_t)l_end[e] * CTR_STRIDE], (unsigned int)(bc[e] >> 32),
                                                sm.errflag, sm.spin_limit);
      c_end[e] = __uint_as_float((unsigned int)(f & 0xffffffffull));
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int o = u * SPAN + o0;
    if (o < p.len) {
      if (inside) {
        const float a = lr * c_end[0];
        v4f xn;
#pragma unroll
        for (int k = 0; k < 4; ++k) xn[k] = X[u][k] - a * UU[u][k];
        st4(x + p.tile0 + o, xn);
        if (LPX) st4_lp(x_lp, p.tile0 + u * SPAN, o0, xn, x_lp_bf16);
      } else {
        int s = sg.find(ti.nseg, o);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          while (s < ti.nseg && o + k >= sg.end[s]) ++s;
          if (s < ti.nseg) {
            const float c = (s == 0) ? c_end[0] : (s == last_seg) ? c_end[1] : sg.coeff[s];
            const float xn = X[u][k] - (lr * c) * UU[u][k];
            x[p.tile0 + o + k] = xn;
            if (LPX) reinterpret_cast<unsigned short*>(x_lp)[p.tile0 + o + k] = float_to_lp(xn, x_lp_bf16);
          }
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Momentum-scale coefficients of Appendix A.5.2, formed once at the end of warmup.  The paper gives
// no formula; the reading taken: sigma_l = ||m_l||_2/sqrt(n_l), k_l = mean_l(sigma_l)/sigma_l over
// the non-empty layers, 1 where sigma_l = 0 or the layer is empty (every layer's RMS becomes the
// mean RMS before the fused buffer is compressed).
//   a: per (tile, layer) segment the fp64 sum of m^2
//   b: one workgroup: per-layer sigma, their mean (fixed order), k_l
// ---------------------------------------------------------------------------------------------
// A workgroup takes R consecutive tiles of the 1024-element tiling (the segment tables are the
// plain kernels'), looks up what it needs to know about all of them, then requests all of them,
// then reduces them one by one: with one 128-bit load per thread in flight, and the table look-ups
// of a tile that meets a layer boundary (three dependent loads) made for every tile after its data
// had arrived, the kernel ran at half the streaming rate.
template <int R>
__global__ __launch_bounds__(BLOCK) void k_momentum_sumsq(const float* __restrict__ m,
                                                          double* __restrict__ seg_sums,
                                                          int64_t n_c, int tpc, int n_tiles, LayerTab lt,
                                                          const int* __restrict__ tile_seg0,
                                                          const int* __restrict__ seg_layer) {
  __shared__ double lds[BLOCK / WAVE];
  const int o = threadIdx.x * 4;
  const int t0 = (int)blockIdx.x * R;
  TilePos P[R];
  int l0[R], s0[R];
  int64_t end0[R];       // end of the layer the tile starts in
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int t = (t0 + r < n_tiles) ? t0 + r : n_tiles - 1;   // (a repeated last tile is skipped below)
    P[r] = tile_pos<SPAN>(n_c, tpc, t);
    l0[r] = lt.first_layer[t];
    s0[r] = tile_seg0[t];
  }
#pragma unroll
  for (int r = 0; r < R; ++r) end0[r] = lt.off[l0[r] + 1];   // off has L+2 entries
  v4f M[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    M[r] = 0.0f;
    if (t0 + r < n_tiles && l0[r] < lt.L && o < P[r].len) M[r] = ld4(m + P[r].tile0 + o);
  }
  // the usual case: all R tiles lie inside one and the same layer -- one reduction for all of them;
  // the sum goes to the first tile's segment and the other segments contribute 0 to the layer
  bool together = (t0 + R <= n_tiles) && (l0[0] < lt.L);
#pragma unroll
  for (int r = 0; r < R; ++r)
    together = together && (l0[r] == l0[0]) && (P[r].len == SPAN) && (P[r].tile0 + SPAN <= end0[r]);
  if (together) {   // uniform
    double acc = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int k = 0; k < 4; ++k) acc += (double)M[r][k] * (double)M[r][k];
    acc = block_sum(acc, lds);
    if (threadIdx.x == 0) {
      seg_sums[s0[0]] = acc;
#pragma unroll
      for (int r = 1; r < R; ++r) seg_sums[s0[r]] = 0.0;
    }
    return;
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (t0 + r >= n_tiles) break;          // uniform
    if (l0[r] >= lt.L) continue;           // uniform: the tile lies in the padding (it has no segment)
    const TilePos& p = P[r];
    if (p.tile0 + p.len <= end0[r]) {      // uniform: the tile lies inside one layer, its one segment
      double acc = 0.0;
      if (o < p.len) {
#pragma unroll
        for (int k = 0; k < 4; ++k) acc += (double)M[r][k] * (double)M[r][k];
      }
      acc = block_sum(acc, lds);
      if (threadIdx.x == 0) seg_sums[s0[r]] = acc;
      continue;
    }
    const int s1 = tile_seg0[p.t + 1];
    for (int s = s0[r]; s < s1; ++s) {
      const int l = seg_layer[s];
      const int64_t a = lt.off[l], b = lt.off[l + 1];
      double acc = 0.0;
      if (o < p.len) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int64_t i = p.tile0 + o + k;
          if (i >= a && i < b) acc += (double)M[r][k] * (double)M[r][k];
        }
      }
      acc = block_sum(acc, lds);
      if (threadIdx.x == 0) seg_sums[s] = acc;
    }
  }
}

// sigma[l] (fp64 scratch, [L]) from the segment sums; one workgroup per layer.
__global__ __launch_bounds__(FBLOCK) void k_layer_rms(const double* __restrict__ seg_sums,
                                                      const int* __restrict__ layer_seg0,
                                                      const int64_t* __restrict__ off,
                                                      double* __restrict__ sigma) {
  __shared__ double lds[FBLOCK / WAVE];
  const int l = blockIdx.x;
  double a = 0.0;
  const int s1 = layer_seg0[l + 1];
  for (int s = layer_seg0[l] + threadIdx.x; s < s1; s += 4 * FBLOCK) {   // four loads in flight per thread
    double v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = (s + u * FBLOCK < s1) ? seg_sums[s + u * FBLOCK] : 0.0;
#pragma unroll
    for (int u = 0; u < 4; ++u) a += v[u];
  }
  a = block_sum<FBLOCK>(a, lds);
  if (threadIdx.x == 0) {
    const int64_t n = off[l + 1] - off[l];
    sigma[l] = (n > 0) ? sqrt(a / (double)n) : 0.0;
  }
}

// mean of sigma over the non-empty layers (one workgroup, fixed order), then k_l.
__global__ __launch_bounds__(FBLOCK) void k_momentum_scale(const double* __restrict__ sigma,
                                                           const int64_t* __restrict__ off, int L,
                                                           float* __restrict__ mom_scale) {
  __shared__ double lds[FBLOCK / WAVE];
  __shared__ double mean_s;
  double a = 0.0, cnt = 0.0;
  for (int l = threadIdx.x; l < L; l += FBLOCK) {
    if (off[l + 1] > off[l]) {
      a += sigma[l];
      cnt += 1.0;
    }
  }
  a = block_sum<FBLOCK>(a, lds);
  cnt = block_sum<FBLOCK>(cnt, lds);
  if (threadIdx.x == 0) mean_s = (cnt > 0.0) ? a / cnt : 0.0;
  __syncthreads();
  const double mean = mean_s;
  for (int l = threadIdx.x; l < L; l += FBLOCK) {
    const double s = sigma[l];
    mom_scale[l] = (s > 0.0) ? (float)(mean / s) : 1.0f;
  }
}

// Diagnostics: a plain streaming copy in the shape of the N-sized kernels above (1024-element
// tiles, one 128-bit nontemporal load and store per thread).  What it reaches is the device's
// practical streaming ceiling, against which the benchmark reports every kernel next to the
// published peak.
__global__ __launch_bounds__(BLOCK) void k_diag_copy(const float* __restrict__ src, float* __restrict__ dst,
                                                     int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * SPAN + threadIdx.x * 4;
  if (i + 4 <= n) {
    st4(dst + i, ld4(src + i));
  } else {
    for (int64_t j = i; j < n; ++j) dst[j] = src[j];
  }
}

__global__ __launch_bounds__(BLOCK) void k_fill(float* __restrict__ p, int64_t n, float v) {
  const int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (i < n) p[i] = v;
}

}  // namespace obk
