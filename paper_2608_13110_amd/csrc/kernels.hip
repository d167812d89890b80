// HIP kernels for gfx950 (CDNA4) of the temporal-boundary contraction.
//
//  k_init     row-0 build-up of the boundary tensor (one write pass)
//  k_resolve  per-batch choice of every update's matrix variant
//  k_pass     one fused window of staircase updates over every tile of the
//             boundary tensor (the hot loop); in place, HBM-streaming
//  k_late_*   the folded late-phase contraction: the Alg. 2 join and the late
//             layers, FP64 accumulation (k_late_mf on FP64 matrix cores,
//             k_late_dot and k_late_out for narrow products), and k_late_ops,
//             the rest of the late program
//  k_one      all of it in one launch for tensors of up to 2^12 entries
//  k_win      the pass over tensors too small to fill the chip
//  k_fold     the join matrix with late removals folded in, once per plan
//  k_logxeb   FP64 log-XEB reduction; samplers
//
// The kernels of the amplitude path are recorded as launches (Launch, see
// kernels.hpp) before they run.  Each such kernel has a body taking its block
// index explicitly, a plain entry point, and (complex64 path) a grouped entry
// point that runs segment blockIdx.z of a table of (argument, grid) segments:
// launches of one kernel for different requests merged into one.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cstdio>
#include <cstring>
#include <vector>

#include "kernels.hpp"

namespace tnc {

// The segment of a grouped launch that this block belongs to, or null when
// the block lies outside its segment's own grid.
template <class A>
__device__ __attribute__((always_inline)) inline const Seg<A>* group_seg(const Seg<A>* segs) {
  const Seg<A>* s = segs + blockIdx.z;
  if (blockIdx.x >= s->gx || blockIdx.y >= s->gy) return nullptr;
  return s;
}

// ---------------------------------------------------------------------------
// Row-0 build-up.  The first row only creates slots: its boundary tensor is
// the product  v[a_0] * prod_{j>=1} seg_j[a_j][a_{j-1}] * f_x[a_{m-1}]
// (copy tensors of the down-bonds joined by the one-qubit segments).
// For h >= 11 each wave writes 2048 consecutive entries, lane l taking the
// entries 64 e + l (e < 32): every store is one contiguous 512-byte run, and
// the factors of bits 0..5 (the lane) and >= 11 (the wave) are multiplied
// once per thread, those of bits 6..10 per entry.  Entries above 2^m are
// zero.
__device__ inline double2 zmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

__device__ __attribute__((always_inline)) inline void init_body(const InitArgs& a, uint32_t bx) {
  __shared__ double2 seg[4 * 64];
  const int nseg = a.m0 - 1;
  for (int i = threadIdx.x; i < 4 * nseg; i += blockDim.x) seg[i] = a.seg[i];
  __syncthreads();
  const int m = a.m0;
  const long long gid = (long long)bx * blockDim.x + threadIdx.x;
  auto sg = [&](int j, unsigned long long i) {
    return seg[4 * (j - 1) + 2 * (int)((i >> j) & 1ull) + (int)((i >> (j - 1)) & 1ull)];
  };
  if (a.h < 11) {
    const long long total = (long long)a.n_batches << a.h;
    if (gid >= total) return;
    const long long batch = gid >> a.h;
    const unsigned long long i = (unsigned long long)gid & ((1ull << a.h) - 1ull);
    float2* out = a.B + gid;
    if (i >> m) {
      *out = make_float2(0.f, 0.f);
      return;
    }
    const int x0 = a.bits[batch * a.n];
    double2 val = a.v[i & 1ull];
    for (int j = 1; j < m; ++j) val = zmul(val, sg(j, i));
    val = zmul(val, a.f[x0][(i >> (m - 1)) & 1ull]);
    *out = make_float2((float)val.x, (float)val.y);
    return;
  }
  const long long wave = gid >> 6;
  const unsigned long long lane = (unsigned long long)(gid & 63);
  if (wave >= (((long long)a.n_batches << a.h) >> 11)) return;
  const long long first = wave << 11;
  const long long batch = first >> a.h;
  const unsigned long long i0 = ((unsigned long long)first & ((1ull << a.h) - 1ull)) | lane;
  float2* out = a.B + first + (long long)lane;
  const int x0 = a.bits[batch * a.n];
  // factors fixed for the thread: bits 0..5 (lane) and >= 11 (wave)
  double2 fixed = a.v[lane & 1ull];
  for (int j = 1; j < m && j <= 5; ++j) fixed = zmul(fixed, sg(j, i0));
  for (int j = 12; j < m; ++j) fixed = zmul(fixed, sg(j, i0));
  const bool f_var = m - 1 >= 6 && m - 1 <= 10;
  if (!f_var) fixed = zmul(fixed, a.f[x0][(i0 >> (m - 1)) & 1ull]);
  const int jhi = m - 1 < 11 ? m - 1 : 11;
  for (int e = 0; e < 32; ++e) {
    const unsigned long long i = i0 + ((unsigned long long)e << 6);
    if (i >> m) {
      out[e << 6] = make_float2(0.f, 0.f);
      continue;
    }
    double2 val = fixed;
    for (int j = 6; j <= jhi; ++j) val = zmul(val, sg(j, i));
    if (f_var) val = zmul(val, a.f[x0][(i >> (m - 1)) & 1ull]);
    out[e << 6] = make_float2((float)val.x, (float)val.y);
  }
}

__global__ __launch_bounds__(kBlock) void k_init(InitArgs a) { init_body(a, blockIdx.x); }

__global__ __launch_bounds__(kBlock) void k_init_g(const Seg<InitArgs>* __restrict__ segs) {
  const Seg<InitArgs>* s = group_seg(segs);
  if (!s) return;
  const InitArgs a = s->a;
  init_body(a, blockIdx.x);
}

// Row-0 build-up into 16-bit block-scaled storage: one workgroup per block
// of 2^blk_bits consecutive entries (the scale block of this writer); the
// FP64 product is rounded to FP32 as in the complex64 path, then the block
// maximum fixes the power-of-two scale.
template <int S>
__global__ __launch_bounds__(kBlock) void k_init16(InitArgs a) {
  constexpr int kMaxPer = 4096 / kBlock;
  __shared__ double2 seg[4 * 64];
  __shared__ uint32_t smax;
  const int nseg = a.m0 - 1;
  for (int i = threadIdx.x; i < 4 * nseg; i += blockDim.x) seg[i] = a.seg[i];
  if (threadIdx.x == 0) smax = 0u;
  __syncthreads();
  const int bb = a.blk_bits;
  const int per_batch_blocks_log = a.h - bb;
  const long long batch = (long long)blockIdx.x >> per_batch_blocks_log;
  const unsigned long long sblk = (unsigned long long)blockIdx.x & ((1ull << per_batch_blocks_log) - 1ull);
  const unsigned long long i0 = sblk << bb;
  const int nper = 1 << bb;
  const int x0 = a.bits[batch * a.n];
  const int m = a.m0;
  float2 val[kMaxPer];
  float amax = 0.f;
#pragma unroll
  for (int q = 0; q < kMaxPer; ++q) {
    const int off = q * kBlock + (int)threadIdx.x;
    val[q] = make_float2(0.f, 0.f);
    if (off >= nper) continue;
    const unsigned long long i = i0 + (unsigned long long)off;
    if (i >> m) continue;
    double2 v = a.v[i & 1ull];
    for (int j = 1; j < m; ++j) {
      const int aj = (int)((i >> j) & 1ull), ajm = (int)((i >> (j - 1)) & 1ull);
      v = zmul(v, seg[4 * (j - 1) + 2 * aj + ajm]);
    }
    v = zmul(v, a.f[x0][(i >> (m - 1)) & 1ull]);
    val[q] = make_float2((float)v.x, (float)v.y);
    amax = fmaxf(amax, fmaxf(fabsf(val[q].x), fabsf(val[q].y)));
  }
  if (amax > 0.f) atomicMax(&smax, __float_as_uint(amax));
  __syncthreads();
  const int e = block_exponent(__uint_as_float(smax));
  const float inv = ldexpf(1.f, -e);
  uint32_t* out = reinterpret_cast<uint32_t*>(a.B) + (batch << a.h) + i0;
#pragma unroll
  for (int q = 0; q < kMaxPer; ++q) {
    const int off = q * kBlock + (int)threadIdx.x;
    if (off < nper) out[off] = pack16<S>(val[q].x, val[q].y, inv);
  }
  if (threadIdx.x == 0) a.scale_out[batch * a.scale_stride + (long long)sblk] = ldexpf(1.f, e);
}

// ---------------------------------------------------------------------------
// Variant resolution: every op's matrix pair for each batch of the group,
// picked once from the batch's output bits, so the pass kernels read their
// matrices at addresses that depend on the op only.
__device__ __attribute__((always_inline)) inline void resolve_body(const ResolveArgs& a, uint32_t bx) {
  const long long gid = (long long)bx * blockDim.x + threadIdx.x;
  const long long total = (long long)a.n_batches * a.n_ops;
  if (gid >= total) return;
  const int b = (int)(gid / a.n_ops);
  const int o = (int)(gid - (long long)b * a.n_ops);
  const DevOp op = a.ops[o];
  const uint8_t* x = a.bits + (size_t)b * a.n;
  const int var = (op.xrow0 >= 0 ? 2 * (x[op.xrow0] & 1) : 0) + (op.xrow1 >= 0 ? (x[op.xrow1] & 1) : 0);
  const float4* src = reinterpret_cast<const float4*>(a.mats + ((size_t)op.mat * 4 + var) * 16);
  float4* dst = reinterpret_cast<float4*>(a.rmats + (size_t)b * a.rstride + (size_t)o * 16);
#pragma unroll
  for (int q = 0; q < 4; ++q) dst[q] = src[q];
}

__global__ __launch_bounds__(kBlock) void k_resolve(ResolveArgs a) { resolve_body(a, blockIdx.x); }

__global__ __launch_bounds__(kBlock) void k_resolve_g(const Seg<ResolveArgs>* __restrict__ segs) {
  const Seg<ResolveArgs>* s = group_seg(segs);
  if (!s) return;
  const ResolveArgs a = s->a;
  resolve_body(a, blockIdx.x);
}

// ---------------------------------------------------------------------------
// The pass kernel.  A tile is 2^T entries of one batch's boundary tensor: the
// global slots [0, lo_bits) and [win_lo, win_lo + win_len).  A block holds
// one tile (T - R = 8 thread bits with 256 threads, 9 with 512) or several
// small ones.  Data path:
//   HBM -> LDS with 16-byte accesses along the contiguous low slots,
//   per phase: LDS -> registers (2^R entries per thread, the phase's target
//   slots as register bits), the phase's updates in registers, registers ->
//   LDS,
//   LDS -> HBM, in place.
// WU: every wave lies inside one tile (one tile per block, or T - R >= 6),
// so the batch and everything read through it are wave-uniform; such
// kernels also run the fused matrix-core phases.
// NT: threads per block (256; 512 for one 2^(R+9)-entry tile per block).
// Resident waves per SIMD the register allocation must allow.  LDS admits five
// 32 KiB blocks of small 16-entry tiles (T - R < 6) per CU, but five waves leave
// 96 registers, and the updates' fused operations need 124: what went to scratch
// cost more than the fifth wave gives.  ms of the passes over the five-slot window
// of a call at w = 24 (59 qubits, k = 8, two batches), five / four / three waves:
// 6.60 / 3.88 / 3.88 (4.74 before the operations were spelled out, with 24 bytes of
// scratch at five), in FP16 at w = 23 (13 batches) 25.0 / 12.4 / 12.8 (20.3).
// Eight-entry complex64 tiles of that kind took 64 registers and eight waves before
// and 75 and six with the fused operations: asked for seven waves they take 72 and no
// scratch (passes of a call at w = 19, 9 batches, 2^7-entry tiles: 1.31 ms, 1.46
// and 1.37; eight waves 1.82, with scratch).  Fused phases keep two.
template <int R, bool WU, int NT, bool C64>
constexpr int pass_waves_per_eu() {
  return WU ? 2 : NT != 256 ? 1 : R == 4 ? 4 : R == 3 && C64 ? 7 : 1;
}

// Blocks are dispatched round-robin over the 8 XCDs; each XCD takes a
// contiguous range of tiles instead, so the blocks in flight on one XCD read
// and write neighbouring runs (measured: 3.7 % more bandwidth on the loads
// and stores alone, about 1 % per pass).
__device__ __attribute__((always_inline)) inline unsigned xcd_block(uint32_t bx, uint32_t gx) {
  return (gx & 7u) == 0u ? (bx & 7u) * (gx >> 3) + (bx >> 3) : bx;
}

// Tensors far larger than the 256 MiB last-level cache are read and written once
// per pass, so their lines are marked as not to be kept (Stream, record_pass): a
// call at w = 28 (2 GiB, k = 8) 139.0 -> 134.5 ms (writes alone 137.3), at w = 30
// (k = 0, 30 qubits) 323 -> 303 ms.  At 1 GiB the marks change nothing (w = 27:
// 39.8 ms both ways), at 256 MiB, where the cache serves the next pass, they cost
// 7 % (bond four, w = 25: 5.39 -> 5.75 ms).  Runs below 128 bytes need the cache to
// join them (128 batches at w = 20, 64-byte runs: 24.7 -> 26.7 ms).
typedef float tnc_f4 __attribute__((ext_vector_type(4)));
typedef uint32_t tnc_u4 __attribute__((ext_vector_type(4)));
template <bool Stream>
__device__ __attribute__((always_inline)) inline float4 hbm_get(const float2* p) {
  if constexpr (Stream) {
    const tnc_f4 v = __builtin_nontemporal_load(reinterpret_cast<const tnc_f4*>(p));
    return make_float4(v.x, v.y, v.z, v.w);
  }
  return *reinterpret_cast<const float4*>(p);
}
template <bool Stream>
__device__ __attribute__((always_inline)) inline void hbm_put(float2* p, float4 v) {
  if constexpr (Stream) __builtin_nontemporal_store(tnc_f4{v.x, v.y, v.z, v.w}, reinterpret_cast<tnc_f4*>(p));
  else *reinterpret_cast<float4*>(p) = v;
}

// LDS slots of the iteration parts it << shift (it < 32) of the entries a
// thread stages: swz is linear, so the slot of it << shift is the XOR of the
// slots of its set bits, taken from five values computed once per thread.
struct IterSlots {
  uint32_t b[5];
  __device__ __attribute__((always_inline)) explicit IterSlots(int shift) {
#pragma unroll
    for (int q = 0; q < 5; ++q) b[q] = swz(1u << (shift + q));
  }
  // `it` is a compile-time constant in the unrolled staging loops
  __device__ __attribute__((always_inline)) uint32_t of(int it) const {
    uint32_t s = 0;
#pragma unroll
    for (int q = 0; q < 5; ++q)
      if ((it >> q) & 1) s ^= b[q];
    return s;
  }
};

template <int R, bool MULTI, bool WU, int NT, int KIND, bool Stream>
__device__ __attribute__((always_inline)) inline void pass_body(const PassArgs& a, float2* lds, uint32_t bx,
                                                                uint32_t gx) {
  constexpr int E = 1 << R;
  const int T = a.T;
  const int TB = T - R;
  const int tid = threadIdx.x;
  const int tile_in_block = MULTI ? (tid >> TB) : 0;
  const uint32_t tt = MULTI ? (uint32_t)(tid & ((1 << TB) - 1)) : (uint32_t)tid;
  const int tiles_per_block = MULTI ? (NT >> TB) : 1;
  const long long tile = (long long)xcd_block(bx, gx) * tiles_per_block + tile_in_block;
  const bool active = tile < a.n_tiles;
  const int tbits = a.h - T;
  long long batch = active ? (tile >> tbits) : 0;
  if constexpr (WU) batch = __builtin_amdgcn_readfirstlane((int)batch);
  const unsigned long long blk = active ? ((unsigned long long)tile & ((1ull << tbits) - 1ull)) : 0ull;
  float2* __restrict__ Bt = a.B + (batch << a.h) + block_offset(blk, a.lo_bits, a.win_lo, a.win_len);
  char* region = reinterpret_cast<char*>(lds) + ((size_t)tile_in_block << (T + 3));
  const int tpt = 1 << TB;

  // LDS slot of entry i = (it * tpt + tt) * 2: the thread part and the
  // (wave-uniform) iteration part occupy disjoint bits, so their slots XOR;
  // the iteration part's slot is the XOR of the slots of its set bits
  const uint32_t st = swz(tt * 2u);
  const IterSlots isl(TB + 1);
  if (active) {
    // every load in flight before the first LDS write
    float4 ld[E / 2];
#pragma unroll
    for (int it = 0; it < E / 2; ++it) {
      const uint32_t i = (uint32_t)(it * tpt + (int)tt) * 2u;
      ld[it] = hbm_get<Stream>(Bt + tile_offset(i, a.lo_bits, a.win_lo));
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int it = 0; it < E / 2; ++it) {
      const uint32_t si = isl.of(it) ^ st;
      *reinterpret_cast<float4*>(region + pair_slot(si)) = pair_order(ld[it], pair_swapped(si));
    }
  }
  __syncthreads();

  PhaseCtx<R> ctx;
  ctx.rm = (const TNC_TBL float*)(a.rmats + (size_t)batch * a.rstride);
  ctx.tb = 0;
  ctx.uniform = WU;
  // the phases address the LDS by whole LDS addresses: the tile's region
  // base with the array's own address ORed in (the pass kernels declare no
  // static LDS, so the dynamic array starts at LDS address 0)
  const uint32_t rbase = lds_address(lds) | ((uint32_t)tile_in_block << (T + 3));
  for (int p = 0; p < a.n_phases; ++p) {
    const DevPhase P = load_phase(a.phases, p);
    phase_dispatch<R, WU, KIND>(reinterpret_cast<char*>(lds), rbase, P, (const TNC_TBL uint32_t*)a.poffs + p * kPhaseOffs,
                          ctx, tt, TB, a.fmats + (size_t)p * kFusedWords);
    __syncthreads();
  }

  if (active) {
#pragma unroll
    for (int it = 0; it < E / 2; ++it) {
      const uint32_t i = (uint32_t)(it * tpt + (int)tt) * 2u;
      const uint32_t si = isl.of(it) ^ st;
      const float4 val = *reinterpret_cast<const float4*>(region + pair_slot(si));
      hbm_put<Stream>(Bt + tile_offset(i, a.lo_bits, a.win_lo), pair_order(val, pair_swapped(si)));
    }
  }
}

// KIND 0: the bond-two phase forms (staircases, DUP, fused); KIND 1: the
// bond-four ones (dense phases and single uncontrolled updates).
template <int R, bool MULTI, bool WU, int NT = kBlock, int KIND = 0, bool Stream = false>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(pass_waves_per_eu<R, WU, NT, KIND == 0>()))) void k_pass(
    PassArgs a) {
  extern __shared__ float2 lds[];
  pass_body<R, MULTI, WU, NT, KIND, Stream>(a, lds, blockIdx.x, gridDim.x);
}

template <int R, bool MULTI, bool WU, int NT = kBlock, int KIND = 0>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(pass_waves_per_eu<R, WU, NT, KIND == 0>()))) void k_pass_g(
    const Seg<PassArgs>* __restrict__ segs) {
  extern __shared__ float2 lds[];
  const Seg<PassArgs>* s = group_seg(segs);
  if (!s) return;
  const PassArgs a = s->a;
  pass_body<R, MULTI, WU, NT, KIND, false>(a, lds, blockIdx.x, s->gx);
}

// The pass kernel on 16-bit block-scaled storage: the same tiles, phases,
// block shapes and XCD-contiguous tile order as k_pass, with the entries
// decoded (value = stored x block scale of the previous writer) on the way
// into LDS, and re-encoded on the way out with a fresh power-of-two scale
// per block of this pass's tiles (taken from the block's largest component
// after the pass).  4 entries (16 bytes) per HBM access, 2 when a thread
// holds only 2 entries.
template <int R, bool MULTI, int S, bool WU, int NT = kBlock, int KIND = 0>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(pass_waves_per_eu<R, WU, NT, false>()))) void k_pass16(
    PassArgs a) {
  extern __shared__ float2 lds[];
  constexpr int E = 1 << R;
  constexpr int U = E >= 4 ? 4 : 2;
  const int T = a.T;
  const int TB = T - R;
  const int tid = threadIdx.x;
  const int tile_in_block = MULTI ? (tid >> TB) : 0;
  const uint32_t tt = MULTI ? (uint32_t)(tid & ((1 << TB) - 1)) : (uint32_t)tid;
  const int tiles_per_block = MULTI ? (NT >> TB) : 1;
  const long long tile = (long long)xcd_block(blockIdx.x, gridDim.x) * tiles_per_block + tile_in_block;
  const bool active = tile < a.n_tiles;
  const int tbits = a.h - T;
  long long batch = active ? (tile >> tbits) : 0;
  if constexpr (WU) batch = __builtin_amdgcn_readfirstlane((int)batch);
  const unsigned long long blk = active ? ((unsigned long long)tile & ((1ull << tbits) - 1ull)) : 0ull;
  const uint64_t boff = block_offset(blk, a.lo_bits, a.win_lo, a.win_len);
  uint32_t* __restrict__ Bw = reinterpret_cast<uint32_t*>(a.B) + (batch << a.h);
  const float* __restrict__ sin = a.scale_in + batch * a.scale_stride;
  char* region = reinterpret_cast<char*>(lds) + ((size_t)tile_in_block << (T + 3));
  uint32_t* smax = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(lds) + ((size_t)tiles_per_block << (T + 3)));
  const int tpt = 1 << TB;
  const int blk_bits = T < 12 ? T : 12;
  const int nblk = 1 << (T - blk_bits);  // scale blocks per tile (1, 2 or 4)
  if (tid < nblk * tiles_per_block) smax[tid] = 0u;

  // A scale slot gathers bit fields of the entry index, and the block part
  // (boff), the thread part (tt) and the iteration part (it) of an entry's
  // index occupy disjoint bits, so its slot is the OR of the three parts'
  // slots; the iteration part is the same for every thread (scalar work).
  const uint64_t slot_t = scale_slot(boff, a.in_map) |
                          scale_slot(tile_offset(tt * (uint32_t)U, a.lo_bits, a.win_lo), a.in_map);
  const uint32_t st = swz(tt * (uint32_t)U);  // LDS slot of the thread part (see k_pass)
  const IterSlots isl(TB + (U == 4 ? 2 : 1));
  if (active) {
    // every load (and its scale) in flight before the first LDS write
    uint4 ld[E / U];
    float scl[E / U];
#pragma unroll
    for (int it = 0; it < E / U; ++it) {
      const uint32_t i = (uint32_t)(it * tpt + (int)tt) * (uint32_t)U;
      const uint64_t g = boff + tile_offset(i, a.lo_bits, a.win_lo);
      const uint64_t slot_i = scale_slot(tile_offset((uint32_t)(it * tpt) * (uint32_t)U, a.lo_bits, a.win_lo), a.in_map);
      scl[it] = sin[slot_t | slot_i];
      if constexpr (U == 4) {
        ld[it] = *reinterpret_cast<const uint4*>(Bw + g);
      } else {
        const uint2 w = *reinterpret_cast<const uint2*>(Bw + g);
        ld[it] = make_uint4(w.x, w.y, 0u, 0u);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int it = 0; it < E / U; ++it) {
      const float sc = scl[it];
      const uint32_t si = isl.of(it) ^ st;  // swz(i); swz(i + 2) = si ^ 2
      const uint4 w = ld[it];
      const float2 e0 = unpack16<S>(w.x, sc), e1 = unpack16<S>(w.y, sc);
      *reinterpret_cast<float4*>(region + pair_slot(si)) =
          pair_order(make_float4(e0.x, e0.y, e1.x, e1.y), pair_swapped(si));
      if constexpr (U == 4) {
        const float2 e2 = unpack16<S>(w.z, sc), e3 = unpack16<S>(w.w, sc);
        *reinterpret_cast<float4*>(region + pair_slot(si ^ 2u)) =
            pair_order(make_float4(e2.x, e2.y, e3.x, e3.y), pair_swapped(si));
      }
    }
  }
  __syncthreads();

  PhaseCtx<R> ctx;
  ctx.rm = (const TNC_TBL float*)(a.rmats + (size_t)batch * a.rstride);
  ctx.tb = 0;
  ctx.uniform = WU;
  for (int p = 0; p < a.n_phases; ++p) {
    const DevPhase P = load_phase(a.phases, p);
    phase_dispatch<R, WU, KIND>(reinterpret_cast<char*>(lds), lds_address(lds) | ((uint32_t)tile_in_block << (T + 3)), P,
                          (const TNC_TBL uint32_t*)a.poffs + p * kPhaseOffs, ctx, tt, TB,
                          a.fmats + (size_t)p * kFusedWords);
    __syncthreads();
  }

  // largest component of each scale block of the tile (the blocks are the
  // tile's highest local bits, so a thread's entries fall in the block of
  // their iteration part: one running maximum per block)
  if (active) {
    float m[4] = {0.f, 0.f, 0.f, 0.f};
    const uint32_t st2 = swz(tt * 2u);
    const IterSlots isl2(TB + 1);
#pragma unroll
    for (int it = 0; it < E / 2; ++it) {
      const uint32_t i = (uint32_t)(it * tpt + (int)tt) * 2u;
      const float4 v = *reinterpret_cast<const float4*>(region + pair_slot(isl2.of(it) ^ st2));  // order irrelevant
      const float am = fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w)));
      const uint32_t q = (i >> blk_bits) & 3u;
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (q == (uint32_t)c) m[c] = fmaxf(m[c], am);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (c < nblk && m[c] > 0.f) atomicMax(&smax[nblk * tile_in_block + c], __float_as_uint(m[c]));
  }
  __syncthreads();
  if (active) {
    float inv[4];
#pragma unroll
    for (int c = 0; c < 4; ++c)
      inv[c] = c < nblk ? ldexpf(1.f, -block_exponent(__uint_as_float(smax[nblk * tile_in_block + c]))) : 1.f;
#pragma unroll
    for (int it = 0; it < E / U; ++it) {
      const uint32_t i = (uint32_t)(it * tpt + (int)tt) * (uint32_t)U;
      const uint64_t g = boff + tile_offset(i, a.lo_bits, a.win_lo);
      const uint32_t q = (i >> blk_bits) & 3u;
      const float iv = q == 0 ? inv[0] : q == 1 ? inv[1] : q == 2 ? inv[2] : inv[3];
      const uint32_t si = isl.of(it) ^ st;
      const float4 v0 = pair_order(*reinterpret_cast<const float4*>(region + pair_slot(si)), pair_swapped(si));
      if constexpr (U == 4) {
        const float4 v1 = pair_order(*reinterpret_cast<const float4*>(region + pair_slot(si ^ 2u)), pair_swapped(si));
        *reinterpret_cast<uint4*>(Bw + g) = make_uint4(pack16<S>(v0.x, v0.y, iv), pack16<S>(v0.z, v0.w, iv),
                                                       pack16<S>(v1.x, v1.y, iv), pack16<S>(v1.z, v1.w, iv));
      } else {
        *reinterpret_cast<uint2*>(Bw + g) = make_uint2(pack16<S>(v0.x, v0.y, iv), pack16<S>(v0.z, v0.w, iv));
      }
    }
    if (tt < (uint32_t)nblk) {
      float* sout = a.scale_out + batch * a.scale_stride + ((long long)blk << (T - blk_bits));
      sout[tt] = ldexpf(1.f, block_exponent(__uint_as_float(smax[nblk * tile_in_block + tt])));
    }
  }
}

// ---------------------------------------------------------------------------
// Launch records.

template <class A>
static void set_arg(Launch* L, const A& a) {
  static_assert(sizeof(A) <= kMaxArgBytes, "kernel argument too large for a launch record");
  std::memset(L->arg, 0, sizeof(L->arg));
  std::memcpy(L->arg, &a, sizeof(A));
  L->arg_bytes = (uint32_t)sizeof(A);
  L->seg_stride = (uint32_t)sizeof(Seg<A>);
}

static hipError_t set_shape(Launch* L, long long blocks_x, unsigned blocks_y, unsigned threads, size_t shmem) {
  if (blocks_x <= 0 || blocks_x > 0x7fffffffLL || blocks_y == 0 || blocks_y > 65535) return hipErrorInvalidValue;
  L->grid = dim3((unsigned)blocks_x, blocks_y, 1);
  L->block = dim3(threads, 1, 1);
  L->shmem = (uint32_t)shmem;
  return hipSuccess;
}

hipError_t record_init(const InitArgs& a, Launch* L) {
  *L = Launch();
  L->cls = 0;
  if (a.store == STORE_C64) {
    if (a.m0 - 1 > 64) return hipErrorInvalidValue;
    const long long threads = a.h < 11 ? ((long long)a.n_batches << a.h) : (((long long)a.n_batches << a.h) >> 5);
    L->fn = reinterpret_cast<const void*>(&k_init);
    L->gfn = reinterpret_cast<const void*>(&k_init_g);
    set_arg(L, a);
    return set_shape(L, (threads + kBlock - 1) / kBlock, 1, kBlock, 0);
  }
  if (a.m0 - 1 > 64 || a.blk_bits > 12 || a.blk_bits < 0 || a.blk_bits > a.h) return hipErrorInvalidValue;
  if (a.store == STORE_F16) L->fn = reinterpret_cast<const void*>(&k_init16<STORE_F16>);
  else if (a.store == STORE_BF16) L->fn = reinterpret_cast<const void*>(&k_init16<STORE_BF16>);
  else return hipErrorInvalidValue;
  set_arg(L, a);
  return set_shape(L, (long long)a.n_batches << (a.h - a.blk_bits), 1, kBlock, 0);
}

hipError_t record_resolve(const ResolveArgs& a, Launch* L) {
  *L = Launch();
  L->cls = 0;
  const long long total = (long long)a.n_batches * a.n_ops;
  if (total <= 0) return hipErrorInvalidValue;
  L->fn = reinterpret_cast<const void*>(&k_resolve);
  L->gfn = reinterpret_cast<const void*>(&k_resolve_g);
  set_arg(L, a);
  return set_shape(L, (total + kBlock - 1) / kBlock, 1, kBlock, 0);
}

template <int R, int NT, bool MULTI, bool WU>
static void pick_pass(Launch* L, int kind) {
  if (kind == 1) {
    L->fn = reinterpret_cast<const void*>(&k_pass<R, MULTI, WU, NT, 1>);
    L->gfn = reinterpret_cast<const void*>(&k_pass_g<R, MULTI, WU, NT, 1>);
  } else {
    L->fn = reinterpret_cast<const void*>(&k_pass<R, MULTI, WU, NT, 0>);
    L->gfn = reinterpret_cast<const void*>(&k_pass_g<R, MULTI, WU, NT, 0>);
  }
}

template <int R, int NT, bool MULTI, bool WU>
static void pick_pass16(Launch* L, int store, int kind) {
  if (kind == 1) {
    if (store == STORE_F16) L->fn = reinterpret_cast<const void*>(&k_pass16<R, MULTI, STORE_F16, WU, NT, 1>);
    else L->fn = reinterpret_cast<const void*>(&k_pass16<R, MULTI, STORE_BF16, WU, NT, 1>);
  } else {
    if (store == STORE_F16) L->fn = reinterpret_cast<const void*>(&k_pass16<R, MULTI, STORE_F16, WU, NT, 0>);
    else L->fn = reinterpret_cast<const void*>(&k_pass16<R, MULTI, STORE_BF16, WU, NT, 0>);
  }
}

constexpr uint64_t kStreamBytes = 2ull << 30;  // (see hbm_get)

// The streaming form of a pass that pick_pass chose: the same updates, and its
// grouped entry point stays the one without marks (a launch without one could not
// stand in a group, not even alone).
template <int NT>
static void pick_stream(Launch* L, int kind) {
  L->fn = kind == 1 ? reinterpret_cast<const void*>(&k_pass<4, false, true, NT, 1, true>)
                    : reinterpret_cast<const void*>(&k_pass<4, false, true, NT, 0, true>);
}

// Block shape of a pass: one 2^(R+9)-entry tile per 512-thread block, one
// 2^(R+8)-entry tile per 256-thread block, or several smaller tiles per
// 256-thread block (their waves lie inside one tile when T - R >= 6).
template <int R>
static hipError_t record_pass_r(const PassArgs& a, Launch* L) {
  const int TB = a.T - R;
  if (TB < 0 || TB > 9) return hipErrorInvalidValue;
  const bool s16 = a.store == STORE_F16 || a.store == STORE_BF16;
  if (!s16 && a.store != STORE_C64) return hipErrorInvalidValue;
  const int NT = TB == 9 ? 512 : kBlock;
  const bool multi = TB < 8;
  const int tiles_per_block = multi ? (kBlock >> TB) : 1;
  const long long blocks = ((long long)a.n_tiles + tiles_per_block - 1) / tiles_per_block;
  size_t lds = (size_t)tiles_per_block << (a.T + 3);
  if (s16) lds += (size_t)4 * NT;  // per-tile block maxima
  if (a.kind != 0 && a.kind != 1) return hipErrorInvalidValue;
  if (TB == 9) {
    if (s16) pick_pass16<R, 512, false, true>(L, a.store, a.kind);
    else pick_pass<R, 512, false, true>(L, a.kind);
  } else if (!multi) {
    if (s16) pick_pass16<R, kBlock, false, true>(L, a.store, a.kind);
    else pick_pass<R, kBlock, false, true>(L, a.kind);
  } else if (TB >= 6) {
    if (s16) pick_pass16<R, kBlock, true, true>(L, a.store, a.kind);
    else pick_pass<R, kBlock, true, true>(L, a.kind);
  } else {
    if (s16) pick_pass16<R, kBlock, true, false>(L, a.store, a.kind);
    else pick_pass<R, kBlock, true, false>(L, a.kind);
  }
  // streaming tensors (whole tiles per block of 16 entries per thread: the tiles
  // that large calls take by size, and the option sets that the tuner picks for them)
  const bool runs = a.lo_bits == 0 || (sizeof(float2) << a.lo_bits) >= 128;
  if constexpr (R == 4) {
    if (!s16 && !multi && runs && ((uint64_t)a.n_tiles << (a.T + 3)) >= kStreamBytes) {
      if (NT == 512) pick_stream<512>(L, a.kind);
      else pick_stream<kBlock>(L, a.kind);
    }
  }
  set_arg(L, a);
  return set_shape(L, blocks, 1, NT, lds);
}

hipError_t record_pass(const PassArgs& a, int R, Launch* L) {
  *L = Launch();
  L->cls = 1;
  switch (R) {
    case 1: return record_pass_r<1>(a, L);
    case 2: return record_pass_r<2>(a, L);
    case 3: return record_pass_r<3>(a, L);
    case 4: return record_pass_r<4>(a, L);
    case 5: return record_pass_r<5>(a, L);
    default: return hipErrorInvalidValue;
  }
}

hipError_t issue(const Launch& L, hipStream_t s) {
  void* args[1] = {const_cast<unsigned char*>(L.arg)};
  return hipLaunchKernel(L.fn, L.grid, L.block, args, L.shmem, s);
}

hipError_t graph_add(const Launch& L, hipGraph_t g, hipGraphNode_t* node, const hipGraphNode_t* dep, size_t n_dep) {
  hipKernelNodeParams kp;
  std::memset(&kp, 0, sizeof(kp));
  void* args[1] = {const_cast<unsigned char*>(L.arg)};
  kp.func = const_cast<void*>(L.fn);
  kp.gridDim = L.grid;
  kp.blockDim = L.block;
  kp.sharedMemBytes = L.shmem;
  kp.kernelParams = args;
  kp.extra = nullptr;
  return hipGraphAddKernelNode(node, g, dep, n_dep, &kp);
}

bool groupable(const Launch& a, const Launch& b) {
  return a.gfn && a.fn == b.fn && a.gfn == b.gfn && a.block.x == b.block.x && a.seg_stride == b.seg_stride;
}

size_t write_segments(const Launch* const* members, int n, unsigned char* dst) {
  size_t off = 0;
  for (int i = 0; i < n; ++i) {
    const Launch& L = *members[i];
    std::memset(dst + off, 0, L.seg_stride);
    const uint32_t g[2] = {L.grid.x, L.grid.y};
    std::memcpy(dst + off, g, sizeof(g));
    std::memcpy(dst + off + kSegHeader, L.arg, L.arg_bytes);
    off += L.seg_stride;
  }
  return off;
}

hipError_t issue_grouped(const Launch* const* members, int n, const void* d_segs, hipStream_t s) {
  if (n < 1 || n > 65535 || !d_segs) return hipErrorInvalidValue;
  const Launch& L0 = *members[0];
  unsigned gx = 0, gy = 0;
  uint32_t shmem = 0;
  for (int i = 0; i < n; ++i) {
    if (!groupable(L0, *members[i])) return hipErrorInvalidValue;
    gx = std::max(gx, members[i]->grid.x);
    gy = std::max(gy, members[i]->grid.y);
    shmem = std::max(shmem, members[i]->shmem);
  }
  void* args[1] = {(void*)&d_segs};
  return hipLaunchKernel(L0.gfn, dim3(gx, gy, (unsigned)n), L0.block, args, shmem, s);
}

// Host emulation of a fused phase, wave by wave, with the lane layout of
// phase_tri: D[4 g + r][j] = sum_k A[4 g + r][k] B[k][j], A[i][k] from the
// operand table of lane i + 16 (k % 4) at step k / 4, B[k][j] the step-(k/4)
// value of lane 16 (k % 4) + j.  FP32 sums in step order.
template <int R>
static void emulate_tri(char* region, const DevPhase& P, const uint32_t* po, const float4* F, const float* rm, int TB) {
  constexpr int E = 1 << R;
  constexpr int G = E / 2;
  const int tpt = 1 << TB;
  auto comp = [](const float4& q, int st) { return st == 0 ? q.x : st == 1 ? q.y : st == 2 ? q.z : q.w; };
  for (int w0 = 0; w0 < tpt; w0 += 64) {
    static thread_local float vx[64][E], vy[64][E];
    uint32_t off[64][E];
    for (int l = 0; l < 64; ++l) {
      const uint32_t tt = (uint32_t)(w0 + l);
      uint32_t vb = 0;
      for (int t = 0; t < TB; ++t)
        if ((tt >> t) & 1u) vb ^= po[kPhaseEntries + t];
      for (int i = 0; i < E; ++i) {
        off[l][i] = vb ^ po[i];
        const float2 x = *reinterpret_cast<const float2*>(region + off[l][i]);
        vx[l][i] = x.x;
        vy[l][i] = x.y;
      }
    }
    for (int j = 0; j < G; ++j) {
      const float4* A = F + (j >= G / 2 ? 64 : 0);
      float out[64][4];
      for (int l = 0; l < 64; ++l) {
        const int g = l / 16, jj = l % 16;
        for (int r = 0; r < 4; ++r) {
          const int i = 4 * g + r;
          float d = 0.f;
          for (int st = 0; st < 4; ++st)
            for (int gg = 0; gg < 4; ++gg) {
              const int src = 16 * gg + jj;
              const float b = st == 0 ? vx[src][2 * j] : st == 1 ? vy[src][2 * j] : st == 2 ? vx[src][2 * j + 1]
                                                                                         : vy[src][2 * j + 1];
              d = std::fma(comp(A[i + 16 * gg], st), b, d);
            }
          out[l][r] = d;
        }
      }
      for (int l = 0; l < 64; ++l) {
        vx[l][2 * j] = out[l][0];
        vy[l][2 * j] = out[l][1];
        vx[l][2 * j + 1] = out[l][2];
        vy[l][2 * j + 1] = out[l][3];
      }
    }
    // the staircase tail (a unit phase: the next step's 4x4s), lane by lane
    for (int l = 0; l < 64; ++l) {
      Regs<R> v;
      for (int i = 0; i < E; ++i) {
        v.x[i] = vx[l][i];
        v.y[i] = vy[l][i];
      }
      if (P.pad == 3) {
        if (P.n_ops == 8) {
          v = op_dense<R, 1, 2>(v, rm + (size_t)(P.op_begin + 4) * 16);
          v = op_dense<R, 0, 2>(v, rm + (size_t)(P.op_begin + 6) * 16);
        }
        for (int i = 0; i < E; ++i) {
          vx[l][i] = v.x[i];
          vy[l][i] = v.y[i];
        }
        continue;
      }
      if (P.n_ops >= 4) v = op_sel<R, 1>(v, rm + (size_t)(P.op_begin + 3) * 16 + 8 * ((l >> 5) & 1));
      if (P.n_ops >= 5) v = op_reg<R, 2, 1>(v, (const TNC_TBL float*)(rm + (size_t)(P.op_begin + 4) * 16));
      if constexpr (R >= 4) {
        if (P.n_ops >= 6) v = op_reg<R, 3, 2>(v, (const TNC_TBL float*)(rm + (size_t)(P.op_begin + 5) * 16));
      }
      if constexpr (R >= 5) {
        if (P.n_ops >= 7) v = op_reg<R, 4, 3>(v, (const TNC_TBL float*)(rm + (size_t)(P.op_begin + 6) * 16));
      }
      for (int i = 0; i < E; ++i) {
        vx[l][i] = v.x[i];
        vy[l][i] = v.y[i];
      }
    }
    for (int l = 0; l < 64; ++l)
      for (int i = 0; i < E; ++i) *reinterpret_cast<float2*>(region + off[l][i]) = make_float2(vx[l][i], vy[l][i]);
  }
}

// Host emulation with the same helpers and the same LDS placement.
template <int R>
static void emulate_pass_r(const PassArgs& a) {
  constexpr int E = 1 << R;
  const int T = a.T, TB = T - R;
  const int tpt = 1 << TB;
  const int tbits = a.h - T;
  std::vector<float2> lds((size_t)1 << T);
  char* region = reinterpret_cast<char*>(lds.data());
  const bool s16 = a.store == STORE_F16 || a.store == STORE_BF16;
  auto dec = [&](uint32_t w, float sc) {
    return a.store == STORE_F16 ? unpack16<STORE_F16>(w, sc) : unpack16<STORE_BF16>(w, sc);
  };
  auto enc = [&](float2 v, float inv) {
    return a.store == STORE_F16 ? pack16<STORE_F16>(v.x, v.y, inv) : pack16<STORE_BF16>(v.x, v.y, inv);
  };
  const int blk_bits = T < 12 ? T : 12;
  for (long long tile = 0; tile < a.n_tiles; ++tile) {
    const long long batch = tile >> tbits;
    const unsigned long long blk = (unsigned long long)tile & ((1ull << tbits) - 1ull);
    const uint64_t boff = block_offset(blk, a.lo_bits, a.win_lo, a.win_len);
    float2* Bt = a.B + (batch << a.h) + boff;
    uint32_t* Bw = reinterpret_cast<uint32_t*>(a.B) + (batch << a.h);
    for (int tt = 0; tt < tpt; ++tt)
      for (int it = 0; it < E / 2; ++it) {
        const uint32_t i = (uint32_t)(it * tpt + tt) * 2u;
        if (s16) {
          const uint64_t g = boff + tile_offset(i, a.lo_bits, a.win_lo);
          const float sc = a.scale_in[batch * a.scale_stride + (long long)scale_slot(g, a.in_map)];
          lds[swz(i)] = dec(Bw[g], sc);
          lds[swz(i + 1u)] = dec(Bw[g + 1], sc);
        } else {
          const float2* src = Bt + tile_offset(i, a.lo_bits, a.win_lo);
          lds[swz(i)] = src[0];
          lds[swz(i + 1u)] = src[1];
        }
      }
    PhaseCtx<R> ctx;
    ctx.rm = (const TNC_TBL float*)(a.rmats + (size_t)batch * a.rstride);
    ctx.tb = 0;
    ctx.uniform = false;
    for (int p = 0; p < a.n_phases; ++p) {
      const DevPhase P = load_phase(a.phases, p);
      if (P.pad == 1 || P.pad == 3) {
        if constexpr (R >= 3)
          emulate_tri<R>(region, P, a.poffs + p * kPhaseOffs, a.fmats + (size_t)p * kFusedWords,
                         a.rmats + (size_t)batch * a.rstride, TB);
        continue;
      }
      for (int tt = 0; tt < tpt; ++tt)
        if (a.kind == 1)
          phase_dispatch<R, false, 1>(region, 0u, P, (const TNC_TBL uint32_t*)a.poffs + p * kPhaseOffs, ctx,
                                      (uint32_t)tt, TB);
        else
          phase_dispatch<R, false, 0>(region, 0u, P, (const TNC_TBL uint32_t*)a.poffs + p * kPhaseOffs, ctx,
                                      (uint32_t)tt, TB);
    }
    if (s16) {
      const int nblk = 1 << (T - blk_bits);
      float amax[4] = {0.f, 0.f, 0.f, 0.f};
      for (uint32_t i = 0; i < (1u << T); ++i) {
        const float2 v = lds[swz(i)];
        float& m = amax[(i >> blk_bits) & 3u];
        m = std::max(m, std::max(std::fabs(v.x), std::fabs(v.y)));
      }
      int ex[4];
      for (int c = 0; c < 4; ++c) ex[c] = block_exponent(amax[c]);
      for (uint32_t i = 0; i < (1u << T); ++i) {
        const uint64_t g = boff + tile_offset(i, a.lo_bits, a.win_lo);
        Bw[g] = enc(lds[swz(i)], std::ldexp(1.f, -ex[(i >> blk_bits) & 3u]));
      }
      float* sout = a.scale_out + batch * a.scale_stride + ((long long)blk << (T - blk_bits));
      for (int c = 0; c < nblk; ++c) sout[c] = std::ldexp(1.f, ex[c]);
      continue;
    }
    for (int tt = 0; tt < tpt; ++tt)
      for (int it = 0; it < E / 2; ++it) {
        const uint32_t i = (uint32_t)(it * tpt + tt) * 2u;
        float2* dst = Bt + tile_offset(i, a.lo_bits, a.win_lo);
        dst[0] = lds[swz(i)];
        dst[1] = lds[swz(i + 1u)];
      }
  }
}

void emulate_pass_host(const PassArgs& a, int R) {
  switch (R) {
    case 1: emulate_pass_r<1>(a); break;
    case 2: emulate_pass_r<2>(a); break;
    case 3: emulate_pass_r<3>(a); break;
    case 4: emulate_pass_r<4>(a); break;
    case 5: emulate_pass_r<5>(a); break;
    default: break;
  }
}

// Host emulation of the phases that the one-launch and latency kernels run on a
// tile in LDS (LDS order), thread by thread: the addresses and control bit that
// one_thread and one_fetch look up, the updates of one_step and one_rest.
template <int R>
static void emulate_one_r(const OnePhase* phases, const OneSlot* slots, int n_phases, const float* mats,
                          const uint8_t* bits, int T, char* tile) {
  for (int p = 0; p < n_phases; ++p) {
    const OnePhase& P = phases[p];
    const float* m[R] = {};
    for (int b = 0; b < P.n_ops; ++b) {
      const OneSlot& s = slots[p * R + b];
      const int var = (s.xrow0 >= 0 ? 2 * (bits[s.xrow0] & 1) : 0) + (s.xrow1 >= 0 ? (bits[s.xrow1] & 1) : 0);
      m[b] = mats + ((size_t)s.op * 4 + var) * 16;
    }
    for (uint32_t tt = 0; tt < (1u << (T - R)); ++tt) {
      const uint32_t vb = P.low[tt & 15u] ^ P.high[tt >> 4];
      Regs<R> v;
      for (int i = 0; i < (1 << R); ++i) {
        const float2 x = *reinterpret_cast<const float2*>(tile + ((vb & ~kOneCtl) ^ P.off[i]));
        v.x[i] = x.x;
        v.y[i] = x.y;
      }
      v = op_sel<R, 0>(v, m[0] + 8 * (vb >> 31));
      if constexpr (R > 1)
        if (P.n_ops > 1) v = op_reg<R, 1, 0>(v, m[1]);
      if constexpr (R > 2)
        if (P.n_ops > 2) v = op_reg<R, 2, 1>(v, m[2]);
      for (int i = 0; i < (1 << R); ++i)
        *reinterpret_cast<float2*>(tile + ((vb & ~kOneCtl) ^ P.off[i])) = make_float2(v.x[i], v.y[i]);
    }
  }
}

void emulate_one_host(const OnePhase* phases, const OneSlot* slots, int n_phases, const float* mats,
                      const uint8_t* bits, float2* B, int T, int R, int lo_bits, int win_lo, uint64_t boff) {
  std::vector<float2> tile(size_t(1) << T);
  auto at = [&](uint32_t i) -> float2& { return B[boff + tile_offset(i, lo_bits, win_lo)]; };
  for (uint32_t i = 0; i < (1u << T); ++i) tile[swz(i)] = at(i);
  char* t = reinterpret_cast<char*>(tile.data());
  switch (R) {
    case 1: emulate_one_r<1>(phases, slots, n_phases, mats, bits, T, t); break;
    case 2: emulate_one_r<2>(phases, slots, n_phases, mats, bits, T, t); break;
    case 3: emulate_one_r<3>(phases, slots, n_phases, mats, bits, T, t); break;
    default: break;
  }
  for (uint32_t i = 0; i < (1u << T); ++i) at(i) = tile[swz(i)];
}

// ---------------------------------------------------------------------------
// Late phase: out[b][r][c] = sum_kk in[b][r][kk] * J[var][kk][c] in FP64.
// J folds the early-region tensor Z_early (first launch), the late layers'
// one- and two-qubit gates and the removal of the crossing bonds between the
// fixed rows and the open band (Alg. 2).  M, K and N are powers of two and
// very uneven: one amplitude per batch sums thousands of products into one
// value, eight open legs are a square 256-column product.  Three kernels
// share the work (record_late):
//   k_late_mf   N >= 4 and 64 rows: tiles on the FP64 matrix cores
//   k_late_dot  fewer of either, with K >= 64: lanes along K
//   k_late_out  K < 64 otherwise: a thread per output
__device__ inline double2 to_d2(float2 v) { return make_double2((double)v.x, (double)v.y); }
__device__ inline double2 to_d2(double2 v) { return v; }

// Entry g of batch b of the first late launch's input, in FP64.
template <typename TIn, int S>
__device__ inline double2 late_in(const LateArgs& a, const TIn* __restrict__ in, int b, uint64_t g) {
  if constexpr (S == STORE_F16 || S == STORE_BF16) {
    const float sc = a.scale_in[(long long)b * a.scale_stride + (long long)scale_slot(g, a.in_map)];
    return to_d2(unpack16<S>(in[g], sc));
  } else {
    return to_d2(in[g]);
  }
}

// Lanes along K: a wave takes RB consecutive rows and NC columns, lane l the
// products kk = l, l + 64, ...; KS waves of the block share a row group and
// split its K.  J is read once per RB rows, the tensor once per column group
// with 512-byte runs.  The 64 lanes' partial sums are halved against each
// other (lane_reduce), the KS waves' sums meet in LDS.  Bound by the read of
// the tensor.  A 64 x 64-tile kernel took 64 columns of arithmetic for these
// one to eight: 282 us for one amplitude at w = 10 and 1582 us for the 2^25
// entries of a bond-four circuit of 26 layers (256 MiB, two columns), against 7 us
// and 55 us (4.9 TB/s) here.  Conditional loads of the rows past M made the
// compiler wait on each (121 -> 177 us, measured with the sums in scratch).
// (one function per halving, so that every index is a constant: as a loop over h
// it was not unrolled at V = 32, and the sums went to scratch memory)
template <int H, int Mask, int V>
__device__ __attribute__((always_inline)) inline void lane_halve(double (&v)[V], int lane) {
  if constexpr (H >= 1) {
    const bool up = (lane & Mask) != 0;
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const double send = up ? v[i] : v[i + H];
      v[i] = (up ? v[i + H] : v[i]) + __shfl_xor(send, Mask);
    }
    lane_halve<H / 2, Mask / 2>(v, lane);
  } else {
#pragma unroll
    for (int mask = Mask; mask >= 1; mask >>= 1) v[0] += __shfl_xor(v[0], mask);
  }
}

template <int V>
__device__ __attribute__((always_inline)) inline double lane_reduce(double (&v)[V], int lane) {
  lane_halve<V / 2, 32>(v, lane);
  return v[0];
}

template <typename TIn, int S, int NC, int RB>
__device__ __attribute__((always_inline)) inline void late_dot_body(const LateArgs& a, uint32_t bx, uint32_t by) {
  constexpr int V = RB * NC * 2;  // real sums of a wave, at most 64
  static_assert(V <= 64, "one sum per lane");
  __shared__ double part[4][V];
  const int b = by;
  const int KS = a.K >= 256 ? 4 : a.K >= 128 ? 2 : 1;
  const int WR = 4 / KS;
  const int groups = a.N / NC;
  const int col0 = (int)(bx % (uint32_t)groups) * NC;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int wk = wave % KS, wr = wave / KS;
  const int row0 = ((int)(bx / (uint32_t)groups) * WR + wr) * RB;
  const int var = a.xrow >= 0 ? (int)(a.bits[(size_t)b * a.n + a.xrow] & 1) : 0;
  const double2* __restrict__ J = a.J + (size_t)var * a.K * a.N + col0;
  const TIn* __restrict__ in = reinterpret_cast<const TIn*>(a.in) + (size_t)b * a.in_batch_stride;
  double v[V];
#pragma unroll
  for (int i = 0; i < V; ++i) v[i] = 0.0;
  // K is a power of two; every row group starts at another slice of it, or all
  // blocks would read the same offsets of their rows at once, which fall on
  // the same few memory channels
  const int slices = a.K / (64 * KS);
  for (int it = 0; it < slices; ++it) {
    const int kk = (((it + (int)(bx / (uint32_t)groups)) & (slices - 1)) * KS + wk) * 64 + lane;
    double2 x[RB], z[NC];
#pragma unroll
    for (int r = 0; r < RB; ++r)
      x[r] = late_in<TIn, S>(a, in, b, (uint64_t)min(row0 + r, a.M - 1) * a.K + kk);  // (no branch: loads in flight)
#pragma unroll
    for (int c = 0; c < NC; ++c) z[c] = J[(size_t)kk * a.N + c];
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        v[2 * (r * NC + c)] += x[r].x * z[c].x - x[r].y * z[c].y;
        v[2 * (r * NC + c) + 1] += x[r].x * z[c].y + x[r].y * z[c].x;
      }
  }
  const double sum = lane_reduce<V>(v, lane);
  // after the halvings lane l holds sum l / (64 / V)
  constexpr int kLanes = 64 / V;
  if (lane % kLanes == 0) part[wave][lane / kLanes] = sum;
  __syncthreads();
  double* out = reinterpret_cast<double*>(a.out + (size_t)b * a.out_batch_stride);
  for (int i = threadIdx.x; i < V * WR; i += kBlock) {
    const int g = i / V, q = i % V;
    double t = 0.0;
    for (int w = 0; w < KS; ++w) t += part[g * KS + w][q];
    const int row = ((int)(bx / (uint32_t)groups) * WR + g) * RB + q / (2 * NC);
    if (row < a.M) out[2 * ((size_t)row * a.N + col0) + q % (2 * NC)] = t;
  }
}

template <typename TIn, int S, int NC, int RB>
__global__ __launch_bounds__(kBlock) void k_late_dot(LateArgs a) {
  late_dot_body<TIn, S, NC, RB>(a, blockIdx.x, blockIdx.y);
}

template <typename TIn, int S, int NC, int RB>
__global__ __launch_bounds__(kBlock) void k_late_dot_g(const Seg<LateArgs>* __restrict__ segs) {
  const Seg<LateArgs>* s = group_seg(segs);
  if (!s) return;
  const LateArgs a = s->a;
  late_dot_body<TIn, S, NC, RB>(a, blockIdx.x, blockIdx.y);
}

// One thread per output (of more than kLateOutBlocks blocks' threads: every so
// many): with K < 64 a row and J's columns stay in the L1 cache, neighbouring
// threads share a row's entries and read J in runs.
constexpr long long kLateOutBlocks = 1 << 23;  // 2^31 threads: a launch has to stay below 2^32
template <typename TIn, int S>
__device__ __attribute__((always_inline)) inline void late_out_body(const LateArgs& a, uint32_t bx, uint32_t by,
                                                                    uint32_t gx) {
  const int b = by;
  const int var = a.xrow >= 0 ? (int)(a.bits[(size_t)b * a.n + a.xrow] & 1) : 0;
  const TIn* __restrict__ in = reinterpret_cast<const TIn*>(a.in) + (size_t)b * a.in_batch_stride;
  for (long long o = (long long)bx * kBlock + threadIdx.x; o < (long long)a.M * a.N; o += (long long)gx * kBlock) {
    const int col = (int)(o % a.N);
    const uint64_t row = (uint64_t)(o / a.N);
    const double2* __restrict__ J = a.J + (size_t)var * a.K * a.N + col;
    double2 acc = make_double2(0.0, 0.0);
#pragma unroll 8
    for (int kk = 0; kk < a.K; ++kk) {
      const double2 x = late_in<TIn, S>(a, in, b, row * a.K + kk);
      const double2 z = J[(size_t)kk * a.N];
      acc.x += x.x * z.x - x.y * z.y;
      acc.y += x.x * z.y + x.y * z.x;
    }
    a.out[(size_t)b * a.out_batch_stride + o] = acc;
  }
}

template <typename TIn, int S>
__global__ __launch_bounds__(kBlock) void k_late_out(LateArgs a) {
  late_out_body<TIn, S>(a, blockIdx.x, blockIdx.y, gridDim.x);
}

template <typename TIn, int S>
__global__ __launch_bounds__(kBlock) void k_late_out_g(const Seg<LateArgs>* __restrict__ segs) {
  const Seg<LateArgs>* s = group_seg(segs);
  if (!s) return;
  const LateArgs a = s->a;
  late_out_body<TIn, S>(a, blockIdx.x, blockIdx.y, s->gx);
}

// The same contraction on the FP64 matrix cores (v_mfma_f64_16x16x4f64):
// a 64 x 64 output tile per 256-thread block, 32 x 32 (2 x 2 MFMA tiles)
// per wave; the complex product takes four real MFMAs per tile and k-step
// (re += ar*br - ai*bi, im += ar*bi + ai*br).  Lane l supplies A[l%16][k]
// and B[k][l%16] with k = l/16 and receives D[l/16 + 4q][l%16], q < 4.
// CT: columns of the block's tile.  Products of 32 or 16 columns take tiles
// of 128 rows by that many, 32 rows per wave, so no wave multiplies padding.
typedef double tnc_d4 __attribute__((ext_vector_type(4)));

template <typename TIn, int S, int CT>
__device__ __attribute__((always_inline)) inline void late_mf_body(const LateArgs& a, uint32_t bx, uint32_t by) {
  constexpr int RT = CT == 64 ? 64 : 128;  // rows of the block's tile
  constexpr int WJ = CT >= 32 ? 2 : 1;     // MFMA columns per wave
  constexpr int QA = RT * 16 / kBlock, QB = CT * 16 / kBlock;
  __shared__ double2 As[16][RT + 1];
  __shared__ double2 Bs[16][CT + 1];
  const int b = by;
  const int tilesN = (a.N + CT - 1) / CT;
  const int tilesM = (a.M + RT - 1) / RT;
  // Consecutive block ids go to different XCDs (round robin over 8); the
  // tilesN column blocks of one row tile are given ids that land on the
  // same XCD, so they share its L2 for the row tile.
  // (with fewer than eight row tiles that would leave XCDs idle: in order)
  const int xcd = bx & 7;
  const int g = bx >> 3;
  const int bn = tilesM < 8 ? bx % tilesN : g % tilesN;
  const int bm = tilesM < 8 ? bx / tilesN : (g / tilesN) * 8 + xcd;
  if (bm >= tilesM) return;
  const int row0 = bm * RT, col0 = bn * CT;
  const int var = a.xrow >= 0 ? (int)a.bits[(size_t)b * a.n + a.xrow] : 0;
  const double2* __restrict__ J = a.J + (size_t)var * a.K * a.N;
  const TIn* __restrict__ in = reinterpret_cast<const TIn*>(a.in) + (size_t)b * a.in_batch_stride;
  const int tid = threadIdx.x;
  const int wave = tid >> 6, lane = tid & 63;
  const int wr = CT == 64 ? (wave >> 1) * 32 : wave * 32, wc = CT == 64 ? (wave & 1) * 32 : 0;
  const int li = lane & 15, lk = lane >> 4;
  tnc_d4 cr[2][WJ], ci[2][WJ];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < WJ; ++j) {
      cr[i][j] = tnc_d4{0.0, 0.0, 0.0, 0.0};
      ci[i][j] = tnc_d4{0.0, 0.0, 0.0, 0.0};
    }
  // the next k-slice of A and B is loaded into registers while the current
  // one is multiplied from LDS
  double2 pa[QA], pb[QB];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      const int e = tid + q * kBlock;
      const int r = e >> 4, kk = e & 15;
      const int row = row0 + r;
      pa[q] = make_double2(0.0, 0.0);
      if (row < a.M && k0 + kk < a.K) pa[q] = late_in<TIn, S>(a, in, b, (uint64_t)row * a.K + k0 + kk);
    }
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int e = tid + q * kBlock;
      const int kb = e / CT, col = col0 + e % CT;
      pb[q] = make_double2(0.0, 0.0);
      if (col < a.N && k0 + kb < a.K) pb[q] = J[(size_t)(k0 + kb) * a.N + col];
    }
  };
  fetch(0);
  for (int k0 = 0; k0 < a.K; k0 += 16) {
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      const int e = tid + q * kBlock;
      As[e & 15][e >> 4] = pa[q];
    }
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int e = tid + q * kBlock;
      Bs[e / CT][e % CT] = pb[q];
    }
    __syncthreads();
    if (k0 + 16 < a.K) fetch(k0 + 16);
#pragma unroll
    for (int kc = 0; kc < 4; ++kc) {
      const int kk = kc * 4 + lk;
      double2 av[2], bv[WJ];
#pragma unroll
      for (int i = 0; i < 2; ++i) av[i] = As[kk][wr + 16 * i + li];
#pragma unroll
      for (int j = 0; j < WJ; ++j) bv[j] = Bs[kk][wc + 16 * j + li];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < WJ; ++j) {
          cr[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[i].x, bv[j].x, cr[i][j], 0, 0, 0);
          cr[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(-av[i].y, bv[j].y, cr[i][j], 0, 0, 0);
          ci[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[i].x, bv[j].y, ci[i][j], 0, 0, 0);
          ci[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[i].y, bv[j].x, ci[i][j], 0, 0, 0);
        }
    }
    __syncthreads();
  }
  double2* out = a.out + (size_t)b * a.out_batch_stride;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < WJ; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row = row0 + wr + 16 * i + lk + 4 * q;
        const int col = col0 + wc + 16 * j + li;
        if (row < a.M && col < a.N) out[(size_t)row * a.N + col] = make_double2(cr[i][j][q], ci[i][j][q]);
      }
}

template <typename TIn, int S, int CT>
__global__ __launch_bounds__(kBlock) void k_late_mf(LateArgs a) { late_mf_body<TIn, S, CT>(a, blockIdx.x, blockIdx.y); }

template <typename TIn, int S, int CT>
__global__ __launch_bounds__(kBlock) void k_late_mf_g(const Seg<LateArgs>* __restrict__ segs) {
  const Seg<LateArgs>* s = group_seg(segs);
  if (!s) return;
  const LateArgs a = s->a;
  late_mf_body<TIn, S, CT>(a, blockIdx.x, blockIdx.y);
}

template <typename TIn, int S, int CT>
static void pick_late_mf(Launch* L) {
  L->fn = reinterpret_cast<const void*>(&k_late_mf<TIn, S, CT>);
  if (S == STORE_C64) L->gfn = reinterpret_cast<const void*>(&k_late_mf_g<TIn, S, CT>);
}

template <typename TIn, int S, int NC, int RB>
static void pick_late_dot(Launch* L) {
  L->fn = reinterpret_cast<const void*>(&k_late_dot<TIn, S, NC, RB>);
  if (S == STORE_C64) L->gfn = reinterpret_cast<const void*>(&k_late_dot_g<TIn, S, NC, RB>);
}

// The kernel and grid of a first late launch.  At least four columns, a K of one
// MFMA slice and 64 rows take the matrix-core tiles, padded to 16 columns.  Below
// that the lanes go along K where K gives every lane of a wave a product, and else
// a thread computes one output.  us of the join, 16-column tile / along K:
//   tensor                 2 columns       4 columns       8 columns
//   2^17 entries, K = 64   18.6 /  7.8     18.4 /  6.8     18.6 /   7.0
//   2^20, K = 256          67.0 /  9.0     67.2 / 10.1     67.2 /  15.2
//   2^24, K = 64           64.3 / 51.3     64.4 / 71.4     65.3 / 136.7
//   2^27, K = 128           604 /  467      604 /  647      619 /  1181
//   2^27, K = 512           629 /  376      628 /  465      640 /  1035
// Two columns are faster along K at every size.  With four and eight a single small
// tensor would be as well, but the rule sees one batch (the groups that a call is
// split into must not change its results), and of many batches or a large tensor
// the tiles take half the time.  (A 64-column vector tile: 217 us at 2^24 entries,
// 1790 at 2^27.)  RB rows share a read of J: as many as leave one sum per lane, no
// more than eight.
template <typename TIn, int S>
static long long pick_late(const LateArgs& a, Launch* L) {
  if (a.N >= 4 && a.K >= 16 && a.M >= 64) {
    // 32 columns of up to 2^14 rows in all (a block per CU at most) take the 64-column
    // tile as well: its blocks have half the rows, and the chain over K, which is all
    // such a launch waits for, is shorter: 256 products, 2^12 rows 61 us against 80 in
    // 128-row tiles, 2^14 rows 62 / 81; 32 products, 2^12 rows 12.1 / 13.6, 2^14 rows
    // 14.7 / 14.7.  From 2^15 rows on the padding counts: 22.1 / 16.2.  (Either adds an
    // output's products in the same order.)
    const bool few = (long long)a.M * a.n_batches <= 1 << 14;
    const int CT = a.N >= 64 || (a.N == 32 && few) ? 64 : a.N >= 32 ? 32 : 16;
    const int RT = CT == 64 ? 64 : 128;
    if (CT == 64) pick_late_mf<TIn, S, 64>(L);
    else if (CT == 32) pick_late_mf<TIn, S, 32>(L);
    else pick_late_mf<TIn, S, 16>(L);
    const long long tilesM = ((long long)a.M + RT - 1) / RT;
    return (tilesM < 8 ? tilesM : (tilesM + 7) / 8 * 8) * ((a.N + CT - 1) / CT);
  }
  if (a.K >= 64) {
    const int NC = std::min(a.N, 8);
    const int RB = NC <= 2 ? 8 : NC == 4 ? 4 : 2;
    if (NC == 1) pick_late_dot<TIn, S, 1, 8>(L);
    else if (NC == 2) pick_late_dot<TIn, S, 2, 8>(L);
    else if (NC == 4) pick_late_dot<TIn, S, 4, 4>(L);
    else pick_late_dot<TIn, S, 8, 2>(L);
    const int rows = RB * (a.K >= 256 ? 1 : a.K >= 128 ? 2 : 4);
    return ((long long)a.M + rows - 1) / rows * (a.N / NC);
  }
  L->fn = reinterpret_cast<const void*>(&k_late_out<TIn, S>);
  if (S == STORE_C64) L->gfn = reinterpret_cast<const void*>(&k_late_out_g<TIn, S>);
  return std::min(kLateOutBlocks, ((long long)a.M * a.N + kBlock - 1) / kBlock);
}

hipError_t record_late(const LateArgs& a, bool in_c64, Launch* L) {
  *L = Launch();
  L->cls = 2;
  if (a.n_batches < 1 || a.M < 1 || a.K < 1 || a.N < 1 || (a.N & (a.N - 1)) != 0 || (a.K & (a.K - 1)) != 0)
    return hipErrorInvalidValue;
  long long blocks;
  if (!in_c64) blocks = pick_late<double2, STORE_C64>(a, L);
  else if (a.store == STORE_F16) blocks = pick_late<uint32_t, STORE_F16>(a, L);
  else if (a.store == STORE_BF16) blocks = pick_late<uint32_t, STORE_BF16>(a, L);
  else if (a.store == STORE_C64) blocks = pick_late<float2, STORE_C64>(a, L);
  else return hipErrorInvalidValue;
  set_arg(L, a);
  return set_shape(L, blocks, (unsigned)a.n_batches, kBlock, 0);
}

// ---------------------------------------------------------------------------
// Late program on the shrinking tensor, FP64.  A block loads 2^j consecutive
// rows of 2^s state entries into LDS; two-qubit gates act on the state bits of
// every live row, a removal sums the lowest remaining row bit against C_u on
// state bit 0 (Alg. 2, the late ContractLayer steps).  After l removals the
// live rows are those whose low l row bits are zero.  The ops are a serial
// chain of LDS round trips, so their latency counts: the program is staged in
// LDS first (read from memory op by op, its header and then its matrix cost
// two cache misses per op), and a thread per group of four entries, up to 512,
// keeps each op to one or two rounds.  w = 17, k = 5, one batch: 120 us for
// both launches before (with the one-qubit gates as ops of their own), 47 us
// now; 64 batches of w = 20, k = 6: 2.60 ms before, 1.23 ms now.
constexpr int kLateStage = 48;  // ops staged at a time (13 KiB)
__device__ inline double2 zfma2(double2 m0, double2 x0, double2 m1, double2 x1) {
  return make_double2(m0.x * x0.x - m0.y * x0.y + m1.x * x1.x - m1.y * x1.y,
                      m0.x * x0.y + m0.y * x0.x + m1.x * x1.y + m1.y * x1.x);
}

__device__ inline int insert_zero(int x, int bit) {
  const int lo = x & ((1 << bit) - 1);
  return ((x - lo) << 1) | lo;
}

// Runs src_prog[0..n_prog) on the 2^j rows of 2^sb entries at st (LDS), the
// program staged at prog (LDS, room for kLateStage ops); bits: the batch's.
// Starts with a barrier (after the caller's writes of st, and of the first ops
// where the caller staged them itself) unless n_prog = 0.
__device__ inline void late_stage(LateOpDev* prog, const LateOpDev* src, int n) {
  const int words = min(kLateStage, n) * (int)(sizeof(LateOpDev) / 16);
  for (int i = threadIdx.x; i < words; i += blockDim.x)
    reinterpret_cast<uint4*>(prog)[i] = reinterpret_cast<const uint4*>(src)[i];
}

__device__ __attribute__((always_inline)) inline void late_run(double2* st, LateOpDev* prog, const LateOpDev* src_prog,
                                                               int n_prog, int sb, int j, const uint8_t* bits,
                                                               bool staged) {
  int l = 0;
  for (int o = 0; o < n_prog; ++o) {
    const int at = o % kLateStage;
    if (at == 0) {  // the next ops of the program (every thread is past the last ones: barrier below)
      if (!(staged && o == 0)) late_stage(prog, src_prog + o, n_prog - o);
      __syncthreads();
    }
    const LateOpDev& op = prog[at];
    const int kind = __builtin_amdgcn_readfirstlane(op.kind);
    const int live = j - l;
    if (kind == 1) {
      const int items = (1 << live) << (sb - 1);
      for (int w = threadIdx.x; w < items; w += blockDim.x) {
        const int r = (w >> (sb - 1)) << l;
        const int t0 = insert_zero(w & ((1 << (sb - 1)) - 1), op.a);
        const int i0 = (r << sb) | t0, i1 = i0 | (1 << op.a);
        const double2 x0 = st[i0], x1 = st[i1];
        st[i0] = zfma2(op.m[0], x0, op.m[1], x1);
        st[i1] = zfma2(op.m[2], x0, op.m[3], x1);
      }
    } else if (kind == 2) {
      const int items = (1 << live) << (sb - 2);
      for (int w = threadIdx.x; w < items; w += blockDim.x) {
        const int r = (w >> (sb - 2)) << l;
        const int t0 = insert_zero(insert_zero(w & ((1 << (sb - 2)) - 1), op.a), op.a + 1);
        const int base = (r << sb) | t0;
        const int idx[4] = {base, base | (1 << (op.a + 1)), base | (1 << op.a), base | (3 << op.a)};
        double2 x[4], y[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = st[idx[u]];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const double2 p0 = zfma2(op.m[4 * q + 0], x[0], op.m[4 * q + 1], x[1]);
          const double2 p1 = zfma2(op.m[4 * q + 2], x[2], op.m[4 * q + 3], x[3]);
          y[q] = make_double2(p0.x + p1.x, p0.y + p1.y);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) st[idx[u]] = y[u];
      }
    } else if (kind == 3) {
      // an output-bit variant (xrow >= 0) takes the second set of matrices
      const double2* m = op.m + ((op.xrow >= 0 && (bits[op.xrow] & 1)) ? 8 : 0);
      const int items = (1 << (live - 1)) << (sb - 1);
      for (int w = threadIdx.x; w < items; w += blockDim.x) {
        const int ra = (w >> (sb - 1)) << (l + 1);
        const int rb = ra | (1 << l);
        const int t0 = (w & ((1 << (sb - 1)) - 1)) << 1;
        const int ia = (ra << sb) | t0, ib = (rb << sb) | t0;
        const double2 x0 = st[ia], x1 = st[ia | 1], y0 = st[ib], y1 = st[ib | 1];
        const double2 o0a = zfma2(m[0], x0, m[1], x1), o0b = zfma2(m[4], y0, m[5], y1);
        const double2 o1a = zfma2(m[2], x0, m[3], x1), o1b = zfma2(m[6], y0, m[7], y1);
        st[ia] = make_double2(o0a.x + o0b.x, o0a.y + o0b.y);
        st[ia | 1] = make_double2(o1a.x + o1b.x, o1a.y + o1b.y);
      }
      ++l;
    } else if (kind == 6) {
      // two slots (l, l+1) at once: row u = bit l + 2 bit (l+1) takes C_u
      const int items = (1 << (live - 2)) << (sb - 1);
      for (int w = threadIdx.x; w < items; w += blockDim.x) {
        const int r0 = (w >> (sb - 1)) << (l + 2);
        const int t0 = (w & ((1 << (sb - 1)) - 1)) << 1;
        double2 o0 = make_double2(0.0, 0.0), o1 = make_double2(0.0, 0.0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int iu = ((r0 | (u << l)) << sb) | t0;
          const double2 x0 = st[iu], x1 = st[iu | 1];
          const double2 p0 = zfma2(op.m[4 * u], x0, op.m[4 * u + 1], x1);
          const double2 p1 = zfma2(op.m[4 * u + 2], x0, op.m[4 * u + 3], x1);
          o0 = make_double2(o0.x + p0.x, o0.y + p0.y);
          o1 = make_double2(o1.x + p1.x, o1.y + p1.y);
        }
        const int i0 = (r0 << sb) | t0;
        st[i0] = o0;
        st[i0 | 1] = o1;
      }
      l += 2;
    }
    __syncthreads();
  }
}

// The final contraction, by all threads of the block (past a barrier after
// the last write of st).
__device__ __attribute__((always_inline)) inline void late_final(const double2* st, double2* out, int final_kind, int k,
                                                                 const double2* dot, int x) {
  if (final_kind == 5) {
    for (int bb = threadIdx.x; bb < (1 << k); bb += blockDim.x) {
      int t = 0;
      for (int q = 0; q < k; ++q) t |= ((bb >> (k - 1 - q)) & 1) << q;
      out[bb] = st[t];
    }
  } else if (threadIdx.x == 0) {
    out[0] = zfma2(dot[2 * x], st[0], dot[2 * x + 1], st[1]);
  }
}

__device__ __attribute__((always_inline)) inline void late_ops_body(const LateOpsArgs& a, double2* st, uint32_t bx,
                                                                    uint32_t by) {
  const long long row_out = bx;
  const int b = by;
  const int sb = a.s;
  const int total = 1 << (sb + a.j);
  const double2* in = a.in + (size_t)b * a.in_batch_stride + ((size_t)row_out << (a.j + sb));
  for (int i = threadIdx.x; i < total; i += blockDim.x) st[i] = in[i];
  const uint8_t* bits = a.bits + (size_t)b * a.n;
  late_run(st, reinterpret_cast<LateOpDev*>(st + total), a.prog, a.n_prog, sb, a.j, bits, false);
  if (a.n_prog == 0) __syncthreads();
  double2* out = a.out + (size_t)b * a.out_batch_stride;
  if (a.final_kind != 0) {
    late_final(st, out, a.final_kind, a.k, &a.dot[0][0], a.final_kind == 4 ? (int)bits[a.final_xrow] & 1 : 0);
  } else {
    for (int t = threadIdx.x; t < (1 << sb); t += blockDim.x) out[((size_t)row_out << sb) + t] = st[t];
  }
}

__global__ __launch_bounds__(512) void k_late_ops(LateOpsArgs a) {
  extern __shared__ double2 st[];
  late_ops_body(a, st, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(512) void k_late_ops_g(const Seg<LateOpsArgs>* __restrict__ segs) {
  extern __shared__ double2 st[];
  const Seg<LateOpsArgs>* s = group_seg(segs);
  if (!s) return;
  const LateOpsArgs a = s->a;
  late_ops_body(a, st, blockIdx.x, blockIdx.y);
}

hipError_t record_late_ops(const LateOpsArgs& a, Launch* L) {
  *L = Launch();
  L->cls = 2;
  if (a.s + a.j > 12 || a.n_batches < 1 || a.n_prog < 0) return hipErrorInvalidValue;
  static_assert(sizeof(LateOpDev) % 16 == 0 && alignof(LateOpDev) <= 16, "staged as 16-byte words");
  const int threads = std::max(64, std::min(512, 1 << std::max(0, a.s + a.j - 2)));
  const size_t lds = (sizeof(double2) << (a.s + a.j)) + sizeof(LateOpDev) * (size_t)std::min(kLateStage, a.n_prog);
  L->fn = reinterpret_cast<const void*>(&k_late_ops);
  L->gfn = reinterpret_cast<const void*>(&k_late_ops_g);
  set_arg(L, a);
  return set_shape(L, a.rows_out, (unsigned)a.n_batches, (unsigned)threads, lds);
}

// ---------------------------------------------------------------------------
// The join matrix with j late removals folded in, once per plan and k: one row
// per block, its 2^k-entry state in LDS.  On the host the fold of three removals
// takes 21 ms at k = 8 and five about 100 ms; here 0.03 ms, so that calls of 2^24
// entries have one too.
__global__ __launch_bounds__(kBlock) void k_fold(const double2* Z, const LateOpDev* src_prog, int n_prog, int k, int j,
                                                 double2* J) {
  extern __shared__ __attribute__((aligned(16))) double2 st[];
  const int dim = 1 << k;
  LateOpDev* prog = reinterpret_cast<LateOpDev*>(st + dim);
  const uint32_t row = blockIdx.x, u = row >> k;
  const double2* in = Z + (size_t)(row & (uint32_t)(dim - 1)) * dim;
  for (int i = threadIdx.x; i < dim; i += blockDim.x) st[i] = in[i];
  int l = 0;
  for (int o = 0; o < n_prog; ++o) {
    if (o % kLateStage == 0) {
      late_stage(prog, src_prog + o, n_prog - o);
      __syncthreads();
    }
    const LateOpDev& op = prog[o % kLateStage];
    const int kind = __builtin_amdgcn_readfirstlane(op.kind);
    if (kind == 2) {
      for (int w = threadIdx.x; w < dim / 4; w += blockDim.x) {
        const int base = insert_zero(insert_zero(w, op.a), op.a + 1);
        const int idx[4] = {base, base | (1 << (op.a + 1)), base | (1 << op.a), base | (3 << op.a)};
        double2 x[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = st[idx[q]];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const double2 p0 = zfma2(op.m[4 * q + 0], x[0], op.m[4 * q + 1], x[1]);
          const double2 p1 = zfma2(op.m[4 * q + 2], x[2], op.m[4 * q + 3], x[3]);
          st[idx[q]] = make_double2(p0.x + p1.x, p0.y + p1.y);
        }
      }
    } else {  // a one-qubit gate, or a removal's matrix on bit 0
      const int bit = kind == 3 ? 0 : op.a;
      const double2* m = op.m + (kind == 3 ? 4 * ((u >> l) & 1u) : 0u);
      for (int w = threadIdx.x; w < dim / 2; w += blockDim.x) {
        const int i0 = insert_zero(w, bit), i1 = i0 | (1 << bit);
        const double2 x0 = st[i0], x1 = st[i1];
        st[i0] = zfma2(m[0], x0, m[1], x1);
        st[i1] = zfma2(m[2], x0, m[3], x1);
      }
      if (kind == 3) ++l;
    }
    __syncthreads();  // (also ahead of the next ops' staging)
  }
  if (n_prog == 0) __syncthreads();
  double2* out = J + (size_t)row * dim;
  for (int i = threadIdx.x; i < dim; i += blockDim.x) out[i] = st[i];
}

hipError_t launch_fold(const double2* Z, const LateOpDev* prog, int n_prog, int k, int j, double2* J, hipStream_t s) {
  if (!Z || !prog || !J || k < 1 || k > 10 || j < 0 || j > 12 || n_prog < 0) return hipErrorInvalidValue;
  const int threads = std::max(64, std::min(kBlock, 1 << std::max(0, k - 2)));
  const size_t lds = (sizeof(double2) << k) + sizeof(LateOpDev) * (size_t)std::min(kLateStage, n_prog);
  void* args[] = {&Z, &prog, &n_prog, &k, &j, &J};
  return hipLaunchKernel(reinterpret_cast<const void*>(&k_fold), dim3(1u << (k + j)), dim3((unsigned)threads), args, lds, s);
}

// ---------------------------------------------------------------------------
// The whole amplitude call in one launch: tensors of up to 2^12 entries, one
// batch per block, from the row-0 build-up to the amplitudes.  As separate
// launches such a call is all latency (build-up, variants, a pass of one tile
// per batch whose phases each wait on cold scalar loads of their matrices, the
// join, the late program).  Here a block keeps its tensor in LDS, and the
// phases' offsets and the matrices of the batch's variants are staged in LDS
// too, kOneChunk phases at a time, so a phase waits on nothing farther than
// LDS.  Few entries per thread (4, or 8 from 2^11 entries on) put the tensor
// on all four SIMDs: an update of 2^10 entries costs a wave two pairs.  Every
// update is the same FP32 arithmetic as in the pass kernel, in the same order.
// Bound by the chain of phases (0.4 us each at w = 10, of which 0.13 us is the
// arithmetic), with many batches by LDS.  Before and now, in us: one amplitude
// at w = 10 432 and 48 (24 qubits), 512 batches at w = 6, k = 3 145 and 17,
// 1024 batches at w = 12, k = 6 775 and 642, at k = 0 24600 and 359.
constexpr int kOneChunk = 64;

// Product initialisation of entry i, multiplied in the order of init_body.
__device__ inline float2 one_init(const double2* c, int h, int m, int x0, uint32_t i) {
  if (i >> m) return make_float2(0.f, 0.f);
  const double2* seg = c + 10;  // (v, f, the final contraction's vectors, then the segments)
  auto sg = [&](int j) { return seg[4 * (j - 1) + 2 * (int)((i >> j) & 1u) + (int)((i >> (j - 1)) & 1u)]; };
  const double2 f = c[2 + 2 * x0 + (int)((i >> (m - 1)) & 1u)];
  double2 val = c[i & 1u];
  if (h < 11) {
    for (int j = 1; j < m; ++j) val = zmul(val, sg(j));
    val = zmul(val, f);
  } else {
    for (int j = 1; j < m && j <= 5; ++j) val = zmul(val, sg(j));
    for (int j = 12; j < m; ++j) val = zmul(val, sg(j));
    const bool f_var = m - 1 >= 6 && m - 1 <= 10;
    if (!f_var) val = zmul(val, f);
    for (int j = 6; j < m && j <= 11; ++j) val = zmul(val, sg(j));
    if (f_var) val = zmul(val, f);
  }
  return make_float2((float)val.x, (float)val.y);
}

// A staged phase: its table, and at a fixed place of its own the matrices of R
// updates (so nothing is addressed by what was just read).
constexpr int kOneLow = 16;
template <int R>
struct OneStage {
  OnePhase P;
  float mats[16 * R];
};

// n 16-byte words from memory to LDS, four loads in flight per thread.
template <class Src, class Dst>
__device__ __attribute__((always_inline)) inline void stage_words(int n, Src src, Dst dst) {
  const int tid = threadIdx.x, nt = blockDim.x;
  for (int i0 = tid; i0 < n; i0 += 4 * nt) {
    uint4 w[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) w[q] = src(min(i0 + q * nt, n - 1));
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (i0 + q * nt < n) dst(i0 + q * nt) = w[q];
  }
}

// What a phase needs besides its entries, in registers: the LDS addresses of
// the thread's entries and the matrices of up to R updates (op 0's picked by
// its control, the others for both values of theirs).
template <int R>
struct OneRegs {
  uint32_t off[1 << R];
  float k[8 + 16 * (R - 1)];
  int n_ops;
};

// The thread's part of a phase's LDS addresses (and kOneCtl).
template <int R>
__device__ __attribute__((always_inline)) inline uint32_t one_thread(const OneStage<R>* S, uint32_t tt) {
  return S->P.low[tt & (kOneLow - 1)] ^ S->P.high[tt / kOneLow];
}

template <int R>
__device__ __attribute__((always_inline)) inline void one_fetch(const OneStage<R>* S, uint32_t base, uint32_t vb,
                                                                OneRegs<R>& r) {
  const float4* m = reinterpret_cast<const float4*>(S->mats);
  auto get = [](float* dst, const float4 x) {
    dst[0] = x.x;
    dst[1] = x.y;
    dst[2] = x.z;
    dst[3] = x.w;
  };
  get(r.k, m[2 * (vb >> 31)]);
  get(r.k + 4, m[2 * (vb >> 31) + 1]);
#pragma unroll
  for (int q = 0; q < 4 * (R - 1); ++q) get(r.k + 8 + 4 * q, m[4 + q]);
  const uint32_t at = base ^ (vb & ~kOneCtl);
#pragma unroll
  for (int q = 0; q < ((1 << R) + 3) / 4; ++q) {
    const uint4 w = reinterpret_cast<const uint4*>(S->P.off)[q];
    const uint32_t o[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (4 * q + e < (1 << R)) r.off[4 * q + e] = at ^ o[e];
  }
  r.n_ops = S->P.n_ops;
}

// (the branches of a phase end in the stores: no values to merge)
template <int R>
TNC_HD inline void one_store(const Regs<R>& v, const OneRegs<R>& c) {
#pragma unroll
  for (int i = 0; i < (1 << R); ++i) lds_put(nullptr, c.off[i], make_float2(v.x[i], v.y[i]));
}

template <int R>
__device__ __attribute__((always_inline)) inline void one_rest(Regs<R> v, const OneRegs<R>& c) {
  if constexpr (R > 1) {
    const int n_ops = __builtin_amdgcn_readfirstlane(c.n_ops);
    if (n_ops == 1) return one_store<R>(v, c);
    v = op_reg<R, 1, 0>(v, (const float*)(c.k + 8));
    if constexpr (R > 2) {
      if (n_ops == 2) return one_store<R>(v, c);
      v = op_reg<R, 2, 1>(v, (const float*)(c.k + 24));
    }
  }
  one_store<R>(v, c);
}

// One phase from c, with the next one's registers into n and the thread part
// of the one after it into vb: their reads go out behind this phase's entries
// and are used after the barrier at the earliest.
template <int R>
__device__ __attribute__((always_inline)) inline void one_step(const OneRegs<R>& c, const OneStage<R>* next,
                                                               const OneStage<R>* next2, uint32_t base, uint32_t tt,
                                                               OneRegs<R>& n, uint32_t& vb) {
  Regs<R> v;
#pragma unroll
  for (int i = 0; i < (1 << R); ++i) {
    const float2 t = lds_get(nullptr, c.off[i]);
    v.x[i] = t.x;
    v.y[i] = t.y;
  }
  __builtin_amdgcn_sched_barrier(0);
  one_fetch<R>(next, base, vb, n);
  vb = one_thread<R>(next2, tt);
  __builtin_amdgcn_sched_barrier(0);
  v = op_sel<R, 0>(v, (const float*)c.k);
  // (the addresses are computed here, ahead of the barrier)
#pragma unroll
  for (int i = 0; i < (1 << R); ++i) asm volatile("" : "+v"(n.off[i]));
  asm volatile("" : "+v"(vb));
  one_rest<R>(v, c);
}

// The phases of a tile in LDS (at address `base`): tables and matrices staged at
// `stage`, kOneChunk phases at a time; sbits: the batch's bits in LDS (written by
// the caller, no barrier since).  fill() writes the tile; it runs once, behind
// the first chunk's loads and ahead of the barrier before the first phase.
// Ends with a barrier.
template <int R, class Fill>
__device__ __attribute__((always_inline)) inline void one_sweep(const OnePhase* tables, const OneSlot* slots,
                                                                const float* all_mats, int n_phases, OneStage<R>* phases,
                                                                const uint8_t* sbits, uint32_t base, uint32_t tt,
                                                                Fill fill) {
  const int tid = threadIdx.x, nt = blockDim.x;
  if (n_phases == 0) {  // no updates
    __syncthreads();
    fill();
    __syncthreads();
  }
  // a matrix float4 per item, at most kItems per thread and chunk (nt >= 64,
  // and 256 or more for R = 3)
  constexpr int kItems = kOneChunk * 4 * R / (R > 2 ? 256 : 64);
  for (int c = 0; c < n_phases; c += kOneChunk) {
    const int np = min(kOneChunk, n_phases - c);
    if (c > 0) __syncthreads();  // every thread is past the last chunk's phases
    constexpr int kHead = sizeof(OnePhase) / 16, kStage = sizeof(OneStage<R>) / 16;
    OneSlot sl[kItems];
#pragma unroll
    for (int q = 0; q < kItems; ++q)
      sl[q] = slots[(size_t)c * R + (min(tid + q * nt, np * R * 4 - 1) >> 2)];
    stage_words(np * kHead, [&](int i) { return reinterpret_cast<const uint4*>(tables + c)[i]; },
                [&](int i) -> uint4& { return reinterpret_cast<uint4*>(phases)[i / kHead * kStage + i % kHead]; });
    if (c == 0) __syncthreads();  // the bits are staged
    float4 w[kItems];
#pragma unroll
    for (int q = 0; q < kItems; ++q) {
      const OneSlot x = sl[q];
      const int i = min(tid + q * nt, np * R * 4 - 1);
      const int b0 = sbits[max((int)x.xrow0, 0)] & 1, b1 = sbits[max((int)x.xrow1, 0)] & 1;
      const int var = (x.xrow0 >= 0 ? 2 * b0 : 0) + (x.xrow1 >= 0 ? b1 : 0);
      w[q] = reinterpret_cast<const float4*>(all_mats + ((size_t)max(x.op, 0) * 4 + var) * 16)[i & 3];
    }
    if (c == 0) fill();  // (while the matrices arrive)
#pragma unroll
    for (int q = 0; q < kItems; ++q) {
      const int i = min(tid + q * nt, np * R * 4 - 1);  // (past the end: the last one again, no branch)
      reinterpret_cast<float4*>(phases[i / (4 * R)].mats)[i % (4 * R)] = w[q];
    }
    __syncthreads();
    // Phase p + 1's offsets and matrices are read while phase p computes: its
    // entries are then the only thing a phase waits for.  Two phases per turn,
    // so the two register sets take turns without copies.
    OneRegs<R> c0, c1;
    one_fetch<R>(phases, base, one_thread<R>(phases, tt), c0);
    uint32_t vb = one_thread<R>(phases + min(1, np - 1), tt);
    for (int p = 0; p < np; p += 2) {
      one_step<R>(c0, phases + min(p + 1, np - 1), phases + min(p + 2, np - 1), base, tt, c1, vb);
      __syncthreads();
      if (p + 1 < np) {
        one_step<R>(c1, phases + min(p + 2, np - 1), phases + min(p + 3, np - 1), base, tt, c0, vb);
        __syncthreads();
      }
    }
  }
}

template <int R>
__device__ __attribute__((always_inline)) inline void one_body(const OneArgs& a, char* lds, uint32_t bx) {
  constexpr int E = 1 << R;
  const int tid = threadIdx.x, nt = blockDim.x;
  const int h = a.h, TB = h - R;
  const uint32_t b = bx;
  const uint8_t* bits = a.bits + (size_t)b * a.n;
  float2* tile = reinterpret_cast<float2*>(lds);
  OneStage<R>* phases = reinterpret_cast<OneStage<R>*>(__builtin_assume_aligned(lds + ((size_t)8 << h), 16));
  const int chunk = min(kOneChunk, max(1, a.n_phases));
  double2* seg = reinterpret_cast<double2*>(phases + chunk);
  uint8_t* sbits = reinterpret_cast<uint8_t*>(seg + 10 + 4 * max(0, a.m0 - 1));
  const uint32_t base = lds_address(lds);
  // a tile of fewer than 64 threads: the wave's other lanes repeat their work
  // (the same values to the same addresses, in the same instruction)
  const uint32_t tt = (uint32_t)tid & ((1u << TB) - 1u);
  // what does not depend on other loads goes out together
  for (int i = tid; i < a.n; i += nt) sbits[i] = bits[i];
  stage_words(10 + 4 * max(0, a.m0 - 1), [&](int i) { return reinterpret_cast<const uint4*>(a.seg)[i]; },
              [&](int i) -> uint4& { return reinterpret_cast<uint4*>(seg)[i]; });
  one_sweep<R>(a.phases, a.slots, a.mats, a.n_phases, phases, sbits, base, tt, [&]() {
    for (uint32_t i = tid; i < (1u << h); i += nt) tile[swz(i)] = one_init(seg, h, a.m0, sbits[0], i);
  });
  // the late program, past the tile and past the states that replace it
  LateOpDev* prog = reinterpret_cast<LateOpDev*>(lds + max((size_t)a.M * a.N * 16, (size_t)8 << h));
  // The join, out[r][c] = sum_kk tile[r K + kk] J[kk][c] in FP64, into
  // registers first: the states then take the tile's place.  Fewer outputs
  // than threads: `part` neighbouring threads share an output's K.
  const int outs = a.M * a.N;
  int part = 1;
  while (outs * part * 2 <= nt && part * 2 <= a.K) part *= 2;
  // (with `part` above 64 the sums meet where the program would go)
  if (!a.join_final && part <= 64) late_stage(prog, a.prog, a.n_prog);
  const int var = a.xrow >= 0 ? (int)(bits[a.xrow] & 1) : 0;
  const double2* __restrict__ J = a.J + (size_t)var * a.K * a.N;
  double2 acc[E];
#pragma unroll
  for (int q = 0; q < E; ++q) {
    acc[q] = make_double2(0.0, 0.0);
    const int o = (tid + q * nt) / part, p = tid & (part - 1);
    if (o < outs) {
      const int row = o / a.N, col = o % a.N;
#pragma unroll 4
      for (int kk = p; kk < a.K; kk += part) {
        const double2 x = to_d2(tile[swz((uint32_t)(row * a.K + kk))]);
        const double2 z = J[(size_t)kk * a.N + col];
        acc[q].x += x.x * z.x - x.y * z.y;
        acc[q].y += x.x * z.y + x.y * z.x;
      }
    }
    for (int m = 1; m < min(part, 64); m <<= 1) {
      acc[q].x += __shfl_xor(acc[q].x, m);
      acc[q].y += __shfl_xor(acc[q].y, m);
    }
  }
  if (part > 64) {  // the waves of an output meet in the staging area
    double2* red = reinterpret_cast<double2*>(phases);
    if ((tid & 63) == 0) red[tid >> 6] = acc[0];
    __syncthreads();
    if ((tid & (part - 1)) == 0)
      for (int w = 1; w < part / 64; ++w) {
        acc[0].x += red[(tid >> 6) + w].x;
        acc[0].y += red[(tid >> 6) + w].y;
      }
  }
  double2* out = a.out + ((size_t)b << a.k);
  double2* st = reinterpret_cast<double2*>(lds);
  if (!a.join_final) __syncthreads();
#pragma unroll
  for (int q = 0; q < E; ++q) {
    const int o = (tid + q * nt) / part;
    if (o < outs && (tid & (part - 1)) == 0) (a.join_final ? out : st)[o] = acc[q];
  }
  if (a.join_final) return;
  late_run(st, prog, a.prog, a.n_prog, a.s, a.j, bits, part <= 64);
  if (a.n_prog == 0) __syncthreads();
  late_final(st, out, a.final_kind, a.k, a.seg + 6, a.final_kind == 4 ? (int)bits[a.final_xrow] & 1 : 0);
}

template <int R>
__global__ __launch_bounds__(512) void k_one(OneArgs a) {
  extern __shared__ __attribute__((aligned(16))) char one_lds[];
  one_body<R>(a, one_lds, blockIdx.x);
}

template <int R>
__global__ __launch_bounds__(512) void k_one_g(const Seg<OneArgs>* __restrict__ segs) {
  extern __shared__ __attribute__((aligned(16))) char one_lds[];
  const Seg<OneArgs>* s = group_seg(segs);
  if (!s) return;
  const OneArgs a = s->a;
  one_body<R>(a, one_lds, blockIdx.x);
}

template <int R>
static void pick_one(Launch* L) {
  L->fn = reinterpret_cast<const void*>(&k_one<R>);
  L->gfn = reinterpret_cast<const void*>(&k_one_g<R>);
}

hipError_t record_one(const OneArgs& a, Launch* L) {
  *L = Launch();
  L->cls = 1;
  const int R = one_reg_bits(a.h);
  if (R == 0 || a.n_batches < 1 || a.n_prog < 0 || a.M < 1 || a.K < 1 || a.N < 1 ||
      (long long)a.M * a.K > (1ll << a.h) || (!a.join_final && a.M * a.N != 1 << (a.j + a.s)))
    return hipErrorInvalidValue;
  const int nt = std::max(64, 1 << (a.h - R));
  if ((long long)a.M * a.N > (long long)nt << R) return hipErrorInvalidValue;  // 2^R outputs per thread
  if (R == 1) pick_one<1>(L);
  else if (R == 2) pick_one<2>(L);
  else pick_one<3>(L);
  if (a.n < 1 || a.n > 1 << 13) return hipErrorInvalidValue;  // the bits are staged
  if (R == 3 && nt < 256) return hipErrorInvalidValue;
  // the tile, a chunk of phases (the waves' partial sums of the join take their
  // place), the build-up's factors, the bits
  const size_t stage = R == 1 ? sizeof(OneStage<1>) : R == 2 ? sizeof(OneStage<2>) : sizeof(OneStage<3>);
  const size_t sweep = ((size_t)8 << a.h) + std::min(kOneChunk, std::max(1, a.n_phases)) * stage +
                       16 * (size_t)(10 + 4 * std::max(0, a.m0 - 1)) + ((size_t)a.n + 15) / 16 * 16;
  const size_t late = a.join_final ? 0 : std::max((size_t)a.M * a.N * 16, (size_t)8 << a.h) +
                                             sizeof(LateOpDev) * (size_t)std::min(kLateStage, a.n_prog);
  set_arg(L, a);
  return set_shape(L, a.n_batches, 1, (unsigned)nt, std::max(sweep, late));
}

// ---------------------------------------------------------------------------
// One pass over a window of a tensor too small to fill the chip (2^13 to 2^20
// entries in all): bound by latency, launch after launch, so the tiles are the
// smallest that still cover the slots with two windows (most CUs, fewest
// entries per thread) and the phases run from LDS as in the one-launch kernel.
// The pass kernel's phases wait on two scalar loads each, cold in every launch.
// The first pass builds its tile up instead of reading it.
// One pass at w = 17, one batch: 7.6 us (36 of them, 128 tiles of 2^10 entries)
// against 17 us on average (16 tiles of 2^13); a call of 41 qubits, k = 5, 782
// us before and 318 us now.
template <int R>
__device__ __attribute__((always_inline)) inline void win_body(const WinArgs& a, char* lds, uint32_t bx) {
  constexpr int E = 1 << R;
  const int tid = threadIdx.x, nt = blockDim.x;
  const int T = a.T, TB = T - R;
  const int tbits = a.h - T;
  const uint32_t tile = xcd_block(bx, (uint32_t)a.n_tiles);
  const uint32_t b = tile >> tbits;
  const uint64_t boff = block_offset(tile & ((1u << tbits) - 1u), a.lo_bits, a.win_lo, a.win_len);
  const uint8_t* bits = a.bits + (size_t)b * a.n;
  float2* __restrict__ B = a.B + ((size_t)b << a.h) + boff;
  OneStage<R>* phases = reinterpret_cast<OneStage<R>*>(__builtin_assume_aligned(lds + ((size_t)8 << T), 16));
  double2* seg = reinterpret_cast<double2*>(phases + min(kOneChunk, max(1, a.n_phases)));
  const int n_seg = 10 + 4 * max(0, a.m0 - 1);
  uint8_t* sbits = reinterpret_cast<uint8_t*>(seg + (a.init ? n_seg : 0));
  const uint32_t tt = (uint32_t)tid & ((1u << TB) - 1u);
  // entry pairs it * 2^(TB + 1) + 2 tt of the tile (HBM order), all loads first
  const uint32_t st = swz(tt * 2u);
  const IterSlots isl(TB + 1);
  float4 ld[E / 2];
  if (!a.init) {
#pragma unroll
    for (int it = 0; it < E / 2; ++it)
      ld[it] = *reinterpret_cast<const float4*>(B + tile_offset(((uint32_t)it << (TB + 1)) + tt * 2u, a.lo_bits, a.win_lo));
  }
  for (int i = tid; i < a.n; i += nt) sbits[i] = bits[i];
  if (a.init)
    stage_words(n_seg, [&](int i) { return reinterpret_cast<const uint4*>(a.seg)[i]; },
                [&](int i) -> uint4& { return reinterpret_cast<uint4*>(seg)[i]; });
  one_sweep<R>(a.phases, a.slots, a.mats, a.n_phases, phases, sbits, lds_address(lds), tt, [&]() {
    if (a.init) {
      float2* t = reinterpret_cast<float2*>(lds);
      for (uint32_t i = tid; i < (1u << T); i += nt)
        t[swz(i)] = one_init(seg, a.h, a.m0, sbits[0], (uint32_t)(boff + tile_offset(i, a.lo_bits, a.win_lo)));
    } else {
#pragma unroll
      for (int it = 0; it < E / 2; ++it) {
        const uint32_t si = isl.of(it) ^ st;
        *reinterpret_cast<float4*>(lds + pair_slot(si)) = pair_order(ld[it], pair_swapped(si));
      }
    }
  });
#pragma unroll
  for (int it = 0; it < E / 2; ++it) {
    const uint32_t si = isl.of(it) ^ st;
    const float4 v = *reinterpret_cast<const float4*>(lds + pair_slot(si));
    *reinterpret_cast<float4*>(B + tile_offset(((uint32_t)it << (TB + 1)) + tt * 2u, a.lo_bits, a.win_lo)) =
        pair_order(v, pair_swapped(si));
  }
}

template <int R>
__global__ __launch_bounds__(512) void k_win(WinArgs a) {
  extern __shared__ __attribute__((aligned(16))) char one_lds[];
  win_body<R>(a, one_lds, blockIdx.x);
}

template <int R>
__global__ __launch_bounds__(512) void k_win_g(const Seg<WinArgs>* __restrict__ segs) {
  extern __shared__ __attribute__((aligned(16))) char one_lds[];
  const Seg<WinArgs>* s = group_seg(segs);
  if (!s) return;
  const WinArgs a = s->a;
  win_body<R>(a, one_lds, blockIdx.x);
}

hipError_t record_win(const WinArgs& a, int R, Launch* L) {
  *L = Launch();
  L->cls = 1;
  const int TB = a.T - R;
  // one thread per 2^R entries, whole waves; pairs of entries in the low slots
  if ((R != 2 && R != 3) || TB < 6 || TB > 9 || (R == 3 && TB < 8) || a.T > a.h || a.h > 31 || a.n_tiles < 1 ||
      a.lo_bits + a.win_len != a.T || (a.lo_bits < 1 && a.win_lo != 0) || a.win_lo < a.lo_bits ||
      a.win_lo + a.win_len > a.h || a.n < 1 || a.n > 1 << 13)
    return hipErrorInvalidValue;
  if (R == 2) {
    L->fn = reinterpret_cast<const void*>(&k_win<2>);
    L->gfn = reinterpret_cast<const void*>(&k_win_g<2>);
  } else {
    L->fn = reinterpret_cast<const void*>(&k_win<3>);
    L->gfn = reinterpret_cast<const void*>(&k_win_g<3>);
  }
  const size_t stage = R == 2 ? sizeof(OneStage<2>) : sizeof(OneStage<3>);
  const size_t lds = ((size_t)8 << a.T) + std::min(kOneChunk, std::max(1, a.n_phases)) * stage +
                     (a.init ? 16 * (size_t)(10 + 4 * std::max(0, a.m0 - 1)) : 0) + ((size_t)a.n + 15) / 16 * 16;
  set_arg(L, a);
  return set_shape(L, a.n_tiles, 1, 1u << TB, lds);
}

// ---------------------------------------------------------------------------
// The complex128 reference sweep: the same product initialisation as k_init
// kept in FP64, then every update of the sweep as its own launch, each
// thread one pair of entries.  A test path (the paper's precision study
// compares complex64 with complex128 runs, Sec. 5.1), not tuned.
__global__ __launch_bounds__(kBlock) void k_init64(InitArgs a) {
  const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long total = (long long)a.n_batches << a.h;
  if (gid >= total) return;
  const long long batch = gid >> a.h;
  const unsigned long long i = (unsigned long long)gid & ((1ull << a.h) - 1ull);
  double2* out = reinterpret_cast<double2*>(a.B) + gid;
  const int m = a.m0;
  if (i >> m) {
    *out = make_double2(0.0, 0.0);
    return;
  }
  const int x0 = a.bits[batch * a.n];
  double2 val = a.v[i & 1ull];
  for (int j = 1; j < m; ++j) {
    const int aj = (int)((i >> j) & 1ull), ajm = (int)((i >> (j - 1)) & 1ull);
    val = zmul(val, a.seg[4 * (j - 1) + 2 * aj + ajm]);
  }
  *out = zmul(val, a.f[x0][(i >> (m - 1)) & 1ull]);
}

__global__ __launch_bounds__(kBlock) void k_op64(Op64Args a) {
  const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long pairs = (long long)a.n_batches << (a.h - 1);
  if (gid >= pairs) return;
  const Op64 op = *a.op;
  const long long batch = gid >> (a.h - 1);
  const unsigned long long p = (unsigned long long)gid & ((1ull << (a.h - 1)) - 1ull);
  const unsigned long long ts = 1ull << op.target;
  const unsigned long long lo = p & (ts - 1ull);
  const unsigned long long i0 = ((p - lo) << 1) | lo, i1 = i0 | ts;
  double2* B = a.B + (batch << a.h);
  if (op.kind == 1) {
    B[i1] = B[i0];
    return;
  }
  const uint8_t* x = a.bits + (size_t)batch * a.n;
  const int var = (op.xrow0 >= 0 ? 2 * (x[op.xrow0] & 1) : 0) + (op.xrow1 >= 0 ? (x[op.xrow1] & 1) : 0);
  const int c = op.control >= 0 ? (int)((i0 >> op.control) & 1ull) : 0;
  const double2* m = op.m[var][c];
  const double2 b0 = B[i0], b1 = B[i1];
  const double2 p0 = zmul(m[0], b0), q0 = zmul(m[1], b1), p1 = zmul(m[2], b0), q1 = zmul(m[3], b1);
  B[i0] = make_double2(p0.x + q0.x, p0.y + q0.y);
  B[i1] = make_double2(p1.x + q1.x, p1.y + q1.y);
}

hipError_t launch_init64(const InitArgs& a, hipStream_t s) {
  if (a.m0 - 1 > 64 || a.h < 1) return hipErrorInvalidValue;
  const long long blocks = (((long long)a.n_batches << a.h) + kBlock - 1) / kBlock;
  if (blocks > 0x7fffffffLL || blocks < 1) return hipErrorInvalidValue;
  InitArgs b = a;
  return hipLaunchKernel(reinterpret_cast<const void*>(&k_init64), dim3((unsigned)blocks), dim3(kBlock),
                         std::array<void*, 1>{&b}.data(), 0, s);
}

hipError_t launch_op64(const Op64Args& a, hipStream_t s) {
  if (a.h < 1) return hipErrorInvalidValue;
  const long long blocks = (((long long)a.n_batches << (a.h - 1)) + kBlock - 1) / kBlock;
  if (blocks > 0x7fffffffLL || blocks < 1) return hipErrorInvalidValue;
  Op64Args b = a;
  return hipLaunchKernel(reinterpret_cast<const void*>(&k_op64), dim3((unsigned)blocks), dim3(kBlock),
                         std::array<void*, 1>{&b}.data(), 0, s);
}

// ---------------------------------------------------------------------------
// FP64 complex fill and sum (the ring's sum over slices).
__global__ __launch_bounds__(kBlock) void k_fill_zero(double2* out, long long count) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) out[i] = make_double2(0.0, 0.0);
}

// A launch whose status is its own (hipGetLastError after a launch would
// also return, and clear, an error the caller had pending).  The arguments
// are the kernel's parameters by value, in order.
template <class... A>
static hipError_t launch_direct(const void* fn, dim3 grid, dim3 block, hipStream_t s, A... args) {
  void* argv[] = {static_cast<void*>(&args)...};
  return hipLaunchKernel(fn, grid, block, argv, 0, s);
}

hipError_t launch_fill_zero(double2* out, long long count, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  return launch_direct(reinterpret_cast<const void*>(&k_fill_zero), dim3((unsigned)((count + kBlock - 1) / kBlock)),
                       dim3(kBlock), s, out, count);
}

// out[i] += sum over r < rows of in[r * stride + i] (FP64).  A block takes W
// consecutive outputs: thread (g, i) sums rows g, g + 256 / W, ..., and the
// groups' sums meet in LDS, in a fixed order.  One thread per output, all rows in
// turn, left 16 threads to read 1024 rows: 240 us, 6 us here with W = 16.  With
// fewer rows than groups the idle threads would cost more than the chain, so W
// grows until every group has a row (launch_accumulate_rows).
__global__ __launch_bounds__(kBlock) void k_accumulate_rows(double2* out, const double2* in, long long stride,
                                                           int rows, long long count, int W) {
  __shared__ double2 part[kBlock];
  const int i = threadIdx.x % W, g = threadIdx.x / W, G = kBlock / W;
  const long long o = (long long)blockIdx.x * W + i;
  double2 acc = make_double2(0.0, 0.0);
  if (o < count) {
#pragma unroll 8
    for (int r = g; r < rows; r += G) {
      const double2 v = in[(long long)r * stride + o];
      acc.x += v.x;
      acc.y += v.y;
    }
  }
  part[threadIdx.x] = acc;
  __syncthreads();
  for (int h = G / 2; h > 0; h >>= 1) {
    if (g < h) {
      part[threadIdx.x].x += part[threadIdx.x + h * W].x;
      part[threadIdx.x].y += part[threadIdx.x + h * W].y;
    }
    __syncthreads();
  }
  if (g == 0 && o < count) {
    out[o].x += part[i].x;
    out[o].y += part[i].y;
  }
}

hipError_t launch_accumulate_rows(double2* out, const double2* in, long long stride, int rows, long long count,
                                  hipStream_t s) {
  if (count <= 0 || rows <= 0) return hipSuccess;
  int W = kBlock;
  while (W > 1 && (W / 2 >= count || (W > 16 && kBlock / W < rows))) W /= 2;
  return launch_direct(reinterpret_cast<const void*>(&k_accumulate_rows), dim3((unsigned)((count + W - 1) / W)),
                       dim3(kBlock), s, out, in, stride, rows, count, W);
}


// Batched sampling (Sec. 4.2, steps 3-4): one block per batch.  Thread t
// holds entries [t E, t E + E) of the batch's 2^k (E = 2^k / 256 or 1),
// their probabilities |Z|^2 in FP64 and their sum; a block scan of those
// sums gives every entry's inclusive prefix; the suffix is the smallest b
// whose prefix exceeds u Q_a (the last suffix if rounding leaves none).
__global__ __launch_bounds__(kBlock) void k_sample_batched(const double2* amps, int k, const double* u, int32_t* bout,
                                                           double* qout) {
  __shared__ double scan[kBlock];
  __shared__ int best;
  const long long batch = blockIdx.x;
  const int B = 1 << k;
  const int E = B > kBlock ? B / kBlock : 1;
  const int t = threadIdx.x;
  const int first = t * E;
  const double2* z = amps + batch * (long long)B;
  double p[kMaxSampleEntries];
  double local = 0.0;
#pragma unroll
  for (int e = 0; e < kMaxSampleEntries; ++e) {
    p[e] = 0.0;
    if (e < E && first + e < B) {
      const double2 v = z[first + e];
      p[e] = v.x * v.x + v.y * v.y;
      local += p[e];
    }
  }
  if (t == 0) best = B - 1;
  scan[t] = local;
  __syncthreads();
  // inclusive Hillis-Steele scan over the thread sums
  for (int off = 1; off < kBlock; off <<= 1) {
    const double add = t >= off ? scan[t - off] : 0.0;
    __syncthreads();
    scan[t] += add;
    __syncthreads();
  }
  const double q = scan[kBlock - 1];
  const double target = u[batch] * q;
  double run = scan[t] - local;  // exclusive prefix of this thread's entries
#pragma unroll
  for (int e = 0; e < kMaxSampleEntries; ++e) {
    if (e < E && first + e < B) {
      run += p[e];
      if (run > target) {
        atomicMin(&best, first + e);
        break;
      }
    }
  }
  __syncthreads();
  if (t == 0) {
    bout[batch] = best;
    qout[batch] = q;
  }
}

// Frugal rejection (Sec. 4.1, steps 2-3): z = 2^n |amp|^2, accepted when
// u < min(1, z / M).
__global__ __launch_bounds__(kBlock) void k_frugal_accept(const double2* amps, long long count, int n, double M,
                                                          const double* u, uint8_t* accept, double* zout) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const double2 v = amps[i];
  const double z = ldexp(v.x * v.x + v.y * v.y, n);
  zout[i] = z;
  accept[i] = u[i] < fmin(1.0, z / M) ? 1 : 0;
}

hipError_t launch_sample_batched(const double2* amps, int n_batches, int k, const double* u, int32_t* b, double* q,
                                 hipStream_t s) {
  if (n_batches <= 0) return hipSuccess;
  return launch_direct(reinterpret_cast<const void*>(&k_sample_batched), dim3((unsigned)n_batches), dim3(kBlock), s,
                       amps, k, u, b, q);
}

hipError_t launch_frugal_accept(const double2* amps, long long count, int n, double M, const double* u,
                                uint8_t* accept, double* z, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  const long long blocks = (count + kBlock - 1) / kBlock;
  return launch_direct(reinterpret_cast<const void*>(&k_frugal_accept), dim3((unsigned)blocks), dim3(kBlock), s, amps,
                       count, n, M, u, accept, z);
}

// log-XEB (Sec. 5.2): F = gamma + n ln 2 + mean_i ln p_i with p_i = |amp|^2
// of the selected component of each batch (sel == nullptr: every component).
// FP64 throughout.  result = {F, SE, F - 1.96 SE, F + 1.96 SE, N}.
__device__ inline void xeb_result(double sum, double sum2, long long total, int n_qubits, double* result) {
  const double N = (double)total;
  const double mean = sum / N;
  const double var = N > 1 ? (sum2 - N * mean * mean) / (N - 1.0) : 0.0;
  const double se = N > 1 ? sqrt(var > 0 ? var : 0.0) / sqrt(N) : 0.0;
  const double gamma = 0.57721566490153286060651209008240243;
  const double F = gamma + (double)n_qubits * 0.69314718055994530941723212145817657 + mean;
  result[0] = F;
  result[1] = se;
  result[2] = F - 1.96 * se;
  result[3] = F + 1.96 * se;
  result[4] = N;
}

// Sums of ln p and (ln p)^2 over this block's share of the components, valid
// in thread 0.
template <int NT>
__device__ inline double2 xeb_block_sums(const double2* amps, int k, const int32_t* sel, long long total) {
  __shared__ double s1[NT], s2[NT];
  double a1 = 0.0, a2 = 0.0;
  for (long long i = (long long)blockIdx.x * NT + threadIdx.x; i < total; i += (long long)gridDim.x * NT) {
    const long long idx = sel ? ((i << k) + sel[i]) : i;
    const double2 z = amps[idx];
    const double lp = log(z.x * z.x + z.y * z.y);
    a1 += lp;
    a2 += lp * lp;
  }
  s1[threadIdx.x] = a1;
  s2[threadIdx.x] = a2;
  __syncthreads();
  for (int off = NT / 2; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) {
      s1[threadIdx.x] += s1[threadIdx.x + off];
      s2[threadIdx.x] += s2[threadIdx.x + off];
    }
    __syncthreads();
  }
  return make_double2(s1[0], s2[0]);
}

// One block: up to 1024 components by 256 threads, up to kXebSingle by 1024 (8192
// components 11.6 us with 256 threads, 8.5 with 1024).
template <int NT>
__global__ __launch_bounds__(NT) void k_logxeb(const double2* amps, long long total, int k, const int32_t* sel,
                                                   int n_qubits, double* result) {
  const double2 s = xeb_block_sums<NT>(amps, k, sel, total);
  if (threadIdx.x == 0) xeb_result(s.x, s.y, total, n_qubits, result);
}

// Many blocks: each adds its two sums to the caller's result buffer, and the
// last to arrive turns them into the result.  The sums go in as integers, two
// words each (k_logxeb_clear zeroes all five): a fixed-point value v is
// hi * q + lo * q / 2^40, q a power of two that keeps the total below 2^62.
// Integer sums do not depend on the order of arrival, so the result is the
// same from run to run, and their 100 bits add no rounding of note.  One block
// of 256 computes 2051 x 256 logarithms in 780 us (one CU), 128 blocks in 17 us.
constexpr int kXebBlocks = 128;  // (their sums meet at five addresses: 512 blocks took 37 us)
// Up to here one block of 1024 threads.  The clearing launch costs the host 2.5
// us, which is what a call costs among others that it waits for.  us per call,
// one block of 256 / one of 1024 / clearing and many blocks:
//   components   calls of log-XEB alone   two of them with both samplers
//         8200   12.0 /  8.6 /  9.6       33.3 / 34.8 / 37.1
//        10240   13.8 / 10.0 /  9.8       33.5 / 34.6 / 37.5
//        20480   25.1 / 17.3 /  9.8       34.8 / 34.9 / 37.9
//        24576   29.6 / 20.1 / 10.0       39.2 / 35.0 / 38.0
// so the many blocks start where the estimators' sequence, on one block of 256,
// would have taken as long as with the second launch.
constexpr long long kXebSingle = 20480;
static_assert(kXebBlocks < (1 << 12), "arrival fields of 16 bits, low words of 40 bits");

// ln p of a finite nonzero double lies in (-746, 710): |sum| < total 2^10 and
// sum of squares < total 2^20; the quantum of the sum (p = 1) or of the squares (p = 2)
__device__ inline int xeb_shift(long long total, int p) { return 64 - __clzll(total) + 10 * p - 62; }

__device__ inline void xeb_add(unsigned long long* acc, double v, int shift) {
  const double u = ldexp(v, -shift);
  const double hi = rint(u);
  atomicAdd(acc, (unsigned long long)(long long)hi);
  atomicAdd(acc + 1, (unsigned long long)(long long)rint(ldexp(u - hi, 40)));
}

__device__ inline double xeb_value(unsigned long long* acc, int shift) {
  const long long hi = (long long)atomicAdd(acc, 0ull), lo = (long long)atomicAdd(acc + 1, 0ull);
  return ldexp((double)hi + ldexp((double)lo, -40), shift);
}

__global__ void k_logxeb_clear(unsigned long long* acc) {
  if (threadIdx.x < 5) acc[threadIdx.x] = 0ull;
}

__global__ __launch_bounds__(kBlock) void k_logxeb_blocks(const double2* amps, long long total, int k,
                                                          const int32_t* sel, int n_qubits, double* result) {
  const double2 s = xeb_block_sums<kBlock>(amps, k, sel, total);
  if (threadIdx.x != 0) return;
  // word 4: arrivals, and how many sums were -inf (a zero probability), +inf, NaN
  unsigned long long* acc = reinterpret_cast<unsigned long long*>(result);
  unsigned long long mark = 1ull;
  if (isfinite(s.x) && isfinite(s.y)) {
    xeb_add(acc, s.x, xeb_shift(total, 1));
    xeb_add(acc + 2, s.y, xeb_shift(total, 2));
  } else {
    mark |= isnan(s.x) ? 1ull << 48 : s.x > 0.0 ? 1ull << 32 : 1ull << 16;
  }
  __threadfence();
  const unsigned long long seen = atomicAdd(acc + 4, mark) + mark;
  if ((seen & 0xffffull) != gridDim.x) return;
  __threadfence();
  double sum = xeb_value(acc, xeb_shift(total, 1)), sum2 = xeb_value(acc + 2, xeb_shift(total, 2));
  if (seen >> 16) {
    if ((seen >> 16) & 0xffffull) sum -= INFINITY;
    if ((seen >> 32) & 0xffffull) sum += INFINITY;
    if (seen >> 48) sum = NAN;
    sum2 = isnan(sum) && (seen >> 48) ? NAN : INFINITY;
  }
  xeb_result(sum, sum2, total, n_qubits, result);
}

hipError_t launch_logxeb(const double2* amps, int n_batches, int k, const int32_t* sel, int n_qubits,
                         double* result, hipStream_t s) {
  const long long total = sel ? (long long)n_batches : (long long)n_batches << k;
  if (total <= 1024)
    return launch_direct(reinterpret_cast<const void*>(&k_logxeb<256>), dim3(1), dim3(256), s, amps, total, k, sel,
                         n_qubits, result);
  if (total <= kXebSingle)
    return launch_direct(reinterpret_cast<const void*>(&k_logxeb<1024>), dim3(1), dim3(1024), s, amps, total, k, sel,
                         n_qubits, result);
  const hipError_t e = launch_direct(reinterpret_cast<const void*>(&k_logxeb_clear), dim3(1), dim3(64), s,
                                     reinterpret_cast<unsigned long long*>(result));
  if (e != hipSuccess) return e;
  // at least four components per thread
  const long long blocks = std::min<long long>(kXebBlocks, (total + 4 * kBlock - 1) / (4 * kBlock));
  return launch_direct(reinterpret_cast<const void*>(&k_logxeb_blocks), dim3((unsigned)blocks), dim3(kBlock), s, amps,
                       total, k, sel, n_qubits, result);
}

}  // namespace tnc
