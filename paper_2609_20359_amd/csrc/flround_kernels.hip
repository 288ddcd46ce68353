// flround_kernels.hip -- gfx950 kernels of the parameter-sync path.
//
// Every kernel here is a bandwidth-bound stream over the flat shard: an
// element is read once, updated with a few dozen fp32 operations and written
// once, so the kernels are built for HBM, not for the matrix cores:
//   * a workgroup is one wave64 and takes one unit of 512 elements, 8 to a
//     lane: 4 of each half of the unit in the passes that write fp32, 8 in a
//     row in the others (kHalves and kWhole say why).  The grid has a workgroup
//     for every unit, and how many a CU holds at once is limited per pass (the
//     launch shapes say why);
//   * all loads of a unit are out before its arithmetic, the layout table's by
//     way of the scalar cache: a wave waits for memory once;
//   * sums over peers and replicas run in ascending index order in fp32, one
//     correctly rounded operation at a time (the file is built with
//     -ffp-contract=off), so results are bitwise those of the definition and
//     do not depend on the grid;
//   * per-segment sums of squares use wave64 butterfly reductions only: each
//     lane squares its elements exactly in double, and each wave writes one
//     double partial per (tile, segment) piece it covers; a small finalize
//     folds the partials per segment (and, for clipping, over the shard) in
//     fixed trees; only units that straddle a segment boundary (rare) resolve
//     segments per element.
#include "flr_internal.h"

#include <mutex>

// Workspace of fl_round_noalloc, for callers that cannot allocate: one array
// per GPU in the code object, held until the process ends.  Host code uses
// only the per-device address that noalloc_scratch() looks up, never this
// name (which on the host side is a stand-in, not a device address).
static __device__ __align__(256) unsigned char scratch[flr::kNoallocScratchBytes];

namespace flr {
namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

// Cache hints.  ld_once: streams read once per pass (peer gradients, FedAvg
// replicas); ld: the read-modify-write state (master, m, v, fp32 gradient);
// st: every store.
#ifndef FLR_NT_ONCE
#define FLR_NT_ONCE 1
#endif
#ifndef FLR_NT_LOADS
#define FLR_NT_LOADS 0
#endif
#ifndef FLR_NT_STORES
#define FLR_NT_STORES 1
#endif

template <typename T>
__device__ __forceinline__ T ld_once(const T* p) {
#if FLR_NT_ONCE
  return __builtin_nontemporal_load(p);
#else
  return *p;
#endif
}

template <typename T>
__device__ __forceinline__ T ld(const T* p) {
#if FLR_NT_LOADS
  return __builtin_nontemporal_load(p);
#else
  return *p;
#endif
}

template <typename T>
__device__ __forceinline__ void st(T* p, T v) {
#if FLR_NT_STORES
  __builtin_nontemporal_store(v, p);
#else
  *p = v;
#endif
}

// Values that no kernel writes while one reads them (layout tables, the clip
// total of an earlier kernel) and that a whole wave reads at one address: by
// way of the constant address space the compiler uses scalar loads, which do
// not queue behind or stall the streams' vector loads.
template <typename T>
__device__ __forceinline__ T ld_uniform(const T* p) {
  return *(const __attribute__((address_space(4))) T*)(uintptr_t)p;
}

// Asks for a step's kernel arguments at the top of the kernel, all together:
// left to itself the compiler loads them where they are first used, block by
// block, and a wave waits for each group in turn before its first data load.
template <int NP>
__device__ __forceinline__ void args_in(const StepArgs& a) {
  asm volatile("" ::"s"(a.carry.partials), "s"(a.L.n), "s"(a.L.n_tiles), "s"(a.L.tiles),
               "s"(a.master), "s"(a.m), "s"(a.v), "s"(a.working), "s"(a.g_in), "s"(a.partials),
               "s"(a.clip_total), "s"(a.grad_scale), "s"(a.s.b1), "s"(a.s.omb1), "s"(a.s.b2),
               "s"(a.s.omb2), "s"(a.s.step_size), "s"(a.s.bc2_sqrt), "s"(a.s.eps),
               "s"(a.s.decay), "s"(a.s.rbc2), "s"(a.grads[0]), "s"(a.grads[1 % NP]), "s"(a.grads[2 % NP]),
               "s"(a.grads[3 % NP]), "s"(a.grads[4 % NP]), "s"(a.grads[5 % NP]),
               "s"(a.grads[6 % NP]), "s"(a.grads[7 % NP]));
}

// Keeps the compiler from moving a stream's loads below the arithmetic before
// it, which it does to save registers; all of a wave's loads have to be out
// before it waits for the first.
__device__ __forceinline__ void loads_out() { __builtin_amdgcn_sched_barrier(0); }

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// fp32 -> bf16 bits, round to nearest even; NaN -> quiet NaN, sign kept: the
// conversion instruction (two values at a time), which gives these bits for
// all 2^32 inputs.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

__device__ __forceinline__ uint32_t to_bf16(float x) { return pack_bf16x2(x, 0.f) & 0xFFFFu; }

__device__ __forceinline__ u32x4 pack_bf16x8(const float x[8]) {
  return u32x4{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(x[4], x[5]),
               pack_bf16x2(x[6], x[7])};
}

// acc[e] = acc[e] + bf16 element e of w (ascending e).
__device__ __forceinline__ void add_bf16x8(float acc[8], u32x4 w) {
  acc[0] = acc[0] + bf16_lo(w.x);
  acc[1] = acc[1] + bf16_hi(w.x);
  acc[2] = acc[2] + bf16_lo(w.y);
  acc[3] = acc[3] + bf16_hi(w.y);
  acc[4] = acc[4] + bf16_lo(w.z);
  acc[5] = acc[5] + bf16_hi(w.z);
  acc[6] = acc[6] + bf16_lo(w.w);
  acc[7] = acc[7] + bf16_hi(w.w);
}

// acc[e] = acc[e] + wt * bf16 element e of w.
__device__ __forceinline__ void fma_free_bf16x8(float acc[8], float wt, u32x4 w) {
  acc[0] = acc[0] + (wt * bf16_lo(w.x));
  acc[1] = acc[1] + (wt * bf16_hi(w.x));
  acc[2] = acc[2] + (wt * bf16_lo(w.y));
  acc[3] = acc[3] + (wt * bf16_hi(w.y));
  acc[4] = acc[4] + (wt * bf16_lo(w.z));
  acc[5] = acc[5] + (wt * bf16_hi(w.z));
  acc[6] = acc[6] + (wt * bf16_lo(w.w));
  acc[7] = acc[7] + (wt * bf16_hi(w.w));
}

// Where a lane's 8 elements lie.  kWhole: 8 in a row, one 16-byte access per
// bf16 stream and two of fp32, each of which covers every other 16 bytes of the
// wave's lines.  kHalves: elements 4l .. 4l + 3 of each half of the unit, so
// that one fp32 access covers whole lines.  Passes that write fp32 run on
// halves: whole, some of their lines left the L2 half written (broadcast receive
// 1.12 of its bytes written, the reduction to fp32 1.10, FedAvg G=4 1.03).
constexpr int kWhole = 4, kHalves = kUnit / 2;  // distance of the second four

template <int kGap = kWhole>
__device__ __forceinline__ void load_f32x8(const float* p, float x[8]) {
  const f32x4 a = ld(reinterpret_cast<const f32x4*>(p));
  const f32x4 b = ld(reinterpret_cast<const f32x4*>(p + kGap));
  x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
  x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
}

template <int kGap = kWhole>
__device__ __forceinline__ void store_f32x8(float* p, const float x[8]) {
  st(reinterpret_cast<f32x4*>(p), f32x4{x[0], x[1], x[2], x[3]});
  st(reinterpret_cast<f32x4*>(p + kGap), f32x4{x[4], x[5], x[6], x[7]});
}

template <int kGap>
__device__ __forceinline__ u32x4 load_bf16x8(const uint16_t* p) {
  if constexpr (kGap == kWhole) {
    return ld_once(reinterpret_cast<const u32x4*>(p));
  } else {
    const u32x2 a = ld_once(reinterpret_cast<const u32x2*>(p));
    const u32x2 b = ld_once(reinterpret_cast<const u32x2*>(p + kGap));
    return u32x4{a.x, a.y, b.x, b.y};
  }
}

template <int kGap>
__device__ __forceinline__ void store_bf16x8(uint16_t* p, const float x[8]) {
  const u32x4 w = pack_bf16x8(x);
  if constexpr (kGap == kWhole) {
    st(reinterpret_cast<u32x4*>(p), w);
  } else {
    st(reinterpret_cast<u32x2*>(p), u32x2{w.x, w.y});
    st(reinterpret_cast<u32x2*>(p + kGap), u32x2{w.z, w.w});
  }
}

// Sum over n bf16 streams of element e of a full vector, streams in ascending
// order: add(acc, k, w) adds stream k's 8 elements w.  N > 0: n == N, all its
// loads issued before the first addition; N == 0: n > kChunk, kChunk streams
// at a time, the next chunk's loads issued before this one's additions.
constexpr int kChunk = 8;

template <int N, int kGap = kWhole, typename Ptr, typename Add>
__device__ __forceinline__ void sum_streams(Ptr ptr, int n, Add add) {
  if constexpr (N > 0) {
    u32x4 w[N];
#pragma unroll
    for (int k = 0; k < N; ++k) w[k] = load_bf16x8<kGap>(ptr(k));
    loads_out();
#pragma unroll
    for (int k = 0; k < N; ++k) add(k, w[k]);
  } else {
    u32x4 w[kChunk];
#pragma unroll
    for (int k = 0; k < kChunk; ++k) w[k] = load_bf16x8<kGap>(ptr(k));
    int k0 = kChunk;
    for (; k0 + kChunk <= n; k0 += kChunk) {
      u32x4 x[kChunk];
#pragma unroll
      for (int k = 0; k < kChunk; ++k) x[k] = load_bf16x8<kGap>(ptr(k0 + k));
      loads_out();
#pragma unroll
      for (int k = 0; k < kChunk; ++k) {
        add(k0 - kChunk + k, w[k]);
        w[k] = x[k];
      }
    }
    u32x4 x[kChunk];
#pragma unroll
    for (int k = 0; k < kChunk - 1; ++k)
      if (k0 + k < n) x[k] = load_bf16x8<kGap>(ptr(k0 + k));
    loads_out();
#pragma unroll
    for (int k = 0; k < kChunk; ++k) add(k0 - kChunk + k, w[k]);
#pragma unroll
    for (int k = 0; k < kChunk - 1; ++k)
      if (k0 + k < n) add(k0 + k, x[k]);
  }
}

// The unit that the shard's end cuts: a lane holds the elements below `left`
// (its own first one is 0).  A group of four is read or written at once where it
// is whole, as in the other units; of the one group cut inside (some = n % 4
// elements) the elements are.  And all loads of a chunk of streams are out before
// its first addition.  One element and stream after another instead, this unit
// took 3 us at 8 streams and 66 at 64, longer than a short pass: with 64 streams
// the reduction of 65,000 elements took 64 us and takes 23 (the call from Python),
// the sums of 1.4e7 346 and 272, the wire format of 3e6 with 8 streams 14.1 and
// 11.1.  The path is short on purpose, as one wave runs it from a cold instruction
// cache: with a branch for each element, and moments of 0 past the end, which sent
// the wave to the long forms of AdamW, eight steps and FedAvg of 426,000 elements
// (R = 4) took 51.5 us and take 39.3.
struct Cut {
  int left, some;
  template <int kGap>
  __device__ __forceinline__ bool whole(int h) const { return left >= h * kGap + 4; }
  template <int kGap>
  __device__ __forceinline__ bool part(int h) const { return some && left == h * kGap + some; }
};

__device__ __forceinline__ Cut cut_at(int64_t end, int64_t base) {
  int some = (int)(end & 3);
  asm volatile("" : "+s"(some));  // (not kept in registers by the whole units)
  return {(int)(end - base), some};
}

// (fill: what the elements past the end come out as)
template <int kGap>
__device__ __forceinline__ void load_f32x8_cut(const float* p, Cut c, float x[8],
                                               float fill = 0.f) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    f32x4 a{fill, fill, fill, fill};
    if (c.whole<kGap>(h)) a = ld(reinterpret_cast<const f32x4*>(p + h * kGap));
    if (c.some && c.part<kGap>(h)) {
#pragma unroll
      for (int e = 0; e < 3; ++e) a[e] = p[h * kGap + (e < c.some ? e : 0)];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) x[4 * h + e] = a[e];
  }
}

template <int kGap>
__device__ __forceinline__ void store_f32x8_cut(float* p, Cut c, const float x[8]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const float* y = x + 4 * h;
    if (c.whole<kGap>(h)) st(reinterpret_cast<f32x4*>(p + h * kGap), f32x4{y[0], y[1], y[2], y[3]});
    if (c.some && c.part<kGap>(h)) {
#pragma unroll
      for (int e = 0; e < 3; ++e)
        if (e < c.some) p[h * kGap + e] = y[e];
    }
  }
}

template <int kGap>
__device__ __forceinline__ void store_bf16x8_cut(uint16_t* p, Cut c, const float x[8]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const float* y = x + 4 * h;
    if (c.whole<kGap>(h))
      st(reinterpret_cast<u32x2*>(p + h * kGap),
         u32x2{pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])});
    if (c.some && c.part<kGap>(h)) {
#pragma unroll
      for (int e = 0; e < 3; ++e)
        if (e < c.some) p[h * kGap + e] = (uint16_t)to_bf16(y[e]);
    }
  }
}

// sum_streams for that unit, of the arrays' elements base (the lane's first) to
// end.  The elements of the group cut inside come stream by lane: lane k loads
// stream k's, and each stream's go to the lane that holds the group.  At most four
// compiled streams at a time: this path shall not cost the others registers.
static_assert(kMaxPeers <= 64, "a lane for each stream");

template <int N, int kGap, typename Array, typename Add>
__device__ __forceinline__ void sum_streams_cut(Array array, int n, int64_t base, int64_t end,
                                                Add add) {
  constexpr int kMost = N == 0 ? kChunk : N <= 4 ? N : 4;
  const Cut c = cut_at(end, base);
  asm volatile("" : "+s"(n));
  const int some = c.some;
  const bool in0 = c.part<kGap>(0), in1 = c.part<kGap>(1);
  uint32_t c0 = 0, c1 = 0;
  if (some && (int)threadIdx.x < n) {
    const uint16_t* p = array((int)threadIdx.x) + (end - some);
    const uint32_t x = p[0], y = p[some > 1 ? 1 : 0], z = p[some > 2 ? 2 : 0];
    c0 = some > 1 ? x | y << 16 : x;
    c1 = some > 2 ? z : 0;
  }
  for (int k0 = 0; k0 < n; k0 += kMost) {
    const uint16_t* p[kMost];
#pragma unroll
    for (int k = 0; k < kMost; ++k) p[k] = array(kMost == N || k0 + k < n ? k0 + k : n - 1);
    u32x4 w[kMost] = {};
    if (c.whole<kGap>(0)) {
#pragma unroll
      for (int k = 0; k < kMost; ++k) {
        const u32x2 x = ld_once(reinterpret_cast<const u32x2*>(p[k] + base));
        w[k].x = x.x;
        w[k].y = x.y;
      }
    }
    if (c.whole<kGap>(1)) {
#pragma unroll
      for (int k = 0; k < kMost; ++k) {
        const u32x2 x = ld_once(reinterpret_cast<const u32x2*>(p[k] + base + kGap));
        w[k].z = x.x;
        w[k].w = x.y;
      }
    }
    loads_out();
#pragma unroll
    for (int k = 0; k < kMost; ++k) {
      if (kMost == N || k0 + k < n) {
        const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)c0, k0 + k);
        const uint32_t y = (uint32_t)__builtin_amdgcn_readlane((int)c1, k0 + k);
        add(k0 + k, u32x4{in0 ? x : w[k].x, in0 ? y : w[k].y, in1 ? x : w[k].z,
                          in1 ? y : w[k].w});
      }
    }
  }
}

// A pause of 256 clocks between a wave's last addition and its stores.  Passes
// that do little else run faster with it on long shards of a few streams (TB/s
// with it and without, on 5e8 elements): to the wire format R=3 6.85 and 6.64,
// R=4 6.81 and 6.48, R=8 6.68 and 6.55, FedAvg G=3 6.69 and 6.61, G=4 6.70 and
// 6.47, G=8 6.63 and 6.57.  FedAvg of one and two loses (6.47 and 6.61, 6.57 and
// 6.67); elsewhere, and on shorter shards, the difference is within noise.
// Twice the pause gave no more, half of it half.  With AdamW between loads and
// stores it makes no difference.
__device__ __forceinline__ void pause() { __builtin_amdgcn_s_sleep(4); }

// Reduced gradient of 8 elements (full vector): peers in ascending order.
template <int RT, int kGap = kWhole>
__device__ __forceinline__ void reduce_vec(const StepArgs& a, int64_t base, float g[8]) {
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  sum_streams<RT, kGap>([&](int r) { return a.grads[r] + base; }, a.R,
                  [&](int, u32x4 w) { add_bf16x8(acc, w); });
#pragma unroll
  for (int e = 0; e < 8; ++e) g[e] = acc[e] * a.grad_scale;
}

// Same for a unit that the shard's end cuts: 0 past it.
template <int RT, int kGap>
__device__ __forceinline__ void reduce_cut(const StepArgs& a, int64_t base, float g[8]) {
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  sum_streams_cut<RT, kGap>([&](int r) { return a.grads[r]; }, a.R, base, a.L.n,
                            [&](int, u32x4 w) { add_bf16x8(acc, w); });
#pragma unroll
  for (int e = 0; e < 8; ++e) g[e] = acc[e] * a.grad_scale;
}

// Fixed-tree sum over one wave64, all lanes active: the butterfly of
// exchanges with lanes 32, 16, 8, 4, 2 and 1 away, in this order, the same in
// every lane.  The first two swap halves and rows between two copies of the
// value, so that a lane's two copies are its own and its partner's; the others
// are DPP moves (once the lanes 8 apart agree, a rotation by 4 within a row
// reaches what the exchange would).  wave_sum_lds is the same tree by way of
// LDS, twelve dependent trips: the same bits, later.
__device__ __forceinline__ double of_words(uint32_t lo, uint32_t hi) {
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

template <int kCtrl>
__device__ __forceinline__ double from_dpp(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)u, kCtrl, 0xF, 0xF, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(u >> 32), kCtrl, 0xF, 0xF, true);
  return of_words(lo, hi);
}

template <int kOff>
__device__ __forceinline__ double add_lane_xor(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t l = (uint32_t)u, h = (uint32_t)(u >> 32);
  if constexpr (kOff == 32) {
    const u32x2 lo = __builtin_amdgcn_permlane32_swap(l, l, false, false);
    const u32x2 hi = __builtin_amdgcn_permlane32_swap(h, h, false, false);
    return of_words(lo.x, hi.x) + of_words(lo.y, hi.y);
  } else if constexpr (kOff == 16) {
    const u32x2 lo = __builtin_amdgcn_permlane16_swap(l, l, false, false);
    const u32x2 hi = __builtin_amdgcn_permlane16_swap(h, h, false, false);
    return of_words(lo.x, hi.x) + of_words(lo.y, hi.y);
  } else if constexpr (kOff == 8) {
    return v + from_dpp<0x128>(v);  // row_ror:8
  } else if constexpr (kOff == 4) {
    return v + from_dpp<0x124>(v);  // row_ror:4
  } else if constexpr (kOff == 2) {
    return v + from_dpp<0x4E>(v);   // quad_perm [2,3,0,1]
  } else {
    return v + from_dpp<0xB1>(v);   // quad_perm [1,0,3,2]
  }
}

//
// kLast: the last exchange, 1 or 2.  With 2 the odd lanes hold the sums of the
// tree's lanes l and l + 32 (see unit_sum), and only they come out right.
template <int kLast = 1>
__device__ __forceinline__ double wave_sum(double v) {
  if constexpr (kLast == 1) {
    v = add_lane_xor<32>(v);
    v = add_lane_xor<16>(v);
    v = add_lane_xor<8>(v);
    v = add_lane_xor<4>(v);
    v = add_lane_xor<2>(v);
    return add_lane_xor<1>(v);
  } else {
    v = add_lane_xor<32>(v);
    v = add_lane_xor<16>(v);
    v = add_lane_xor<8>(v);
    v = add_lane_xor<4>(v);
    return add_lane_xor<2>(v);
  }
}

template <int kLast = 1>
__device__ __forceinline__ double wave_sum_lds(double v) {
#pragma unroll
  for (int off = 32; off >= kLast; off >>= 1) v = v + __shfl_xor(v, off, 64);
  return v;
}

// Clip coefficient from the whole-shard sum of squares: min(1, max / (norm +
// 1e-6)) in double, rounded once to float; a NaN norm gives NaN, as torch's
// clamp does.
__device__ __forceinline__ float clip_coef(double total, float max_norm) {
  const double c = (double)max_norm / (__builtin_sqrt(total) + 1e-6);
  return (float)(c >= 1.0 ? 1.0 : c);
}

// Segments a and b of the elements i and k, searching [lo, hi] (segments
// overlapping the unit or tile): both at a time, as each step waits for a load.
// UNIFORM: the same for the whole wave, by scalar loads.  One after the other and
// by vector loads, a step of 1e6 elements in segments of 37 took 10.1 us (R = 1)
// and takes 9.4, of 1.4e7 in segments of 700 8 to 11 % longer.
template <bool UNIFORM>
__device__ __forceinline__ void find_segs(const int64_t* off, int lo, int hi, int64_t i,
                                          int64_t k, int& a, int& b) {
  int a1 = hi, b1 = hi;
  a = b = lo;
  while (a < a1 || b < b1) {
    const int am = (a + a1 + 1) >> 1, bm = (b + b1 + 1) >> 1;
    const int64_t x = UNIFORM ? ld_uniform(off + am) : off[am];
    const int64_t y = UNIFORM ? ld_uniform(off + bm) : off[bm];
    if (a < a1) {
      if (x <= i) a = am; else a1 = am - 1;
    }
    if (b < b1) {
      if (y <= k) b = bm; else b1 = bm - 1;
    }
  }
}

// Fixed-tree total of the (piece, wave) partials of finalize chunk c: thread
// j folds pieces j, j + 256, ... (each piece's kWaves slots in order), a
// wave64 butterfly, then the 4 wave totals in order.  Called by all threads
// of the workgroup; the result is valid in thread 0.  The partials were
// written by an earlier kernel.
__device__ __forceinline__ double chunk_fold(const int64_t* chunk_p0, const double* partials,
                                             int64_t c, double* red) {
  const int64_t p0 = chunk_p0[c];
  const int64_t p1 = chunk_p0[c + 1];
  double acc = 0.0;
  for (int64_t p = p0 + threadIdx.x; p < p1; p += kBlock) {
    const double* q = partials + p * kWaves;
    const f64x2 w0 = *reinterpret_cast<const f64x2*>(q);
    const f64x2 w1 = *reinterpret_cast<const f64x2*>(q + 2);
    acc = acc + w0.x;
    acc = acc + w0.y;
    acc = acc + w1.x;
    acc = acc + w1.y;
  }
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  const double sum = ((red[0] + red[1]) + red[2]) + red[3];
  __syncthreads();
  return sum;
}

// Fixed-tree total of n_seg per-segment values: thread t adds values t,
// t + 256, ... in order, a wave64 butterfly, then the 4 wave totals in order.
// Called by all threads; the result is valid in thread 0.
template <typename Get>
__device__ __forceinline__ double total_fold(int64_t n_seg, Get get, double* red) {
  double acc = 0.0;
  for (int64_t s = threadIdx.x; s < n_seg; s += kBlock) acc = acc + get(s);
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  const double sum = ((red[0] + red[1]) + red[2]) + red[3];
  __syncthreads();
  return sum;
}

// The chunk total of chunk_fold by one wave64: each lane stands for threads
// lane, lane + 64, lane + 128 and lane + 192 of that tree, so the bits are the
// same.  Their four loads go out together: with one after another the fold of
// a short pass (512 pieces) outlasts the pass that carries it.
__device__ __forceinline__ double chunk_fold_wave(const int64_t* chunk_p0, const double* partials,
                                                  int64_t c) {
  const int64_t p0 = chunk_p0[c];
  const int64_t p1 = chunk_p0[c + 1];
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (int64_t p = p0 + threadIdx.x; p < p1; p += 256) {
    f64x2 w0[4], w1[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t pk = p + 64 * k < p1 ? p + 64 * k : p;
      w0[k] = *reinterpret_cast<const f64x2*>(partials + pk * kWaves);
      w1[k] = *reinterpret_cast<const f64x2*>(partials + pk * kWaves + 2);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (p + 64 * k < p1) {
        acc[k] = acc[k] + w0[k].x;
        acc[k] = acc[k] + w0[k].y;
        acc[k] = acc[k] + w1[k].x;
        acc[k] = acc[k] + w1[k].y;
      }
    }
  }
  double w[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) w[k] = wave_sum(acc[k]);
  return ((w[0] + w[1]) + w[2]) + w[3];
}

// A carried finalize (see Carry): the first kCarryMaxChunks workgroups of a
// kernel launched with that many more fold the previous pass's partials, one
// chunk each, with the tree of k_seg_chunks, and write each segment's float
// sum; returns true in those (which then have nothing else to do).  Every
// workgroup calls it first; the others take their units from index
// blockIdx.x - carried.  Workgroups go to the eight XCDs round robin, so with
// eight in front every unit stays on the XCD that has it without a carry: at
// small shard sizes the next pass finds the unit in that XCD's L2.  In front,
// the fold runs while the others stream, also when the grid does not fit on
// the chip at once.  The partials come from an earlier kernel of the same
// stream, so plain loads see them.
static_assert(kCarryMaxChunks % 8 == 0, "carriers must not move units to other XCDs");

__device__ __forceinline__ bool run_carry(const Carry& c) {
  if (c.partials == nullptr || blockIdx.x >= kCarryMaxChunks) return false;
  if (blockIdx.x < c.n_chunks) {
    const double sum = chunk_fold_wave(c.chunk_p0, c.partials, blockIdx.x);
    if (threadIdx.x == 0) c.out[blockIdx.x] = (float)sum;
  }
  return true;
}

__device__ __forceinline__ int carried(const Carry& c) {
  return c.partials != nullptr ? kCarryMaxChunks : 0;
}

// The segments of one unit: ti its tile, lo..hi the segments it overlaps
// (lo > hi past the shard's end).  Of a tile of few segments (2 to 64) each lane
// asks for one, all at once: end is where it ends (elements from the unit's first,
// within 0 to kUnit), decays has a bit for each.  What a wave then needs of them it
// has in registers; with a search instead, a chain of eight loads, the one unit of
// the last tile that several segments share outlasted the others of a short pass:
// eight steps and FedAvg of 426,000 elements (R = 4, a layer's nine segments) took
// 55.8 us and 51.5 with this.
struct UnitSegs {
  TileInfo ti;
  int lo, hi;
  int end;
  uint64_t decays;
  __device__ __forceinline__ bool few() const { return ti.nseg <= 64; }
};

__device__ __forceinline__ UnitSegs unit_segs(const LayoutDev& L, const TileInfo& ti, int64_t u,
                                              int lane) {
  UnitSegs s;
  s.ti = ti;
  s.lo = s.hi = ti.seg0;
  s.end = kUnit;
  s.decays = 0;
  // (expected paths are marked where a short round gains from it, by up to 1 %)
  if (__builtin_expect(ti.nseg > 1, 0)) {
    const int64_t b = u * kUnit;
    const int64_t left = L.n - b;
    const int n = left < kUnit ? (int)left : kUnit;
    if (left <= 0) {   // (segments 0 and 1 exist: the tile has several)
      s.lo = 1;
      s.hi = 0;
    } else if (s.few()) {
      int decay = 0;
      if (lane < ti.nseg) {
        const int64_t end = L.seg_off[ti.seg0 + 1 + lane] - b;
        decay = L.seg_decay[ti.seg0 + lane];
        s.end = end < 0 ? 0 : end < kUnit ? (int)end : kUnit;
      }
      s.decays = __ballot(decay);
      s.lo += __popcll(__ballot(s.end <= 0));
      s.hi += __popcll(__ballot(s.end < n));
    } else {
      find_segs<true>(L.seg_off, ti.seg0, ti.seg0 + ti.nseg - 1, b, b + n - 1, s.lo, s.hi);
    }
  }
  return s;
}

// Segment of each of a lane's elements, for a unit of several; -1 past the
// shard's end.
template <int kGap>
__device__ __forceinline__ void lane_segs(const LayoutDev& L, const UnitSegs& us, int64_t u,
                                          int lane, int seg[8]) {
  const int at = lane * (kGap == kWhole ? kVec : 4);
  const int64_t base = u * kUnit + at;
  if (us.few()) {
#pragma unroll
    for (int e = 0; e < 8; ++e) seg[e] = us.lo;
#pragma unroll 1
    for (int j = us.lo; j < us.hi; ++j) {
      const int end = __builtin_amdgcn_readlane(us.end, j - us.ti.seg0) - at;
#pragma unroll
      for (int e = 0; e < 8; ++e) seg[e] += (e / 4) * kGap + e % 4 >= end;
    }
    if (base - at + kUnit > L.n) {
      const int left = (int)(L.n - base);
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if ((e / 4) * kGap + e % 4 >= left) seg[e] = -1;
    }
    return;
  }
  int s[2];
  find_segs<false>(L.seg_off, us.lo, us.hi, base, base + kGap, s[0], s[1]);
  int64_t next[2] = {L.seg_off[s[0] + 1], L.seg_off[s[1] + 1]};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t i = base + h * kGap + e;
      if (i < L.n)
        while (i >= next[h]) next[h] = L.seg_off[++s[h] + 1];
      seg[4 * h + e] = i < L.n ? s[h] : -1;
    }
  }
}

// Whether segment seg decays, for one of the unit's.
__device__ __forceinline__ bool decays(const LayoutDev& L, const UnitSegs& us, int seg) {
  return us.few() ? (us.decays >> (seg - us.ti.seg0)) & 1 : L.seg_decay[seg] != 0;
}

// acc + x * x in double: a float's square is exact, so fused is the same.
template <typename T>
__device__ __forceinline__ double add_square(double acc, T x) {
  return __builtin_fma((double)x, (double)x, acc);
}

// One partial, valid in lane kSumLane: the exact double squares of 8
// consecutive elements summed in order, then the butterfly over the 64 groups
// of 8.  On halves a lane has 4 of a group of each half, its first 4 if the lane
// is even: the odd lanes go on from their neighbour's sums with their own 4 and
// add the two halves' groups, lanes 32 apart in the tree.  So the tree over
// element indices is the same in every pass, and the clip total has the same
// bits with and without a gradient scratch.  Four steps of the 8B shard take
// 28.41 ms with it and 28.41 when each lane summed what it holds, the 1 Mi round
// 31.6 and 31.4 us; moving the elements between the lanes instead, 28.58 ms.
template <int kGap>
constexpr int kSumLane = kGap == kWhole ? 0 : 1;

template <int kGap, bool LDS, typename T>
__device__ __forceinline__ double unit_sum(const T g[8]) {
  if constexpr (kGap == kWhole) {
    double acc = 0.0;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc = add_square(acc, g[e]);
    return LDS ? wave_sum_lds(acc) : wave_sum(acc);
  } else {
    double h0 = 0.0, h1 = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      h0 = add_square(h0, g[e]);
      h1 = add_square(h1, g[4 + e]);
    }
    h0 = from_dpp<0xB1>(h0);
    h1 = from_dpp<0xB1>(h1);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      h0 = add_square(h0, g[e]);
      h1 = add_square(h1, g[4 + e]);
    }
    return LDS ? wave_sum_lds<2>(h0 + h1) : wave_sum<2>(h0 + h1);
  }
}

// Sums of squares of unit u: one partial per (piece, unit) of its tile; 0 for
// the tile's segments that the unit does not touch.  (g is 0 past the shard's
// end, and so are here the other segments' elements: adding 0 changes no bit.)
template <int kGap, bool LDS = false, typename T>
__device__ __forceinline__ void unit_sumsq(double* partials, const UnitSegs& us, int64_t u,
                                           int lane, const int seg[8], const T g[8]) {
  double* out = partials + (int64_t)us.ti.piece0 * kWaves + u % kWaves;
  if (__builtin_expect(us.lo == us.hi, 1)) {
    const double tot = unit_sum<kGap, LDS>(g);
    if (lane == kSumLane<kGap>) out[(int64_t)(us.lo - us.ti.seg0) * kWaves] = tot;
  } else {
    for (int sj = us.lo; sj <= us.hi; ++sj) {
      T of[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) of[e] = seg[e] == sj ? g[e] : T(0);
      const double tot = unit_sum<kGap, LDS>(of);
      if (lane == kSumLane<kGap>) out[(int64_t)(sj - us.ti.seg0) * kWaves] = tot;
    }
  }
  for (int j = lane; j < us.ti.nseg; j += 64)
    if (us.ti.seg0 + j < us.lo || us.ti.seg0 + j > us.hi) out[(int64_t)j * kWaves] = 0.0;
}

// A streaming workgroup is one wave; its first unit (or group of units) and
// its stride, behind the carriers.
struct Place {
  int lane;
  int64_t at, stride;
};

__device__ __forceinline__ Place place(const Carry& c) {
  const int64_t first = carried(c);
  return {(int)threadIdx.x, blockIdx.x - first, (int64_t)gridDim.x - first};
}

// AdamW on 8 elements: p already decayed, g clipped; m, v and p updated.
//
// The division and the two correctly rounded operations before it are a third
// of the step's instructions as the compiler expands them, most of it for
// operands at the ends of the range.  When no lane of the wave has one (kLo,
// kHi below, and s.rbc2, which the host sets when eps and bc2_sqrt allow), the
// same results come cheaper:
//  - sqrt: x * rsq(x) with one correction by its exact residual.  That it is the
//    correctly rounded root rests on the values the instruction returns, so the
//    tests compare every float of the range;
//  - / bc2_sqrt: by its correctly rounded reciprocal and two corrections (the
//    first makes the quotient faithful, the second by Markstein's theorem
//    correctly rounded);
//  - mn / den: reciprocal, one Newton step, two corrections: the operations of
//    the full division where its scaling does nothing.
// Per round: 8B shard (R = 8, A = 4) 29.62 to 29.16 ms, 1 Mi elements (R = 4,
// from cache) 37.8 to 37.1 us; together with the rounding instruction.
constexpr float kMnLo = 0x1p-60f, kMnHi = 0x1p30f, kVnLo = 0x1p-100f, kVnHi = 0x1p60f;

__device__ __forceinline__ void adam8(const AdamScalars& s, const float g[8], float p[8],
                                      float m[8], float v[8]) {
  float m_lo = kMnHi, m_hi = 0.f, v_lo = kVnHi, v_hi = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    m[e] = (s.b1 * m[e]) + (s.omb1 * g[e]);
    v[e] = (s.b2 * v[e]) + (s.omb2 * (g[e] * g[e]));
    const float am = __builtin_fabsf(m[e]);
    m_lo = __builtin_fminf(m_lo, am);
    m_hi = __builtin_fmaxf(m_hi, am);
    v_lo = __builtin_fminf(v_lo, v[e]);
    v_hi = __builtin_fmaxf(v_hi, v[e]);
  }
  // (a NaN is in neither minimum nor maximum; it comes out NaN either way)
  const bool in_range = m_lo >= kMnLo && m_hi <= kMnHi && v_lo >= kVnLo && v_hi <= kVnHi;
  if (s.rbc2 > 0.f && __all(in_range)) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float y = __builtin_amdgcn_rsqf(v[e]);
      float r = v[e] * y;
      r = __builtin_fmaf(__builtin_fmaf(-r, r, v[e]), 0.5f * y, r);
      float q = r * s.rbc2;
      q = __builtin_fmaf(__builtin_fmaf(-s.bc2_sqrt, q, r), s.rbc2, q);
      q = __builtin_fmaf(__builtin_fmaf(-s.bc2_sqrt, q, r), s.rbc2, q);
      const float den = q + s.eps;
      float z = __builtin_amdgcn_rcpf(den);
      z = __builtin_fmaf(__builtin_fmaf(-den, z, 1.0f), z, z);
      float u = m[e] * z;
      u = __builtin_fmaf(__builtin_fmaf(-den, u, m[e]), z, u);
      u = __builtin_fmaf(__builtin_fmaf(-den, u, m[e]), z, u);
      p[e] = p[e] - (s.step_size * u);
    }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float den = (__builtin_sqrtf(v[e]) / s.bc2_sqrt) + s.eps;
      p[e] = p[e] - (s.step_size * (m[e] / den));
    }
  }
}

// The AdamW step on the fp32 state, and the bf16 working copy.
// MODE 0: fused with the reduction of the R peer gradients; 2: of the fp32
// gradient g_in.  The gradient is scaled by the clip coefficient when
// a.clip_total is set.  SUMS 1: per-piece sums of squares of g (before
// clipping); 2: the same, exchanged by way of LDS.
// Elements on halves: the 8B shard's step (R = 8) runs at 6.38 TB/s and 6.24 on
// whole vectors, the 1 Mi round takes 31.7 and 34.0 us.  RT kMany (the generic
// count, for more than 24 peers): on whole vectors, as twice the loads cost more
// than whole lines give (R = 64 5.56 TB/s on halves, 5.62 whole).
constexpr int kMany = 99;

// Waves a SIMD has registers for, at least: what a short pass, which has no other
// limit, can use.  (The compiler would take a few registers more for paths that one
// wave runs.)
template <int RT, int SUMS>
constexpr int kStepWaves = RT != 0 && RT != kMany ? 5 : SUMS == 0 ? 4 : 3;

template <int RT, int MODE, int SUMS>
__global__ void __launch_bounds__(64, (kStepWaves<RT, SUMS>)) k_step(const StepArgs a) {
  constexpr int kGap = RT == kMany ? kWhole : kHalves;
  constexpr int kStreams = RT == kMany ? 0 : RT;
  args_in<MODE == 2 ? 1 : kStreams == 0 ? 8 : kStreams>(a);
  if (run_carry(a.carry)) return;
  const Place w = place(a.carry);
  const int lane = w.lane;
  const int64_t n_units = a.L.n_tiles * kWaves;  // past n too: their partials are 0
  for (int64_t u = w.at; u < n_units; u += w.stride) {
    const int64_t base = u * kUnit + lane * (kGap == kWhole ? kVec : 4);
    const bool full = (u + 1) * kUnit <= a.L.n;

    // asked for before the streams, so that it is there when they are
    i32x4 tile = ld_uniform(reinterpret_cast<const i32x4*>(a.L.tiles) + u / kWaves);
    const bool clip = a.clip_total != nullptr;
    double total =
        ld_uniform(clip ? a.clip_total : reinterpret_cast<const double*>(a.L.tiles));

    float g[8];
    float p[8], m[8], v[8];
    if (__builtin_expect(full, 1)) {
      load_f32x8<kGap>(a.master + base, p);
      load_f32x8<kGap>(a.m + base, m);
      load_f32x8<kGap>(a.v + base, v);
      if constexpr (MODE == 2) {
        load_f32x8<kGap>(a.g_in + base, g);
        loads_out();
      } else {
        reduce_vec<kStreams, kGap>(a, base, g);
      }
    } else {
      // (moments of 1 past the end keep the wave on the short forms)
      const Cut c = cut_at(a.L.n, base);
      load_f32x8_cut<kGap>(a.master + base, c, p);
      load_f32x8_cut<kGap>(a.m + base, c, m, 1.f);
      load_f32x8_cut<kGap>(a.v + base, c, v, 1.f);
      if constexpr (MODE == 2) load_f32x8_cut<kGap>(a.g_in + base, c, g);
      else reduce_cut<kStreams, kGap>(a, base, g);
    }

    // (not looked at before the streams' loads are out)
    asm volatile("" : "+s"(tile), "+s"(total));
    const TileInfo ti{tile.x, tile.y, tile.z, tile.w};
    const UnitSegs us = unit_segs(a.L, ti, u, lane);
    int seg[8];
    if (us.lo != us.hi) lane_segs<kGap>(a.L, us, u, lane, seg);

    const AdamScalars& s = a.s;
    const float coef = clip ? clip_coef(total, a.clip_max) : 1.0f;
    float gc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) gc[e] = clip ? g[e] * coef : g[e];
    float d[8];
    if (us.lo == us.hi) {
      const bool dec = us.ti.nseg == 1 ? us.ti.decay : decays(a.L, us, us.lo);
      const float du = dec ? s.decay : 1.0f;
#pragma unroll
      for (int e = 0; e < 8; ++e) d[e] = du;
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) d[e] = seg[e] >= 0 && decays(a.L, us, seg[e]) ? s.decay : 1.0f;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) p[e] = p[e] * d[e];
    adam8(s, gc, p, m, v);
    if (__builtin_expect(full, 1)) {
      store_f32x8<kGap>(a.master + base, p);
      store_f32x8<kGap>(a.m + base, m);
      store_f32x8<kGap>(a.v + base, v);
      if (MODE == 0 || a.working) store_bf16x8<kGap>(a.working + base, p);
    } else {
      const Cut c = cut_at(a.L.n, base);
      store_f32x8_cut<kGap>(a.master + base, c, p);
      store_f32x8_cut<kGap>(a.m + base, c, m);
      store_f32x8_cut<kGap>(a.v + base, c, v);
      if (MODE == 0 || a.working) store_bf16x8_cut<kGap>(a.working + base, c, p);
    }
    if constexpr (SUMS != 0) unit_sumsq<kGap, SUMS == 2>(a.partials, us, u, lane, seg, g);
  }
}

// The reduction of the R peer gradients alone.  OUT 1: to fp32 (g_out); 3: to
// the bf16 wire format (wire_out); 4: no output but the sums of squares.
// SUMSQ: per-piece sums of squares of g.  A wave takes NV consecutive units of
// a tile, all their loads issued first: a pass of few streams has too little
// in flight per wave otherwise.
template <int RT, int OUT, bool SUMSQ, int NV>
__global__ void __launch_bounds__(64) k_reduce(const StepArgs a) {
  if (run_carry(a.carry)) return;
  const Place w = place(a.carry);
  const int lane = w.lane;
  // an fp32 output is written on halves
  constexpr int kGap = OUT == 1 ? kHalves : kWhole;
  const int at = lane * (OUT == 1 ? 4 : kVec);
  const int64_t n_groups = a.L.n_tiles * (kWaves / NV);
  for (int64_t b = w.at; b < n_groups; b += w.stride) {
    const int64_t u0 = b * NV;
    i32x4 tile{};
    if constexpr (SUMSQ) tile = ld_uniform(reinterpret_cast<const i32x4*>(a.L.tiles) + u0 / kWaves);
    float g[NV][8];
    if ((u0 + NV) * kUnit <= a.L.n) {
      if constexpr (NV == 1) {
        reduce_vec<RT, kGap>(a, u0 * kUnit + at, g[0]);
      } else {
        u32x4 x[NV][RT];
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
          for (int r = 0; r < RT; ++r)
            x[i][r] = ld_once(reinterpret_cast<const u32x4*>(a.grads[r] + (u0 + i) * kUnit +
                                                             lane * kVec));
        loads_out();
#pragma unroll
        for (int i = 0; i < NV; ++i) {
          float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int r = 0; r < RT; ++r) add_bf16x8(acc, x[i][r]);
#pragma unroll
          for (int e = 0; e < 8; ++e) g[i][e] = acc[e] * a.grad_scale;
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < NV; ++i)
        reduce_cut<RT, kGap>(a, (u0 + i) * kUnit + at, g[i]);
    }
    if constexpr (OUT == 3) pause();
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int64_t base = (u0 + i) * kUnit + at;
      const bool full = (u0 + i + 1) * kUnit <= a.L.n;
      // (before the stores: where the paths of one and of several segments meet
      // the compiler waits for the searches' loads, and so for stores before them)
      UnitSegs us{};
      int seg[8];
      if constexpr (SUMSQ) {
        if (i == 0) asm volatile("" : "+s"(tile));
        us = unit_segs(a.L, TileInfo{tile.x, tile.y, tile.z, tile.w}, u0 + i, lane);
        if (us.lo != us.hi) lane_segs<kGap>(a.L, us, u0 + i, lane, seg);
      }
      // The sums work on copies made before the stores: an instruction that writes
      // a register which a store before it has yet to read waits for that, 0.2 us
      // (R = 8 on 2.7e7 elements 97.7 us so and 91.0 with copies).
      double d[8];
      if constexpr (SUMSQ) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          d[e] = (double)g[i][e];
          if constexpr (OUT == 1) asm volatile("" : "+v"(d[e]));
        }
      }
      if constexpr (OUT == 1) {
        if (full) store_f32x8<kGap>(a.g_out + base, g[i]);
      } else if constexpr (OUT == 3) {
        if (full) st(reinterpret_cast<u32x4*>(a.wire_out + base), pack_bf16x8(g[i]));
      }
      if constexpr (OUT != 4) {
        if (!full) {
          if constexpr (OUT == 1) store_f32x8_cut<kGap>(a.g_out + base, cut_at(a.L.n, base), g[i]);
          else store_bf16x8_cut<kGap>(a.wire_out + base, cut_at(a.L.n, base), g[i]);
        }
      }
      if constexpr (SUMSQ) unit_sumsq<kGap>(a.partials, us, u0 + i, lane, seg, d);
    }
  }
}

// FedAvg: master = sum_g w_g * f32(rep_g), ascending g; working = bf16(master).
// OUTER: the outer optimiser step on that average instead:
//   delta = prev - xbar; buf = mu * buf + delta;
//   d = nesterov ? delta + mu * buf : buf; p = prev - eta * d;
//   master = prev = p; working = bf16(p).
template <int GT, bool OUTER>
__global__ void __launch_bounds__(64) k_fedavg(const FedArgs a) {
  if (run_carry(a.carry)) return;
  const Place w = place(a.carry);
  const int64_t n_units = (a.n + kUnit - 1) / kUnit;
  for (int64_t u = w.at; u < n_units; u += w.stride) {
    const int64_t base = u * kUnit + w.lane * 4;
    const bool full = (u + 1) * kUnit <= a.n;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float prev[8] = {}, buf[8] = {};
    if (full) {
      if constexpr (OUTER) {
        load_f32x8<kHalves>(a.prev + base, prev);
        load_f32x8<kHalves>(a.buf + base, buf);
      }
      sum_streams<GT, kHalves>([&](int k) { return a.reps[k] + base; }, a.G,
                               [&](int k, u32x4 x) { fma_free_bf16x8(acc, a.w[k], x); });
    } else {
      if constexpr (OUTER) {
        load_f32x8_cut<kHalves>(a.prev + base, cut_at(a.n, base), prev);
        load_f32x8_cut<kHalves>(a.buf + base, cut_at(a.n, base), buf);
      }
      sum_streams_cut<GT, kHalves>([&](int k) { return a.reps[k]; }, a.G, base, a.n,
                                   [&](int k, u32x4 x) { fma_free_bf16x8(acc, a.w[k], x); });
    }
    if constexpr (OUTER) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float delta = prev[e] - acc[e];
        const float b = (a.mu * buf[e]) + delta;
        const float d = a.nesterov ? (delta + (a.mu * b)) : b;
        acc[e] = prev[e] - (a.eta * d);
        buf[e] = b;
      }
    }
    if constexpr (!OUTER) pause();
    if (full) {
      store_f32x8<kHalves>(a.master + base, acc);
      store_bf16x8<kHalves>(a.working + base, acc);
      if constexpr (OUTER) {
        store_f32x8<kHalves>(a.prev + base, acc);
        store_f32x8<kHalves>(a.buf + base, buf);
      }
    } else {
      const Cut c = cut_at(a.n, base);
      store_f32x8_cut<kHalves>(a.master + base, c, acc);
      store_bf16x8_cut<kHalves>(a.working + base, c, acc);
      if constexpr (OUTER) {
        store_f32x8_cut<kHalves>(a.prev + base, c, acc);
        store_f32x8_cut<kHalves>(a.buf + base, c, buf);
      }
    }
  }
}

// Per-segment totals of the (piece, wave) partials, in double, in fixed
// trees that do not depend on the grid.  Stage 1: one workgroup per chunk of
// up to kChunkPieces pieces of one segment; thread j folds pieces j, j+256,
// ... (each piece's kWaves slots in order), then a wave64 butterfly and the 4
// wave totals in order.  Stage 2: one thread per segment adds its chunks in
// order (double per segment, and its float rounding if requested); skipped
// when every segment is one chunk.  Stage 3 (whole-shard total, for
// clipping): one workgroup folds the segments.
// DIRECT (every segment is a single chunk, so chunk c is segment c): the
// chunk sum is the segment's total; write it, and its float rounding if
// requested, in place of stage 2 (which would add it to 0.0: the same bits).
template <bool DIRECT>
__global__ void __launch_bounds__(kBlock) k_seg_chunks(const LayoutDev L, const double* partials,
                                                       double* chunk_sums, float* out) {
  __shared__ double red[4];
  for (int64_t c = blockIdx.x; c < L.n_chunks; c += gridDim.x) {
    const double sum = chunk_fold(L.chunk_p0, partials, c, red);
    if (threadIdx.x == 0) {
      chunk_sums[c] = sum;
      if (DIRECT && out) out[c] = (float)sum;
    }
  }
}

__global__ void __launch_bounds__(kBlock) k_seg_totals(const LayoutDev L, const double* chunk_sums,
                                                       double* seg_dbl, float* out) {
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  for (int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x; s < L.n_seg; s += stride) {
    double acc = 0.0;
    for (int64_t c = L.seg_chunk0[s]; c < L.seg_chunk0[s + 1]; ++c) acc = acc + chunk_sums[c];
    seg_dbl[s] = acc;
    if (out) out[s] = (float)acc;
  }
}

__global__ void __launch_bounds__(kBlock) k_total(const int64_t n_seg, const double* seg_dbl,
                                                  double* total) {
  __shared__ double red[4];
  const double tot = total_fold(n_seg, [&](int64_t s) { return seg_dbl[s]; }, red);
  if (threadIdx.x == 0) *total = tot;
}

// Broadcast receive: master = recv; working = bf16(recv).
__global__ void __launch_bounds__(64) k_bcast_recv(const BcastArgs a) {
  if (run_carry(a.carry)) return;
  const Place at = place(a.carry);
  const int64_t n = a.n;
  const int64_t n_units = (n + kUnit - 1) / kUnit;
  for (int64_t ui = at.at; ui < n_units; ui += at.stride) {
    const int64_t base = ui * kUnit + at.lane * 4;
    if ((ui + 1) * kUnit <= n) {
      const f32x4 u = ld_once(reinterpret_cast<const f32x4*>(a.recv + base));
      const f32x4 w = ld_once(reinterpret_cast<const f32x4*>(a.recv + base + kHalves));
      loads_out();
      const float x[8] = {u.x, u.y, u.z, u.w, w.x, w.y, w.z, w.w};
      store_f32x8<kHalves>(a.master + base, x);
      store_bf16x8<kHalves>(a.working + base, x);
    } else {
      const Cut c = cut_at(n, base);
      float x[8];
      load_f32x8_cut<kHalves>(a.recv + base, c, x);
      store_f32x8_cut<kHalves>(a.master + base, c, x);
      store_bf16x8_cut<kHalves>(a.working + base, c, x);
    }
  }
}

// Workgroups as Shape says, behind the carriers of a carried finalize.
template <typename Args>
hipError_t launch(const void* fn, const Args& a, Shape sh, hipStream_t st) {
  void* args[] = {const_cast<Args*>(&a)};
  const unsigned g = sh.grid + (a.carry.partials != nullptr ? (unsigned)kCarryMaxChunks : 0u);
  return hipLaunchKernel(fn, dim3(g), dim3(64), args, sh.lds, st);
}

// The exchange by way of LDS (SUMS 2) is asked for from 3 to 12 streams.
template <int RT, int SUMS>
hipError_t step_of(const StepArgs& a, Shape sh, hipStream_t st) {
  if constexpr (SUMS == 2 && (RT == 1 || RT == 2 || RT == kMany)) return hipErrorInvalidValue;
  else return launch((const void*)k_step<RT, 0, SUMS>, a, sh, st);
}

template <int SUMS>
hipError_t dispatch_step(const StepArgs& a, Shape sh, hipStream_t st) {
  switch (a.R) {
    case 1: return step_of<1, SUMS>(a, sh, st);
    case 2: return step_of<2, SUMS>(a, sh, st);
    case 3: return step_of<3, SUMS>(a, sh, st);
    case 4: return step_of<4, SUMS>(a, sh, st);
    case 5: return step_of<5, SUMS>(a, sh, st);
    case 6: return step_of<6, SUMS>(a, sh, st);
    case 7: return step_of<7, SUMS>(a, sh, st);
    case 8: return step_of<8, SUMS>(a, sh, st);
    default: return a.R > 24 ? step_of<kMany, SUMS>(a, sh, st) : step_of<0, SUMS>(a, sh, st);
  }
}

// Several units per workgroup (sh.units) where the passes of one or two peers
// ask for them.
template <int RT, int OUT, bool SUMSQ>
hipError_t reduce_units(const StepArgs& a, Shape sh, hipStream_t st) {
  if constexpr (OUT == 4 && (RT == 1 || RT == 2)) {
    if (sh.units == 4) return launch((const void*)k_reduce<RT, OUT, SUMSQ, 4>, a, sh, st);
  }
  if constexpr (OUT == 3 && RT == 1) {
    if (sh.units == 2) return launch((const void*)k_reduce<RT, OUT, SUMSQ, 2>, a, sh, st);
  }
  if (sh.units != 1) return hipErrorInvalidValue;
  return launch((const void*)k_reduce<RT, OUT, SUMSQ, 1>, a, sh, st);
}

template <int OUT, bool SUMSQ>
hipError_t dispatch_reduce(const StepArgs& a, Shape sh, hipStream_t st) {
  switch (a.R) {
    case 1: return reduce_units<1, OUT, SUMSQ>(a, sh, st);
    case 2: return reduce_units<2, OUT, SUMSQ>(a, sh, st);
    case 3: return reduce_units<3, OUT, SUMSQ>(a, sh, st);
    case 4: return reduce_units<4, OUT, SUMSQ>(a, sh, st);
    case 5: return reduce_units<5, OUT, SUMSQ>(a, sh, st);
    case 6: return reduce_units<6, OUT, SUMSQ>(a, sh, st);
    case 7: return reduce_units<7, OUT, SUMSQ>(a, sh, st);
    case 8: return reduce_units<8, OUT, SUMSQ>(a, sh, st);
    default: return reduce_units<0, OUT, SUMSQ>(a, sh, st);
  }
}

}  // namespace

hipError_t launch_local_step(const StepArgs& a, Shape sh, hipStream_t st) {
  if (!a.partials) return dispatch_step<0>(a, sh, st);
  return a.sum_by_lds ? dispatch_step<2>(a, sh, st) : dispatch_step<1>(a, sh, st);
}

hipError_t launch_reduce(const StepArgs& a, Shape sh, hipStream_t st) {
  return a.partials ? dispatch_reduce<1, true>(a, sh, st) : dispatch_reduce<1, false>(a, sh, st);
}

hipError_t launch_reduce_wire(const StepArgs& a, Shape sh, hipStream_t st) {
  return dispatch_reduce<3, false>(a, sh, st);
}

hipError_t launch_bcast_recv(const BcastArgs& a, Shape sh, hipStream_t st) {
  return launch((const void*)k_bcast_recv, a, sh, st);
}

hipError_t launch_adamw(const StepArgs& a, Shape sh, hipStream_t st) {
  return launch((const void*)k_step<1, 2, 0>, a, sh, st);
}

template <bool OUTER>
hipError_t dispatch_fedavg(const FedArgs& a, Shape sh, hipStream_t st) {
  switch (a.G) {
    case 1: return launch((const void*)k_fedavg<1, OUTER>, a, sh, st);
    case 2: return launch((const void*)k_fedavg<2, OUTER>, a, sh, st);
    case 3: return launch((const void*)k_fedavg<3, OUTER>, a, sh, st);
    case 4: return launch((const void*)k_fedavg<4, OUTER>, a, sh, st);
    case 5: return launch((const void*)k_fedavg<5, OUTER>, a, sh, st);
    case 6: return launch((const void*)k_fedavg<6, OUTER>, a, sh, st);
    case 7: return launch((const void*)k_fedavg<7, OUTER>, a, sh, st);
    case 8: return launch((const void*)k_fedavg<8, OUTER>, a, sh, st);
    default: return launch((const void*)k_fedavg<0, OUTER>, a, sh, st);
  }
}

hipError_t launch_fedavg(const FedArgs& a, Shape sh, hipStream_t st) {
  return a.prev ? dispatch_fedavg<true>(a, sh, st) : dispatch_fedavg<false>(a, sh, st);
}

hipError_t launch_seg_finalize(const LayoutDev& L, const double* partials, double* chunk_sums,
                               double* seg_dbl, float* out, double* total, hipStream_t st) {
  if (L.n_seg == 0) return hipSuccess;
  const int g1 = (int)(L.n_chunks < 65535 ? L.n_chunks : 65535);
  const bool direct = L.n_chunks == L.n_seg;
  double* stage1 = direct ? seg_dbl : chunk_sums;
  void* a1[] = {const_cast<LayoutDev*>(&L), &partials, &stage1, &out};
  hipError_t e = hipLaunchKernel(direct ? (const void*)k_seg_chunks<true>
                                        : (const void*)k_seg_chunks<false>,
                                 dim3((unsigned)g1), dim3(kBlock), a1, 0, st);
  if (e != hipSuccess) return e;
  if (direct) {
    if (!total) return hipSuccess;
    int64_t n_seg = L.n_seg;
    void* a3[] = {&n_seg, &seg_dbl, &total};
    return hipLaunchKernel((const void*)k_total, dim3(1), dim3(kBlock), a3, 0, st);
  }
  const int64_t b2 = (L.n_seg + kBlock - 1) / kBlock;
  const int g2 = (int)(b2 < 65535 ? b2 : 65535);
  void* a2[] = {const_cast<LayoutDev*>(&L), &chunk_sums, &seg_dbl, &out};
  e = hipLaunchKernel((const void*)k_seg_totals, dim3((unsigned)g2), dim3(kBlock), a2, 0, st);
  if (e != hipSuccess || !total) return e;
  int64_t n_seg = L.n_seg;
  void* a3[] = {&n_seg, &seg_dbl, &total};
  return hipLaunchKernel((const void*)k_total, dim3(1), dim3(kBlock), a3, 0, st);
}

hipError_t launch_zero_total(double* total, hipStream_t st) {
  int64_t n_seg = 0;
  const double* none = nullptr;
  void* a3[] = {&n_seg, &none, &total};
  return hipLaunchKernel((const void*)k_total, dim3(1), dim3(kBlock), a3, 0, st);
}

hipError_t launch_sumsq_only(const StepArgs& a, Shape sh, hipStream_t st) {
  return dispatch_reduce<4, true>(a, sh, st);
}

hipError_t noalloc_scratch(int device, void** ptr) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  if (device < 0 || device >= kMaxDevices || !ptr) return hipErrorInvalidValue;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[device]) {
    void* p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    addr[device] = p;
  }
  *ptr = addr[device];
  return hipSuccess;
}

}  // namespace flr
