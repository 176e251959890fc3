// gfx950 kernels of libdisdp: the W-way reduction of a shard's gradient
// contributions (the SmartSwitch's aggregation in DisDP, Sections III-A and
// III-C, in fp32 or in the integer format of Section III-B), optionally
// fused with the parameter server's mixed-precision Adam step and its bf16
// parameter copy (Section III-D, step 5).
//
// The path is a pure HBM stream: per element it reads W contributions and
// 12 bytes of state and writes 12 bytes of state and 2 bytes of copy, with
// a few dozen ALU operations in between.  No MFMA: there is no contraction.
// Design for CDNA4:
//   * one lane owns 4 consecutive elements, so every stream moves in 16-byte
//     (fp32) or 8-byte (bf16) vector accesses and each wave instruction
//     covers 1 KiB / 512 B of contiguous memory;
//   * a block owns a tile of one group per lane; all loads of a lane (W
//     contributions and p, m, v) are issued before any arithmetic, so each
//     lane keeps W + 3 vector loads in flight;
//   * one tile per block over a grid that covers the shard, so every byte is
//     read once and written once;
//   * data are touched once, so loads and stores carry the non-temporal hint;
//   * no atomics, no cross-lane traffic: each element's reduction is one
//     lane's serial chain in worker order, which makes results independent
//     of grid size and identical to an element-wise evaluation.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>
#include <cstdlib>
#include <cstring>

#include "disdp_launch.h"

// One rounding per written operation: never contract a*b+c into an FMA.
#pragma clang fp contract(off)

// Launch shapes.  The default ("solo") shape -- one-wave (64-lane) blocks
// each owning one tile of 64 four-element groups, non-temporal loads and
// stores, tiles in natural order -- was the best or tied-best in
// interleaved A/B runs on MI355X over the 7B/8, 13B/16 and 175B/64 shards;
// the alternatives measured were within 2% or slower (persistent grids, more
// groups per lane, 128- to 1024-lane blocks, wave-contiguous groups,
// XCD-chunked tile orders, hints on one side only).  One-wave blocks beat
// 256-lane blocks at the same resident waves by 2-6%: a retiring wave frees
// its slot at once instead of waiting for the slowest wave of its block.
// The "shared" shape (four-wave blocks, one occupancy cap per mode) is for
// a GPU whose compute kernels run on other streams at the same time: a
// retiring four-wave block leaves a hole a compute workgroup can take, so
// the chip is shared more evenly (see launch_shape below).
#define DISDP_LAUNCH_BOUNDS __launch_bounds__(256)
#define DISDP_WAVE_LAUNCH_BOUNDS __launch_bounds__(64)

namespace disdp {
namespace {

constexpr int kWave = 64;
constexpr int kMaxBlock = 256;   // lanes per block of the shared shape

// Vector types of the 4-element groups, declared only 4-byte aligned: a
// group of an array that starts off its natural vector boundary (arrays with
// unrelated misalignments) is one 16- or 8-byte access at a 4-byte-aligned
// address, which the global memory instructions take as they are (for
// naturally aligned groups the machine code is the same).
typedef float f32x4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2), aligned(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4), aligned(4)));

// A byte of global memory.  Every array is in the global address space,
// whatever struct its pointer came from (pinned host memory included: it has
// one address for both sides).
typedef __attribute__((address_space(1))) char *GlobalBytes;

// Non-temporal group loads and stores (every byte is touched once).  Typedefs
// and overloads, not templates: deducing the vector type would drop the
// typedef's 4-byte alignment.
#define DISDP_NT_ACCESS(T)                                                                 \
    typedef __attribute__((address_space(1))) T Global_##T;                                \
    __device__ __forceinline__ T ld_##T(GlobalBytes p)                                     \
    {                                                                                      \
        return __builtin_nontemporal_load(reinterpret_cast<const Global_##T *>(p));        \
    }                                                                                      \
    __device__ __forceinline__ void st(GlobalBytes p, T v)                                 \
    {                                                                                      \
        __builtin_nontemporal_store(v, reinterpret_cast<Global_##T *>(p));                 \
    }
DISDP_NT_ACCESS(f32x4)
DISDP_NT_ACCESS(u32x2)
DISDP_NT_ACCESS(i32x4)
#undef DISDP_NT_ACCESS

// Single elements, by plain accesses.
template <class T>
__device__ __forceinline__ T ld_one(GlobalBytes p)
{
    return *reinterpret_cast<const __attribute__((address_space(1))) T *>(p);
}
template <class T>
__device__ __forceinline__ void st_one(GlobalBytes p, T v)
{
    *reinterpret_cast<__attribute__((address_space(1))) T *>(p) = v;
}

// ---- element operations ---------------------------------------------------

// bf16 bits -> fp32: the bf16 pattern is the upper half of the fp32 one.
__device__ __forceinline__ float widen_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float widen_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// fp32 -> bf16 bits, round to nearest even; NaN -> quiet NaN with its sign.
__device__ __forceinline__ uint32_t to_bf16(float x)
{
    const uint32_t u = __float_as_uint(x);
    const uint32_t rounded = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
    const uint32_t qnan = ((u >> 16) & 0x8000u) | 0x7fc0u;
    return (u & 0x7fffffffu) > 0x7f800000u ? qnan : rounded;
}

// Four floats -> bf16 as to_bf16, two per register.  The hardware conversion
// (two floats an instruction) rounds to nearest even and keeps denormals as
// to_bf16 does; only its NaNs differ (they keep payload bits).
__device__ __forceinline__ u32x2 to_bf16x4(const float (&p)[4])
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 lo = __builtin_convertvector((f32x2{p[0], p[1]}), bf16x2);
    const bf16x2 hi = __builtin_convertvector((f32x2{p[2], p[3]}), bf16x2);
    u32x2 w = {__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
    if (__builtin_expect(__builtin_isunordered(p[0], p[1]) || __builtin_isunordered(p[2], p[3]),
                         0))
        w = u32x2{to_bf16(p[0]) | (to_bf16(p[1]) << 16), to_bf16(p[2]) | (to_bf16(p[3]) << 16)};
    return w;
}

// Contribution -> int32 at scale 2^k: exact scaling, rint (ties to even),
// saturation, NaN -> 0 (the integer switch format, Section III-B), in three
// instructions and no branches.
__device__ __forceinline__ int32_t quantize(float x, float scale)
{
    const float r = __builtin_rintf(x * scale);
    // The hardware conversion already has the format's saturation: a float
    // at or above 2^31 (+inf included) gives INT32_MAX, one below -2^31
    // (-inf included) INT32_MIN, NaN 0, anything else its (integral) value.
    // A C++ cast leaves those cases undefined, hence the instruction itself.
    int32_t q;
    asm("v_cvt_i32_f32 %0, %1" : "=v"(q) : "v"(r));
    return q;
}

__device__ __forceinline__ int32_t saturate32(int64_t s)
{
    const int64_t hi = s > INT32_MAX ? int64_t(INT32_MAX) : s;
    return static_cast<int32_t>(hi < INT32_MIN ? int64_t(INT32_MIN) : hi);
}

// The step constants of a launch: by value in the arguments, or read from
// memory when the kernel runs; either way by scalar loads (the constant
// address space) issued while the contributions are in flight.  Left to
// itself the compiler selects between the two addresses first, and each wave
// then waits for one more round trip to memory after its contributions have
// arrived; the empty asm keeps the reads under the (uniform) branch.
template <class A>
__device__ __forceinline__ StepScalars step_scalars_of(const A &a)
{
    StepScalars s = a.s;
    if (a.s_dev) {
        typedef const __attribute__((address_space(4))) float *ConstFloats;
        const ConstFloats c = (ConstFloats)(uintptr_t)a.s_dev;
        s = StepScalars{c[0], c[1], c[2], c[3], c[4], c[5], c[6], c[7], c[8], c[9]};
        asm volatile("" : "+s"(s.b1), "+s"(s.omb1), "+s"(s.b2), "+s"(s.omb2), "+s"(s.bc1),
                          "+s"(s.bc2), "+s"(s.decay), "+s"(s.lr), "+s"(s.eps),
                          "+s"(s.grad_scale));
    }
    return s;
}

// One AdamW step on one element (decoupled decay, bias-corrected moments,
// eps outside the square root), in the compiler's correctly rounded division
// and square root, for any values.
__device__ __forceinline__ void adamw(const StepScalars &s, float agg, float &p, float &m,
                                      float &v)
{
    const float g = agg * s.grad_scale;
    const float mi = s.b1 * m + s.omb1 * g;
    const float vi = s.b2 * v + s.omb2 * (g * g);
    const float mh = mi / s.bc1;
    const float vh = vi / s.bc2;
    const float d = sqrtf(vh) + s.eps;
    p = p * s.decay - s.lr * (mh / d);
    m = mi;
    v = vi;
}

// What a lane derives from the step constants while its loads are in
// flight, for the short forms of the two divisions by a bias correction c:
// zh = 1/c correctly rounded and zl = 1/c - zh.  `tame`: the constants lie
// where those forms hold (see adamw4).  `zero_v`: 1 when a second moment of
// zero is among them, that is when eps alone can be the divisor, else 0.
struct Reciprocals {
    float zh1, zl1, zh2, zl2;
    uint32_t zero_v;
    bool tame;
};

__device__ __forceinline__ Reciprocals reciprocals(const StepScalars &s)
{
    Reciprocals r;
    r.zh1 = 1.0f / s.bc1;
    r.zl1 = __builtin_fmaf(-s.bc1, r.zh1, 1.0f) * r.zh1;
    r.zh2 = 1.0f / s.bc2;
    r.zl2 = __builtin_fmaf(-s.bc2, r.zh2, 1.0f) * r.zh2;
    // not sunk to their use behind the waits for the loads
    asm volatile("" : "+v"(r.zh1), "+v"(r.zl1), "+v"(r.zh2), "+v"(r.zl2));
    // as integers (scalar compares): a sign bit or a NaN is above the ends
    constexpr uint32_t kLo = (127u - 24u) << 23, kOne = 127u << 23;
    constexpr uint32_t kEpsLo = (127u - 48u) << 23, kEps = (127u + 40u) << 23;
    r.zero_v = __float_as_uint(s.eps) >= kEpsLo ? 1 : 0;
    r.tame = __float_as_uint(s.bc1) - kLo <= kOne - kLo &&
             __float_as_uint(s.bc2) - kLo <= kOne - kLo && __float_as_uint(s.eps) <= kEps;
    return r;
}

// x / c, correctly rounded, for 2^-24 <= c <= 1 and 2^-96 <= |x| <= 2^60 or x
// = +0 (the quotient is +0 whatever the sign of zl; -0 would lose its sign).
// q is x * (1/c) with 1/c held in two floats, so within 0.5 + 2^-21 units of
// the quotient; the remainder x - q*c is then exact, and as zh is the
// correctly rounded 1/c one more step rounds correctly (Markstein, "Computation
// of elementary functions on the IBM RISC System/6000 processor", 1990).
__device__ __forceinline__ float div_const(float x, float c, float zh, float zl)
{
    const float q = __builtin_fmaf(x, zh, x * zl);
    return __builtin_fmaf(__builtin_fmaf(-q, c, x), zh, q);
}

// sqrt(x), correctly rounded on gfx950 for 2^-100 <= x <= 2^100 and +0: one
// correction of x * v_rsq_f32(x).  The correction depends on the significand
// and the exponent's parity only, that is 2^24 cases: tests/test_adam_range_gpu.py
// has each of them at four scales.
__device__ __forceinline__ float sqrt_mid(float x)
{
    constexpr uint32_t kLo = (127u - 100u) << 23;
    const uint32_t u = __float_as_uint(x);   // 1/sqrt(0) would be infinite
    const float y = __builtin_amdgcn_rsqf(__uint_as_float(u > kLo ? u : kLo));
    const float g = x * y;
    return __builtin_fmaf(__builtin_fmaf(-g, g, x), 0.5f * y, g);
}

// n / d as the compiler's correctly rounded division computes it where no
// operand needs scaling: 2^-60 <= |n| <= 2^44, 2^-48 <= d <= 2^46.
__device__ __forceinline__ float div_mid(float n, float d)
{
    float y = __builtin_amdgcn_rcpf(d);
    y = __builtin_fmaf(__builtin_fmaf(-d, y, 1.0f), y, y);
    float q = n * y;
    q = __builtin_fmaf(__builtin_fmaf(-d, q, n), y, q);
    return __builtin_fmaf(__builtin_fmaf(-d, q, n), y, q);
}

// adamw on the four elements of a lane, the same bits in fewer instructions
// (a W = 8 fp32 group 316 -> 230 vector instructions, 30 of them while its
// loads are in flight).
// The kernel is bound by memory at shard sizes, but a launch of a few
// megabytes runs its waves in step -- all load, all compute, all store -- and
// the arithmetic adds to its time.  The short divisions and square root need
// the moments in a middle range (2^-60..2^20 for |m|, 2^-96..2^60 for v) or
// exactly zero, as those of padding, unused rows and frozen weights are; a
// wave with an element outside it (a denormal, -0, infinity or NaN included)
// takes the general form whole.  A branch per lane would run both forms in
// such a wave: with 5% of the elements far, W = 8 fp32 at n = 2.5e7 took 237-242
// us that way, 219 this way, 215 with none far (the general form for
// all, at the occupancy it likes: 218).  Zeros in the short form cost 15
// instructions: 215 us with 0, 5% or 100% of the elements at zero, against 214
// and 219 (5%); 1% on a call over 1M elements.  (Looking for zeros only after the
// check without them failed saved half of that 1% and cost waves with far
// moments 2-4%.)
__device__ __forceinline__ void adamw4(const StepScalars &s, const Reciprocals &r,
                                       const float (&agg)[4], float (&p)[4], float (&m)[4],
                                       float (&v)[4])
{
    constexpr uint32_t kMLo = (127u - 60u) << 23, kMHi = (127u + 20u) << 23;
    constexpr uint32_t kVLo = (127u - 96u) << 23, kVHi = (127u + 60u) << 23;
    float mi[4], vi[4];
    // Ends of the moments' bits: of m with the sign below them, so that -0 is 1.
    // One less, +0 is above every lower end.
    uint32_t lo_m = ~0u, hi_m = 0, lo_v = ~0u, hi_v = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float g = agg[e] * s.grad_scale;
        mi[e] = s.b1 * m[e] + s.omb1 * g;
        vi[e] = s.b2 * v[e] + s.omb2 * (g * g);
        const uint32_t um = __builtin_rotateleft32(__float_as_uint(mi[e]), 1);
        const uint32_t uv = __float_as_uint(vi[e]);
        lo_m = um - 1 < lo_m ? um - 1 : lo_m;
        hi_m = um > hi_m ? um : hi_m;
        lo_v = uv - r.zero_v < lo_v ? uv - r.zero_v : lo_v;
        hi_v = uv > hi_v ? uv : hi_v;
    }
    const bool mid = r.tame && lo_m >= 2 * kMLo - 1 && hi_m <= 2 * kMHi + 1 &&
                     lo_v >= kVLo - r.zero_v && hi_v <= kVHi;
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!mid) == 0, 1)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float mh = div_const(mi[e], s.bc1, r.zh1, r.zl1);
            const float vh = div_const(vi[e], s.bc2, r.zh2, r.zl2);
            const float d = sqrt_mid(vh) + s.eps;
            p[e] = p[e] * s.decay - s.lr * div_mid(mh, d);
            m[e] = mi[e];
            v[e] = vi[e];
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            adamw(s, agg[e], p[e], m[e], v[e]);
    }
}

// ---- addressing --------------------------------------------------------------

// Arrays are reached through 64-bit bases in scalar registers.
typedef uint64_t Base;

// Four consecutive elements per lane: lane `lane` has group grp0 + lane of
// its arrays (grp0 uniform, so an access is a scalar base and a 32-bit lane
// offset).  grp0 is negative in the tile of a head's groups.
struct Tile {
    static constexpr int kN = 4;
    int64_t grp0;
    uint32_t lane;
    // the group's first byte in an array of `esz`-byte elements
    __device__ __forceinline__ GlobalBytes at(Base base, int esz) const
    {
        return reinterpret_cast<GlobalBytes>(base + grp0 * (4 * esz)) + lane * (4 * esz);
    }
};

// One element per lane, element `i` (negative in a head).
struct Single {
    static constexpr int kN = 1;
    int64_t i;
    __device__ __forceinline__ GlobalBytes at(Base base, int esz) const
    {
        return reinterpret_cast<GlobalBytes>(base + i * esz);
    }
};

// What one element of a contribution holds once loaded: a float (fp32 or
// widened bf16), or an int32 already in the switch's integer format.
template <int GT>
struct Contrib {
    using type = float;
};
template <>
struct Contrib<kGradI32> {
    using type = int32_t;
};

template <int GT>
__device__ __forceinline__ void load_grad(Base base, Tile t, typename Contrib<GT>::type (&x)[4])
{
    if constexpr (GT == kGradBF16) {
        const u32x2 h = ld_u32x2(t.at(base, 2));
        x[0] = widen_lo(h.x);
        x[1] = widen_hi(h.x);
        x[2] = widen_lo(h.y);
        x[3] = widen_hi(h.y);
    } else if constexpr (GT == kGradI32) {
        const i32x4 v = ld_i32x4(t.at(base, 4));
        x[0] = v.x;
        x[1] = v.y;
        x[2] = v.z;
        x[3] = v.w;
    } else {
        const f32x4 v = ld_f32x4(t.at(base, 4));
        x[0] = v.x;
        x[1] = v.y;
        x[2] = v.z;
        x[3] = v.w;
    }
}

template <int GT>
__device__ __forceinline__ void load_grad(Base base, Single t, typename Contrib<GT>::type (&x)[1])
{
    if constexpr (GT == kGradBF16)
        x[0] = widen_lo(ld_one<uint16_t>(t.at(base, 2)));
    else
        x[0] = ld_one<typename Contrib<GT>::type>(t.at(base, 4));
}

__device__ __forceinline__ void load_f32(Base base, Tile t, float (&x)[4])
{
    const f32x4 v = ld_f32x4(t.at(base, 4));
    x[0] = v.x;
    x[1] = v.y;
    x[2] = v.z;
    x[3] = v.w;
}
__device__ __forceinline__ void load_f32(Base base, Single t, float (&x)[1])
{
    x[0] = ld_one<float>(t.at(base, 4));
}

__device__ __forceinline__ void store_f32(Base base, Tile t, const float (&x)[4])
{
    st(t.at(base, 4), f32x4{x[0], x[1], x[2], x[3]});
}
__device__ __forceinline__ void store_f32(Base base, Single t, const float (&x)[1])
{
    st_one(t.at(base, 4), x[0]);
}

__device__ __forceinline__ void store_i32(Base base, Tile t, const int32_t (&x)[4])
{
    st(t.at(base, 4), i32x4{x[0], x[1], x[2], x[3]});
}
__device__ __forceinline__ void store_i32(Base base, Single t, const int32_t (&x)[1])
{
    st_one(t.at(base, 4), x[0]);
}

__device__ __forceinline__ void store_bf16(Base base, Tile t, const float (&x)[4])
{
    st(t.at(base, 2), to_bf16x4(x));
}
__device__ __forceinline__ void store_bf16(Base base, Single t, const float (&x)[1])
{
    st_one(t.at(base, 2), static_cast<uint16_t>(to_bf16(x[0])));
}

// ---- the reduction of one element over its W contributions ----------------

// Accumulator of one element: fp32 running sum, or exact 64-bit integer sum.
template <int MODE>
struct Acc {
    float f;
    int64_t s;
    __device__ __forceinline__ void first(float x, float qscale)
    {
        if constexpr (MODE == kAggFP32)
            f = x;
        else
            s = quantize(x, qscale);
    }
    __device__ __forceinline__ void next(float x, float qscale)
    {
        if constexpr (MODE == kAggFP32)
            f = f + x;
        else
            s += quantize(x, qscale);
    }
    // contributions already in the integer format (fixed mode only)
    __device__ __forceinline__ void first(int32_t q, float)
    {
        static_assert(MODE == kAggFixed, "int32 contributions are summed as integers");
        s = q;
    }
    __device__ __forceinline__ void next(int32_t q, float)
    {
        static_assert(MODE == kAggFixed, "int32 contributions are summed as integers");
        s += q;
    }
    // (fp32 aggregate, int32 aggregate)
    __device__ __forceinline__ float result(float dqscale, int32_t &ai) const
    {
        if constexpr (MODE == kAggFP32) {
            ai = 0;
            return f;
        } else {
            ai = saturate32(s);
            return static_cast<float>(ai) * dqscale;
        }
    }
};

// ---- one lane's elements ------------------------------------------------------

// The arrays and constants of one call, as a kernel holds them in scalar
// registers.  A base of 0 is an output that is not wanted.
template <int W>
struct Arrays {
    Base g[W > 0 ? W : 1];
    Base p, m, v, p16, agg_f32, agg_i32;
    float qscale, dqscale;
};

// The outputs of one lane's elements: the aggregate where wanted, and with
// the optimizer the updated state.
template <int MODE, bool ADAM, class A, class At, int N = At::kN>
__device__ __forceinline__ void finish(const A &a, At at, const float (&agg)[N],
                                       const int32_t (&ai)[N], float (&p)[N], float (&m)[N],
                                       float (&v)[N], const StepScalars &sc, const Reciprocals &rc)
{
    if (a.agg_f32)
        store_f32(a.agg_f32, at, agg);
    if constexpr (MODE == kAggFixed) {
        if (a.agg_i32)
            store_i32(a.agg_i32, at, ai);
    }
    if constexpr (ADAM) {
        if constexpr (N == 4)
            adamw4(sc, rc, agg, p, m, v);
        else
            adamw(sc, agg[0], p[0], m[0], v[0]);
        store_f32(a.p, at, p);
        store_f32(a.m, at, m);
        store_f32(a.v, at, v);
        if (a.p16)
            store_bf16(a.p16, at, p);
    }
}

// K contributions from `g` on into the accumulators: all K loads issued, then
// the additions in worker order.  No branch separates the loads, so none
// waits for the one before (a conditional load per contribution made the
// compiler wait after each).  `first`: g[0] is contribution 0.  `shift`:
// bytes to add to each base.
template <int K, int GT, int MODE, class At, int N = At::kN>
__device__ __forceinline__ void accumulate(const Base *g, int64_t shift, At at, float qscale,
                                           bool first, Acc<MODE> (&acc)[N])
{
    typename Contrib<GT>::type c[K][N];
#pragma unroll
    for (int j = 0; j < K; ++j)
        load_grad<GT>(g[j] + shift, at, c[j]);
#pragma unroll
    for (int j = 0; j < K; ++j) {
#pragma unroll
        for (int e = 0; e < N; ++e) {
            if (j == 0 && first)
                acc[e].first(c[j][e], qscale);
            else
                acc[e].next(c[j][e], qscale);
        }
    }
}

// The whole of one lane's elements, W known at compile time: every load
// first, then the arithmetic, then the stores.
template <int W, int GT, int MODE, bool ADAM, class Step, class At, int N = At::kN>
__device__ __forceinline__ void process(const Arrays<W> &a, const Step &step, At at)
{
    typename Contrib<GT>::type c[W][N];
    float p[N], m[N], v[N];
    StepScalars sc;
    Reciprocals rc;
#pragma unroll
    for (int w = 0; w < W; ++w)
        load_grad<GT>(a.g[w], at, c[w]);
    if constexpr (ADAM) {
        load_f32(a.p, at, p);
        load_f32(a.m, at, m);
        load_f32(a.v, at, v);
        sc = step_scalars_of(step);
        if constexpr (N == 4)
            rc = reciprocals(sc);
    }
    float agg[N];
    int32_t ai[N];
#pragma unroll
    for (int e = 0; e < N; ++e) {
        Acc<MODE> acc;
        acc.first(c[0][e], a.qscale);
#pragma unroll
        for (int w = 1; w < W; ++w)
            acc.next(c[w][e], a.qscale);
        agg[e] = acc.result(a.dqscale, ai[e]);
    }
    finish<MODE, ADAM>(a, at, agg, ai, p, m, v, sc, rc);
}

// The same for W known only at run time (W <= 64): contributions in chunks of
// 128 bytes per lane (8 fp32 or int32, 16 bf16), then the remaining W mod
// chunk in pieces of 8, 4, 2 and 1.  `g`: the W bases, in the arguments;
// `shift` bytes are added to each.
template <int GT, int MODE, bool ADAM, class Step, class At, int N = At::kN>
__device__ __forceinline__ void process_rt(const Arrays<0> &a, const Base *g, int W,
                                           const Step &step, At at, int64_t shift = 0)
{
    constexpr int kChunk = GT == kGradBF16 ? 16 : 8;
    float p[N], m[N], v[N];
    StepScalars sc;
    Reciprocals rc;
    if constexpr (ADAM) {
        load_f32(a.p, at, p);
        load_f32(a.m, at, m);
        load_f32(a.v, at, v);
        sc = step_scalars_of(step);
        if constexpr (N == 4)
            rc = reciprocals(sc);
    }
    Acc<MODE> acc[N];
    int w0 = 0;
    for (; w0 + kChunk <= W; w0 += kChunk)
        accumulate<kChunk, GT, MODE>(g + w0, shift, at, a.qscale, w0 == 0, acc);
    const int rest = W - w0;
    if constexpr (kChunk > 8) {
        if (rest & 8) {
            accumulate<8, GT, MODE>(g + w0, shift, at, a.qscale, w0 == 0, acc);
            w0 += 8;
        }
    }
    if (rest & 4) {
        accumulate<4, GT, MODE>(g + w0, shift, at, a.qscale, w0 == 0, acc);
        w0 += 4;
    }
    if (rest & 2) {
        accumulate<2, GT, MODE>(g + w0, shift, at, a.qscale, w0 == 0, acc);
        w0 += 2;
    }
    if (rest & 1)
        accumulate<1, GT, MODE>(g + w0, shift, at, a.qscale, w0 == 0, acc);
    float agg[N];
    int32_t ai[N];
#pragma unroll
    for (int e = 0; e < N; ++e)
        agg[e] = acc[e].result(a.dqscale, ai[e]);
    finish<MODE, ADAM>(a, at, agg, ai, p, m, v, sc, rc);
}

// ---- kernels -----------------------------------------------------------------

// How the elements of one contiguous piece are dealt out: n_groups groups of
// four from the (advanced) pointers on, `tail` elements after them and `head`
// elements (0-255) before them.  The head's whole groups are a tile of their
// own in front of the others, and the up to six elements that belong to no
// group go one to a lane to a block of their own: no lane does two things
// after another.  (Done by the lanes of block 0 after their group, up to 255
// head elements one by one made a launch of 2M elements 2 us longer.)
struct Split {
    int64_t n_groups;
    int lead;        // blocks in front of the tile of group 0
    int singles;     // whether the first of them is the block of single elements
    int head, tail;
    int together;    // log2 of how many tiles in a row fall to one XCD
};

__host__ __device__ constexpr Split make_split(int64_t n_groups, int head, int tail, int together)
{
    const int singles = (head & 3) || tail ? 1 : 0;
    return Split{n_groups, singles + (head >= 4 ? 1 : 0), singles, head, tail, together};
}

// The kernel arguments: what a wave needs before its loads first, the
// contributions right behind the state.
template <int W>
struct VectorArgs {
    Split split;
    int lanes_log2;            // lanes per block
    int W_rt;                  // W where it is known at run time only
    Base p, m, v;
    Base g[W > 0 ? W : kMaxW];
    Base p16, agg_f32, agg_i32;
    float qscale, dqscale;
    StepScalars s;
    const StepScalars *s_dev;  // when set, the step constants are read here
};

template <int W, class K>
__device__ __forceinline__ Arrays<W> arrays_of(const K &k)
{
    Arrays<W> a;
    if constexpr (W > 0) {
#pragma unroll
        for (int w = 0; w < W; ++w)
            a.g[w] = k.g[w];
    }
    a.p = k.p;
    a.m = k.m;
    a.v = k.v;
    a.p16 = k.p16;
    a.agg_f32 = k.agg_f32;
    a.agg_i32 = k.agg_i32;
    a.qscale = k.qscale;
    a.dqscale = k.dqscale;
    return a;
}

// Block `block` of a piece split as `sp`, in blocks of 2^lanes_log2 lanes: its
// lanes' elements through f(Tile) or f(Single).
template <class F>
__device__ __forceinline__ void deal(const Split &sp, int block, int lanes_log2, F &&f)
{
    const int lane = threadIdx.x;
    if (sp.singles && block == 0) {
        const bool in_head = lane < (sp.head & 3), in_tail = lane >= 4 && lane < 4 + sp.tail;
        if (in_head || in_tail)
            f(Single{in_head ? int64_t(lane) - sp.head : 4 * sp.n_groups + lane - 4});
        return;
    }
    // Blocks go to the 8 XCDs in turn: 2^together tiles in a row are every
    // eighth of 8 << together blocks (where those are whole).
    int tile = block - sp.lead;
    const int last = tile | ((8 << sp.together) - 1);
    if (sp.together && tile >= 0 && (int64_t(last) + 1) << lanes_log2 <= sp.n_groups)
        tile = last - (8 << sp.together) + 1 + ((tile & 7) << sp.together) +
               ((tile >> 3) & ((1 << sp.together) - 1));
    const int64_t grp0 = int64_t(tile) << lanes_log2;
    // lanes [from, to) have a group: every lane but in the last tile and the
    // head's (the one with grp0 < 0)
    const int64_t left = sp.n_groups - grp0;
    const unsigned to = left < kMaxBlock ? static_cast<unsigned>(left) : kMaxBlock;
    const unsigned from = grp0 < 0 ? (1u << lanes_log2) - (sp.head >> 2) : 0;
    if (lane - from < to - from)
        f(Tile{grp0, threadIdx.x});
}

// Vector kernel.  W > 0: compile-time worker count; W == 0: run-time worker
// count.  One 4-element group per lane, one tile of groups per block (64
// lanes, or 256 in the shared shape).  Every pointer is on a 4-byte
// boundary; the front end chose the head.
template <int W, int GT, int MODE, bool ADAM>
__global__ DISDP_LAUNCH_BOUNDS void vector_kernel(VectorArgs<W> k)
{
    const Arrays<W> a = arrays_of<W>(k);
    // Everything that a wave's loads depend on is read here at once.  Left
    // alone the compiler reads the split first, and the bases behind the
    // branches on it: a second and third scalar round trip before the loads.
    if constexpr (W > 0) {
#define G(i) "s"(a.g[i < W ? i : W - 1])
        asm volatile("" ::"s"(k.split.n_groups), "s"(k.split.lead), "s"(k.split.singles),
                     "s"(k.split.head), "s"(k.split.tail), "s"(k.split.together),
                     "s"(k.lanes_log2), "s"(a.p), "s"(a.m),
                     "s"(a.v), G(0), G(1), G(2), G(3), G(4), G(5), G(6), G(7), G(8), G(9),
                     G(10), G(11), G(12), G(13), G(14), G(15));
#undef G
    }
    deal(k.split, blockIdx.x, k.lanes_log2, [&](auto at) {
        if constexpr (W > 0)
            process<W, GT, MODE, ADAM>(a, k, at);
        else
            process_rt<GT, MODE, ADAM>(a, k.g, k.W_rt, k, at);
    });
}

// Element-wise kernel, for an array not aligned to its element size or bf16
// arrays that no head puts on 4-byte boundaries together: `n` elements, one
// per lane, grid-stride.
template <int GT, int MODE, bool ADAM>
__global__ DISDP_LAUNCH_BOUNDS void element_kernel(VectorArgs<0> k, int64_t n)
{
    const Arrays<0> a = arrays_of<0>(k);
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += stride)
        process_rt<GT, MODE, ADAM>(a, k.g, k.W_rt, k, Single{i});
}

// ---- several tensors in one launch ------------------------------------------

// Arguments of a launch over `count` tensors.  A block finds its tensor in two
// steps of 16 first blocks each (`coarse` holds every 16th; unused entries
// are ~0), each step one scalar read and 16 compares -- a binary search is
// a chain of up to 8 dependent reads in front of every wave's loads.  In
// `table`: the first blocks of the tensors (32 bits, a multiple of 16
// entries), their shapes (32 bits), then from `rows_at` on the base addresses:
// a row of W + 4 per tensor (contributions, p, m, v, bf16 copy or 0), or for
// tensors that lie at one element offset in every array ("flat": slices of
// flat buffers) their 64-bit element offsets and one row for all.  The whole
// stays within 4 KiB of kernel arguments.
constexpr int kMultiTable = 3840;
constexpr int kMultiMost = 240;  // above what the table holds (flat, 16 bytes a tensor)
struct MultiLaunch {
    uint32_t coarse[16];
    int count, W, rows_at, flat;
    int64_t zero;              // the offset of a tensor with a row of its own
    float qscale, dqscale;
    StepScalars s;
    const StepScalars *s_dev;
    alignas(8) unsigned char table[kMultiTable];
};
static_assert(sizeof(MultiLaunch) <= 4096, "kernel arguments above 4 KiB");

// A tensor's shape beside its number of blocks: head (8 bits), tail (2 bits)
// and the groups of its last tile (7 bits, 0: it has no tile).
__host__ __device__ constexpr uint32_t pack_shape(int head, int tail, int last)
{
    return static_cast<uint32_t>(head) | static_cast<uint32_t>(tail) << 8 |
           static_cast<uint32_t>(last) << 10;
}

// How many of 16 ascending first blocks are at most `block`: two scalar
// instructions each (the compiler's own form goes through vector registers).
__device__ __forceinline__ int count_upto(const uint32_t *first, uint32_t block)
{
    uint32_t c = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i)
        asm("s_cmp_le_u32 %1, %2\n\ts_addc_u32 %0, %0, 0"
            : "+s"(c)
            : "s"(first[i]), "s"(block)
            : "scc");
    return static_cast<int>(c);
}

// Fused aggregation + AdamW over the tensors of `k`: each as in
// vector_kernel with one-wave blocks.
template <int W, int GT, int MODE>
__global__ DISDP_WAVE_LAUNCH_BOUNDS void multi_kernel(MultiLaunch k)
{
    // Three rounds of scalar reads, each issued whole: the header and the
    // coarse list, 16 first blocks, all that belongs to tensor j.
    const uint32_t block = blockIdx.x;
    const uint32_t *first = reinterpret_cast<const uint32_t *>(k.table);
    const int count = k.count, rows_at = k.rows_at, flat = k.flat;
    const int Wn = W > 0 ? W : k.W;
    const int j16 = 16 * (count_upto(k.coarse, block) - 1);
    asm volatile("" ::"s"(count), "s"(rows_at), "s"(flat), "s"(Wn));
    const int j = j16 + count_upto(first + j16, block) - 1;
    const int64_t *offsets = reinterpret_cast<const int64_t *>(k.table + rows_at);
    const Base *row = reinterpret_cast<const Base *>(offsets) + (flat ? count : j * (Wn + 4));
    const int64_t off = *(flat ? offsets + j : &k.zero);
    const uint32_t here = first[j], end = first[j + 1];
    const uint32_t shape = first[((count + 16) & ~15) + j];
    if constexpr (W > 0) {
#define G(i) "s"(row[i < W + 4 ? i : W + 3])
        asm volatile("" ::"s"(off), "s"(here), "s"(end), "s"(shape), G(0), G(1), G(2), G(3), G(4),
                     G(5), G(6), G(7), G(8), G(9), G(10), G(11), G(12), G(13), G(14), G(15), G(16),
                     G(17), G(18), G(19));
#undef G
    }
    const int last = shape >> 10;
    Split sp = make_split(0, shape & 255, (shape >> 8) & 3, 0);
    if (last)
        sp.n_groups = (int64_t(end - here) - sp.lead - 1) * kWave + last;
    constexpr int kGradBytes = GT == kGradBF16 ? 2 : 4;
    Arrays<W> a;
    if constexpr (W > 0) {
#pragma unroll
        for (int w = 0; w < W; ++w)
            a.g[w] = row[w] + off * kGradBytes;
    }
    a.p = row[Wn] + off * 4;
    a.m = row[Wn + 1] + off * 4;
    a.v = row[Wn + 2] + off * 4;
    a.p16 = row[Wn + 3] ? row[Wn + 3] + off * 2 : 0;
    a.agg_f32 = 0;
    a.agg_i32 = 0;
    a.qscale = k.qscale;
    a.dqscale = k.dqscale;
    deal(sp, static_cast<int>(block - here), 6, [&](auto at) {
        if constexpr (W > 0)
            process<W, GT, MODE, true>(a, k, at);
        else
            process_rt<GT, MODE, true>(a, row, Wn, k, at, off * kGradBytes);
    });
}

// ---- the format conversion as a producer ------------------------------------

// out = quantize(g), a tile to a one-wave block; the head's groups and the
// single elements are dealt out by the blocks in front, as in vector_kernel.  A
// lane has one load only, so the time between a wave's start and that load
// counts: with the general deal() for every tile the 13B/16 contribution took
// 743 us, this way 722 (two or four tiles a wave: 775, 793).
struct QuantizeVectorArgs {
    Base g, out;
    int64_t n_groups;
    int lead;          // blocks in front of the tiles
    float qscale;
    Split edges;       // of no tiles: the head and the single elements
};

template <int GT, class At>
__device__ __forceinline__ void quantize_at(const QuantizeVectorArgs &k, At at)
{
    constexpr int N = At::kN;
    float x[N];
    int32_t y[N];
    load_grad<GT>(k.g, at, x);
#pragma unroll
    for (int e = 0; e < N; ++e)
        y[e] = quantize(x[e], k.qscale);
    store_i32(k.out, at, y);
}

template <int GT>
__global__ DISDP_WAVE_LAUNCH_BOUNDS void quantize_vector_kernel(QuantizeVectorArgs k)
{
    const int block = static_cast<int>(blockIdx.x) - k.lead;
    if (block >= 0) {
        const Tile at{int64_t(block) * kWave, threadIdx.x};
        if (at.grp0 + at.lane < k.n_groups)
            quantize_at<GT>(k, at);
    } else {
        deal(k.edges, static_cast<int>(blockIdx.x), 6, [&](auto at) {
            constexpr bool kTile = decltype(at)::kN == 4;
            if constexpr (kTile)
                quantize_at<GT>(k, at);
            else
                quantize_at<GT>(k, Single{at.i < 0 ? at.i : at.i + 4 * k.n_groups});
        });
    }
}

template <int GT>
__global__ DISDP_WAVE_LAUNCH_BOUNDS void quantize_element_kernel(QuantizeArgs q)
{
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kWave;
    const Base g = reinterpret_cast<Base>(q.g), out = reinterpret_cast<Base>(q.out);
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * kWave + threadIdx.x; i < q.n;
         i += stride) {
        float x[1];
        load_grad<GT>(g, Single{i}, x);
        const int32_t y[1] = {quantize(x[0], q.qscale)};
        store_i32(out, Single{i}, y);
    }
}

// ---- host side: grid sizing and dispatch --------------------------------------

// Resident waves per CU, by the bytes of loads a lane keeps in flight (4
// elements of each contribution; p, m and v with the optimizer).  What streams
// best is the fewest waves that still cover the memory's latency: the tiles
// in flight are then the shortest stretch of every array.  One wave too few
// costs up to 14%, one too many 1-3%.  0 = as many as fit.
//
// Every entry is the cap whose worst case was best, of 24 to 28: the planned
// slab, arrays in allocations of their own, and scattered offsets, at n = 1e7,
// 2.5e7, 5e7 and 2e8 on two cards, and with 5% of the moments far from the short
// arithmetic's range; caps interleaved in one process.  Figures: how
// far the time lies above the best cap's, worst / mean in percent, in
// brackets the caps next to the chosen one.
//
// Fused: fp32 W = 1 (64 B) 10: 2.5 / 0.4 (9: 8.0 / 2.2; 11: 4.7 / 0.9); W = 2
// (80) 9: 2.0 / 0.3 (8: 10.4 / 2.3; 10: 2.4 / 0.8); W = 3 (96) 8: 2.3 / 0.4 (7:
// 3.1 / 1.7; 9: 1.9 / 0.5); W = 4 (112) 8: 2.4 / 0.6 (7: 3.3 / 0.6); W = 5, 6
// (128, 144) 7: 3.9 / 1.1 (6: 5.8 / 1.4); W = 7, 8 (160, 176) 6: 3.9 / 0.7 (5: 9.2
// / 2.2; 7: 5.0 / 2.1); W = 12 (240) 5: 3.8 / 0.9 (4: 4.8 / 0.9); W = 16 (304) 4:
// 5.6 / 0.4 (5: 5.6 / 1.9); bf16 W = 2, 4, 8, 12, 16 at 10, 9, 8, 7, 6: 2.6, 2.5,
// 4.0, 1.4, 2.0 / 0.4-0.8.
// From kLargeElems on, float or int32 contributions that are not converted want
// one fewer between 112 and 240 B (W = 8 on slabs of 2e8 to 9.3e8 elements 5:
// 0.4 on average, 6: 1.2; in allocations of their own, n = 8.75e8, 6 is 1.4
// behind; 1% on a list of 1.04e8); below it one fewer costs W = 8 up to 9 (n =
// 5e7), and 3 with far moments.
// Converting bf16, twice the conversions per byte, it wants one more, above 144 B
// two (W = 2, 4, 8, 12, 16 at 11, 10, 9, 8, 8: 1.8, 4.1, 3.0, 2.1, 1.9 / 0.3-0.8; W =
// 4 at 8: 12.2 / 6.6).  An aggregate written too wants two more (W = 8, 8 waves:
// 1.7 / 0.2; 6: 4.5 / 2.1).
constexpr int64_t kLargeElems = 100000000;
constexpr int fused_waves(int lane_bytes, bool converts_bf16, bool large)
{
    const int waves = lane_bytes <= 64    ? 10
                      : lane_bytes <= 80  ? 9
                      : lane_bytes <= 112 ? 8
                      : lane_bytes <= 144 ? 7
                      : lane_bytes <= 176 ? 6
                      : lane_bytes <= 240 ? 5
                                          : 4;
    if (converts_bf16)
        return waves + (lane_bytes <= 144 ? 1 : 2);
    return large && lane_bytes >= 112 && lane_bytes <= 240 ? waves - 1 : waves;
}

// The aggregation alone reads nearly all it moves and wants more loads in
// flight, by the same measure: fp32 W = 1, 2 (16, 32 B) uncapped: 0.5 / 0.1 (24,
// 20: 5.9, 5.8); W = 3 18: 3.2 / 0.9; W = 4 14: 3.6 / 0.9 (12: 6.5; 16: 3.1 / 1.3);
// W = 6 10: 2.0 / 0.4; W = 8 8: 1.2 / 0.1 (7: 4.5; 9: 1.7); W = 12, 16 6: 0.5, 1.2;
// bf16 W = 4 uncapped 2.3 / 0.3; W = 8, 12, 16 14, 10, 9: 1.3, 1.1, 2.1.
// Converting bf16, W = 16 11: 2.4 / 0.5 (10: 3.0 / 0.7).
constexpr int aggregate_waves(int lane_bytes, bool bf16, bool converts_bf16)
{
    const int waves = lane_bytes <= 32    ? 0
                      : lane_bytes <= 48  ? 18
                      : lane_bytes <= 64  ? 14
                      : lane_bytes <= 96  ? 10
                      : lane_bytes <= 128 ? 8 + bf16
                                          : 6;
    return converts_bf16 && lane_bytes >= 112 ? waves + 2 : waves;
}

// The run-time worker-count kernels, whose lanes keep chunks of 128 bytes in
// flight and then the smaller pieces of the remainder, one after another: the more
// pieces, the more waves.  By the same measure (worst / mean).
// Fused bf16: W = 9, 11, 13, 15 11, 12, 12, 13: 1.7, 2.7, 1.9, 2.1 (10 for all: 3.2,
// 8.5, 6.5, 9.4); W = 17, 19, 23, 24, 28, 31 9, 10, 11, 7, 9, 11: 3.0, 1.1, 0.6, 1.0, 2.2,
// 1.8 (7 for all: 7.1, 9.9, 10.5, 1.0, 3.4, 10.4); W = 33, 39, 47, 63, 64 8, 9, 9, 9, 7:
// 0.9, 0.1, 0.2, 0.8, 1.3.  Converting: W = 9, 11, 15 1.4, 2.1, 1.5; W = 17, 19, 23, 24,
// 31, 39 10, 11, 12, 9, 12, 11: 1.2, 1.9, 0.8, 0.9, 0.2, 0.7.
// Fused fp32: W = 9, 11, 15 8: 1.3, 0.7, 1.0; W = 17, 20, 23 6, 5, 7: 1.4, 0.9, 1.3; W
// = 24, 27, 31 4, 6, 6: 0.6, 2.1, 1.3 (4 for all: 0.6, 8.6, 11.4); W = 33, 47, 63, 64 5, 5,
// 5, 4: 0.7, 0.7, 3.8, 4.3.  Converting: W = 9, 15 8: 3.3, 1.4; W = 19, 23, 24, 31, 63 7,
// 7, 5, 7, 6: 1.6, 1.4, 2.1, 0.7, 2.6.
// The aggregation alone, bf16: W = 9, 15 16: 0.6, 0.5; W = 17, 20, 23 12, 12, 14: 1.1,
// 2.1, 0.2; W = 24, 31, 32, 33, 39, 64 9, 13, 8, 10, 11, 8: 1.1, 1.5, 3.4, 0.9, 0.5,
// 1.4 (W = 32, 48, 64 at n = 1e7 to 1e8 8: 0.4% ahead of 9 on average); fp32: W = 9,
// 15 9: 1.5, 1.5; W = 17, 23 7: 1.0, 2.6; W = 24, 31 6: 2.4, 1.1; W = 32, 64 5: 1.1, 1.7.
int runtime_w_waves(int W, int gt, int mode, bool adam)
{
    const bool converts = mode == kAggFixed && gt != kGradI32;
    if (gt == kGradBF16) {
        const int pieces = __builtin_popcount(W & 7);   // of fewer than 8
        if (W < 16)
            return adam ? 9 + __builtin_popcount(W) : 16;
        if (!adam)
            return (pieces == 0 ? 9 - (W >= 32)
                    : W >= 32   ? 9 + (pieces + 1) / 2
                                : 10 + pieces + (W < 24)) +
                   2 * converts;
        if (W >= 32 || pieces == 0)
            return 7 + (pieces + 1) / 2 + 2 * converts;
        return 8 + pieces + converts;
    }
    if (!adam)
        return W < 16 ? 9 : W < 24 ? 7 : W < 32 ? 6 : 5;
    if (W < 16)
        return 8;
    const int pieces = __builtin_popcount(W & 3);       // of fewer than 4
    return (W < 24 || converts ? 5 : 4) + (W < 32 ? pieces : pieces > 0);
}

// The caps above pay once a launch is many rounds of resident waves; one of a
// few rounds ends sooner with every wave resident (fused, W = 8, n = 1e6,
// uncapped 10.6 us, 5 waves 11.1; fp32 W = 1, n = 1e6 5.7 against 6.5; W = 16
// bf16, n = 1e6 11.5 against 12.3; from about 5 rounds on -- W = 8, n = 1.5e6
// -- they are within 2%, at 12 rounds the cap is 4% ahead).
constexpr int kUncappedRounds = 5;

// The launch shape of the vector kernels for one call.
//   solo   (default): one-wave blocks, occupancy caps from the tables above
//          -- the fastest shape when the kernel has the GPU to itself.
//   shared (DISDP_LAUNCH_SHAPE=shared in the environment): four-wave blocks,
//          two of them per CU (three or four for fixed-point kernels that
//          convert float contributions).  Next to a bf16 GEMM loop on another
//          stream of the same (unmasked) GPU, the solo shape's stream of
//          one-wave blocks refills every slot a retiring block frees and the
//          GEMM slows about 10x while the fused call slows 1.1x; a retiring
//          four-wave block leaves four wave slots and half the LDS, which a
//          GEMM workgroup can take, and the two slow each other about evenly
//          (measured 1.7x and 2.0x; with three blocks the hole is too small
//          and the GEMM slows 10x again), at 3-5% below the solo shape's rate
//          when alone (W = 8 fp32, n = 2e8, 2 blocks 6.50 TB/s, 3 6.32).
// The variable is read on every call, so a process can switch between
// calls; any other value means solo.
struct Shape {
    int lanes;        // lanes per block
    bool shared;
};

Shape launch_shape()
{
    const char *s = std::getenv("DISDP_LAUNCH_SHAPE");
    if (s && std::strcmp(s, "shared") == 0)
        return Shape{kMaxBlock, true};
    return Shape{kWave, false};
}

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

constexpr int shared_waves(bool adam, bool converts)
{
    return !converts ? 8 : adam ? 12 : 16;
}

// Dynamic LDS bytes a vector-kernel block reserves so that at most
// `blocks_per_cu` blocks fit on a CU (0 = no cap), cached per device.
int occupancy_lds_bytes(int blocks_per_cu)
{
    constexpr int kMaxCap = 64;
    if (blocks_per_cu <= 0 || blocks_per_cu > kMaxCap)
        return 0;
    static std::atomic<int> cached[64][kMaxCap + 1];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64)
        return 0;
    int b = cached[dev][blocks_per_cu].load(std::memory_order_relaxed);
    if (b == 0) {
        int per_cu = 0, per_block = 0;
        if (hipDeviceGetAttribute(&per_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor,
                                  dev) != hipSuccess ||
            hipDeviceGetAttribute(&per_block, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) !=
                hipSuccess ||
            per_cu <= 0) {
            b = -1;  // unknown: launch without a cap
        } else {
            // in whole LDS allocation units (1280 bytes on gfx950), so that
            // `blocks_per_cu` blocks fit and not one fewer
            constexpr int kLdsUnit = 1280;
            b = per_cu / blocks_per_cu / kLdsUnit * kLdsUnit;
            if (b > per_block)
                b = per_block;
            if (b <= 0)
                b = -1;
        }
        cached[dev][blocks_per_cu].store(b, std::memory_order_relaxed);
    }
    return b > 0 ? b : 0;
}

int cu_count()
{
    static std::atomic<int> cached[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64)
        return 256;
    int c = cached[dev].load(std::memory_order_relaxed);
    if (c <= 0) {
        if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            c <= 0)
            c = 256;
        cached[dev].store(c, std::memory_order_relaxed);
    }
    return c;
}

// CUs `stream` may run on: the number of bits of its CU mask among the
// device's CUs (hipExtStreamCreateWithCUMask), or all of them when the
// runtime cannot say.  An error the query records is cleared only when no
// error was pending before it, so a caller's own pending error survives.
int stream_cus(hipStream_t stream)
{
    const int total = cu_count();
    constexpr int kMaxWords = 32;  // masks of up to 1024 CUs
    const int words = (total + 31) / 32;
    uint32_t mask[kMaxWords] = {};
    if (words > kMaxWords)
        return total;
    const hipError_t pending = hipPeekAtLastError();
    if (hipExtStreamGetCUMask(stream, words, mask) != hipSuccess) {
        if (pending == hipSuccess)
            (void)hipGetLastError();
        return total;
    }
    int c = 0;
    for (int i = 0; i < total; ++i)
        c += (mask[i / 32] >> (i % 32)) & 1u;
    return c > 0 ? c : total;
}

// Resident-block cap per CU for a launch of `lanes`-lane blocks on
// `stream`: `base_waves` is the cap in waves for the whole chip.  What
// streams best is a number of resident waves chip-wide, so on a stream
// restricted to fewer CUs each CU takes proportionally more, up to
// kMaxScaledWaves (the register limit of the W = 8 kernels).  Measured on
// the 7B/8 shard with 32 / 64 / 128 CUs: 20 waves per CU streamed 41% / 35%
// / 19% faster than the full-chip cap of the time (12 waves per CU, in
// 4-wave blocks).
constexpr int kMaxScaledWaves = 20;
int blocks_per_cu_cap(int base_waves, int lanes, hipStream_t stream)
{
    if (base_waves <= 0)
        return 0;
    const int total = cu_count();
    const int mine = stream_cus(stream);
    int waves = base_waves;
    if (mine < total) {
        const int scaled = (base_waves * total + mine - 1) / mine;
        waves = scaled < kMaxScaledWaves ? scaled
                                         : (base_waves > kMaxScaledWaves ? base_waves : kMaxScaledWaves);
    }
    const int blocks = waves / (lanes / kWave);
    return blocks > 0 ? blocks : 1;
}

// A dispatch counts its work-items in 32 bits per dimension, so a grid of
// `block`-lane blocks holds at most (2^32 - 1) / block of them.
constexpr int64_t kMaxGridLanes = 0xffffffffLL;
int64_t max_blocks(int block) { return kMaxGridLanes / block; }
int64_t clamp_grid(int64_t blocks, int block)
{
    return blocks < 1 ? 1 : blocks > max_blocks(block) ? max_blocks(block) : blocks;
}

Base base_of(const void *p) { return reinterpret_cast<Base>(p); }

// The arguments common to the vector and element kernels, but for the split.
template <int W>
VectorArgs<W> vector_args(const LaunchArgs &a, int lanes)
{
    VectorArgs<W> k{};
    k.p = base_of(a.p);
    k.m = base_of(a.m);
    k.v = base_of(a.v);
    k.p16 = base_of(a.p16);
    k.agg_f32 = base_of(a.agg_f32);
    k.agg_i32 = base_of(a.agg_i32);
    k.qscale = a.qscale;
    k.dqscale = a.dqscale;
    k.lanes_log2 = lanes == kWave ? 6 : 8;
    k.W_rt = a.W;
    k.s = a.s;
    k.s_dev = a.s_dev;
    for (int w = 0; w < a.W; ++w)
        k.g[w] = base_of(a.g[w]);
    return k;
}

// Moves every array of `k` on by `elems` elements.
template <int W>
void advance(VectorArgs<W> &k, int64_t elems, int grad_bytes)
{
    for (Base *b : {&k.p, &k.m, &k.v, &k.agg_f32, &k.agg_i32})
        if (*b)
            *b += elems * 4;
    if (k.p16)
        k.p16 += elems * 2;
    for (int w = 0; w < k.W_rt; ++w)
        k.g[w] += elems * grad_bytes;
}

// Whether the contributions lie `step` bytes or a multiple of it apart, give or
// take 4 MiB: any two neighbours of them, or every two.
bool multiples_apart(const LaunchArgs &a, uintptr_t step, bool every)
{
    constexpr uintptr_t kNear = uintptr_t(4) << 20;
    for (int w = 1; w < a.W; ++w) {
        const uintptr_t apart = reinterpret_cast<uintptr_t>(a.g[w]) -
                                reinterpret_cast<uintptr_t>(a.g[w - 1]);
        if (((apart + kNear) % step <= 2 * kNear) != every)
            return !every;
    }
    return every;
}

// Waves for the fused kernels of 7 to 16 four-byte contributions that lie a
// multiple of 256 MiB apart (a flat buffer of 2^26 or 2^27 elements each, the planned
// slab at 5.0e7 to 5.8e7), where the same tile of every array falls to the
// same channels.  Against the table's caps: W = 8, 12, 16 at n = 2^26 0.3, 4.5, 8.0%
// faster, 2^27 1.8, 1.5, 3.0%, the slab at 5e7 0.5, 2.5, 4.5%; from 1 GiB apart on it
// loses as often (n = 2^28: 1.8, 3.9, -4.5%).
constexpr int kSameChannelWaves = 8;
bool same_channels(const LaunchArgs &a)
{
    constexpr uintptr_t kMiB = uintptr_t(1) << 20;
    const uintptr_t first = reinterpret_cast<uintptr_t>(a.g[0]);
    const uintptr_t second = reinterpret_cast<uintptr_t>(a.g[a.W > 1 ? 1 : 0]);
    const uintptr_t apart = first < second ? second - first : first - second;
    return apart >= 128 * kMiB && apart < 896 * kMiB && multiples_apart(a, 256 * kMiB, true);
}

// Tiles in a row that one XCD takes, as a log2: 1 for large launches over many
// bf16 contributions.  A bf16 tile is 512 bytes of each; two neighbours on one
// XCD make a 1 KiB read of it, as one fp32 tile is (together / one by one, each
// at its own best cap, TB/s, on two or more layouts each): fused W = 16
// 6.74 / 6.51 (n = 2.5e7), 6.60 / 6.43 (2e8), 6.51 / 6.49 (5e8); W = 12
// 6.55 / 6.49; W = 20, 32, 64 6.53 / 6.34, 6.32 / 6.13, 6.11 / 5.99; the
// aggregation alone W = 16, 24, 32, 64 6.39 / 6.32, 6.27 / 6.10, 6.29 / 6.05,
// 6.06 / 5.88; fixed point, fused W = 16 6.51 / 6.35.  Fewer contributions
// gain under 1% or lose (W = 4, 8; the aggregation of 4 and 8: -2%), a launch
// of a few rounds loses (fused W = 16, n = 4e6 -1.5%, 1e6 -5%; at 17 rounds, the
// aggregation of 16 at n = 1e7, -5%, at 22, n = 1.3e7, 4% ahead), fp32 too (W =
// 1, 4, 8: -1%, -1%, -2%).  Above 7e8 elements it pays on one slab and loses on
// allocations of their own: W = 16 at 8e8 0 and -10%, 1e9 +2 and -3%, 2e9 -2 and
// -1%; W = 12 -9% at 8e8, W = 32 -7% at 1.25e9; at 6e8 it gains 1-4% on both.
// It also loses when the arrays lie a multiple of 64 MiB apart, where the same
// tile of every array falls to the same channels: fused W = 16, arrays 128 and
// 256 pages of 2 MiB apart 5.2 / 6.2 and 5.1 / 6.3, 127 and 129 pages 5.4 / 6.2
// and 4.9 / 6.2, 32 pages 6.2 / 6.3 (4 and 8 tiles together did not do better
// over the layouts).
int tiles_together(const LaunchArgs &a, bool adam, int base_waves)
{
    constexpr int kRounds = 20;
    constexpr int64_t kMostElems = 700000000;
    if (a.gdtype != kGradBF16 || a.W < (adam ? 12 : 16) || a.n > kMostElems ||
        ceil_div(a.n >> 2, kWave) <= int64_t(kRounds) * base_waves * cu_count())
        return 0;
    return multiples_apart(a, uintptr_t(64) << 20, false) ? 0 : 1;
}

template <int W, int GT, int MODE, bool ADAM>
hipError_t launch_vector(const LaunchArgs &a, Shape shape, hipStream_t stream)
{
    // bytes of loads one lane keeps in flight: 4 elements of each
    // contribution, plus p, m and v with the optimizer (run-time W: many)
    constexpr int kGradBytes = GT == kGradBF16 ? 2 : 4;
    constexpr int kLaneBytes = W > 0 ? 4 * (W * kGradBytes + (ADAM ? 12 : 0)) : 1 << 30;
    constexpr bool kConverts = MODE == kAggFixed && GT != kGradI32;
    int base, together = 0;
    if (shape.shared) {
        base = shared_waves(ADAM, kConverts);
    } else {
        base = W == 0 ? runtime_w_waves(a.W, GT, MODE, ADAM)
               : ADAM ? fused_waves(kLaneBytes, kConverts && GT == kGradBF16,
                                    GT != kGradBF16 && !kConverts && a.n >= kLargeElems)
                      : aggregate_waves(kLaneBytes, GT == kGradBF16,
                                        kConverts && GT == kGradBF16);
        if (ADAM && W >= 7 && kGradBytes == 4 && base < kSameChannelWaves && same_channels(a))
            base = kSameChannelWaves;
        together = tiles_together(a, ADAM, base);
        if (ADAM && (a.agg_f32 || a.agg_i32))
            base += 2;
        if (ceil_div(a.n >> 2, kWave) <= int64_t(kUncappedRounds) * base * cu_count())
            base = 0;
    }
    const int lds = occupancy_lds_bytes(blocks_per_cu_cap(base, shape.lanes, stream));
    VectorArgs<W> k = vector_args<W>(a, shape.lanes);
    int64_t left = a.n >> 2;  // groups; a launch per 1.7e10 elements
    int head = a.head;
    do {
        const int64_t most = (max_blocks(shape.lanes) - 2) * shape.lanes;
        const int64_t now = left < most ? left : most;
        left -= now;
        k.split = make_split(now, head, left ? 0 : static_cast<int>(a.n & 3), together);
        const int64_t blocks = k.split.lead + ceil_div(now, shape.lanes);
        void *args[] = {&k};
        const hipError_t e = hipLaunchKernel(
            reinterpret_cast<const void *>(&vector_kernel<W, GT, MODE, ADAM>),
            dim3(static_cast<unsigned>(blocks)), dim3(shape.lanes), args, static_cast<size_t>(lds),
            stream);
        if (e != hipSuccess)
            return e;
        advance(k, 4 * now, kGradBytes);
        head = 0;
    } while (left > 0);
    return hipSuccess;
}

// The element kernel walks the shard grid-stride with 32 waves per CU (its
// registers allow that many resident).
constexpr int kElementWavesPerCu = 32;

template <int GT, int MODE, bool ADAM>
hipError_t dispatch_w(const LaunchArgs &a, bool vec, Shape shape, hipStream_t stream)
{
    if (!vec) {
        const int64_t cap = static_cast<int64_t>(cu_count()) * kElementWavesPerCu /
                            (shape.lanes / kWave);
        const int64_t need = ceil_div(a.n, shape.lanes);
        VectorArgs<0> k = vector_args<0>(a, shape.lanes);
        int64_t n = a.n;
        void *args[] = {&k, &n};
        return hipLaunchKernel(reinterpret_cast<const void *>(&element_kernel<GT, MODE, ADAM>),
                               dim3(static_cast<unsigned>(need < cap ? need : cap)),
                               dim3(shape.lanes), args, 0, stream);
    }
    switch (a.W) {
    case 1: return launch_vector<1, GT, MODE, ADAM>(a, shape, stream);
    case 2: return launch_vector<2, GT, MODE, ADAM>(a, shape, stream);
    case 3: return launch_vector<3, GT, MODE, ADAM>(a, shape, stream);
    case 4: return launch_vector<4, GT, MODE, ADAM>(a, shape, stream);
    case 5: return launch_vector<5, GT, MODE, ADAM>(a, shape, stream);
    case 6: return launch_vector<6, GT, MODE, ADAM>(a, shape, stream);
    case 7: return launch_vector<7, GT, MODE, ADAM>(a, shape, stream);
    case 8: return launch_vector<8, GT, MODE, ADAM>(a, shape, stream);
    case 12: return launch_vector<12, GT, MODE, ADAM>(a, shape, stream);
    case 16: return launch_vector<16, GT, MODE, ADAM>(a, shape, stream);
    default: return launch_vector<0, GT, MODE, ADAM>(a, shape, stream);
    }
}

template <bool ADAM>
hipError_t dispatch(const LaunchArgs &a, bool vec, Shape shape, hipStream_t stream)
{
    if (a.gdtype == kGradI32)  // the front end admits int32 only in fixed mode
        return dispatch_w<kGradI32, kAggFixed, ADAM>(a, vec, shape, stream);
    if (a.gdtype == kGradF32)
        return a.mode == kAggFP32 ? dispatch_w<kGradF32, kAggFP32, ADAM>(a, vec, shape, stream)
                                  : dispatch_w<kGradF32, kAggFixed, ADAM>(a, vec, shape, stream);
    return a.mode == kAggFP32 ? dispatch_w<kGradBF16, kAggFP32, ADAM>(a, vec, shape, stream)
                              : dispatch_w<kGradBF16, kAggFixed, ADAM>(a, vec, shape, stream);
}

}  // namespace

hipError_t launch(const LaunchArgs &a, Kind kind, bool vector_path, hipStream_t stream)
{
    const Shape shape = launch_shape();
    return kind == kAggregateAdam ? dispatch<true>(a, vector_path, shape, stream)
                                  : dispatch<false>(a, vector_path, shape, stream);
}

namespace {

// Tensor `c` of a batch as a call of its own.
LaunchArgs single_of(const MultiArgs &a, int c)
{
    LaunchArgs one{};
    void *const *ptr = a.ptr + c * (a.W + 4);
    for (int w = 0; w < a.W; ++w)
        one.g[w] = ptr[w];
    one.p = static_cast<float *>(ptr[a.W]);
    one.m = static_cast<float *>(ptr[a.W + 1]);
    one.v = static_cast<float *>(ptr[a.W + 2]);
    one.p16 = static_cast<uint16_t *>(ptr[a.W + 3]);
    one.n = a.n[c];
    one.head = a.head[c];
    one.W = a.W;
    one.gdtype = a.gdtype;
    one.mode = a.mode;
    one.frac_bits = a.frac_bits;
    one.qscale = a.qscale;
    one.dqscale = a.dqscale;
    one.s = a.s;
    one.s_dev = a.s_dev;
    return one;
}

// Whether tensor `c` lies as far from tensor `base` in every array, counted in
// elements.
bool same_offset(const MultiArgs &a, int base, int c, int grad_bytes)
{
    const int per = a.W + 4;
    void *const *x = a.ptr + base * per, *const *y = a.ptr + c * per;
    if ((x[a.W + 3] == nullptr) != (y[a.W + 3] == nullptr))
        return false;
    const int64_t off = (static_cast<char *>(y[a.W]) - static_cast<char *>(x[a.W])) / 4;
    for (int k = 0; k < per; ++k) {
        const int esz = k < a.W ? grad_bytes : k == a.W + 3 ? 2 : 4;
        if (x[k] && static_cast<char *>(y[k]) - static_cast<char *>(x[k]) != off * esz)
            return false;
    }
    return true;
}

// Bytes of a MultiLaunch table: first blocks, shapes, then the rows.
constexpr int multi_slots(int count) { return (count + 1 + 15) & ~15; }
constexpr int multi_rows_at(int count) { return (4 * (multi_slots(count) + count) + 7) & ~7; }
constexpr int multi_bytes(int count, int W, bool flat)
{
    return multi_rows_at(count) + (flat ? 8 * count + 8 * (W + 4) : 8 * (W + 4) * count);
}

// what include/disdp.h states for W = 8
static_assert(multi_bytes(36, 8, false) <= kMultiTable && multi_bytes(37, 8, false) > kMultiTable &&
                  multi_bytes(232, 8, true) <= kMultiTable &&
                  multi_bytes(233, 8, true) > kMultiTable &&
                  multi_bytes(kMultiMost, 1, true) > kMultiTable,
              "tensors of a launch");

// The many-tensor kernel always runs one-wave blocks.  A launch takes the
// next tensors that fit its arguments: as slices of flat buffers when at
// least as many in a row are (232 against 36 tensors with rows of their own at
// W = 8), and a tensor that is alone goes to the vector kernel, which has no
// tensor to look up.
template <int W, int GT, int MODE>
hipError_t launch_multi_w(const MultiArgs &a, hipStream_t stream)
{
    constexpr int kGradBytes = GT == kGradBF16 ? 2 : 4;
    constexpr int kLaneBytes = W > 0 ? 4 * (W * kGradBytes + 12) : 1 << 30;
    constexpr bool kConverts = MODE == kAggFixed && GT != kGradI32;
    // one wave more than one tensor's kernel: they look their tensor up
    // before their loads (122 tensors of 15.7M elements, W = 4 bf16, 10 waves
    // 87.3 us, 8 89.8, 12 88.1)
    const int base = 1 + (W == 0 ? runtime_w_waves(a.W, GT, MODE, true)
                                 : fused_waves(kLaneBytes, kConverts && GT == kGradBF16, false));
    const int lds = occupancy_lds_bytes(blocks_per_cu_cap(base, kWave, stream));
    const int per = a.W + 4;
    int general = 1;  // tensors a launch holds with rows of their own
    while (general < kMultiMost && multi_bytes(general + 1, a.W, false) <= kMultiTable)
        ++general;
    MultiLaunch k;
    k.W = a.W;
    k.zero = 0;
    k.qscale = a.qscale;
    k.dqscale = a.dqscale;
    k.s = a.s;
    k.s_dev = a.s_dev;
    for (int i = 0; i < a.count;) {
        const int left = a.count - i;
        int run = 1;
        while (run < left && run < kMultiMost && multi_bytes(run + 1, a.W, true) <= kMultiTable &&
               same_offset(a, i, i + run, kGradBytes))
            ++run;
        k.flat = run >= (general < left ? general : left);
        const int most = k.flat ? run : general < left ? general : left;
        // as many of them as one grid holds
        int64_t blocks = 0;
        int take = 0;
        Split sp[kMultiMost];
        for (; take < most; ++take) {
            const int64_t n = a.n[i + take];
            sp[take] = make_split(n >> 2, a.head[i + take], static_cast<int>(n & 3), 0);
            const int64_t add = sp[take].lead + ceil_div(sp[take].n_groups, kWave);
            if (blocks + add > max_blocks(kWave))
                break;
            blocks += add;
        }
        if (take <= 1) {
            const hipError_t e =
                launch_vector<W, GT, MODE, true>(single_of(a, i), Shape{kWave, false}, stream);
            if (e != hipSuccess)
                return e;
            ++i;
            continue;
        }
        const int slots = multi_slots(take);
        k.count = take;
        k.rows_at = multi_rows_at(take);
        uint32_t *first = reinterpret_cast<uint32_t *>(k.table);
        uint32_t at = 0;
        for (int j = 0; j < take; ++j) {
            const int64_t tiles = ceil_div(sp[j].n_groups, kWave);
            first[j] = at;
            first[slots + j] =
                pack_shape(sp[j].head, sp[j].tail,
                           static_cast<int>(tiles ? sp[j].n_groups - (tiles - 1) * kWave : 0));
            at += static_cast<uint32_t>(sp[j].lead + tiles);
        }
        first[take] = at;
        for (int j = take + 1; j < slots; ++j)
            first[j] = ~0u;
        for (int j = 0; j < 16; ++j)
            k.coarse[j] = 16 * j < slots ? first[16 * j] : ~0u;
        int64_t *rows = reinterpret_cast<int64_t *>(k.table + k.rows_at);
        if (k.flat) {
            const char *p0 = static_cast<const char *>(a.ptr[i * per + a.W]);
            for (int j = 0; j < take; ++j)
                rows[j] = (static_cast<const char *>(a.ptr[(i + j) * per + a.W]) - p0) / 4;
            rows += take;
        }
        std::memcpy(rows, a.ptr + i * per, sizeof(void *) * per * (k.flat ? 1 : take));
        void *args[] = {&k};
        const hipError_t e = hipLaunchKernel(
            reinterpret_cast<const void *>(&multi_kernel<W, GT, MODE>),
            dim3(static_cast<unsigned>(blocks)), dim3(kWave), args, static_cast<size_t>(lds),
            stream);
        if (e != hipSuccess)
            return e;
        i += take;
    }
    return hipSuccess;
}

template <int GT, int MODE>
hipError_t launch_multi_gm(const MultiArgs &a, hipStream_t stream)
{
    switch (a.W) {
    case 1: return launch_multi_w<1, GT, MODE>(a, stream);
    case 2: return launch_multi_w<2, GT, MODE>(a, stream);
    case 3: return launch_multi_w<3, GT, MODE>(a, stream);
    case 4: return launch_multi_w<4, GT, MODE>(a, stream);
    case 5: return launch_multi_w<5, GT, MODE>(a, stream);
    case 6: return launch_multi_w<6, GT, MODE>(a, stream);
    case 7: return launch_multi_w<7, GT, MODE>(a, stream);
    case 8: return launch_multi_w<8, GT, MODE>(a, stream);
    case 12: return launch_multi_w<12, GT, MODE>(a, stream);
    case 16: return launch_multi_w<16, GT, MODE>(a, stream);
    default: return launch_multi_w<0, GT, MODE>(a, stream);
    }
}

}  // namespace

hipError_t launch_multi(const MultiArgs &a, hipStream_t stream)
{
    if (a.gdtype == kGradI32)  // the front end admits int32 only in fixed mode
        return launch_multi_gm<kGradI32, kAggFixed>(a, stream);
    if (a.gdtype == kGradF32)
        return a.mode == kAggFP32 ? launch_multi_gm<kGradF32, kAggFP32>(a, stream)
                                  : launch_multi_gm<kGradF32, kAggFixed>(a, stream);
    return a.mode == kAggFP32 ? launch_multi_gm<kGradBF16, kAggFP32>(a, stream)
                              : launch_multi_gm<kGradBF16, kAggFixed>(a, stream);
}

hipError_t launch_quantize(const QuantizeArgs &q, bool vector_path, hipStream_t stream)
{
    const bool bf16 = q.gdtype == kGradBF16;
    if (!vector_path) {
        const void *fn = bf16 ? reinterpret_cast<const void *>(&quantize_element_kernel<kGradBF16>)
                              : reinterpret_cast<const void *>(&quantize_element_kernel<kGradF32>);
        void *args[] = {const_cast<QuantizeArgs *>(&q)};
        return hipLaunchKernel(
            fn, dim3(static_cast<unsigned>(clamp_grid(ceil_div(q.n, kWave), kWave))), dim3(kWave),
            args, 0, stream);
    }
    const void *fn = bf16 ? reinterpret_cast<const void *>(&quantize_vector_kernel<kGradBF16>)
                          : reinterpret_cast<const void *>(&quantize_vector_kernel<kGradF32>);
    QuantizeVectorArgs k{base_of(q.g), base_of(q.out), 0, 0, q.qscale, {}};
    int64_t left = q.n >> 2;  // as in launch_vector
    int head = q.head;
    do {
        const int64_t most = (max_blocks(kWave) - 2) * kWave;
        const int64_t now = left < most ? left : most;
        left -= now;
        k.n_groups = now;
        k.edges = make_split(0, head, left ? 0 : static_cast<int>(q.n & 3), 0);
        k.lead = k.edges.lead;
        const int64_t blocks = k.lead + ceil_div(now, kWave);
        void *args[] = {&k};
        const hipError_t e = hipLaunchKernel(fn, dim3(static_cast<unsigned>(blocks)), dim3(kWave),
                                             args, 0, stream);
        if (e != hipSuccess)
            return e;
        k.g += 4 * now * (bf16 ? 2 : 4);
        k.out += 4 * now * 4;
        head = 0;
    } while (left > 0);
    return hipSuccess;
}

}  // namespace disdp
