// Device code of the capture-and-stage path for gfx950 (MI355X).
//
// capture_kernel is the producer of the paper's Ring^2 (section 4.2, steps 1-2;
// section 5 "Device-to-device kernel"; section 4.4 gather-compact): it copies the
// selected rows of one observed tensor into the device byte ring and publishes the
// record; or, in one launch, the rows of up to kMaxBatch tensors of one layout that share a
// selection, one record each, laid down as single launches in the same order would (a
// launch costs microseconds whatever it moves, and only more bytes per launch amortise
// that).  The paper's kernel (1-64 blocks, grid-stride 16-byte copies, last block
// publishes) is prior art for other hardware; here
//   * every workgroup scans the per-request row counts for itself (DPP prefix sums of 64
//     requests at a time, kept in LDS; capture_rows_kernel: every wavefront, in registers),
//     so row -> (request, token) needs no pre-pass launch;
//   * rows are read with 16-byte vector loads and written with non-temporal
//     16-byte stores (the ring is not read again by the GPU, so it should not
//     displace the model's working set from the 4 MB per-XCD L2);
//   * downcasts and fp32 row summaries happen in the same pass, summaries reduced
//     by DPP (no matrix cores: nothing here is a contraction);
//   * the record's place in the ring comes from a device-resident head, and the
//     drop-newest decision from the drained mark as an earlier launch read it from a
//     word the host keeps current, both double buffered along the chain of launches:
//     every workgroup reads the same values with no atomic and no workgroup has to be
//     "the last one" (a compare-and-swap on one word from a thousand workgroups
//     measured 7 us here);
//   * there is no fence and no completion counter in the kernel: on this GPU a
//     device-scope fence writes back a whole L2, once per wavefront that issues it
//     (measured: 19 us for a 64-workgroup capture, 300 us for 2048 workgroups).
//     One lane of one workgroup writes where the head stands into this launch's commit slot in
//     device memory, and the host fetches a slot only behind an event recorded after
//     the launch (the kernel-end release makes payload and slot visible);
//   * a small capture is a chain of dependent trips to memory and little else, so every
//     kernel here fetches its argument lines, its control words and its first rows in
//     as few trips as their dependencies allow (see touch_argument_lines, fetch_control,
//     lds_barrier), and the common small shapes have a short straight-line kernel of
//     their own (capture_decode_kernel).
#include "dmi_internal.h"
#include "dmi_debug.h"

#include <hip/hip_ext.h>
#include <hip/hip_fp16.h>

#include <cstddef>
#include <cstring>
#include <type_traits>

namespace dmi {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

enum OutMode { OUT_RAW = 0, OUT_FP16 = 1, OUT_FP8 = 2, OUT_NONE = 3 };

// ---------------------------------------------------------------- atomics
__device__ __forceinline__ uint64_t ld_agent(const uint64_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// a word the host writes (pinned host memory): every read crosses the host link
__device__ __forceinline__ uint64_t ld_system(const uint64_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// the same the other way: past every cache, and on its way at once
__device__ __forceinline__ void st_system(uint64_t *p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---------------------------------------------------------------- wavefront helpers
// Workgroup barrier that orders LDS traffic only.  __syncthreads() also makes every
// wavefront wait until all of its global stores have been acknowledged, a round trip to
// memory of a microsecond or more; values handed over through LDS do not need that, and
// nothing here reads global memory written by another lane of the same launch.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A value that is the same in every lane, said to be.
__device__ __forceinline__ uint64_t uniform_u64(uint64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}
// Wavefront reductions with DPP (data-parallel primitives: the cross-lane operand rides on the
// ALU instruction, no trip through LDS).  quad_perm / row_half_mirror / row_mirror combine the 16
// lanes of a row, row_bcast15 / row_bcast31 carry row totals forward; lane 63 ends up with the
// total, which is read back as a scalar.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xF, false);
}
// Inclusive prefix sums over the wavefront (all 64 lanes of it), the same way: within rows of 16 lanes by shifts of
// 1, 2, 4 and 8, then the rows' totals carried forward.  Shuffles through LDS take six dependent trips of 60 ns.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v)
{
    v += dpp_u32<0x111, 0xF>(v);        // row_shr:1
    v += dpp_u32<0x112, 0xF>(v);        // row_shr:2
    v += dpp_u32<0x114, 0xF>(v);        // row_shr:4
    v += dpp_u32<0x118, 0xF>(v);        // row_shr:8
    v += dpp_u32<0x142, 0xA>(v);        // row_bcast15 into rows 1, 3
    v += dpp_u32<0x143, 0xC>(v);        // row_bcast31 into rows 2, 3
    return v;
}
__device__ __forceinline__ float wave_sum(float v)
{
    v += __uint_as_float(dpp_u32<0xB1, 0xF>(__float_as_uint(v)));      // quad_perm [1,0,3,2]
    v += __uint_as_float(dpp_u32<0x4E, 0xF>(__float_as_uint(v)));      // quad_perm [2,3,0,1]
    v += __uint_as_float(dpp_u32<0x141, 0xF>(__float_as_uint(v)));     // row_half_mirror
    v += __uint_as_float(dpp_u32<0x140, 0xF>(__float_as_uint(v)));     // row_mirror
    v += __uint_as_float(dpp_u32<0x142, 0xA>(__float_as_uint(v)));     // row_bcast15 into rows 1, 3
    v += __uint_as_float(dpp_u32<0x143, 0xC>(__float_as_uint(v)));     // row_bcast31 into rows 2, 3
    return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), 63));
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
    uint32_t o;
    o = dpp_u32<0xB1, 0xF>(v);  v = o > v ? o : v;
    o = dpp_u32<0x4E, 0xF>(v);  v = o > v ? o : v;
    o = dpp_u32<0x141, 0xF>(v); v = o > v ? o : v;
    o = dpp_u32<0x140, 0xF>(v); v = o > v ? o : v;
    o = dpp_u32<0x142, 0xA>(v); v = o > v ? o : v;
    o = dpp_u32<0x143, 0xC>(v); v = o > v ? o : v;
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// The same over groups of `width` consecutive lanes (a power of two from 4 to 64, the same in every
// lane): the last lane of each group ends up with the group's total.  The steps are those above in
// the same order, so a group's total has the bits that wave_sum gives for the group alone.
__device__ __forceinline__ float group_sum(float v, uint32_t width)
{
    v += __uint_as_float(dpp_u32<0xB1, 0xF>(__float_as_uint(v)));
    v += __uint_as_float(dpp_u32<0x4E, 0xF>(__float_as_uint(v)));
    if (width >= 8u) v += __uint_as_float(dpp_u32<0x141, 0xF>(__float_as_uint(v)));
    if (width >= 16u) v += __uint_as_float(dpp_u32<0x140, 0xF>(__float_as_uint(v)));
    if (width >= 32u) v += __uint_as_float(dpp_u32<0x142, 0xA>(__float_as_uint(v)));
    if (width == 64u) v += __uint_as_float(dpp_u32<0x143, 0xC>(__float_as_uint(v)));
    return v;
}
__device__ __forceinline__ uint32_t group_max_u32(uint32_t v, uint32_t width)
{
    uint32_t o;
    o = dpp_u32<0xB1, 0xF>(v);  v = o > v ? o : v;
    o = dpp_u32<0x4E, 0xF>(v);  v = o > v ? o : v;
    if (width >= 8u)  { o = dpp_u32<0x141, 0xF>(v); v = o > v ? o : v; }
    if (width >= 16u) { o = dpp_u32<0x140, 0xF>(v); v = o > v ? o : v; }
    if (width >= 32u) { o = dpp_u32<0x142, 0xA>(v); v = o > v ? o : v; }
    if (width == 64u) { o = dpp_u32<0x143, 0xC>(v); v = o > v ? o : v; }
    return v;
}

// ---------------------------------------------------------------- conversions
// bf16 -> fp8 E4M3FN (OCP: bias 7, max 448, no inf, S.1111.111 NaN), round to
// nearest even, saturating.  Integer arithmetic on the bf16 bit pattern; used on the
// element-wise path (rows that cannot be moved as 16-byte vectors).
__device__ __forceinline__ uint32_t bf16_to_fp8(uint32_t b)
{
    const uint32_t sign = (b >> 8) & 0x80u;
    const uint32_t a = b & 0x7FFFu;
    const uint32_t e = a >> 7;
    uint32_t code;
    if (e >= 121u) {
        // normal in fp8 (|x| >= 2^-6): rebias 127 -> 7, drop 4 mantissa bits with RNE
        const uint32_t x = a - (120u << 7);
        code = (x + 7u + ((x >> 4) & 1u)) >> 4;
        code = code > 0x7Eu ? 0x7Eu : code;
    } else {
        // fp8 subnormal: |x| / 2^-9 = (128 + m) >> (125 - e), RNE; vanishes for shifts > 8
        const uint32_t sh = 125u - e;
        const uint32_t s = sh > 9u ? 9u : sh;
        const uint32_t v = 128u + (a & 0x7Fu);
        code = (v + (1u << (s - 1u)) - 1u + ((v >> s) & 1u)) >> s;
    }
    if (a > 0x7F80u) code = 0x7Fu;
    return sign | code;
}

// Two bf16 (one 32-bit word) -> two fp8 E4M3FN codes in the low or high half of `acc`.
// gfx950's packed convert rounds to nearest even into the OCP format, subnormals
// included, but does not saturate (values that round beyond 448, and infinities, come
// out as NaN) and drops a NaN's sign; so magnitudes are clamped to 448 first with a
// packed 16-bit minimum, and words holding a NaN are patched afterwards.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef short s16x2_t __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ s16x2_t bf16x2_to_fp8x2(uint32_t w, s16x2_t acc, bool hi, uint32_t &nan)
{
    const uint32_t mag = w & 0x7FFF7FFFu;
    const u16x2_t lim = {0x43E0u, 0x43E0u};                                   // 448.0
    const u16x2_t cl = __builtin_elementwise_min(__builtin_bit_cast(u16x2_t, mag), lim);
    const uint32_t x = __builtin_bit_cast(uint32_t, cl) | (w & 0x80008000u);
    const bf16x2_t v = __builtin_bit_cast(bf16x2_t, x);
    const u16x2_t inf = {0x7F80u, 0x7F80u};
    nan |= __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2_t, mag), inf));
    return hi ? __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(acc, v, 1.0f, true)
              : __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(acc, v, 1.0f, false);
}

// Eight bf16 -> eight fp8.
__device__ __forceinline__ u32x2 bf16x8_to_fp8x8(u32x4 v)
{
    uint32_t nan = 0;
    s16x2_t lo = {0, 0}, hi = {0, 0};
    lo = bf16x2_to_fp8x2(v.x, lo, false, nan);
    lo = bf16x2_to_fp8x2(v.y, lo, true, nan);
    hi = bf16x2_to_fp8x2(v.z, hi, false, nan);
    hi = bf16x2_to_fp8x2(v.w, hi, true, nan);
    u32x2 o = {__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
    if (__builtin_expect(nan != 0u, 0)) {       // a NaN somewhere in the eight: sign | 0x7F
        for (uint32_t i = 0; i < 8u; i++) {
            const uint32_t word = i < 4u ? (i < 2u ? v.x : v.y) : (i < 6u ? v.z : v.w);
            const uint32_t e = (i & 1u ? word >> 16 : word) & 0xFFFFu, sh = 8u * (i & 3u);
            if ((e & 0x7FFFu) <= 0x7F80u) continue;
            const uint32_t code = ((e >> 8) & 0x80u) | 0x7Fu;
            if (i < 4u) o.x = (o.x & ~(0xFFu << sh)) | (code << sh);
            else o.y = (o.y & ~(0xFFu << sh)) | (code << sh);
        }
    }
    return o;
}

// bf16 -> fp16: exact widening to f32, then the hardware's round-to-nearest-even
// convert (overflow to inf, gradual underflow); NaN -> sign | 0x7E00.
__device__ __forceinline__ uint32_t bf16_to_fp16(uint32_t b)
{
    const float f = __uint_as_float(b << 16);
    uint32_t h = (uint32_t)__half_as_ushort(__float2half_rn(f));
    if ((b & 0x7FFFu) > 0x7F80u) h = ((b >> 15) << 15) | 0x7E00u;
    return h;
}

__device__ __forceinline__ float widen16(uint32_t bits, uint32_t src_dtype)
{
    return src_dtype == 1u ? __uint_as_float(bits << 16)
                           : __half2float(__ushort_as_half((unsigned short)bits));
}

// ---------------------------------------------------------------- units
// A unit is what one lane moves per access: 16 source bytes, or one element where rows are shorter than that
// and not 16-byte movable.
template <int NB> struct UnitT;
template <> struct UnitT<16> { typedef u32x4 T; };
template <> struct UnitT<8>  { typedef u32x2 T; };
template <> struct UnitT<4>  { typedef uint32_t T; };
template <> struct UnitT<2>  { typedef uint16_t T; };
template <> struct UnitT<1>  { typedef uint8_t T; };

struct RingW {
    uint8_t *ring;
    uint64_t cap;
    uint64_t base;      // physical offset of the record's first byte
};

template <typename T>
__device__ __forceinline__ void ring_store(const RingW &w, uint64_t off, T v)
{
    uint64_t p = w.base + off;
    if (p >= w.cap) p -= w.cap;
    // streaming stores for the vectors a wavefront lays down as whole lines; small scalars (a
    // summary value per workgroup, pad bytes) are left to L2 to merge: as streaming stores of a
    // fraction of a line they cost a launch microseconds
    if constexpr (sizeof(T) >= 8) __builtin_nontemporal_store(v, reinterpret_cast<T *>(w.ring + p));
    else *reinterpret_cast<T *>(w.ring + p) = v;
}

// The same at any address, also across the end of the ring: rows that do not sit on a 16-byte grid are moved in
// 16-byte units all the same (the memory system takes such accesses; only a unit that wraps is taken apart).
template <bool LOOSE, typename T>
__device__ __forceinline__ void store_out(uint8_t *p, T v)
{
    typedef T __attribute__((aligned(LOOSE ? 1 : sizeof(T)))) any_t;
    __builtin_nontemporal_store(v, reinterpret_cast<any_t *>(p));
}
template <bool LOOSE, typename T>
__device__ __forceinline__ void unit_store(const RingW &w, uint64_t off, T v)
{
    if constexpr (!LOOSE) {
        ring_store<T>(w, off, v);
    } else {
        uint64_t p = w.base + off;
        if (p >= w.cap) p -= w.cap;
        if (p + sizeof(T) <= w.cap) {
            store_out<true>(w.ring + p, v);
        } else {
            constexpr uint32_t n = sizeof(T) / 4u;
            const auto words = __builtin_bit_cast(typename UnitT<sizeof(T)>::T, v);
            for (uint32_t i = 0; i < sizeof(T); i++) {
                uint32_t word = words[0];
                for (uint32_t k = 1; k < n; k++) word = i / 4u == k ? words[k] : word;
                uint64_t q = p + i;
                if (q >= w.cap) q -= w.cap;
                w.ring[q] = (uint8_t)(word >> (8u * (i & 3u)));
            }
        }
    }
}

// Per-lane partial row summaries.  Sum of squares and sum are fp32; the largest magnitude is
// kept as the bit pattern of |x| in the source format (sign-magnitude formats order like
// unsigned integers, and a NaN, whose pattern is above infinity's, wins the maximum and so
// surfaces as NaN).  16-bit sources keep two independent 16-bit maxima in one word.
struct Accum {
    float ss, s;
    uint32_t am;
};

typedef _Float16 h16x2_t __attribute__((ext_vector_type(2)));

// two 16-bit elements in one word: v_dot2 does x0*x0 + x1*x1 + acc (and x0 + x1 + acc with a
// vector of ones) without unpacking; v_pk_max_u16 tracks the magnitudes
__device__ __forceinline__ void accum_pair(Accum &a, uint32_t w, bool is_bf16)
{
    if (is_bf16) {
        const bf16x2_t x = __builtin_bit_cast(bf16x2_t, w);
        const bf16x2_t one = __builtin_bit_cast(bf16x2_t, 0x3F803F80u);
        a.ss = __builtin_amdgcn_fdot2_f32_bf16(x, x, a.ss, false);
        a.s = __builtin_amdgcn_fdot2_f32_bf16(x, one, a.s, false);
    } else {
        const h16x2_t x = __builtin_bit_cast(h16x2_t, w);
        const h16x2_t one = __builtin_bit_cast(h16x2_t, 0x3C003C00u);
        a.ss = __builtin_amdgcn_fdot2(x, x, a.ss, false);
        a.s = __builtin_amdgcn_fdot2(x, one, a.s, false);
    }
    a.am = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2_t, a.am),
                                                                  __builtin_bit_cast(u16x2_t, w & 0x7FFF7FFFu)));
}

__device__ __forceinline__ void accum_f32(Accum &a, uint32_t bits)
{
    const float x = __uint_as_float(bits);
    a.ss = fmaf(x, x, a.ss);
    a.s += x;
    const uint32_t m = bits & 0x7FFFFFFFu;
    a.am = m > a.am ? m : a.am;
}

// one 16-bit element (element-wise path)
__device__ __forceinline__ void accum_16(Accum &a, uint32_t bits, uint32_t src_dtype)
{
    const float x = widen16(bits, src_dtype);
    a.ss = fmaf(x, x, a.ss);
    a.s += x;
    const uint32_t m = bits & 0x7FFFu;
    a.am = m > a.am ? m : a.am;
}

// the lane's magnitude maximum as one value comparable across lanes
template <int ES_IN, int VEC>
__device__ __forceinline__ uint32_t fold_am(uint32_t am)
{
    if constexpr (ES_IN == 2 && VEC == 8) return (am & 0xFFFFu) > (am >> 16) ? (am & 0xFFFFu) : (am >> 16);
    else return am;
}

__device__ __forceinline__ float am_value(uint32_t m, uint32_t src_dtype)
{
    if (src_dtype == 3u) return __uint_as_float(m);
    return widen16(m, src_dtype);
}

// One source unit as the record stores it.
template <int ES_IN, int VEC, int OUT>
__device__ __forceinline__ auto convert_unit(typename UnitT<ES_IN * VEC>::T v)
{
    if constexpr (OUT == OUT_FP16 && ES_IN == 2 && VEC == 8) {
        const uint32_t wd[4] = {v.x, v.y, v.z, v.w};
        uint32_t ow[4];
#pragma unroll
        for (int k = 0; k < 4; k++)
            ow[k] = bf16_to_fp16(wd[k] & 0xFFFFu) | (bf16_to_fp16(wd[k] >> 16) << 16);
        return u32x4{ow[0], ow[1], ow[2], ow[3]};
    } else if constexpr (OUT == OUT_FP8 && ES_IN == 2 && VEC == 8) {
        return bf16x8_to_fp8x8(v);
    } else if constexpr (OUT == OUT_FP16 && ES_IN == 2) {
        return (uint16_t)bf16_to_fp16(v);
    } else if constexpr (OUT == OUT_FP8 && ES_IN == 2) {
        return (uint8_t)bf16_to_fp8(v);
    } else {
        static_assert(OUT == OUT_RAW, "a source of this size is stored as it is");
        return v;
    }
}

// Convert one source unit and store it.
template <int ES_IN, int VEC, int OUT, bool LOOSE = false>
__device__ __forceinline__ void emit_unit(const RingW &w, uint64_t out_off, typename UnitT<ES_IN * VEC>::T v)
{
    if constexpr (OUT != OUT_NONE) unit_store<LOOSE && (VEC > 1)>(w, out_off, convert_unit<ES_IN, VEC, OUT>(v));
}

// Add one step's units (four per lane; a lane without that unit has zeros) to the row's partial summaries:
// every unit summed by itself, the four combined in pairs: shorter chains than one running sum.  (The norms' error
// against 64 bits is that of another order: 3.4 -> 4.0e-8 for 64 rows of 512 units, 4.1 -> 4.2e-8 for 32, and
// 16 -> 9.3e-8 for rows of 1024 fp32 units.)
template <int ES_IN, int VEC>
__device__ __forceinline__ void accum_units(Accum &acc, const typename UnitT<ES_IN * VEC>::T (&v)[4],
                                            uint32_t src_dtype)
{
    Accum u[4];
    for (uint32_t k = 0; k < 4; k++) u[k] = Accum{0.f, 0.f, 0u};
    if constexpr (ES_IN == 2 && VEC == 8) {
        // (the source type is asked for once: a branch per word costs more than the arithmetic it chooses)
        auto all = [&](auto is_bf16) {
#pragma unroll
            for (uint32_t k = 0; k < 4; k++) {
                accum_pair(u[k], v[k].x, is_bf16.value);
                accum_pair(u[k], v[k].y, is_bf16.value);
                accum_pair(u[k], v[k].z, is_bf16.value);
                accum_pair(u[k], v[k].w, is_bf16.value);
            }
        };
        if (src_dtype == 1u) all(std::true_type()); else all(std::false_type());
    } else {
#pragma unroll
        for (uint32_t k = 0; k < 4; k++) {
            if constexpr (VEC == 4) {
                accum_f32(u[k], v[k].x);
                accum_f32(u[k], v[k].y);
                accum_f32(u[k], v[k].z);
                accum_f32(u[k], v[k].w);
            } else if constexpr (ES_IN == 4) {
                accum_f32(u[k], v[k]);
            } else {
                accum_16(u[k], v[k], src_dtype);
            }
        }
    }
    acc.ss += (u[0].ss + u[1].ss) + (u[2].ss + u[3].ss);
    acc.s += (u[0].s + u[1].s) + (u[2].s + u[3].s);
    if constexpr (ES_IN == 2 && VEC == 8) {
        auto mx = [](uint32_t x, uint32_t y) {
            return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2_t, x),
                                                                          __builtin_bit_cast(u16x2_t, y)));
        };
        acc.am = mx(acc.am, mx(mx(u[0].am, u[1].am), mx(u[2].am, u[3].am)));
    } else {
        const uint32_t a = u[0].am > u[1].am ? u[0].am : u[1].am, b = u[2].am > u[3].am ? u[2].am : u[3].am;
        const uint32_t m = a > b ? a : b;
        acc.am = m > acc.am ? m : acc.am;
    }
}

// A unit of VEC elements with its first n set to zero.
template <int VEC>
__device__ __forceinline__ u32x4 without_first(u32x4 v, uint32_t n)
{
#pragma unroll
    for (uint32_t i = 0; i < 4; i++) {
        const uint32_t per = VEC / 4u;      // elements of a 32-bit word
        const uint32_t gone = n <= i * per ? 0u : n - i * per < per ? n - i * per : per;
        v[i] &= gone == 0u ? 0xFFFFFFFFu : gone == per ? 0u : 0xFFFF0000u;
    }
    return v;
}

template <int ES_IN, int VEC, int OUT>
__host__ __device__ constexpr uint32_t out_unit_bytes()
{
    return OUT == OUT_NONE ? 0u : OUT == OUT_FP8 ? (uint32_t)VEC : (uint32_t)(ES_IN * VEC);
}

// ---------------------------------------------------------------- LDS layout
struct LdsMap {
    uint32_t hdr, heads, red, bcast, pref, btot, pref_all, btot_all, tab, rb, total_words;
};

__host__ __device__ inline LdsMap lds_map(uint32_t n_reqs, bool index_mode, bool table_in_lds)
{
    LdsMap m;
    const uint32_t nb = (n_reqs + 63u) / 64u;
    uint32_t p = 0;
    m.hdr = p; p += 16;
    m.heads = p; p += 8;
    m.red = p; p += 12;
    m.bcast = p; p += 12;          // head, tail, ring offset of the head, policy flags, seq, step id
    m.pref = p; p += n_reqs + 1;
    m.btot = p; p += nb + 1;
    m.pref_all = p; m.btot_all = p;
    if (index_mode) { p += n_reqs + 1; m.btot_all = p; p += nb + 1; }
    p = (p + 3u) & ~3u;
    m.tab = p; m.rb = p;
    if (table_in_lds) { p += 4 * n_reqs; m.rb = p; p += n_reqs; }
    m.total_words = p;
    return m;
}

uint32_t capture_lds_bytes(uint32_t n_reqs, bool index_mode, bool table_in_lds)
{
    return lds_map(n_reqs, index_mode, table_in_lds).total_words * 4u;
}

// Where one output row comes from.
struct RowRef {
    const uint8_t *base;    // dense: first byte of the row; paged: first byte of the slot
    uint64_t ok;            // 0 if a device-side index left the source (a full word: the struct
                            // is copied around and should stay in registers)
};

// Control words of one launch, fetched by one lane per workgroup.  Every load is issued
// before any result is used, whether or not this launch needs it: loads issued together
// cost one trip to memory, loads issued as their conditions become known cost one each.
struct RawControl {
    uint64_t head, head_at, tail_for, sp_seq, sp_step, sp_floor;
    uint64_t cap[3], drop[3];
    uint32_t sp_flags;
};
struct Control {
    uint64_t head, tail, seq, step_id;
    uint32_t flags;
};

// Issues the loads and touches none of the results, so that the caller can put more
// loads behind them before the first wait.
__device__ __forceinline__ RawControl fetch_control(const DevCtrl *c, uint32_t par, const StepParams *step)
{
    RawControl r;
    // a launch outside a replayable step reads (and ignores) the head of the control block instead
    const StepParams *spp = step ? step : reinterpret_cast<const StepParams *>(c);
    r.head = c->head[par];
    r.head_at = c->head_at[par];
    r.tail_for = c->tail_for[par];
    r.sp_seq = spp->seq_base; r.sp_step = spp->step_id; r.sp_floor = spp->tail_floor;
    r.sp_flags = spp->flags;
    r.cap[0] = c->captured_records; r.cap[1] = c->captured_rows; r.cap[2] = c->captured_bytes;
    r.drop[0] = c->dropped_records; r.drop[1] = c->dropped_rows; r.drop[2] = c->dropped_bytes;
    return r;
}

__device__ __forceinline__ Control resolve_control(const RawControl &r, bool in_step, uint32_t node,
                                                   uint64_t tail_floor, uint64_t seq, uint64_t step_id, uint32_t flags)
{
    Control o;
    o.head = r.head;
    o.seq = in_step ? r.sp_seq + node : seq;
    o.step_id = in_step ? r.sp_step : step_id;
    o.flags = in_step ? r.sp_flags : flags;
    const uint64_t floor = in_step ? r.sp_floor : tail_floor;
    o.tail = (o.flags & kStepDropNewest) && r.tail_for > floor ? r.tail_for : floor;
    return o;
}

// How many of a launch's n records, all of one size, fit behind the head it found (a prefix of them).
__device__ __forceinline__ uint64_t records_that_fit(uint64_t n, uint64_t head, uint64_t tail, uint64_t record_bytes,
                                                     uint64_t cap, bool drop_newest)
{
    if (!drop_newest) return n;
    const uint64_t used = head - tail, fit = used < cap ? (cap - used) / record_bytes : 0u;
    return fit < n ? fit : n;
}

// One lane of a launch leaves head and counters for the next launch and fills the commit slot of its last record
// (slot: NULL in a replayable step, where it follows from the sequence number).  Device memory only; it becomes visible to
// the next launch, and to the copy that fetches the slot, with the kernel-end release.
__device__ __forceinline__ void publish_launch(DevCtrl *c, uint32_t par, uint64_t head, uint64_t head_at, const uint64_t (&captured)[3],
                                               const uint64_t (&dropped)[3], uint64_t record_bytes, uint64_t n_rows,
                                               uint64_t n_fit, uint64_t n_drop, uint64_t cap, uint64_t last_seq, CommitSlot *slot)
{
    const uint64_t cap3[3] = {captured[0] + n_fit, captured[1] + n_fit * n_rows, captured[2] + n_fit * record_bytes};
    const uint64_t drop3[3] = {dropped[0] + n_drop, dropped[1] + n_drop * n_rows, dropped[2] + n_drop * record_bytes};
    if (n_drop) { c->dropped_records = drop3[0]; c->dropped_rows = drop3[1]; c->dropped_bytes = drop3[2]; }
    if (n_fit) { c->captured_records = cap3[0]; c->captured_rows = cap3[1]; c->captured_bytes = cap3[2]; }
    const uint64_t at = head_at + n_fit * record_bytes;     // (what is kept fits the ring: less than one lap further on)
    c->head[par ^ 1u] = head + n_fit * record_bytes;
    c->head_at[par ^ 1u] = at < cap ? at : at - cap;
    CommitSlot *h = slot ? slot : &c->slots[last_seq % kCommitSlots];
    h->head = head + n_fit * record_bytes;
    h->captured_records = cap3[0]; h->captured_rows = cap3[1]; h->captured_bytes = cap3[2];
    h->dropped_records = drop3[0]; h->dropped_rows = drop3[1]; h->dropped_bytes = drop3[2];
    h->seq_plus1 = last_seq + 1u;
}

// Fetch every line of a by-value kernel argument block now, together, along with this
// workgroup's entry of the batch block (its tensor and observation point).
template <typename T>
__device__ __forceinline__ void touch_argument_lines(const T &a, const uint8_t *src, uint32_t point)
{
    const uint32_t *p = reinterpret_cast<const uint32_t *>(&a);
    constexpr uint32_t n = (sizeof(T) + 63u) / 64u;
    static_assert(n <= 10, "argument block larger than expected");
    auto at = [p](uint32_t line) { return p[(line < n ? line : n - 1u) * 16u]; };
    asm volatile("" ::"s"(at(0)), "s"(at(1)), "s"(at(2)), "s"(at(3)), "s"(at(4)), "s"(at(5)), "s"(at(6)), "s"(at(7)),
                 "s"(at(8)), "s"(at(9)), "s"((uint32_t)(uintptr_t)src), "s"((uint32_t)((uintptr_t)src >> 32)), "s"(point));
}

// ---------------------------------------------------------------- capture kernel
// How a launch of the general kernel goes through its rows (kernels of their own, or the registers of one would cost the
// others a workgroup per compute unit).  Without summaries: units dealt to lanes in order, whatever row they are of.
// With summaries: a workgroup per row; several rows per wavefront, at most 256 units each (ONCE: read past the
// memory-side cache); a wavefront per row.
enum RowMode { ROWS_FLAT = 0, SUMM_ROWS = 1, SUMM_SHORT = 2, SUMM_WAVE = 3, SUMM_SHORT_ONCE = 4 };

// The request table of a launch into the caller's memory, where the launch carries it: in the second block of
// the kernel's own arguments, `first` bytes in.  Memory like any other to lanes that read entries of their own; and
// constant, so that what a whole workgroup reads (its row) comes through the scalar cache.
typedef __attribute__((address_space(1))) const uint32_t global_u32;
typedef __attribute__((address_space(4))) const uint32_t constant_u32;
__device__ __forceinline__ global_u32 *inline_table(uint32_t first)
{
    return (global_u32 *)((uintptr_t)__builtin_amdgcn_kernarg_segment_ptr() + first + offsetof(IntoArgs, words));
}
__device__ __forceinline__ constant_u32 *inline_table_uniform(uint32_t first)
{
    return (constant_u32 *)((uintptr_t)__builtin_amdgcn_kernarg_segment_ptr() + first + offsetof(IntoArgs, words));
}
static_assert(offsetof(IntoArgs, words) % 16u == 0 && sizeof(CaptureKernelArgs) % 16u == 0, "read as 16-byte entries");

// Entry r of such a table of n, and its first source row.  (Whether it lies by columns is a bit of a word that the launch's first trip to its
// arguments has brought along, and what else says how lies behind the words, read where it is, through the scalar cache: the block's arrays by
// name would be copied out of it first.  With a word of its own to ask for, and the words moved for it, the general kernel took 4.72 us for 64
// short rows with statistics, and not 4.38; like this 4.38, and no kernel needs a variant for such tables.)
__device__ __forceinline__ constant_u32 *inline_block(uint32_t first)
{
    return (constant_u32 *)((uintptr_t)__builtin_amdgcn_kernarg_segment_ptr() + first);
}
__device__ __forceinline__ u32x4 inline_entry(uint32_t first, uint32_t n_words, uint32_t n, uint32_t r)
{
    global_u32 *const w = inline_table(first);
    if (!(n_words & kByColumn)) return *(__attribute__((address_space(1))) const u32x4 *)(w + 4u * r);
    constant_u32 *const b = inline_block(first);
    const uint32_t even = b[offsetof(IntoArgs, even) / 4u];
    u32x4 e;
    uint32_t at = 0;
#pragma unroll
    for (uint32_t k = 0; k < 4u; k++) {
        if (even >> k & 1u) {
            e[k] = b[offsetof(IntoArgs, base) / 4u + k] + r * b[offsetof(IntoArgs, stride) / 4u + k];
        } else {
            e[k] = w[at + r];
            at += n;
        }
        asm volatile("" : "+v"(e[k]) : : "memory");     // one after the other: all their scalar registers at once are more than there are
    }
    return e;
}
__device__ __forceinline__ uint32_t inline_row(uint32_t first, uint32_t n_words, uint32_t n, uint32_t r)
{
    if (!(n_words & kByColumn)) return inline_table(first)[4u * n + r];
    constant_u32 *const b = inline_block(first);
    if (b[offsetof(IntoArgs, even) / 4u] & 16u)
        return b[offsetof(IntoArgs, base) / 4u + 4u] + r * b[offsetof(IntoArgs, stride) / 4u + 4u];
    return inline_table(first)[b[offsetof(IntoArgs, rows_at) / 4u] + r];
}

// LOOSE: rows of at least 16 bytes that do not sit on a 16-byte grid.  They are moved in 16-byte units too,
// a row's (or head's) last unit ending where the row does and so covering some elements a second time: those
// are stored twice with the same value and left out of the second unit's sums.
template <int ES_IN, int VEC, int OUT, int MODE, typename SRC, bool LOOSE>
__global__ void __launch_bounds__(kThreads) capture_kernel(const CaptureKernelArgs a, const SRC b)
{
    constexpr bool INTO = std::is_same<SRC, IntoArgs>::value;
    constexpr bool SHORT_ROWS = MODE == SUMM_SHORT || MODE == SUMM_SHORT_ONCE;
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    __shared__ float row_sums[SHORT_ROWS || MODE == SUMM_WAVE ? 4 * 192 : 1];   // per wavefront: totals of 64 rows
    const uint32_t y = INTO ? 0u : blockIdx.y;      // which tensor of the batch this workgroup works on
    const uint8_t *const src = b.src[y];
    const uint32_t point_id = b.point[y];
    touch_argument_lines(a, src, point_id);         // all of it in one trip, not one by one
    // entry r of the request table; where request r's rows begin (a row, or a row of the block table)
    auto table_entry = [&](uint32_t r) -> uint4 {
        if constexpr (INTO)
            if (b.n_words) {
                const u32x4 e = inline_entry(sizeof(CaptureKernelArgs), b.n_words, a.n_reqs, r);
                return make_uint4(e.x, e.y, e.z, e.w);
            }
        return a.req_table[r];
    };
    auto row_first = [&](uint32_t r) -> uint32_t {
        if constexpr (INTO)
            if (b.n_words) return inline_row(sizeof(CaptureKernelArgs), b.n_words, a.n_reqs, r);
        return a.row0[r];
    };
    constexpr uint32_t NB_IN = ES_IN * VEC;
    constexpr uint32_t NB_OUT = out_unit_bytes<ES_IN, VEC, OUT>();
    constexpr uint32_t ES_OUT = OUT == OUT_NONE ? 0u : OUT == OUT_FP8 ? 1u : (uint32_t)ES_IN;
    typedef typename UnitT<NB_IN>::T unit_t;
    // a unit as it is loaded: device memory (said explicitly, or a choice between two pointers costs the load its
    // type), at any address if the rows are
    typedef __attribute__((address_space(1))) const unit_t __attribute__((aligned(LOOSE ? ES_IN : ES_IN * VEC))) global_unit_t;

    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t n_reqs = a.n_reqs;
    const bool index_mode = a.row_index != nullptr;
    const bool simple = a.simple != 0;          // no keep mask and one row per request
    const LdsMap m = lds_map(simple ? 0u : n_reqs, index_mode, a.table_in_lds != 0);
    uint32_t *pref = lds + m.pref, *btot = lds + m.btot;
    uint32_t *pref_all = lds + m.pref_all, *btot_all = lds + m.btot_all;
    uint4 *ltab = reinterpret_cast<uint4 *>(lds + m.tab);
    uint32_t *lrb = lds + m.rb;
    const uint32_t nb = (n_reqs + 63u) / 64u;
    const uint32_t par = a.par_in;

    // -- control words: lane 0 of the last wavefront fetches head, tail copy, running counters
    //    and (for a replayable step) the step's parameters, all at once and whether or not this
    //    workgroup will need them, while the first wavefronts start on the request table.
    //    Every dependent trip to memory costs most of a microsecond, and a small capture is
    //    made of little else.  Head and tail are double buffered along the chain of launches:
    //    this launch reads what the previous one left and writes the other copy, so the
    //    values are the same for every workgroup with no atomic and no waiting.
    constexpr uint32_t kCtlTid = kThreads - 64u;
    uint64_t cnt_cap[3] = {0, 0, 0}, cnt_drop[3] = {0, 0, 0}, tail_now = 0, seq = a.seq;
    RawControl raw = {};
    if (!INTO && tid == kCtlTid)    // issued here, used just before the barrier below
        raw = fetch_control(a.ctrl, par, a.step);
    auto publish_control = [&]() {
        const Control ct = resolve_control(raw, a.step != nullptr, a.node, a.tail_floor, a.seq, a.step_id,
                                           a.drop_newest);
        seq = ct.seq;
        for (int i = 0; i < 3; i++) { cnt_cap[i] = raw.cap[i]; cnt_drop[i] = raw.drop[i]; }
        lds[m.bcast + 4] = (uint32_t)raw.head_at;
        lds[m.bcast + 5] = (uint32_t)(raw.head_at >> 32);
        lds[m.bcast + 0] = (uint32_t)ct.head;
        lds[m.bcast + 1] = (uint32_t)(ct.head >> 32);
        lds[m.bcast + 2] = (uint32_t)ct.tail;
        lds[m.bcast + 3] = (uint32_t)(ct.tail >> 32);
        lds[m.bcast + 6] = ct.flags;
        lds[m.bcast + 8] = (uint32_t)ct.seq;
        lds[m.bcast + 9] = (uint32_t)(ct.seq >> 32);
        lds[m.bcast + 10] = (uint32_t)ct.step_id;
        lds[m.bcast + 11] = (uint32_t)(ct.step_id >> 32);
    };
    if (tid < 8) lds[m.heads + tid] = a.heads_sel[tid];

    if (!simple) {
        // -- per-request kept row counts -> exclusive prefix sums (a wavefront's 64 by DPP)
        for (uint32_t b = wave; b < nb; b += kThreads / 64u) {
            const uint32_t r = b * 64u + lane;
            uint32_t cnt = 0, cnt_all = 0;
            if (r < n_reqs) {
                uint4 e = table_entry(r);
                cnt_all = e.w;
                const bool keep = a.keep_mask ? a.keep_mask[r] != 0 : true;
                cnt = keep ? cnt_all : 0u;
                if (a.table_in_lds) {
                    e.w = cnt;
                    ltab[r] = e;
                    lrb[r] = row_first(r);
                }
            }
            const uint32_t inc = wave_incl_scan(cnt);
            if (r < n_reqs) pref[r] = inc - cnt;
            if (lane == 63u) { btot[b] = inc; if (nb == 1u) pref[n_reqs] = inc; }
            if (index_mode) {
                const uint32_t inc_all = wave_incl_scan(cnt_all);
                if (r < n_reqs) pref_all[r] = inc_all - cnt_all;
                if (lane == 63u) { btot_all[b] = inc_all; if (nb == 1u) pref_all[n_reqs] = inc_all; }
            }
        }
        // up to 64 requests: one wavefront has done it all, and the barrier in front of the
        // geometry below is the only one needed
        if (nb != 1u) {
        lds_barrier();
        if (wave == 0) {
            uint32_t carry = 0, carry_all = 0;
            for (uint32_t b0 = 0; b0 < nb; b0 += 64u) {
                const uint32_t b = b0 + lane;
                const uint32_t v = b < nb ? btot[b] : 0u;
                const uint32_t inc = wave_incl_scan(v);
                if (b < nb) btot[b] = carry + inc - v;
                carry += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
                if (index_mode) {
                    const uint32_t va = b < nb ? btot_all[b] : 0u;
                    const uint32_t ia = wave_incl_scan(va);
                    if (b < nb) btot_all[b] = carry_all + ia - va;
                    carry_all += (uint32_t)__builtin_amdgcn_readlane((int)ia, 63);
                }
            }
            if (lane == 0) {
                btot[nb] = carry;
                if (index_mode) btot_all[nb] = carry_all;
            }
        }
        lds_barrier();
        for (uint32_t r = tid; r < n_reqs; r += kThreads) {
            pref[r] += btot[r >> 6];
            if (index_mode) pref_all[r] += btot_all[r >> 6];
        }
        if (tid == 0) {
            pref[n_reqs] = btot[nb];
            if (index_mode) pref_all[n_reqs] = btot_all[nb];
        }
        }
    }
    // first element of a segment's unit (a segment is a row, or a head's part of a paged row)
    auto elem_in_seg = [&](uint32_t c) -> uint64_t {
        const uint64_t e = (uint64_t)c * VEC;
        if constexpr (LOOSE) return e + VEC <= a.seg_elems ? e : a.seg_elems - VEC;
        else return e;
    };
    constexpr uint32_t U = 4;                               // loads in flight per lane
    constexpr uint32_t CH = U * kThreads;                   // units of one step of a workgroup
    const uint32_t cpr = (a.units_per_row + CH - 1u) / CH;  // SUMM_ROWS: steps of a workgroup per row
    const uint32_t wv = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave);
    const uint32_t wave_at = blockIdx.x * (kThreads / 64u) + wv, n_waves = gridDim.x * (kThreads / 64u);
    // summaries: the lanes that share a row; lane l takes units l, l + row_lanes, ..., four at a time
    const uint32_t row_lanes = MODE == ROWS_FLAT ? kThreads : a.row_lanes;
    if (INTO && tid < 12u) lds[m.bcast + tid] = tid == 8u    ? (uint32_t)a.seq
                                                : tid == 9u  ? (uint32_t)(a.seq >> 32)
                                                : tid == 10u ? (uint32_t)a.step_id
                                                : tid == 11u ? (uint32_t)(a.step_id >> 32)
                                                             : 0u;      // head, tail, policy: none
    if (!INTO && tid == kCtlTid) {
        // the drained-up-to mark for the next launch's drop decision: workgroup 0 reads it where
        // the host keeps it (a read across the host link, issued after every other load of this
        // lane so that none of them queues behind it; nothing in this launch waits for it but
        // the closing stores of this one lane)
        const uint64_t *ts = blockIdx.x == 0 && y == 0 && a.tail_src ? a.tail_src : &a.ctrl->tail;
        tail_now = ld_system(ts);
        publish_control();
    }
    lds_barrier();

    // -- record geometry
    // (what comes out of LDS here is the same in every lane, and said to be, so that it and all that follows from it --
    // sizes, places in the ring -- is scalar arithmetic in scalar registers)
    auto lds_word = [&](uint32_t i) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)lds[i]); };
    auto lds_pair = [&](uint32_t i) { return (uint64_t)lds_word(i) | ((uint64_t)lds_word(i + 1u) << 32); };
    const uint32_t n_rows = simple ? n_reqs : lds_word(m.pref + n_reqs);
    const uint32_t es_out = OUT == OUT_NONE ? 0u : OUT == OUT_FP8 ? 1u : (uint32_t)ES_IN;
    const uint64_t table_bytes = ((uint64_t)n_reqs * 16u + 63u) & ~63ull;
    const uint64_t payload_bytes = (uint64_t)n_rows * a.row_elems * es_out;
    const uint64_t off_payload = 64u + table_bytes;
    const uint64_t off_sum = off_payload + ((payload_bytes + 63u) & ~63ull);
    const uint64_t sum_arr = ((uint64_t)n_rows * 4u + 63u) & ~63ull;
    const uint32_t n_sum = __popc(a.summary_mask & 7u);
    const uint64_t record_bytes = off_sum + (uint64_t)n_sum * sum_arr;

    // Record y of the launch lies y records behind the head the launch found: all records of a
    // batch have the same size, so record y fits iff the y before it did, and then they were kept.
    const uint64_t head0 = lds_pair(m.bcast);
    const uint64_t head = head0 + (uint64_t)y * record_bytes;
    const uint32_t flags = lds_word(m.bcast + 6u);
    const bool publisher = !INTO && blockIdx.x == 0 && y == 0 && tid == kCtlTid;
    if (!INTO && (flags & kStepSkip)) {
        // a sampled-out replay: no record, no sequence number; the chain of head and tail
        // copies still has to reach the next launch
        if (publisher) {
            a.ctrl->head[par ^ 1u] = head0;
            a.ctrl->head_at[par ^ 1u] = raw.head_at;
            a.ctrl->tail_for[par ^ 1u] = tail_now > raw.tail_for ? tail_now : raw.tail_for;
        }
        return;
    }
    const uint64_t tail = lds_pair(m.bcast + 2u);
    const bool drop_newest = (flags & kStepDropNewest) != 0;
    const bool dropped = !INTO && (a.force_drop != 0u || (drop_newest && head - tail + record_bytes > a.cap));

    // ---- publish: one lane of the launch leaves head, tail and counters for the next launch and
    //      fills the commit slot of the launch's last record, early, so that it overlaps the copy.
    //      Everything here is device memory; it becomes visible to the next launch and to the copy
    //      that fetches the slot with the kernel-end release.
    if (publisher) {
        if (a.note) st_system(a.note, head0);
        const uint64_t last_seq = seq + gridDim.y + a.n_tail_drop - 1u;
        a.ctrl->tail_for[par ^ 1u] = tail_now > raw.tail_for ? tail_now : raw.tail_for;
        // (a loop of one lane over a uniform index: the points come straight out of the argument block)
        for (uint32_t i = 0; i < a.n_tail_drop; i++)
            atomicAdd(&a.ctrl->point_drops[b.point[gridDim.y + i] & 4095u], 1u);
        const uint64_t n_fit = a.force_drop ? 0u : records_that_fit(gridDim.y, head0, tail, record_bytes, a.cap, drop_newest);
        publish_launch(a.ctrl, par, head0, raw.head_at, cnt_cap, cnt_drop, record_bytes, n_rows, n_fit,
                       gridDim.y - n_fit + a.n_tail_drop, a.cap, last_seq, a.step ? nullptr : a.cslot);
    }
    if (dropped && blockIdx.x == 0 && tid == kCtlTid)
        atomicAdd(&a.ctrl->point_drops[point_id & 4095u], 1u);

    // Whoever issued a launch of several records made sure they fit the ring together (or the
    // ones that do not are dropped), so y records past the head are less than one lap away.
    RingW w;
    w.ring = a.ring;
    w.cap = a.cap;
    w.base = lds_pair(m.bcast + 4u) + (uint64_t)y * record_bytes;
    if (w.base >= w.cap) w.base -= w.cap;

    // row g -> request r (largest r with pref[r] <= g; requests with no rows are skipped
    // because their successor shares the same prefix) -> source location
    // (LDS is read through a pointer that says so: where the table may live either in LDS or
    // in global memory the compiler otherwise merges the two reads into one untyped load,
    // which counts as a global one and makes every wait for it a wait for the row loads too)
    typedef __attribute__((address_space(3))) uint32_t lds_u32;
    const lds_u32 *const L = (const lds_u32 *)lds;
    // In two halves: what has to be loaded to find the row (its index, or its block in the cache), and
    // where that puts it, so that a caller can put other loads in between.
    struct RowTok {
        uint32_t at;        // dense: the row; paged: the physical block (signed where it was loaded)
        uint32_t slot;
    };
    // (where a wavefront works on one row at a time, all of this but a load's result is scalar)
    constexpr bool ROW_PER_WAVE = MODE == SUMM_WAVE || MODE == SUMM_ROWS;
    auto rd = [&](uint32_t i) -> uint32_t { return ROW_PER_WAVE ? (uint32_t)__builtin_amdgcn_readfirstlane((int)L[i]) : L[i]; };
    // Row g's request, for all lanes at once: they look at 64 requests (or 64 evenly spaced ones of more) together: one trip
    // through LDS and a ballot where a binary search takes five of them for 32 requests.
    auto find_request = [&](uint32_t g) -> uint32_t {
        uint32_t lo = 0, span = n_reqs;                 // in [lo, lo + span)
        while (span > 1u) {
            const uint32_t apart = (span + 63u) >> 6, i = lane * apart;
            const uint32_t p = i < span ? L[m.pref + lo + i] : 0xFFFFFFFFu;
            const uint32_t k = (uint32_t)__popcll(__ballot(p <= g)) - 1u;
            lo += k * apart;
            span = span - k * apart < apart ? span - k * apart : apart;
        }
        return lo;
    };
    // `hint`: a request at or in front of row g's, from a caller that goes through rows in ascending order;
    // the row's request comes back in it.
    auto locate_begin = [&](uint32_t g, uint32_t &hint) -> RowTok {
        uint32_t r = g, j = 0;
        if (!simple) {
            uint32_t lo = hint;
            if constexpr (ROW_PER_WAVE) {
                if (rd(m.pref + hint + 1u) <= g) lo = find_request(g);
            } else {
                uint32_t hi = L[m.pref + hint + 1u] > g ? hint + 1u : n_reqs;
                while (hi - lo > 1u) {
                    const uint32_t mid = (lo + hi) >> 1;
                    if (L[m.pref + mid] <= g) lo = mid; else hi = mid;
                }
            }
            r = lo;
            hint = r;
            j = g - rd(m.pref + r);
        }
        RowTok k = {0u, 0u};
        if (!a.paged) {
            if (index_mode) {
                k.at = (uint32_t)a.row_index[simple ? g : rd(m.pref_all + r) + j];
            } else if (a.table_in_lds) {        // (the host keeps every listed row below 2^32)
                k.at = rd(m.rb + r) + j * rd(m.tab + 4u * r + 2u);
            } else {
                k.at = row_first(r);
                if (j) k.at += j * table_entry(r).z;
            }
        } else {
            uint32_t tok0, tstep, seq_row;
            if (a.table_in_lds) {
                tok0 = rd(m.tab + 4u * r + 1u); tstep = rd(m.tab + 4u * r + 2u); seq_row = rd(m.rb + r);
            } else {
                const uint4 e = table_entry(r);
                tok0 = e.y; tstep = e.z; seq_row = row_first(r);
            }
            const uint32_t t = tok0 + j * tstep;            // host keeps token positions below 2^31
            const uint32_t lb = a.bs_shift < 32u ? t >> a.bs_shift : t / a.block_size;
            k.slot = t - lb * a.block_size;
            k.at = (uint32_t)a.block_table[(int64_t)seq_row * a.bt_stride + (int64_t)lb];
        }
        return k;
    };
    auto locate_end = [&](const RowTok &k) -> RowRef {
        const uint32_t word = ROW_PER_WAVE ? (uint32_t)__builtin_amdgcn_readfirstlane((int)k.at) : k.at;
        const int64_t at = a.paged || index_mode ? (int64_t)(int32_t)word : (int64_t)word;
        RowRef ref;
        ref.ok = at >= 0 && at < a.n_src_rows;
        if (!a.paged) ref.base = src + (ref.ok ? at : 0) * a.row_stride_b;
        else ref.base = src + (ref.ok ? at : 0) * a.block_stride_b + (int64_t)k.slot * a.slot_stride_b;
        return ref;
    };
    // Consecutive rows of a wavefront, from `from` on, none behind the last one asked for.  Where the table is in LDS the next
    // row of a request is a stride further on, and only the next request's first row has to be looked up; rows with an
    // index (or a table) in memory are asked for a row ahead.
    const bool walks = !simple && !index_mode && !a.paged && a.table_in_lds != 0;
    struct Walk {
        const uint8_t *base;
        int64_t step;
        uint32_t g, last, r, end;
        RowTok ask;
    };
    auto walk_into = [&](Walk &q, uint32_t j) {         // request q.r's row j
        q.end = rd(m.pref + q.r + 1u);
        const uint32_t tok_step = rd(m.tab + 4u * q.r + 2u);
        q.step = (int64_t)tok_step * a.row_stride_b;
        q.base = src + (int64_t)(uint64_t)(rd(m.rb + q.r) + j * tok_step) * a.row_stride_b;      // (the host has checked these rows)
    };
    auto walk_from = [&](Walk &q, uint32_t from, uint32_t last) -> RowRef {
        q.g = from;
        q.last = last;
        q.r = simple ? 0u : find_request(from);
        if (walks) {
            walk_into(q, from - rd(m.pref + q.r));
            return RowRef{q.base, 1u};
        }
        const RowRef ref = locate_end(locate_begin(from, q.r));
        q.ask = locate_begin(from < last ? from + 1u : last, q.r);
        return ref;
    };
    auto walk_on = [&](Walk &q) -> RowRef {
        q.g++;
        if (walks) {
            if (q.g < q.end) {
                q.base += q.step;
            } else {
                do q.r++; while (rd(m.pref + q.r + 1u) <= q.g);
                walk_into(q, 0u);
            }
            return RowRef{q.base, 1u};
        }
        const RowRef ref = locate_end(q.ask);
        q.ask = locate_begin(q.g < q.last ? q.g + 1u : q.last, q.r);
        return ref;
    };
    auto locate = [&](uint32_t g) -> RowRef {
        uint32_t first = 0;
        return locate_end(locate_begin(g, first));
    };
    auto unit_ptr = [&](const RowRef &ref, uint32_t c) -> const uint8_t * {
        if (!a.paged) return ref.base + elem_in_seg(c) * ES_IN;
        const uint32_t seg = a.seg_shift < 32u ? c >> a.seg_shift : c / a.seg_units;
        const uint32_t cc = c - seg * a.seg_units;
        return ref.base + (int64_t)L[m.heads + seg] * a.head_stride_b + elem_in_seg(cc) * ES_IN;
    };
    // where unit c of row g goes, in bytes from the record's start
    auto out_at = [&](uint64_t g, uint32_t c) -> uint64_t {
        if constexpr (LOOSE) {
            const uint32_t seg = !a.paged ? 0u : a.seg_shift < 32u ? c >> a.seg_shift : c / a.seg_units;
            return off_payload + (g * a.row_elems + (uint64_t)seg * a.seg_elems + elem_in_seg(c - seg * a.seg_units)) * ES_OUT;
        }
        return off_payload + (g * a.units_per_row + c) * NB_OUT;
    };
    // a unit as the row's sums see it: without the elements that the unit in front of it holds as well
    auto sum_part = [&](unit_t v, uint32_t c) -> unit_t {
        if constexpr (LOOSE) {
            const uint32_t cc = !a.paged ? c : a.seg_shift < 32u ? c & ((1u << a.seg_shift) - 1u) : c % a.seg_units;
            return without_first<VEC>(v, cc + 1u == a.seg_units ? a.seg_units * VEC - a.seg_elems : 0u);
        }
        return v;
    };
    // Loads are never put under a condition of their own: the compiler then waits for each
    // one before it issues the next (a register copy where the branches join), and four
    // loads in flight become four trips to memory.  A unit that is not wanted (past the
    // end, or of a row whose index left the source) is read from the control block's zeros.
    const uint8_t *const safe_src = reinterpret_cast<const uint8_t *>(a.ctrl->zeros);
    auto load_unit = [&](const RowRef &ref, uint32_t c, bool want) -> unit_t {
        const uint8_t *p = want ? unit_ptr(ref, want ? c : 0u) : safe_src;
        return *(global_unit_t *)p;
    };
    auto zero_unless = [](bool keep, unit_t v) -> unit_t { return keep ? v : unit_t{}; };

    // Row totals of a wavefront's 64 rows at most, [from, upto), from its part of LDS to the record.
    float *const stash = row_sums + (SHORT_ROWS || MODE == SUMM_WAVE ? wave * 192u : 0u);       // [3][64]
    auto flush_totals = [&](uint64_t from, uint64_t upto) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (from + lane < upto) {
            uint64_t o = off_sum + (from + lane) * 4u;
            if (a.summary_mask & 1u) { ring_store<float>(w, o, sqrtf(stash[lane])); o += sum_arr; }
            if (a.summary_mask & 2u) { ring_store<float>(w, o, stash[64u + lane] / (float)a.row_elems); o += sum_arr; }
            if (a.summary_mask & 4u) ring_store<float>(w, o, am_value(__float_as_uint(stash[128u + lane]), a.src_dtype));
        }
        __builtin_amdgcn_wave_barrier();
    };

    if (!dropped) {
        // ---- header, request table and all pad bytes: workgroup 0.  The header is put
        //      together in LDS and leaves as four 16-byte stores.
        if (blockIdx.x == 0) {
            if (tid == 0) {
                uint32_t *h = lds + m.hdr;
                h[0] = 0x32494D44u;
                h[1] = 1u | (64u << 16);
                const uint64_t seq_y = ((uint64_t)lds[m.bcast + 8] | ((uint64_t)lds[m.bcast + 9] << 32)) + y;
                h[2] = (uint32_t)seq_y;          h[3] = (uint32_t)(seq_y >> 32);
                h[4] = lds[m.bcast + 10];        h[5] = lds[m.bcast + 11];      // step id
                h[6] = point_id;
                h[7] = a.src_dtype | (a.out_dtype << 8) | (a.summary_mask << 16) | (a.rec_flags << 24);
                h[8] = n_reqs;  h[9] = n_rows;  h[10] = a.row_elems;  h[11] = a.rank_tag;
                h[12] = (uint32_t)record_bytes;  h[13] = (uint32_t)(record_bytes >> 32);
                h[14] = (uint32_t)payload_bytes; h[15] = (uint32_t)(payload_bytes >> 32);
            }
            lds_barrier();
            if (tid < 4) {
                const uint32_t *h = lds + m.hdr + 4 * tid;
                u32x4 v = {h[0], h[1], h[2], h[3]};
                ring_store<u32x4>(w, 16u * tid, v);
            }
            const uint32_t tab_slots = (uint32_t)(table_bytes / 16u);
            for (uint32_t r = tid; r < tab_slots; r += kThreads) {
                u32x4 v = {0u, 0u, 0u, 0u};
                if (r < n_reqs) {
                    uint4 e;
                    if (a.table_in_lds) e = ltab[r];
                    else { e = table_entry(r); if (!simple) e.w = pref[r + 1] - pref[r]; }
                    v.x = e.x; v.y = e.y; v.z = e.z; v.w = e.w;
                }
                ring_store<u32x4>(w, 64u + 16ull * r, v);
            }
            {
                const uint32_t pad = (uint32_t)(off_sum - off_payload - payload_bytes);
                if (tid < pad) ring_store<uint8_t>(w, off_payload + payload_bytes + tid, (uint8_t)0);
                const uint32_t spad = (uint32_t)(sum_arr - (uint64_t)n_rows * 4u) / 4u;
                for (uint32_t k = tid; k < n_sum * spad; k += kThreads) {
                    const uint32_t arr = k / spad, i = k - arr * spad;
                    ring_store<uint32_t>(w, off_sum + arr * sum_arr + (uint64_t)n_rows * 4u + 4ull * i, 0u);
                }
            }
        }

        if constexpr (MODE == ROWS_FLAT) {
            if constexpr (OUT != OUT_NONE) {
                // ---- units dealt flat: the n_rows x units_per_row units are dealt to lanes in order,
                //      so stores stay fully coalesced; 4 loads in flight per lane.
                //      A wavefront's 64 units of one slice lie in at most 64/upr + 2 rows.  When
                //      the rows of its four slices fit the 64 lanes, each lane locates one row
                //      (all of them in a single pass) and every unit picks up its row's place by
                //      shuffle: locating a row costs on the order of a hundred instructions, and
                //      done per unit that, not memory, is what the launch spends its time on.
                const uint32_t total = (uint32_t)((uint64_t)n_rows * a.units_per_row);  // host keeps it below 2^32
                const uint32_t upr = a.units_per_row;
                auto row_of = [&](uint32_t u) { return a.upr_shift < 32u ? u >> a.upr_shift : u / upr; };
                const bool shared_locate = 64u / upr + 2u <= 16u;
                const uint32_t slice_stride = gridDim.x * kThreads;
                for (uint64_t t0 = (uint64_t)blockIdx.x * kThreads; t0 < total; t0 += (uint64_t)slice_stride * U) {
                    unit_t v[U];
                    bool live[U], okk[U];
                    uint32_t my_lo = 0, my_hi = 0, my_ok = 0, my_first = 0;
                    if (shared_locate) {
                        const uint32_t sl = lane >> 4, j = lane & 15u;
                        const uint64_t us = t0 + (uint64_t)sl * slice_stride + wave * 64u;
                        if (us < total) {
                            const uint32_t ue = us + 63u < total ? (uint32_t)us + 63u : total - 1u;
                            my_first = row_of((uint32_t)us);
                            const uint32_t g = my_first + j;
                            if (g <= row_of(ue)) {
                                const RowRef ref = locate(g);
                                my_lo = (uint32_t)(uintptr_t)ref.base;
                                my_hi = (uint32_t)((uintptr_t)ref.base >> 32);
                                my_ok = ref.ok ? 1u : 0u;
                                // a bad row is counted where its first unit lies
                                const uint64_t fu = (uint64_t)g * upr;
                                if (!ref.ok && fu >= us && fu <= ue)
                                    atomicAdd((unsigned long long *)&a.ctrl->bad_rows, 1ull);
                            }
                        }
                    }
#pragma unroll
                    for (uint32_t k = 0; k < U; k++) {
                        const uint64_t u = t0 + (uint64_t)k * slice_stride + tid;
                        live[k] = u < total;
                        const uint32_t u32 = live[k] ? (uint32_t)u : total - 1u;
                        const uint32_t g = row_of(u32);
                        const uint32_t c = u32 - g * upr;
                        RowRef ref;
                        if (shared_locate) {
                            // executed by all 64 lanes: a shuffle reads nothing useful from a lane that is off
                            const uint32_t first_k = __shfl(my_first, (int)(k << 4), 64);
                            const int src = (int)(((k << 4) + (g - first_k)) & 63u);
                            const uint32_t lo = __shfl(my_lo, src, 64), hi = __shfl(my_hi, src, 64);
                            ref.ok = __shfl(my_ok, src, 64);
                            ref.base = reinterpret_cast<const uint8_t *>(((uint64_t)hi << 32) | lo);
                            if (!live[k]) ref.ok = 0;
                        } else {
                            ref.base = nullptr;
                            ref.ok = 0;
                            if (live[k]) {
                                ref = locate(g);
                                if (!ref.ok && c == 0) atomicAdd((unsigned long long *)&a.ctrl->bad_rows, 1ull);
                            }
                        }
                        okk[k] = live[k] && ref.ok != 0;
                        v[k] = load_unit(ref, c, okk[k]);
                    }
#pragma unroll
                    for (uint32_t k = 0; k < U; k++) {
                        const uint64_t u = t0 + (uint64_t)k * slice_stride + tid;
                        const uint32_t g = LOOSE ? row_of((uint32_t)u) : 0u;    // (else a record's units just follow each other)
                        if (live[k])
                            emit_unit<ES_IN, VEC, OUT, LOOSE>(
                                w, LOOSE ? out_at(g, (uint32_t)u - g * upr) : off_payload + u * NB_OUT,
                                zero_unless(okk[k], v[k]));
                    }
                }
            }
        } else if constexpr (SHORT_ROWS) {
            // ---- summaries of short rows (up to 256 units): 4 to 64 lanes share a row, each with up to four
            //      of its units, so one step of a wavefront is 64 / row_lanes whole rows and a row costs one
            //      reduction over few lanes (a row of 32 units used to take a wavefront of its own, half of its
            //      lanes and three of its four loads idle, and a reduction over all 64 lanes).  A wavefront works through
            //      consecutive rows: each starts its search where the row before it was found.  What finding a
            //      row has to load (its block) is asked for a step before the row's own loads, and totals wait in
            //      LDS until 64 rows are together: memory operations of a wavefront complete in order, so a row's
            //      place asked for behind a step's loads, or a store inside the loop, would make every step wait.
            //      Bound: HBM reads.  8 caches x 72.7 k rows of 32 units, norms and largest magnitudes:
            //      297 -> 69 us (1.0 -> 4.4 TB/s read), 66 -> 60 us past the memory-side cache, which holds less than a launch like
            //      this reads.
            const uint32_t lpr = row_lanes, lg = 31u - (uint32_t)__builtin_clz(lpr);
            const uint32_t rpi = 64u >> lg;                             // rows per step, at most 16
            const uint32_t sub_r = lane >> lg, l_r = lane & (lpr - 1u);
            const uint32_t per = n_rows ? ((n_rows - 1u) / n_waves / rpi + 1u) * rpi : 0u;
            const uint64_t r0 = (uint64_t)wave_at * per;
            const uint64_t r1 = r0 + per < n_rows ? r0 + per : n_rows;
            // where this lane's units lie in a row does not change from row to row
            bool in_row[U];
            int64_t unit_off[U];
#pragma unroll
            for (uint32_t k = 0; k < U; k++) {
                const uint32_t c = l_r + k * lpr;
                in_row[k] = c < a.units_per_row;
                const RowRef zero = {nullptr, 1};
                unit_off[k] = (int64_t)(uintptr_t)unit_ptr(zero, in_row[k] ? c : 0u);
            }
            const uint8_t *const zeros = reinterpret_cast<const uint8_t *>(a.ctrl->zeros);
            uint32_t n_bad = 0, hint = 0;
            auto begin = [&](uint64_t g) -> RowTok {    // (behind the last row: that one again)
                const uint64_t x = g + sub_r;
                return locate_begin((uint32_t)(x < r1 ? x : r1 - 1u), hint);
            };
            auto end = [&](const RowTok &k, uint64_t g) -> RowRef {
                RowRef ref = locate_end(k);
                const bool live = g + sub_r < r1;
                n_bad += live && l_r == 0u && !ref.ok ? 1u : 0u;
                ref.ok = live && ref.ok ? 1u : 0u;
                return ref;
            };
            // a lane with nothing to load (behind the row's end, or the rows', or a bad row) reads zeros
            auto load = [&](const RowRef &ref, unit_t (&v)[U]) {
#pragma unroll
                for (uint32_t k = 0; k < U; k++) {
                    const uint8_t *ptr = ref.ok && in_row[k] ? ref.base + unit_off[k] : zeros;
                    v[k] = MODE == SUMM_SHORT_ONCE ? __builtin_nontemporal_load((global_unit_t *)ptr) : *(global_unit_t *)ptr;
                }
            };
            auto process = [&](const unit_t (&v)[U], uint64_t g0) {
                const uint64_t g = g0 + sub_r;
                if constexpr (OUT != OUT_NONE) {
#pragma unroll
                    for (uint32_t k = 0; k < U; k++)
                        if (g < r1 && in_row[k]) emit_unit<ES_IN, VEC, OUT, LOOSE>(w, out_at(g, l_r + k * lpr), v[k]);
                }
                Accum acc = {0.f, 0.f, 0u};
                unit_t sv[U];
#pragma unroll
                for (uint32_t k = 0; k < U; k++) sv[k] = sum_part(v[k], l_r + k * lpr);
                accum_units<ES_IN, VEC>(acc, sv, a.src_dtype);           // (what is not the row's was read as zeros)
                const uint32_t at = (uint32_t)(g - r0) & 63u;
                const bool last = l_r == lpr - 1u;
                if (a.summary_mask & 1u) {
                    const float ss = group_sum(acc.ss, lpr);
                    if (last) stash[at] = ss;
                }
                if (a.summary_mask & 2u) {
                    const float sm = group_sum(acc.s, lpr);
                    if (last) stash[64u + at] = sm;
                }
                if (a.summary_mask & 4u) {
                    const uint32_t am = group_max_u32(fold_am<ES_IN, VEC>(acc.am), lpr);
                    if (last) stash[128u + at] = __uint_as_float(am);
                }
                const uint64_t done = g0 + rpi - r0;
                if ((done & 63u) == 0u) flush_totals(r0 + done - 64u, g0 + rpi < r1 ? g0 + rpi : r1);
                else if (g0 + rpi >= r1) flush_totals(r0 + (done & ~63ull), r1);
            };
            if (r0 < r1) {
                unit_t va[U], vb[U];
                uint64_t g = r0;
                const RowTok k0 = begin(g), k1 = begin(g + rpi);
                RowRef next = end(k0, g);
                load(next, va);
                next = end(k1, g + rpi);
                for (;;) {
                    RowTok k = begin(g + 2u * rpi);
                    load(next, vb);
                    process(va, g);
                    next = end(k, g + 2u * rpi);
                    g += rpi;
                    if (g >= r1) break;
                    k = begin(g + 2u * rpi);
                    load(next, va);
                    process(vb, g);
                    next = end(k, g + 2u * rpi);
                    g += rpi;
                    if (g >= r1) break;
                }
                if (n_bad) atomicAdd((unsigned long long *)&a.ctrl->bad_rows, (unsigned long long)n_bad);
            }
        } else if constexpr (MODE == SUMM_WAVE) {
            // ---- summaries, a wavefront per row (paged rows, or of more than 64 ragged requests): where a launch has rows enough
            //      to fill the GPU that way, a row costs no barrier and a workgroup lives for four rows or more
            //      instead of one, so its prologue weighs less.
            //      The sums are taken in the order in which a workgroup takes them (the decode-shaped kernel, and
            //      the path below): the row's lanes in parts of 64, each lane's (at most four) units, then the lanes
            //      of a part, then the (at most four) parts.  A step is one part of a row; its loads are issued
            //      before the step in front of it is worked on.
            //      Bound: HBM reads.  80 x 256 rows of 512 units, statistics only: 64 -> 35 us
            //      (4.8 TB/s); plan_grid() has more figures, and says where the line lies.
            const uint32_t per = n_rows ? (n_rows - 1u) / n_waves + 1u : 0u;
            const uint64_t r0 = (uint64_t)wave_at * per;
            const uint64_t r1 = r0 + per < n_rows ? r0 + per : n_rows;
            const uint32_t parts = row_lanes >> 6;
            auto wave_unit = [&](uint32_t part, uint32_t t) { return part * 64u + lane + t * row_lanes; };
            const uint8_t *const zeros = reinterpret_cast<const uint8_t *>(a.ctrl->zeros);
            struct Step { uint64_t g; uint32_t part; RowRef ref; };
            uint32_t n_bad = 0;
            Walk walk;
            // a lane with nothing to load reads zeros
            auto load = [&](const Step &s, unit_t (&v)[U]) {
                const bool ok = s.g < r1 && s.ref.ok;
#pragma unroll
                for (uint32_t t = 0; t < U; t++) {
                    const uint32_t c = wave_unit(s.part, t);
                    const uint8_t *ptr = ok && c < a.units_per_row ? unit_ptr(s.ref, c) : zeros;
                    v[t] = *(global_unit_t *)ptr;
                }
            };
            uint32_t row_am = 0;
            float ss[2] = {0.f, 0.f}, sm[2] = {0.f, 0.f};      // of parts 0 and 1; of the last part, or of 2 and 3
            auto process = [&](const Step &s, const unit_t (&v)[U]) {
                unit_t sv[U];
#pragma unroll
                for (uint32_t t = 0; t < U; t++) {
                    const uint32_t c = wave_unit(s.part, t);
                    if constexpr (OUT != OUT_NONE) {
                        if (c < a.units_per_row) emit_unit<ES_IN, VEC, OUT, LOOSE>(w, out_at(s.g, c), v[t]);
                    }
                    sv[t] = sum_part(v[t], c);
                }
                Accum acc = {0.f, 0.f, row_am};
                accum_units<ES_IN, VEC>(acc, sv, a.src_dtype);
                row_am = acc.am;
                if (a.summary_mask & 1u) {
                    float r = wave_sum(acc.ss);
                    if (s.part & 1u) r = ss[1] + r;
                    if (s.part < 2u) ss[0] = r;
                    ss[1] = r;
                }
                if (a.summary_mask & 2u) {
                    float r = wave_sum(acc.s);
                    if (s.part & 1u) r = sm[1] + r;
                    if (s.part < 2u) sm[0] = r;
                    sm[1] = r;
                }
                if (s.part + 1u < parts) return;
                const uint32_t at = (uint32_t)(s.g - r0) & 63u;         // the row is complete
                const uint32_t am = wave_max_u32(fold_am<ES_IN, VEC>(row_am));
                const bool both = parts > 2u;
                if (lane == 0) {
                    stash[at] = both ? ss[0] + ss[1] : ss[0];
                    stash[64u + at] = both ? sm[0] + sm[1] : sm[0];
                    stash[128u + at] = __uint_as_float(am);
                }
                row_am = 0;
                if (at == 63u || s.g + 1u >= r1) flush_totals(s.g - at, s.g + 1u);
            };
            if (r0 < r1) {
                unit_t va[U], vb[U];
                auto next = [&](const Step &s) -> Step {        // (behind the last row: steps that read zeros)
                    Step n = s;
                    if (++n.part < parts) return n;
                    n.part = 0;
                    if (++n.g >= r1) return n;
                    n.ref = walk_on(walk);
                    n_bad += n.ref.ok ? 0u : 1u;
                    return n;
                };
                Step s;
                s.g = r0;
                s.part = 0;
                s.ref = walk_from(walk, (uint32_t)r0, (uint32_t)r1 - 1u);
                load(s, va);
                n_bad += s.ref.ok ? 0u : 1u;
                for (;;) {
                    Step n = next(s);
                    load(n, vb);
                    process(s, va);
                    if (n.g >= r1) break;
                    s = next(n);
                    load(s, va);
                    process(n, vb);
                    if (s.g >= r1) break;
                }
                if (n_bad && lane == 0) atomicAdd((unsigned long long *)&a.ctrl->bad_rows, (unsigned long long)n_bad);
            }
        } else {
            // ---- summaries, a workgroup per row: a step is 4 units per lane of one row; rows longer than
            //      that take several steps.  Steps are software pipelined (the next step's loads are issued before
            //      this step is converted, stored and accumulated), across row boundaries too.
            float *red = reinterpret_cast<float *>(lds + m.red);
            auto fetch = [&](uint64_t g, uint32_t pass, RowRef &ref, unit_t (&v)[U]) {
                if (pass == 0) {
                    ref = locate((uint32_t)g);
                    if (!ref.ok && tid == 0) atomicAdd((unsigned long long *)&a.ctrl->bad_rows, 1ull);
                }
#pragma unroll
                for (uint32_t k = 0; k < U; k++) {
                    const uint32_t c = tid + (pass * U + k) * row_lanes;
                    v[k] = load_unit(ref, c, ref.ok != 0 && tid < row_lanes && c < a.units_per_row);
                }
            };
            uint64_t g = blockIdx.x;
            uint32_t pass = 0;
            if (g < n_rows) {
                RowRef ref = {nullptr, 0};
                unit_t v[U];
                fetch(g, pass, ref, v);
                Accum acc = {0.f, 0.f, 0u};
                for (;;) {
                    uint64_t nxt_g = g;
                    uint32_t nxt_pass = pass + 1u;
                    if (nxt_pass == cpr) { nxt_pass = 0; nxt_g += gridDim.x; }
                    const bool more = nxt_g < n_rows;
                    RowRef ref_n = ref;             // a later pass of the same row keeps the row
                    unit_t v_n[U];
                    if (more) fetch(nxt_g, nxt_pass, ref_n, v_n);
                    unit_t sv[U];
#pragma unroll
                    for (uint32_t k = 0; k < U; k++) {
                        const uint32_t c = tid + (pass * U + k) * row_lanes;
                        if (OUT != OUT_NONE && tid < row_lanes && c < a.units_per_row)
                            emit_unit<ES_IN, VEC, OUT, LOOSE>(w, out_at(g, c), v[k]);
                        sv[k] = sum_part(v[k], c);
                    }
                    const bool mine = (uint32_t)__builtin_amdgcn_readfirstlane((int)tid) < row_lanes;
                    if (mine) accum_units<ES_IN, VEC>(acc, sv, a.src_dtype);
                    if (pass == cpr - 1u) {         // the row is complete: reduce and store its summaries
                        uint32_t am = 0;
                        if (mine) {
                            acc.ss = wave_sum(acc.ss);
                            acc.s = wave_sum(acc.s);
                            am = wave_max_u32(fold_am<ES_IN, VEC>(acc.am));
                        }
                        lds_barrier();        // the previous row's readers are done with red[]
                        if (lane == 0) {
                            red[wave] = acc.ss;
                            red[4 + wave] = acc.s;
                            reinterpret_cast<uint32_t *>(red)[8 + wave] = am;
                        }
                        lds_barrier();
                        acc.ss = (red[0] + red[1]) + (red[2] + red[3]);
                        acc.s = (red[4] + red[5]) + (red[6] + red[7]);
                        const uint32_t *ra = reinterpret_cast<const uint32_t *>(red) + 8;
                        const uint32_t m01 = ra[0] > ra[1] ? ra[0] : ra[1], m23 = ra[2] > ra[3] ? ra[2] : ra[3];
                        am = m01 > m23 ? m01 : m23;
                        if (tid == 0) {
                            uint64_t o = off_sum + g * 4u;
                            if (a.summary_mask & 1u) { ring_store<float>(w, o, sqrtf(acc.ss)); o += sum_arr; }
                            if (a.summary_mask & 2u) { ring_store<float>(w, o, acc.s / (float)a.row_elems); o += sum_arr; }
                            if (a.summary_mask & 4u) { ring_store<float>(w, o, am_value(am, a.src_dtype)); }
                        }
                        acc = Accum{0.f, 0.f, 0u};
                    }
                    if (!more) break;
                    g = nxt_g;
                    pass = nxt_pass;
                    ref = ref_n;
#pragma unroll
                    for (uint32_t k = 0; k < U; k++) v[k] = v_n[k];
                }
            }
        }
    }
}


// ---------------------------------------------------------------- decode-shaped capture
// The common case of the paper's workloads (every layer's hidden state at a decode step):
// bf16 rows, one per request, no keep mask.  Everything about the record except its place
// in the ring is known on the host, so the kernel is straight-line: a workgroup per row
// issues its loads at once, an extra workgroup writes header, table and pads and publishes.
// A small capture is bound by instructions issued and dependent memory trips, not by
// bytes; the general kernel above executes several times as many instructions per row.
// Kernel arguments of the decode-shaped kernel.  The scalar cache is cold at every launch,
// so each 64-byte line of the argument block costs a trip to memory when it is first
// touched, and the compiler, left alone, puts each argument load next to its first use:
// a chain of such trips, one after another, that is longer than the copy itself.  What
// every workgroup needs therefore sits in the first two lines, what only the extra
// workgroup needs in the third, and all three are fetched together at the top.
struct DecodeArgs {
    // line 0
    uint64_t spare0;
    int64_t row_stride_b;
    const int32_t *rows;            // row per request (int32 indices or uint32 first rows), unless consecutive
    uint8_t *ring;
    uint64_t cap;
    DevCtrl *ctrl;
    const StepParams *step;
    uint64_t tail_floor;
    // line 1
    uint64_t record_bytes, off_payload, off_sum, sum_arr;
    uint32_t n_src_rows, n_reqs, units_per_row, row_first;
    uint32_t flags;                 // kDec*
    uint32_t node, summary_mask, row_elems;
    // line 2
    uint64_t seq, step_id;
    const uint4 *req_table;
    CommitSlot *cslot;
    uint64_t payload_bytes;
    uint32_t rows_at;               // launches into the caller's memory: the word of their table from which on rows are listed
    uint32_t hdr7, rank_tag, pad;
    const uint64_t *tail_src;       // where the extra workgroup reads the drained-up-to mark (may be NULL)
    // line 3
    const uint8_t *keep_mask;       // keep vector (MASK variants): request r is captured iff keep_mask[r] != 0
    uint32_t n_wg_rows;             // row workgroups = rows listed (= n_reqs unless requests list several rows)
    uint32_t unit_stride;           // lane l < unit_stride takes units l, l + unit_stride, ...: all lanes of the
                                    // workgroup, or with summaries the general kernel's row_lanes (the sums are
                                    // then taken in the same order there and here)
    uint64_t *note;                 // where the extra workgroup says where it found the head (may be NULL)
    uint64_t spare[5];
};
static_assert(sizeof(DecodeArgs) == 256, "four lines");
constexpr uint32_t kDecDropNewest = 1u, kDecConsecutive = 2u, kDecIndexed = 4u, kDecParIn = 8u, kDecRowMap = 16u;

// MASK: the paper's best-effort path (section 4.4): a batch-aligned keep vector, read when the
// kernel runs, decides per request.  Every workgroup reads the whole vector (at most 1024
// bytes) together with its other loads, the wavefronts ballot it into 16 words of LDS, and
// each workgroup derives from those the record's row count and its own row's place.  The
// row itself is loaded before the vector is known and thrown away if the request is out.
// Eight workgroups per compute unit: 64 vector registers at most.  With 65 to 69 (what one lane keeps for the next launch has to be
// looked after: the place of the head comes back out of LDS) seven fit: 32 tensors of 64 x 4096 raw with summaries 10.5 / 9.9 us on cold
// rows, 9.1 / 8.0 on others, 4096 rows of one tensor 24.3 / 21.2, to fp8 without summaries 20.8 / 18.4.
template <int OUT, bool SUMM, bool MASK, typename SRC>
__global__ void __launch_bounds__(kThreads, 8) capture_decode_kernel(const DecodeArgs a, const SRC b)
{
    constexpr bool INTO = std::is_same<SRC, IntoArgs>::value;
    __shared__ uint32_t sh[32];
    __shared__ uint64_t kept_bits[16];      // MASK: bit i of word q = request 64 q + i is kept
    const uint32_t y = INTO ? 0u : blockIdx.y;      // which tensor of the batch
    const uint8_t *const src = b.src[y];
    const uint32_t point_id = b.point[y];
    touch_argument_lines(a, src, point_id);
    constexpr uint32_t U = 4;
    constexpr uint32_t NB_OUT = out_unit_bytes<2, 8, OUT>();
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t par = (a.flags & kDecParIn) ? 1u : 0u;
    const bool meta_wg = blockIdx.x == a.n_wg_rows;
    const uint32_t ustr = SUMM ? a.unit_stride : kThreads;
    constexpr uint32_t kCtlTid = kThreads - 64u;

    // control words first (they depend on nothing but the arguments), then the row
    uint64_t cnt_cap[3] = {0, 0, 0}, cnt_drop[3] = {0, 0, 0}, tail_now = 0, seq = a.seq;
    RawControl raw = {};
    if (!INTO && tid == kCtlTid) raw = fetch_control(a.ctrl, par, a.step);
    uint32_t kb[4] = {0u, 0u, 0u, 0u};
    if constexpr (MASK) {
#pragma unroll
        for (uint32_t k = 0; k < 4; k++) {
            const uint32_t r = tid + k * kThreads;
            kb[k] = a.keep_mask[r < a.n_reqs ? r : 0u];
        }
    }
    u32x4 v[U];
    bool ok = false;
    if (!meta_wg) {
        const uint32_t g = blockIdx.x;
        // the usual decode layout (request i in row first + i) saves the dependent trip to the table
        int64_t row;
        if (a.flags & kDecConsecutive) {
            row = (int64_t)a.row_first + g;
        } else {
            bool in_args = false;
            uint32_t at = 0;
            if constexpr (INTO) {       // the row of every request, or of every listed row behind those
                in_args = b.n_words && !(a.flags & kDecIndexed);
                if (in_args) at = inline_table_uniform(sizeof(DecodeArgs))[a.rows_at + g];
            }
            // (the same in every lane, and said so here: the wait for it then stays on this branch, and the common case
            // above does not wait for the control words before it loads its row)
            if (!in_args) at = (uint32_t)__builtin_amdgcn_readfirstlane(a.rows[g]);
            row = a.flags & kDecIndexed ? (int64_t)(int32_t)at : (int64_t)at;
        }
        ok = row >= 0 && row < (int64_t)a.n_src_rows;
        const uint8_t *base = src + (ok ? row : 0) * a.row_stride_b;
#pragma unroll
        for (uint32_t k = 0; k < U; k++) v[k] = u32x4{0u, 0u, 0u, 0u};
        if (ok) {
            // straight-line loads: lanes past the end of the row fetch zeros, or (where nothing is summed) its first
            // unit again and ignore it (a load under its own condition makes the compiler wait between loads)
#pragma unroll
            for (uint32_t k = 0; k < U; k++) {
                const uint32_t c = tid + k * ustr;
                if constexpr (SUMM) {
                    const uint8_t *p = tid < ustr && c < a.units_per_row ? base + (uint64_t)c * 16u
                                                                         : reinterpret_cast<const uint8_t *>(a.ctrl->zeros);
                    v[k] = *(__attribute__((address_space(1))) const u32x4 *)p;
                } else {
                    v[k] = *reinterpret_cast<const u32x4 *>(base + (uint64_t)(c < a.units_per_row ? c : 0u) * 16u);
                }
            }
        }
    }
    if constexpr (MASK) {
#pragma unroll
        for (uint32_t k = 0; k < 4; k++) {
            const uint32_t r = tid + k * kThreads;
            const uint64_t b = __ballot(r < a.n_reqs && kb[k] != 0u);
            if (lane == 0) kept_bits[k * 4u + wave] = b;
        }
    }
    if (INTO && tid < 28u && (tid < 8u || tid >= 24u))      // head, tail, policy: none
        sh[tid] = tid == 24u   ? (uint32_t)a.seq
                  : tid == 25u ? (uint32_t)(a.seq >> 32)
                  : tid == 26u ? (uint32_t)a.step_id
                  : tid == 27u ? (uint32_t)(a.step_id >> 32)
                               : 0u;
    if (!INTO && tid == kCtlTid) {
        // the drained-up-to mark for the next launch's drop decision, read where the host keeps
        // it by the extra workgroup's lane, after every other load of that lane
        const uint64_t *ts = meta_wg && y == 0 && a.tail_src ? a.tail_src : &a.ctrl->tail;
        tail_now = ld_system(ts);
        const Control ct = resolve_control(raw, a.step != nullptr, a.node, a.tail_floor, a.seq, a.step_id,
                                           a.flags & kDecDropNewest);
        seq = ct.seq;
        for (int i = 0; i < 3; i++) { cnt_cap[i] = raw.cap[i]; cnt_drop[i] = raw.drop[i]; }
        sh[0] = (uint32_t)ct.head;  sh[1] = (uint32_t)(ct.head >> 32);
        sh[2] = (uint32_t)ct.tail;  sh[3] = (uint32_t)(ct.tail >> 32);
        sh[4] = (uint32_t)raw.head_at;  sh[5] = (uint32_t)(raw.head_at >> 32);
        sh[6] = ct.flags;
        sh[24] = (uint32_t)ct.seq;      sh[25] = (uint32_t)(ct.seq >> 32);
        sh[26] = (uint32_t)ct.step_id;  sh[27] = (uint32_t)(ct.step_id >> 32);
    }
    // Summaries are taken before the one barrier of this kernel, which then hands over both
    // the control words and the wavefronts' partial sums: the rows arrive later than the
    // control words anyway, and a second barrier behind the stores would put the summary
    // stores a good half microsecond behind the row stores.
    if constexpr (SUMM) {
        Accum acc = {0.f, 0.f, 0u};
        if (!meta_wg) {
            // (wavefronts without a part of the row have nothing to add, and with eight of them on a SIMD their
            // vector instructions would be the others' time)
            uint32_t am = 0;
            if ((uint32_t)__builtin_amdgcn_readfirstlane((int)tid) < ustr) {
                accum_units<2, 8>(acc, v, a.hdr7 & 0xFFu);
                if (a.summary_mask & 1u) acc.ss = wave_sum(acc.ss);
                if (a.summary_mask & 2u) acc.s = wave_sum(acc.s);
                if (a.summary_mask & 4u) am = wave_max_u32(fold_am<2, 8>(acc.am));
            }
            float *red = reinterpret_cast<float *>(sh + 8);
            if (lane == 0) {
                red[wave] = acc.ss;
                red[4 + wave] = acc.s;
                sh[16 + wave] = am;
            }
        }
    }
    lds_barrier();
    const uint64_t head0 = (uint64_t)sh[0] | ((uint64_t)sh[1] << 32);
    const uint64_t tail = (uint64_t)sh[2] | ((uint64_t)sh[3] << 32);
    const uint64_t head_at = (uint64_t)sh[4] | ((uint64_t)sh[5] << 32);
    const uint32_t flags = sh[6];
    const bool publisher = !INTO && meta_wg && y == 0 && tid == kCtlTid;
    if (!INTO && (flags & kStepSkip)) {    // sampled-out replay: pass head and tail on, capture nothing
        if (publisher) {
            a.ctrl->head[par ^ 1u] = head0;
            a.ctrl->head_at[par ^ 1u] = head_at;
            a.ctrl->tail_for[par ^ 1u] = tail_now > raw.tail_for ? tail_now : raw.tail_for;
        }
        return;
    }
    // record geometry: known on the host, or from the keep vector
    uint32_t n_rows = a.n_wg_rows, my_row = blockIdx.x;
    bool kept = true;
    uint64_t record_bytes = a.record_bytes, payload_bytes = a.payload_bytes, off_sum = a.off_sum, sum_arr = a.sum_arr;
    if constexpr (MASK) {
        const uint32_t q_me = blockIdx.x >> 6;
        n_rows = 0;
        my_row = 0;
#pragma unroll
        for (uint32_t q = 0; q < 16; q++) {
            const uint32_t pc = (uint32_t)__popcll(kept_bits[q]);
            n_rows += pc;
            if (q < q_me) my_row += pc;
        }
        if (!meta_wg) {
            const uint64_t mine = kept_bits[q_me & 15u], bit = 1ull << (blockIdx.x & 63u);
            kept = (mine & bit) != 0;
            my_row += (uint32_t)__popcll(mine & (bit - 1u));
        }
        payload_bytes = (uint64_t)n_rows * a.units_per_row * NB_OUT;
        off_sum = a.off_payload + ((payload_bytes + 63u) & ~63ull);
        sum_arr = ((uint64_t)n_rows * 4u + 63u) & ~63ull;
        record_bytes = off_sum + (uint64_t)__popc(a.summary_mask & 7u) * sum_arr;
    }
    // record y of the launch lies y records behind the head the launch found (all records of a
    // batch have one size: record y fits iff the y before it did, and then they were kept)
    const bool drop_newest = (flags & kStepDropNewest) != 0;
    const uint64_t head = head0 + (uint64_t)y * record_bytes;
    const bool dropped = !INTO && drop_newest && head - tail + record_bytes > a.cap;
    RingW w;
    w.ring = a.ring;
    w.cap = a.cap;
    w.base = head_at + (uint64_t)y * record_bytes;
    if (w.base >= w.cap) w.base -= w.cap;   // the issuer made sure a launch's records fit the ring together

    if (meta_wg) {
        if (publisher) {
            if (a.note) st_system(a.note, head0);
            a.ctrl->tail_for[par ^ 1u] = tail_now > raw.tail_for ? tail_now : raw.tail_for;
            const uint64_t n_fit = records_that_fit(gridDim.y, head0, tail, record_bytes, a.cap, drop_newest);
            publish_launch(a.ctrl, par, head0, head_at, cnt_cap, cnt_drop, record_bytes, n_rows, n_fit, gridDim.y - n_fit, a.cap,
                           seq + gridDim.y - 1u, a.step ? nullptr : a.cslot);
        }
        if (dropped && tid == kCtlTid) atomicAdd(&a.ctrl->point_drops[point_id & 4095u], 1u);
        if (dropped) return;
        if (tid < 4) {
            u32x4 hv;
            const uint64_t seq_y = ((uint64_t)sh[24] | ((uint64_t)sh[25] << 32)) + y;
            if (tid == 0) hv = u32x4{0x32494D44u, 1u | (64u << 16), (uint32_t)seq_y, (uint32_t)(seq_y >> 32)};
            else if (tid == 1) hv = u32x4{sh[26], sh[27], point_id, a.hdr7};
            else if (tid == 2) hv = u32x4{a.n_reqs, n_rows, a.row_elems, a.rank_tag};
            else hv = u32x4{(uint32_t)record_bytes, (uint32_t)(record_bytes >> 32), (uint32_t)payload_bytes,
                            (uint32_t)(payload_bytes >> 32)};
            ring_store<u32x4>(w, 16u * tid, hv);
        }
        const uint32_t tab_slots = (uint32_t)((a.off_payload - 64u) / 16u);
        for (uint32_t r = tid; r < tab_slots; r += kThreads) {
            u32x4 tv = {0u, 0u, 0u, 0u};
            if (r < a.n_reqs) {
                bool have = false;
                if constexpr (INTO)
                    if (b.n_words) {
                        tv = inline_entry(sizeof(DecodeArgs), b.n_words, a.n_reqs, r);
                        have = true;
                    }
                if (!have) {
                    const uint4 e = a.req_table[r];
                    tv.x = e.x; tv.y = e.y; tv.z = e.z; tv.w = e.w;
                }
                if constexpr (MASK) tv.w = (uint32_t)((kept_bits[(r >> 6) & 15u] >> (r & 63u)) & 1ull);
            }
            ring_store<u32x4>(w, 64u + 16ull * r, tv);
        }
        const uint32_t pad = (uint32_t)(off_sum - a.off_payload - payload_bytes);
        if (tid < pad) ring_store<uint8_t>(w, a.off_payload + payload_bytes + tid, (uint8_t)0);
        const uint32_t n_sum = __popc(a.summary_mask & 7u);
        const uint32_t spad = (uint32_t)(sum_arr - (uint64_t)n_rows * 4u) / 4u;
        for (uint32_t k = tid; k < n_sum * spad; k += kThreads) {
            const uint32_t arr = k / spad, i = k - arr * spad;
            ring_store<uint32_t>(w, off_sum + arr * sum_arr + (uint64_t)n_rows * 4u + 4ull * i, 0u);
        }
        return;
    }

    if (dropped || !kept) return;
    const uint32_t g = my_row;
    if (!ok && tid == 0) atomicAdd((unsigned long long *)&a.ctrl->bad_rows, 1ull);
    const uint64_t row_off = a.off_payload + (uint64_t)g * a.units_per_row * NB_OUT;
#pragma unroll
    for (uint32_t k = 0; k < U; k++) {
        const uint32_t c = tid + k * ustr;
        if ((!SUMM || tid < ustr) && c < a.units_per_row)
            emit_unit<2, 8, OUT>(w, row_off + (uint64_t)c * NB_OUT, v[k]);
    }
    if constexpr (SUMM) {
        if (tid == 0) {
            const float *red = reinterpret_cast<const float *>(sh + 8);
            const float ss = (red[0] + red[1]) + (red[2] + red[3]);
            const float sm = (red[4] + red[5]) + (red[6] + red[7]);
            const uint32_t m01 = sh[16] > sh[17] ? sh[16] : sh[17], m23 = sh[18] > sh[19] ? sh[18] : sh[19];
            const uint32_t am = m01 > m23 ? m01 : m23;
            uint64_t o = off_sum + (uint64_t)g * 4u;
            if (a.summary_mask & 1u) { ring_store<float>(w, o, sqrtf(ss)); o += sum_arr; }
            if (a.summary_mask & 2u) { ring_store<float>(w, o, sm / (float)a.row_elems); o += sum_arr; }
            if (a.summary_mask & 4u) { ring_store<float>(w, o, am_value(am, a.hdr7 & 0xFFu)); }
        }
    }
}

// ---------------------------------------------------------------- dense rows that a launch finds by itself
// Dense rows of one row per request or of up to 64 ragged requests: the largest records there are (ragged prompts, the
// tensors of a batch).  Without summaries, of at least kLongRowUnits units: a wavefront takes up to 256 consecutive units of one row, and everything but its
// lanes' places in them is the same for the whole wavefront and kept in scalar registers.
// Bound: HBM.  What a launch loses on top is the time until its first loads leave, and the unequal ends of its
// workgroups.  Time stamps in the general kernel, which took these rows before, showed 5 us in front of the first loads of
// a full GPU where memory answers in 0.6: a thousand instructions (fetched cold), scans and searches through LDS, a
// barrier.  So there is hardly anything in front of the loads here: each wavefront scans the request table by itself
// (at most 64 requests, one per lane; none at all where requests have one row each), there is no LDS and no
// barrier, and header, table and publishing are a workgroup of their own, whose code the others do not run through.  It is the first
// one of its record: a table of many requests takes it several trips, and as the last one to start it kept the GPU waiting (4096
// requests x 4096 fp32 stored 32.7 us and 27.4 like this, 2048 x 14336 bf16 26.4 and 23.5, 1024 x 14336 15.1 and 13.7).  And there is one step to a wavefront, many more workgroups than fit at once, and no
// software pipeline: eight workgroups per compute unit hide each other's trips (55 to 58 registers; two steps in
// a pipeline take 93, five workgroups).  Steps per wavefront 1 / 2 / 4: 19.1 / 20.4 / 23.7 us; units per lane 2 / 4 / 8:
// 21.8 / 18.8 / 20.0 (9.3 k rows x 4096 bf16 -> fp8).
// Kernel times, before and after: bf16 -> fp8, 32 requests: 9.3 k x 4096 (every fourth token) 23.5 -> 18.8 us (6.1 TB/s),
// 9.3 k x 14336 85 -> 69.4 (5.8 TB/s), 37 k x 4096 93 -> 79, 9.3 k x 2304 25 -> 13, 2000 x 4096 9.1 -> 5.9; raw: 9.3 k x 4096
// 28.6 -> 24.2, 9.3 k x 14336 106 -> 92; one row per request, 80 tensors of 256 x 8192 raw in one launch 111 -> 107.
// Under best effort the head, which tells whether the record fits, is asked for with everything else and looked at when the first
// rows have been asked for: waited for in front of them it cost the launch of 80 tensors of 256 x 8192 raw 6 us (cold, all kept:
// 116.5 -> 109.9, under the completeness policy 111; the general kernel 114).  A record that is dropped has read a step for nothing.
// ONCE: launches that read more than the memory-side cache holds do so past it (non-temporal loads; plan_grid() has the figures).
// With summaries (SUMM), of more than 128 units: a wavefront per row, or a workgroup per row with a quarter of it to each
// wavefront (plan_grid() says which, with figures); lanes, parts and the order of the sums are the general and the
// decode-shaped kernel's, so a row's summaries have the same bits wherever it is captured.  80 tensors of 256 x 8192,
// statistics alone: 61 -> 49.5 us (6.8 TB/s read).
// Shorter rows, and in large launches those that leave many of a step's lanes idle, are dealt flat by the general kernel (plan_grid()
// says which, with figures), and so are rows of more than 64 ragged requests.
struct RowsArgs {
    // lines 0 and 1, for summaries also the start of line 2: what the row workgroups need
    int64_t row_stride_b, n_src_rows;
    const uint4 *req_table;
    const uint32_t *row0;           // first source row of each request
    const uint8_t *keep_mask;
    const int32_t *row_index;
    uint8_t *ring;
    uint64_t cap;
    DevCtrl *ctrl;
    const StepParams *step;
    uint64_t tail_floor;
    uint32_t flags;                 // kRows*
    uint32_t n_reqs, units_per_row, row_elems;
    uint32_t parts, parts_magic, parts_shift;   // steps per row; x / parts = (x * parts_magic >> 32) >> parts_shift, x below 2^31
    uint32_t row_groups;            // workgroups that move rows (gridDim.x - 1: the first one does not)
    uint32_t row_first;
    uint32_t summary_mask, src_dtype, row_lanes, passes;     // summaries: lanes that share a row, as in the general kernel
    uint32_t pad;
    // the rest of line 2: header and publishing
    uint64_t seq, step_id;
    CommitSlot *cslot;
    const uint64_t *tail_src;
    uint32_t node, hdr7, rank_tag, n_tail_drop;
    uint64_t *note;
    uint32_t rows_at;               // launches into the caller's memory: the word of their table from which on rows are listed
    uint32_t spare;
};
static_assert(sizeof(RowsArgs) % 16u == 0, "the block behind it is read as 16-byte entries");
constexpr uint32_t kRowsSimple = 1u;        // no keep vector, one row per request
constexpr uint32_t kRowsConsecutive = 2u;   // and request i's row is row_first + i
constexpr uint32_t kRowsDropNewest = 4u, kRowsParIn = 8u;

// SUMM: 0 no summaries, 1 a wavefront per row, 2 a workgroup per row.
template <int ES_IN, int OUT, int SUMM, typename SRC, bool LOOSE, bool ONCE>
__global__ void __launch_bounds__(kThreads) capture_rows_kernel(const RowsArgs a, const SRC b)
{
    constexpr bool INTO = std::is_same<SRC, IntoArgs>::value;
    constexpr int VEC = 16 / ES_IN;
    constexpr uint32_t U = 4, SU = U * 64u;                 // units of a step
    constexpr uint32_t NB_IN = 16u, NB_OUT = out_unit_bytes<ES_IN, VEC, OUT>(), ES_OUT = NB_OUT / VEC;
    typedef typename UnitT<ES_IN * VEC>::T unit_t;
    typedef __attribute__((address_space(1))) const unit_t __attribute__((aligned(LOOSE ? ES_IN : ES_IN * VEC))) global_unit_t;
    typedef __attribute__((address_space(4))) const uint64_t constant_u64;
    typedef __attribute__((address_space(1))) const uint64_t global_u64;
    typedef __attribute__((address_space(4))) const int32_t constant_i32;
    const uint32_t y = INTO ? 0u : blockIdx.y;
    const uint8_t *const src = b.src[y];
    const uint32_t lane = threadIdx.x & 63u, wv = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const bool simple = (a.flags & kRowsSimple) != 0u, meta = blockIdx.x == 0u;
    const uint32_t group = blockIdx.x - 1u;                 // of the workgroups that move rows
    const bool index_mode = a.row_index != nullptr;
    const uint32_t n_reqs = a.n_reqs, par = a.flags & kRowsParIn ? 1u : 0u;

    // -- control words.  Where the record lies is asked for here, by vector loads (said to be), and waited for when the
    //    first rows are on their way; what decides whether there is a record at all comes through the scalar cache.
    uint64_t head_v = 0, at_v = 0, tail = 0;
    uint32_t policy = 0;
    if constexpr (!INTO) {
        uint64_t ctrl_v = (uint64_t)(uintptr_t)a.ctrl;
        asm volatile("" : "+v"(ctrl_v));
        head_v = ((global_u64 *)(ctrl_v + offsetof(DevCtrl, head)))[par];
        at_v = ((global_u64 *)(ctrl_v + offsetof(DevCtrl, head_at)))[par];
        policy = a.flags & kRowsDropNewest ? kStepDropNewest : 0u;
        tail = a.tail_floor;
        if (a.step) {
            policy = (uint32_t)((constant_u64 *)a.step)[3];
            tail = ((constant_u64 *)a.step)[2];
        }
        if (policy & kStepDropNewest) {
            const uint64_t seen = ((constant_u64 *)a.ctrl->tail_for)[par];
            tail = seen > tail ? seen : tail;
        }
    }

    // -- the request table, a request per lane: kept rows in front of it, first source row, rows between two of its rows
    u32x4 entry = {0u, 0u, 0u, 0u};
    uint32_t first_row = 0, kept = 0, upto = 0, listed_upto = 0;
    uint32_t n_rows = n_reqs;
    if (!simple) {
        const uint32_t r = lane < n_reqs ? lane : 0u;
        bool have = false;
        if constexpr (INTO) {
            if (b.n_words) {
                // (at most 64 requests: their table fits as it is)
                entry = *(__attribute__((address_space(1))) const u32x4 *)(inline_table(sizeof(RowsArgs)) + 4u * r);
                first_row = inline_table(sizeof(RowsArgs))[4u * n_reqs + r];
                have = true;
            }
        }
        if (!have) {
            const uint4 e = a.req_table[r];
            entry = u32x4{e.x, e.y, e.z, e.w};
            first_row = a.row0[r];
        }
        const bool keep = a.keep_mask ? a.keep_mask[r] != 0 : true;
        const uint32_t listed = lane < n_reqs ? entry.w : 0u;
        kept = keep ? listed : 0u;
        upto = wave_incl_scan(kept);
        n_rows = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
        if (index_mode) listed_upto = wave_incl_scan(listed);
    }
    auto of_request = [](uint32_t v, uint32_t r) { return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)r); };

    // -- record geometry, and whether the record fits
    const uint64_t row_in = (uint64_t)a.row_elems * ES_IN, row_out = (uint64_t)a.row_elems * ES_OUT;
    const uint64_t off_payload = 64u + (((uint64_t)n_reqs * 16u + 63u) & ~63ull);
    const uint64_t payload_bytes = n_rows * row_out;
    const uint64_t off_sum = off_payload + ((payload_bytes + 63u) & ~63ull), sum_arr = ((uint64_t)n_rows * 4u + 63u) & ~63ull;
    const uint32_t n_sum = SUMM ? (uint32_t)__popc(a.summary_mask) : 0u;
    const uint64_t record_bytes = off_sum + n_sum * sum_arr;
    // (where the launch found the head is what it waits for longest: not before the first rows are on their way)
    auto dropped = [&]() -> bool {
        if constexpr (INTO) return false;
        return (policy & kStepDropNewest) && uniform_u64(head_v) + (y + 1ull) * record_bytes - tail > a.cap;
    };
    RingW w;
    w.ring = a.ring;
    w.cap = a.cap;
    w.base = 0;
    auto settle = [&]() {
        if constexpr (!INTO) {
            w.base = uniform_u64(at_v) + (uint64_t)y * record_bytes;    // (the issuer made sure a launch's records fit the ring together)
            if (w.base >= w.cap) w.base -= w.cap;
        }
    };

    if (!meta) {
        if (!INTO && (policy & kStepSkip)) return;
        if constexpr (SUMM != 0) {
            if (dropped()) return;
        }
        const uint32_t n_steps = n_rows * a.parts;          // (the host keeps rows x units below 2^32)
        const uint8_t *const zeros = reinterpret_cast<const uint8_t *>(a.ctrl->zeros);
        struct Step { uint32_t g, part; const uint8_t *base; bool ok; };
        auto listed_row = [&](uint32_t i) -> int64_t {      // a row that is listed somewhere
            if constexpr (INTO)
                if (b.n_words && !index_mode) return (int64_t)inline_table_uniform(sizeof(RowsArgs))[a.rows_at + i];
            const int32_t v = ((constant_i32 *)(index_mode ? a.row_index : reinterpret_cast<const int32_t *>(a.row0)))[i];
            return index_mode ? (int64_t)v : (int64_t)(uint32_t)v;
        };
        auto step_at = [&](uint32_t s) -> Step {
            Step st;
            st.g = a.parts == 1u ? s : __umulhi(s, a.parts_magic) >> a.parts_shift;
            st.part = s - st.g * a.parts;
            int64_t row;
            if (simple) {
                row = a.flags & kRowsConsecutive ? (int64_t)a.row_first + st.g : listed_row(st.g);
            } else {
                const uint32_t r = (uint32_t)__popcll(__ballot(lane < n_reqs && upto - kept <= st.g)) - 1u;
                const uint32_t j = st.g - (of_request(upto, r) - of_request(kept, r));      // the request's kept row j
                if (index_mode) row = listed_row(of_request(listed_upto, r) - of_request(entry.w, r) + j);
                else row = (int64_t)(uint64_t)(of_request(first_row, r) + j * of_request(entry.z, r));
            }
            st.ok = row >= 0 && row < a.n_src_rows;
            st.base = src + (st.ok ? row : 0) * a.row_stride_b;
            return st;
        };
        uint32_t n_bad = 0;
        if constexpr (SUMM != 0) {
            constexpr bool WG = SUMM == 2;              // a workgroup per row, a part of it to each wavefront
            __shared__ float red[WG ? 12 : 1];
            const uint32_t rl = a.row_lanes, parts = rl >> 6;
            const uint32_t rows_at_once = a.row_groups * (WG ? 1u : kThreads / 64u);
            for (uint64_t g = WG ? group : group * (kThreads / 64u) + wv; g < n_rows; g += rows_at_once) {
                const Step st = step_at((uint32_t)g);
                n_bad += st.ok || (WG && wv != 0u) ? 0u : 1u;
                float ss[4] = {0.f, 0.f, 0.f, 0.f}, sm[4] = {0.f, 0.f, 0.f, 0.f};       // of each part
                uint32_t am = 0;
                auto one_part = [&](uint32_t part) -> Accum {
                    Accum acc = {0.f, 0.f, 0u};
#pragma unroll 1
                    for (uint32_t pass = 0; pass < a.passes; pass++) {
                        const uint32_t c0 = pass * U * rl + part * 64u + lane;
                        u32x4 v[U];
#pragma unroll
                        for (uint32_t t = 0; t < U; t++) {          // (a lane with nothing to load reads zeros)
                            const uint32_t c = c0 + t * rl;
                            const uint64_t e = (uint64_t)c * VEC, last = (uint64_t)a.row_elems - VEC;
                            const uint8_t *p = st.ok && c < a.units_per_row ? st.base + (LOOSE && e > last ? last : e) * ES_IN : zeros;
                            v[t] = ONCE ? __builtin_nontemporal_load((global_unit_t *)p) : *(global_unit_t *)p;
                        }
                        settle();
                        if constexpr (OUT != OUT_NONE) {
#pragma unroll
                            for (uint32_t t = 0; t < U; t++) {
                                const uint32_t c = c0 + t * rl;
                                const uint64_t e = (uint64_t)c * VEC, last = (uint64_t)a.row_elems - VEC;
                                if (c < a.units_per_row)
                                    emit_unit<ES_IN, VEC, OUT, LOOSE>(w, off_payload + g * row_out + (LOOSE && e > last ? last : e) * ES_OUT, v[t]);
                            }
                        }
                        if constexpr (LOOSE) {          // the last unit's elements that the one in front of it has as well
#pragma unroll
                            for (uint32_t t = 0; t < U; t++)
                                if (c0 + t * rl + 1u == a.units_per_row) v[t] = without_first<VEC>(v[t], a.units_per_row * VEC - a.row_elems);
                        }
                        accum_units<ES_IN, VEC>(acc, v, a.src_dtype);
                    }
                    if (a.summary_mask & 1u) acc.ss = wave_sum(acc.ss);
                    if (a.summary_mask & 2u) acc.s = wave_sum(acc.s);
                    if (a.summary_mask & 4u) acc.am = wave_max_u32(fold_am<ES_IN, VEC>(acc.am));
                    return acc;
                };
                if constexpr (WG) {
                    Accum acc = {0.f, 0.f, 0u};
                    if (wv < parts) acc = one_part(wv);
                    if (g >= rows_at_once) lds_barrier();       // (the row before this one has been read)
                    if (lane == 0) {
                        red[wv] = acc.ss;
                        red[4 + wv] = acc.s;
                        red[8 + wv] = __uint_as_float(acc.am);
                    }
                    lds_barrier();
#pragma unroll
                    for (uint32_t i = 0; i < 4; i++) {
                        ss[i] = red[i];
                        sm[i] = red[4 + i];
                        const uint32_t x = __float_as_uint(red[8 + i]);
                        am = x > am ? x : am;
                    }
                } else {
#pragma unroll
                    for (uint32_t part = 0; part < 4u; part++) {
                        if (part >= parts) break;
                        const Accum acc = one_part(part);
                        ss[part] = acc.ss;
                        sm[part] = acc.s;
                        am = acc.am > am ? acc.am : am;
                    }
                }
                if (lane == 0 && (!WG || wv == 0u)) {           // (the order in which every kernel here takes them)
                    uint64_t o = off_sum + g * 4u;
                    if (a.summary_mask & 1u) { ring_store<float>(w, o, sqrtf((ss[0] + ss[1]) + (ss[2] + ss[3]))); o += sum_arr; }
                    if (a.summary_mask & 2u) { ring_store<float>(w, o, ((sm[0] + sm[1]) + (sm[2] + sm[3])) / (float)a.row_elems); o += sum_arr; }
                    if (a.summary_mask & 4u) ring_store<float>(w, o, am_value(am, a.src_dtype));
                }
            }
        } else {
            // where a lane's unit t of a step lies, in bytes from the step's first (a row that is not a whole number of
            // units ends with one that reaches back, which is why other parts than the first count from a unit earlier);
            // lanes behind the end of the row get its last unit
            auto lane_at = [&](uint32_t part, uint32_t t, uint64_t row_bytes, uint32_t nb) -> uint32_t {
                const uint32_t back = LOOSE && part ? nb : 0u;
                const uint64_t rest = row_bytes - (uint64_t)part * (SU * nb);
                const uint32_t last = (rest < SU * nb ? (uint32_t)rest : SU * nb) + back - nb;
                const uint32_t off = (lane + t * 64u) * nb + back;
                return off < last ? off : last;
            };
            auto load = [&](const Step &st, u32x4 (&v)[U]) {    // (a row that lies outside the source: zeros)
                const uint8_t *const base = st.ok ? st.base + (uint64_t)st.part * (SU * NB_IN) - (LOOSE && st.part ? NB_IN : 0u) : zeros;
                const uint32_t mask = st.ok ? ~0u : 0u;
#pragma unroll
                for (uint32_t t = 0; t < U; t++) {
                    const uint8_t *p = base + (lane_at(st.part, t, row_in, NB_IN) & mask);
                    v[t] = ONCE ? __builtin_nontemporal_load((global_unit_t *)p) : *(global_unit_t *)p;
                }
            };
            auto store = [&](const Step &st, const u32x4 (&v)[U]) {
                const uint32_t c0 = st.part * SU;
                const uint64_t pos = off_payload + st.g * row_out + (uint64_t)c0 * NB_OUT - (LOOSE && st.part ? NB_OUT : 0u);
                uint64_t p = w.base + pos;
                if (p >= w.cap) p -= w.cap;
                if (p + (SU + 1u) * NB_OUT <= w.cap) {          // all of it in front of the ring's end: no lane needs to look
#pragma unroll
                    for (uint32_t t = 0; t < U; t++) {
                        const auto o = convert_unit<ES_IN, VEC, OUT>(v[t]);
                        if (c0 + lane + t * 64u < a.units_per_row) store_out<LOOSE>(w.ring + p + lane_at(st.part, t, row_out, NB_OUT), o);
                    }
                } else {
#pragma unroll
                    for (uint32_t t = 0; t < U; t++)
                        if (c0 + lane + t * 64u < a.units_per_row)
                            unit_store<LOOSE>(w, pos + lane_at(st.part, t, row_out, NB_OUT), convert_unit<ES_IN, VEC, OUT>(v[t]));
                }
            };
            // (one step each, unless a replayed step's selection has grown since its grid was made)
            for (uint64_t s = group * (kThreads / 64u) + wv; s < n_steps; s += a.row_groups * (kThreads / 64u)) {
                const Step st = step_at((uint32_t)s);
                u32x4 v[U];
                load(st, v);
                if (dropped()) return;
                settle();
                n_bad += st.part == 0u && !st.ok ? 1u : 0u;     // a bad row is counted where it begins
                store(st, v);
            }
        }
        if (n_bad && lane == 0) atomicAdd((unsigned long long *)&a.ctrl->bad_rows, (unsigned long long)n_bad);
        return;
    }

    // -- the first workgroup: header, request table, pads; and, of the launch's first record, the chain of launches
    settle();
    const uint64_t head0 = uniform_u64(head_v), at0 = uniform_u64(at_v);
    const uint32_t tid = threadIdx.x, point_id = b.point[y];
    uint64_t seq = a.seq, step_id = a.step_id;
    if constexpr (!INTO) {
        if (a.step) {
            seq = ((constant_u64 *)a.step)[0] + a.node;
            step_id = ((constant_u64 *)a.step)[1];
        }
        if (y == 0 && tid == kThreads - 64u) {
            DevCtrl *c = a.ctrl;
            const uint64_t tail_now = ld_system(a.tail_src ? a.tail_src : &c->tail);
            const RawControl raw = fetch_control(c, par, nullptr);
            c->tail_for[par ^ 1u] = tail_now > raw.tail_for ? tail_now : raw.tail_for;
            if (policy & kStepSkip) {
                c->head[par ^ 1u] = head0;
                c->head_at[par ^ 1u] = at0;
            } else {
                if (a.note) st_system(a.note, head0);
                const uint64_t n_fit = records_that_fit(gridDim.y, head0, tail, record_bytes, a.cap, (policy & kStepDropNewest) != 0u);
                publish_launch(c, par, head0, at0, raw.cap, raw.drop, record_bytes, n_rows, n_fit, gridDim.y - n_fit + a.n_tail_drop,
                               a.cap, seq + gridDim.y + a.n_tail_drop - 1u, a.step ? nullptr : a.cslot);
                for (uint32_t i = 0; i < a.n_tail_drop; i++) atomicAdd(&c->point_drops[b.point[gridDim.y + i] & 4095u], 1u);
            }
        }
        if (policy & kStepSkip) return;
        if (dropped()) {
            if (tid == 0) atomicAdd(&a.ctrl->point_drops[point_id & 4095u], 1u);
            return;
        }
    }
    if (tid < 4u) {
        const uint64_t seq_y = seq + y;
        u32x4 hv;
        if (tid == 0) hv = u32x4{0x32494D44u, 1u | (64u << 16), (uint32_t)seq_y, (uint32_t)(seq_y >> 32)};
        else if (tid == 1) hv = u32x4{(uint32_t)step_id, (uint32_t)(step_id >> 32), point_id, a.hdr7};
        else if (tid == 2) hv = u32x4{n_reqs, n_rows, a.row_elems, a.rank_tag};
        else hv = u32x4{(uint32_t)record_bytes, (uint32_t)(record_bytes >> 32), (uint32_t)payload_bytes, (uint32_t)(payload_bytes >> 32)};
        ring_store<u32x4>(w, 16u * tid, hv);
    }
    const uint32_t tab_slots = (uint32_t)((off_payload - 64u) / 16u);
    if (!simple) {                          // (one request per lane: the first wavefront's own)
        if (tid < tab_slots) {
            const u32x4 tv = {entry.x, entry.y, entry.z, kept};
            ring_store<u32x4>(w, 64u + 16ull * tid, tid < n_reqs ? tv : u32x4{0u, 0u, 0u, 0u});
        }
    } else {
        typedef __attribute__((address_space(1))) const u32x4 global_entry;
        global_entry *table = (global_entry *)a.req_table;
        if constexpr (INTO)
            if (b.n_words) table = (global_entry *)inline_table(sizeof(RowsArgs));
        uint32_t slots = tab_slots;
        if constexpr (INTO)
            if (b.n_words & kByColumn) {
                for (uint32_t r = tid; r < tab_slots; r += kThreads) {
                    const u32x4 tv = inline_entry(sizeof(RowsArgs), b.n_words, n_reqs, r < n_reqs ? r : n_reqs - 1u);
                    ring_store<u32x4>(w, 64u + 16ull * r, r < n_reqs ? tv : u32x4{0u, 0u, 0u, 0u});
                }
                slots = 0;
            }
        // (up to 4096 of them: four trips in flight)
        for (uint32_t r0 = tid; r0 < slots; r0 += 4u * kThreads) {
            u32x4 tv[4];
#pragma unroll
            for (uint32_t k = 0; k < 4; k++) {
                const uint32_t r = r0 + k * kThreads;
                tv[k] = table[r < n_reqs ? r : n_reqs - 1u];
            }
#pragma unroll
            for (uint32_t k = 0; k < 4; k++) {
                const uint32_t r = r0 + k * kThreads;
                if (r < tab_slots) ring_store<u32x4>(w, 64u + 16ull * r, r < n_reqs ? tv[k] : u32x4{0u, 0u, 0u, 0u});
            }
        }
    }
    const uint32_t pad = (uint32_t)(off_sum - off_payload - payload_bytes);
    if (tid < pad) ring_store<uint8_t>(w, off_payload + payload_bytes + tid, (uint8_t)0);
    const uint32_t spad = (uint32_t)(sum_arr - (uint64_t)n_rows * 4u) / 4u;
    if (tid < n_sum * 16u && (tid & 15u) < spad)
        ring_store<uint32_t>(w, off_sum + (tid >> 4) * sum_arr + (uint64_t)n_rows * 4u + 4u * (tid & 15u), 0u);
}

// ---------------------------------------------------------------- small kernels
// Words for device memory, carried by the launch.  Up to 896 of them in 3.6 KB of arguments, larger tables 3072 at a time:
// a launch of 12 KB of arguments takes the host as long as one of 4 KB (3.3 us; 24 KB: 6.9).
template <uint32_t N>
struct UploadChunk {
    uint32_t w[N];
};

template <uint32_t N>
__global__ void __launch_bounds__(kThreads) upload_kernel(uint32_t *dst, const UploadChunk<N> c, uint32_t n)
{
    for (uint32_t i = threadIdx.x; i < n; i += kThreads) dst[i] = c.w[i];
}

// Start of a replayable step (an ordinary launch in front of the graph's): the step's
// parameter block, and head / tail_for carried over to the copy its first launch reads.
__global__ void step_begin_kernel(DevCtrl *ctrl, StepParams *step, const StepParams v, uint32_t par_from,
                                  uint32_t par_to, const uint64_t *host_tail)
{
    if (threadIdx.x != 0) return;
    *step = v;
    if (host_tail) ctrl->tail = ld_system(host_tail);    // the step's launches read this copy
    if (par_from != par_to) {
        ctrl->head[par_to] = ctrl->head[par_from];
        ctrl->head_at[par_to] = ctrl->head_at[par_from];
        ctrl->tail_for[par_to] = ctrl->tail_for[par_from];
    }
}

// Fetch one commit slot into pinned host memory: a small launch of its own on the producer's
// stream, so the capture kernel itself never writes across PCIe (such a store is
// acknowledged only after some 4-5 microseconds, and a kernel cannot retire before its
// stores have been).
__global__ void fetch_slot_kernel(const CommitSlot *src, CommitSlot *dst_host)
{
    const uint32_t i = threadIdx.x;
    if (i < sizeof(CommitSlot) / 8u)
        reinterpret_cast<volatile uint64_t *>(dst_host)[i] = reinterpret_cast<const uint64_t *>(src)[i];
}

// Drain by kernel: 16-byte loads from the device ring, 16-byte stores into the pinned host ring (posted PCIe writes).
// Bound by the link.  The stores go past L2 by their own cache policy (system scope), for two reasons.  What L2 takes in first
// leaves it by eviction, in whatever order and as parts of lines: 16.8 MB 322 us with plain non-temporal stores, 311 like this (the
// copy engine: 322 with the host's wait in front of it).  And a store that has been acknowledged has arrived: a workgroup that has
// waited for its own can say so itself, in a word of its own in pinned memory (`done`, one per workgroup), with no fence, no
// counter and nothing behind the kernel.  A host that polls those words sees 4 KB, captured and copied, 10.0 us after it has issued both,
// 0.6 MB after 21.4, 4.2 MB after 85; by an event behind the kernel 14.2, 25.6 and 92.
// 64 workgroups: with 16 the same 16.8 MB take 313 us.
__global__ void __launch_bounds__(kThreads) drain_kernel(const DrainSpans d, uint64_t *done, uint64_t tick)
{
    constexpr int kSystem = 1 | 2 | 16;         // sc0, nt, sc1: write through, do not keep
#pragma unroll
    for (uint32_t i = 0; i < 3; i++) {
        const uint8_t *const src = d.span[i].src;
        const uint32_t n = d.span[i].n;
        const __amdgpu_buffer_rsrc_t host = __builtin_amdgcn_make_buffer_rsrc(d.span[i].dst, 0, (int)n, 0x00027000);
        for (uint32_t o = (blockIdx.x * kThreads + threadIdx.x) * 16u; o < n; o += gridDim.x * kThreads * 16u) {
            const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src + o));
            __builtin_amdgcn_raw_buffer_store_b128(v, host, (int)o, 0, kSystem);
        }
    }
    if (!done) return;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // this wavefront's stores have arrived
    __syncthreads();                                    // and so have the others'
    if (threadIdx.x == 0) st_system(done + blockIdx.x, tick);
}

// ---------------------------------------------------------------- launchers
// A benchmark may ask for the next capture launch of its thread to be timed by the hardware itself:
// the two events then take the dispatch's own start and end time stamps (what a profiler reports
// as the kernel's duration), not the times at which markers around the launch were reached.
static thread_local hipEvent_t t_time_start = nullptr, t_time_stop = nullptr;

extern "C" dmi_status_t dmi_debug_time_next_launch(void *start_event, void *stop_event)
{
    t_time_start = static_cast<hipEvent_t>(start_event);
    t_time_stop = static_cast<hipEvent_t>(stop_event);
    return DMI_OK;
}

#define DMI_LAUNCH_CAPTURE(in_step, kernel, grid, lds, stream, ...)                                                   \
    do {                                                                                                              \
        if (t_time_start && t_time_stop && !(in_step)) {                                                              \
            hipExtLaunchKernelGGL(kernel, grid, dim3(kThreads), lds, stream, t_time_start, t_time_stop, 0, __VA_ARGS__); \
            t_time_start = t_time_stop = nullptr;                                                                     \
        } else {                                                                                                      \
            hipLaunchKernelGGL(kernel, grid, dim3(kThreads), lds, stream, __VA_ARGS__);                                \
        }                                                                                                             \
    } while (0)

template <int ES_IN, int OUT, int SUMM, bool LOOSE, typename SRC>
static hipError_t launch_rows(const CaptureArgs &a, const SRC &b, uint32_t grid, hipStream_t s)
{
    if (a.paged || (!a.simple && a.n_reqs > 64u)) return hipErrorInvalidValue;
    if constexpr (std::is_same<SRC, IntoArgs>::value)
        if ((b.n_words & kByColumn) && !a.simple) return hipErrorInvalidValue;
    RowsArgs d;
    std::memset(&d, 0, sizeof d);
    d.row_stride_b = a.row_stride_b;
    d.n_src_rows = a.n_src_rows;
    d.req_table = a.req_table;
    d.row0 = a.row0;
    d.keep_mask = a.keep_mask;
    d.row_index = a.row_index;
    d.ring = a.ring;
    d.cap = a.cap;
    d.ctrl = a.ctrl;
    d.step = a.step;
    d.tail_floor = a.tail_floor;
    d.flags = (a.simple ? kRowsSimple : 0u) | (a.rows_consecutive ? kRowsConsecutive : 0u) |
              (a.drop_newest ? kRowsDropNewest : 0u) | (a.par_in ? kRowsParIn : 0u);
    d.n_reqs = a.n_reqs;
    d.units_per_row = a.units_per_row;
    d.row_elems = a.row_elems;
    d.parts = SUMM ? 1u : (a.units_per_row + 255u) / 256u;      // (with summaries a wavefront takes the row)
    d.summary_mask = a.summary_mask;
    d.src_dtype = a.src_dtype;
    d.row_lanes = a.row_lanes;
    d.passes = SUMM ? (a.units_per_row + 4u * a.row_lanes - 1u) / (4u * a.row_lanes) : 0u;
    if (d.parts > 1u) {             // magic = ceil(2^(31 + l) / parts) with l = ceil(log2(parts)): exact for 31 bits
        d.parts_shift = 31u - (uint32_t)__builtin_clz(d.parts - 1u);
        d.parts_magic = (uint32_t)(((1ull << (32u + d.parts_shift)) + d.parts - 1u) / d.parts);
    }
    d.row_groups = grid;
    if constexpr (std::is_same<SRC, IntoArgs>::value) d.rows_at = b.n_words & kByColumn ? b.rows_at : 4u * a.n_reqs;
    d.row_first = a.row_first;
    d.seq = a.seq;
    d.step_id = a.step_id;
    d.cslot = a.cslot;
    d.tail_src = a.tail_src;
    d.note = a.note;
    d.node = a.node;
    d.hdr7 = a.src_dtype | (a.out_dtype << 8) | (a.summary_mask << 16) | (a.rec_flags << 24);
    d.rank_tag = a.rank_tag;
    d.n_tail_drop = a.n_tail_drop;
    const dim3 g(grid + 1u, a.n_batch);
    if constexpr (!LOOSE) {
        if (a.read_once) {
            DMI_LAUNCH_CAPTURE(a.step != nullptr, (capture_rows_kernel<ES_IN, OUT, SUMM, SRC, LOOSE, true>), g, 0, s, d, b);
            return hipGetLastError();
        }
    }
    DMI_LAUNCH_CAPTURE(a.step != nullptr, (capture_rows_kernel<ES_IN, OUT, SUMM, SRC, LOOSE, false>), g, 0, s, d, b);
    return hipGetLastError();
}

template <int ES_IN, int VEC, int OUT, bool LOOSE, typename SRC>
static hipError_t launch_t(const CaptureArgs &a, const SRC &b, uint32_t grid, hipStream_t s)
{
    const dim3 g(grid, a.n_batch);
    const CaptureKernelArgs &k = a;
    if (VEC == 1 && a.units_per_row >= kThreads) return hipErrorInvalidValue;   // rows go by elements only if they are short
    if (a.summary_mask && a.row_lanes <= 64u && !(a.step_per_wave && !a.force_drop)) {
        if constexpr (OUT == OUT_NONE && VEC > 1 && !LOOSE) {
            if (a.read_once) {
                DMI_LAUNCH_CAPTURE(a.step != nullptr, (capture_kernel<ES_IN, VEC, OUT, SUMM_SHORT_ONCE, SRC, LOOSE>), g, a.lds_bytes, s, k, b);
                return hipGetLastError();
            }
        }
        DMI_LAUNCH_CAPTURE(a.step != nullptr, (capture_kernel<ES_IN, VEC, OUT, SUMM_SHORT, SRC, LOOSE>), g, a.lds_bytes, s, k, b);
    } else if (a.summary_mask) {
        if constexpr (VEC > 1) {
            if (a.step_per_wave && !a.force_drop)
                return a.wave_rows ? launch_rows<ES_IN, OUT, 1, LOOSE>(a, b, grid, s) : launch_rows<ES_IN, OUT, 2, LOOSE>(a, b, grid, s);
            if (a.wave_rows && a.units_per_row > 1024u) return hipErrorInvalidValue;    // four units for each of 256 lanes
            if (a.wave_rows)
                DMI_LAUNCH_CAPTURE(a.step != nullptr, (capture_kernel<ES_IN, VEC, OUT, SUMM_WAVE, SRC, LOOSE>), g, a.lds_bytes, s, k, b);
            else
                DMI_LAUNCH_CAPTURE(a.step != nullptr, (capture_kernel<ES_IN, VEC, OUT, SUMM_ROWS, SRC, LOOSE>), g, a.lds_bytes, s, k, b);
        } else {
            return hipErrorInvalidValue;
        }
    } else if constexpr (OUT != OUT_NONE) {
        if constexpr (VEC > 1)
            if (a.step_per_wave && !a.force_drop) return launch_rows<ES_IN, OUT, 0, LOOSE>(a, b, grid, s);
        DMI_LAUNCH_CAPTURE(a.step != nullptr, (capture_kernel<ES_IN, VEC, OUT, ROWS_FLAT, SRC, LOOSE>), g, a.lds_bytes, s, k, b);
    }
    return hipGetLastError();
}

template <typename SRC>
static hipError_t launch_no_rows(const CaptureArgs &a, const SRC &b, uint32_t grid, hipStream_t s)
{
    const dim3 g(grid, a.n_batch);
    const CaptureKernelArgs &k = a;
    DMI_LAUNCH_CAPTURE(a.step != nullptr, (capture_kernel<2, 8, OUT_NONE, ROWS_FLAT, SRC, false>), g, a.lds_bytes, s, k, b);
    return hipGetLastError();
}

template <int ES_IN, int VEC, bool LOOSE, typename SRC>
static hipError_t launch_o(const CaptureArgs &a, const SRC &b, uint32_t grid, hipStream_t s)
{
    const bool raw = a.out_dtype == a.src_dtype;
    if (a.out_dtype == 0) {
        // (neither rows nor summaries: header and request table alone, whatever the source)
        if (!a.summary_mask) return launch_no_rows(a, b, grid, s);
        return launch_t<ES_IN, VEC, OUT_NONE, LOOSE>(a, b, grid, s);
    }
    if (raw) return launch_t<ES_IN, VEC, OUT_RAW, LOOSE>(a, b, grid, s);
    if constexpr (ES_IN == 2) {
        if (a.out_dtype == 2) return launch_t<ES_IN, VEC, OUT_FP16, LOOSE>(a, b, grid, s);
        if (a.out_dtype == 4) return launch_t<ES_IN, VEC, OUT_FP8, LOOSE>(a, b, grid, s);
    }
    return hipErrorInvalidValue;
}

template <typename SRC>
static hipError_t launch_any(const CaptureArgs &a, const SRC &b, uint32_t grid, bool vec16, hipStream_t s)
{
    if (grid == 0 || grid > kMaxGrid || a.n_batch == 0 || a.n_batch > kMaxBatch) return hipErrorInvalidValue;
    const bool four = a.src_dtype == 3;
    if (!vec16 && a.loose) return four ? launch_o<4, 4, true>(a, b, grid, s) : launch_o<2, 8, true>(a, b, grid, s);
    if (four) return vec16 ? launch_o<4, 4, false>(a, b, grid, s) : launch_o<4, 1, false>(a, b, grid, s);
    return vec16 ? launch_o<2, 8, false>(a, b, grid, s) : launch_o<2, 1, false>(a, b, grid, s);
}

hipError_t launch_capture(const CaptureArgs &a, const BatchArgs &b, uint32_t grid, bool vec16, hipStream_t s)
{
    return launch_any(a, b, grid, vec16, s);
}

template <int OUT, typename SRC>
static hipError_t launch_decode_t(const DecodeArgs &d, const SRC &b, uint32_t n_batch, bool summaries, hipStream_t s)
{
    const dim3 grid(d.n_wg_rows + 1u, n_batch);
    if (d.keep_mask) {
        if (summaries)
            DMI_LAUNCH_CAPTURE(d.step != nullptr, (capture_decode_kernel<OUT, true, true, SRC>), grid, 0, s, d, b);
        else
            DMI_LAUNCH_CAPTURE(d.step != nullptr, (capture_decode_kernel<OUT, false, true, SRC>), grid, 0, s, d, b);
    } else {
        if (summaries)
            DMI_LAUNCH_CAPTURE(d.step != nullptr, (capture_decode_kernel<OUT, true, false, SRC>), grid, 0, s, d, b);
        else
            DMI_LAUNCH_CAPTURE(d.step != nullptr, (capture_decode_kernel<OUT, false, false, SRC>), grid, 0, s, d, b);
    }
    return hipGetLastError();
}

template <typename SRC>
static hipError_t launch_decode_any(const CaptureArgs &a, const SRC &b, hipStream_t s)
{
    if (a.n_src_rows < 0 || a.n_src_rows > 0xFFFFFFFFll) return hipErrorInvalidValue;
    if (a.n_batch == 0 || a.n_batch > kMaxBatch) return hipErrorInvalidValue;
    DecodeArgs d;
    std::memset(&d, 0, sizeof d);
    d.row_stride_b = a.row_stride_b;
    d.rows = a.row_index ? a.row_index : reinterpret_cast<const int32_t *>(a.row_map ? a.row_map : a.row0);
    d.n_wg_rows = a.hdr[9];         // rows listed
    d.unit_stride = a.row_lanes ? a.row_lanes : kThreads;
    d.ring = a.ring;
    d.cap = a.cap;
    d.ctrl = a.ctrl;
    d.step = a.step;
    d.tail_floor = a.tail_floor;
    d.record_bytes = a.record_bytes;
    d.off_payload = a.off_payload;
    d.off_sum = a.off_sum;
    d.sum_arr = a.sum_arr;
    d.n_src_rows = (uint32_t)a.n_src_rows;
    d.n_reqs = a.n_reqs;
    d.units_per_row = a.units_per_row;
    d.row_first = a.row_first;
    d.flags = (a.drop_newest ? kDecDropNewest : 0u) | (a.rows_consecutive ? kDecConsecutive : 0u) |
              (a.row_index ? kDecIndexed : 0u) | (a.par_in ? kDecParIn : 0u) | (a.row_map ? kDecRowMap : 0u);
    d.node = a.node;
    if constexpr (std::is_same<SRC, IntoArgs>::value) d.rows_at = b.n_words & kByColumn ? b.rows_at : (a.row_map ? 5u : 4u) * a.n_reqs;
    d.summary_mask = a.summary_mask;
    d.row_elems = a.row_elems;
    d.seq = a.seq;
    d.step_id = a.step_id;
    d.req_table = a.req_table;
    d.cslot = a.cslot;
    d.payload_bytes = a.payload_bytes;
    d.hdr7 = a.hdr[7];
    d.rank_tag = a.rank_tag;
    d.tail_src = a.tail_src;
    d.note = a.note;
    d.keep_mask = a.keep_mask;
    if (a.keep_mask && a.n_reqs > 1024u) return hipErrorInvalidValue;
    const bool summ = a.summary_mask != 0;
    if (a.out_dtype == a.src_dtype) return launch_decode_t<OUT_RAW>(d, b, a.n_batch, summ, s);
    switch (a.out_dtype) {
    case 0: return launch_decode_t<OUT_NONE>(d, b, a.n_batch, summ, s);
    case 2: return launch_decode_t<OUT_FP16>(d, b, a.n_batch, summ, s);
    case 4: return launch_decode_t<OUT_FP8>(d, b, a.n_batch, summ, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_capture_decode(const CaptureArgs &a, const BatchArgs &b, hipStream_t s)
{
    return launch_decode_any(a, b, s);
}

hipError_t launch_capture_into(const CaptureArgs &a, const IntoArgs &b, bool decode, uint32_t grid, bool vec16,
                               hipStream_t s)
{
    if (a.n_batch != 1u || a.step) return hipErrorInvalidValue;
    return decode ? launch_decode_any(a, b, s) : launch_any(a, b, grid, vec16, s);
}

template <uint32_t N>
static hipError_t launch_upload_chunk(uint32_t *dst, const uint32_t *words, uint32_t n, hipStream_t s)
{
    UploadChunk<N> c;
    std::memcpy(c.w, words, n * 4u);
    hipLaunchKernelGGL((upload_kernel<N>), dim3(1), dim3(kThreads), 0, s, dst, c, n);
    return hipGetLastError();
}

hipError_t launch_upload(uint32_t *dst, const uint32_t *words, uint32_t n_words, hipStream_t s)
{
    for (uint32_t o = 0; o < n_words;) {
        const uint32_t left = n_words - o, n = left < 3072u ? left : 3072u;
        const hipError_t e = n <= 896u ? launch_upload_chunk<896>(dst + o, words + o, n, s)
                                       : launch_upload_chunk<3072>(dst + o, words + o, n, s);
        if (e != hipSuccess) return e;
        o += n;
    }
    return hipSuccess;
}

hipError_t launch_fetch_slot(const CommitSlot *src, CommitSlot *dst_host, hipStream_t s)
{
    hipLaunchKernelGGL(fetch_slot_kernel, dim3(1), dim3(64), 0, s, src, dst_host);
    return hipGetLastError();
}

hipError_t launch_step_begin(DevCtrl *ctrl, StepParams *step, StepParams v, uint32_t par_from, uint32_t par_to,
                             const uint64_t *host_tail, hipStream_t s)
{
    hipLaunchKernelGGL(step_begin_kernel, dim3(1), dim3(64), 0, s, ctrl, step, v, par_from, par_to, host_tail);
    return hipGetLastError();
}

hipError_t launch_drain_kernel(const uint8_t *ring, uint64_t cap, uint8_t *host_ring, uint64_t host_cap,
                               uint64_t from, uint64_t nbytes, uint32_t grid, uint64_t *done, uint64_t tick, hipStream_t s)
{
    if (grid == 0 || grid > kDrainGroups || nbytes > cap || nbytes > host_cap || (from | nbytes | cap | host_cap) % 64u) return hipErrorInvalidValue;
    do {
        DrainSpans d;
        std::memset(&d, 0, sizeof d);
        const uint64_t n = drain_spans(ring, cap, host_ring, host_cap, from, nbytes, d);
        from += n;
        nbytes -= n;
        hipLaunchKernelGGL(drain_kernel, dim3(grid), dim3(kThreads), 0, s, d, nbytes ? nullptr : done, tick);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    } while (nbytes);
    return hipSuccess;
}

}  // namespace dmi
