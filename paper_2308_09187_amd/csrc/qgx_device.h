// Device-side helpers for the gfx950 kernels: the counter-based generator, wavefront scans and
// reductions, and small bit utilities.  64-wide wavefronts throughout.
#pragma once

#include "qgx_internal.h"

namespace qgx {

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & (kWave - 1)); }
// The same, worked out where it stands: no register holds it from the kernel's start until then.
__device__ __forceinline__ int late_lane_id()
{
    uint32_t all = 0xFFFFFFFFu;
    asm volatile("" : "+s"(all));
    return (int)__builtin_amdgcn_mbcnt_hi(all, __builtin_amdgcn_mbcnt_lo(all, 0u));
}
__device__ __forceinline__ int wave_id() { return (int)(threadIdx.x >> 6); }

// Philox4x32 with 10 rounds (Salmon, Moraes, Dror, Shaw, SC'11).  The key schedule is uniform
// across the wave, so the compiler keeps it in scalar registers; the two 32x32->64 products per
// round are the cost.  The two exclusive ors of a word are one three-operand instruction (coding 8 x 2^24
// coordinates 170 -> 163 us, with buckets of 1024 111 -> 105, the kernel that forms its own input 2.11 -> 2.07 ms).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return (uint32_t)__builtin_amdgcn_bitop3_b32((int)a, (int)b, (int)c, 0x96);
}

struct PhiloxKeys { uint32_t a[10], b[10]; };             // the keys of the ten rounds

__device__ __forceinline__ PhiloxKeys philox_keys(uint32_t k0, uint32_t k1)
{
    PhiloxKeys k;
#pragma unroll
    for (uint32_t r = 0; r < 10; ++r) { k.a[r] = k0 + r * 0x9E3779B9u; k.b[r] = k1 + r * 0xBB67AE85u; }
    return k;
}

__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              const PhiloxKeys& key, uint32_t (&out)[4])
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, key.a[r]);
        const uint32_t n2 = xor3((uint32_t)(p0 >> 32), c3, key.b[r]);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// Two standard normal draws from two words of a Philox block (Box-Muller): u1 = (2 (w >> 9) + 1) 2^-24 in
// (0, 1), u2 = (w' >> 8) 2^-24 in [0, 1), r = sqrt(-2 ln u1), (r cos 2 pi u2, r sin 2 pi u2).  Both
// uniforms are exact in binary32; logarithm, root, sine and cosine are the hardware's (v_log_f32 in base
// 2, v_sin_f32 and v_cos_f32 take their argument in turns), good to about 1e-6, which is ample for noise.
__device__ __forceinline__ float2 box_muller(uint32_t w_radius, uint32_t w_angle)
{
    // (1 + m 2^-23 less 1 - 2^-24, m = w >> 9: exact, and two instructions where a conversion of 2 m + 1 takes four)
    const float u1 = __uint_as_float(__builtin_amdgcn_alignbit(0x7Fu, w_radius, 9)) - 0x1.fffffep-1f;
    const float u2 = (float)(w_angle >> 8) * 0x1p-24f;
    const float r = __builtin_amdgcn_sqrtf(-1.3862943611198906f * __builtin_amdgcn_logf(u1));   // -2 ln 2 * log2 u1
    return make_float2(r * __builtin_amdgcn_cosf(u2), r * __builtin_amdgcn_sinf(u2));
}

// Between two phases in which the lanes of a wave exchange data through LDS without a workgroup barrier.
// The hardware runs a wave's LDS instructions in the order they were issued; this keeps the compiler from
// moving them across the boundary, or from making one side of the exchange part of a branch that only
// some lanes take.  No instruction is emitted.
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Inclusive prefix sum over the 64 lanes of a wave with DPP row shifts and row broadcasts: four
// shifted adds inside each row of 16 lanes, then lane 15 of a row into the next row, then lane 31
// into the upper half.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);   // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);   // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);   // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);   // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);   // row_bcast:15 -> rows 1,3
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);   // row_bcast:31 -> rows 2,3
    return x;
}

// The value of the lane before; lane 0 gets `first`.
__device__ __forceinline__ uint32_t wave_shift_in(uint32_t x, uint32_t first)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)first, (int)x, 0x138, 0xf, 0xf, false);   // wave_shr:1
}

// x of lane (i xor D), for a value that is already the same in all lanes that differ in bits above D only; these steps never
// leave the vector registers.  (A shuffle through LDS takes some 130 clocks, and a wave's binary64 sum needs twelve.)
template <int D>
__device__ __forceinline__ uint32_t xor_lane(uint32_t x)
{
    constexpr int ctrl = D == 8 ? 0x128 : D == 4 ? 0x124 : D == 2 ? 0x4E : 0xB1;   // row_ror:8, row_ror:4, quad_perm [2,3,0,1], [1,0,3,2]
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, ctrl, 0xf, 0xf, true);
}

struct LanePair { uint32_t a, b; };                        // the two values that lanes i and i xor D have, in both
template <int D>
__device__ __forceinline__ LanePair lane_pair(uint32_t x)
{
    if constexpr (D == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        return LanePair{(uint32_t)r[0], (uint32_t)r[1]};
    } else if constexpr (D == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        return LanePair{(uint32_t)r[0], (uint32_t)r[1]};
    } else {
        return LanePair{x, xor_lane<D>(x)};
    }
}

// The wave's sum, maximum and so on in every lane, lanes i and i xor 32, 16, 8, 4, 2, 1 joined in turn.
template <int D, typename Op>
__device__ __forceinline__ uint32_t wave_join_u32(uint32_t x, Op op)
{
    const LanePair p = lane_pair<D>(x);
    x = op(p.a, p.b);
    if constexpr (D > 1) return wave_join_u32<D / 2>(x, op);
    else return x;
}

template <int D = 32>
__device__ __forceinline__ double wave_sum(double x)
{
    const LanePair lo = lane_pair<D>((uint32_t)__double2loint(x)), hi = lane_pair<D>((uint32_t)__double2hiint(x));
    x = __hiloint2double((int)hi.a, (int)lo.a) + __hiloint2double((int)hi.b, (int)lo.b);
    if constexpr (D > 1) return wave_sum<D / 2>(x);
    else return x;
}

__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t x)
{
    return wave_join_u32<32>(x, [](uint32_t a, uint32_t b) { return a + b; });
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x)
{
    return wave_join_u32<32>(x, [](uint32_t a, uint32_t b) { return max(a, b); });
}

__device__ __forceinline__ float wave_max(float x)
{
    return __uint_as_float(wave_join_u32<32>(__float_as_uint(x), [](uint32_t a, uint32_t b) {
        return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b)));
    }));
}

__device__ __forceinline__ uint32_t wave_or(uint32_t x)
{
    return wave_join_u32<32>(x, [](uint32_t a, uint32_t b) { return a | b; });
}

// A 16-byte load of data that is read once: marked non-temporal, so that it does not push what is
// reused (the coded streams a later kernel reads back) out of the caches.
typedef float nt_f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 nt_load4(const float* p)
{
    const nt_f32x4 r = __builtin_nontemporal_load(reinterpret_cast<const nt_f32x4*>(p));
    return make_float4(r.x, r.y, r.z, r.w);
}

// An address that is the same in every lane of the wave, in scalar registers.
__device__ __forceinline__ uintptr_t uniform_address(const void* p)
{
    const uintptr_t x = reinterpret_cast<uintptr_t>(p);
    return ((uintptr_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32)) << 32) |
           (uintptr_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
}

typedef uint32_t nt_u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 nt_load4u(const uint4* p)
{
    const nt_u32x4 r = __builtin_nontemporal_load(reinterpret_cast<const nt_u32x4*>(p));
    return make_uint4(r.x, r.y, r.z, r.w);
}

typedef uint32_t lds_u32x2 __attribute__((ext_vector_type(2)));

// Memory as a buffer: a load from past its end gives zeros.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* first, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(uniform_address(first)), 0, (int)bytes, 0x00027000);
}

// A chunk's coordinates in registers: 16 rows of 256, four to a lane.  Its whole groups of four coordinates are a buffer, outside of
// which a load gives zeros (a row's place is part of the lane's offset, which the bounds apply to; the scalar one is not checked
// by what the compiler promises): no branch whatever the chunk's length, so that the compiler knows how many loads are under way.
// Vectors of an odd length put a worker's rows at any multiple of 4 bytes, which 16-byte loads take.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t chunk_rows(const float* first, uint32_t len)
{
    return buffer_of(first, (len & ~3u) * (uint32_t)sizeof(float));
}

__device__ __forceinline__ float4 load_row(__amdgpu_buffer_rsrc_t rows, int r, int lane)
{
    constexpr int kNonTemporal = 2;                          // (read once: see nt_load4)
    const nt_u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(rows, lane * 16 + r * 1024, 0, kNonTemporal);
    return make_float4(__uint_as_float(x.x), __uint_as_float(x.y), __uint_as_float(x.z), __uint_as_float(x.w));
}

__device__ __forceinline__ void load_rows(float4 (&v)[kRows], __amdgpu_buffer_rsrc_t rows, int lane)
{
#pragma unroll
    for (int r = 0; r < kRows; ++r) v[r] = load_row(rows, r, lane);
}

// The last one to three coordinates of a vector whose length is no multiple of four (only a worker's last chunk has such).
__device__ __forceinline__ void load_rest(float4 (&v)[kRows], const float* __restrict__ first, uint32_t len, int lane)
{
    if ((len & 3u) == 0u) return;
    const uint32_t at = len & ~3u;                           // (all wave-uniform)
    float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
    x.x = first[at];
    if ((len & 3u) > 1u) x.y = first[at + 1u];
    if ((len & 3u) > 2u) x.z = first[at + 2u];
#pragma unroll
    for (int r = 0; r < kRows; ++r)
        if (r == (int)(at >> 8) && (uint32_t)lane == (at & 255u) >> 2) v[r] = x;
}

// The largest magnitude of four and one; a NaN among them is the result (two instructions).
__device__ __forceinline__ float largest_of(const float4& x, float m)
{
    m = __builtin_elementwise_maximum(__builtin_elementwise_maximum(fabsf(x.x), fabsf(x.y)), m);
    return __builtin_elementwise_maximum(__builtin_elementwise_maximum(fabsf(x.z), fabsf(x.w)), m);
}

// Coordinates i0 .. i0 + 3 (i0 a multiple of 4) of F(z) = M z + b, from what they take.
struct GameOperands { float4 z, b; float2 a; };

__device__ __forceinline__ float4 game_operator_row(const GameArgs& G, const GameOperands& o)
{
    float4 f;
    f.x = (G.mu * o.z.x + o.a.x * o.z.y) + o.b.x;
    f.y = (G.mu * o.z.y - o.a.x * o.z.x) + o.b.y;
    f.z = (G.mu * o.z.z + o.a.y * o.z.w) + o.b.z;
    f.w = (G.mu * o.z.w - o.a.y * o.z.z) + o.b.w;
    return f;
}

__device__ __forceinline__ float4 game_operator_row(const GameArgs& G, uint32_t i0)
{
    return game_operator_row(G, GameOperands{*reinterpret_cast<const float4*>(G.z + i0), *reinterpret_cast<const float4*>(G.b + i0),
                                             *reinterpret_cast<const float2*>(G.a + (i0 >> 1))});
}

// A chunk's operands as buffers, zeros past its end (its length is a multiple of four).
struct GameRows { __amdgpu_buffer_rsrc_t z, b, a; };

__device__ __forceinline__ GameRows game_rows(const GameArgs& G, uint32_t first, uint32_t len)
{
    return GameRows{buffer_of(G.z + first, len * sizeof(float)), buffer_of(G.b + first, len * sizeof(float)),
                    buffer_of(G.a + (first >> 1), len / 2u * sizeof(float))};
}

__device__ __forceinline__ GameOperands load_game_operands(const GameRows& rows, int r, int lane)
{
    const nt_u32x4 z = __builtin_amdgcn_raw_buffer_load_b128(rows.z, lane * 16 + r * 1024, 0, 0);
    const nt_u32x4 b = __builtin_amdgcn_raw_buffer_load_b128(rows.b, lane * 16 + r * 1024, 0, 0);
    const lds_u32x2 a = __builtin_amdgcn_raw_buffer_load_b64(rows.a, lane * 8 + r * 512, 0, 0);
    auto f = [](uint32_t x) { return __uint_as_float(x); };
    return GameOperands{make_float4(f(z.x), f(z.y), f(z.z), f(z.w)), make_float4(f(b.x), f(b.y), f(b.z), f(b.w)), make_float2(f(a.x), f(a.y))};
}

// The same four coordinates of worker k's dual vector in call `call_id`: F(z) + sigma N, the noise from the
// Philox block with key (seed_lo, seed_hi) and counter (i0 / 4, 1, k, call_id).  F: game_operator_row.
__device__ __forceinline__ float4 game_noisy_row(const GameArgs& G, float4 F, uint32_t i0, uint32_t k, uint32_t call_id)
{
    uint32_t w[4];
    philox4x32_10(i0 >> 2, 1u, k, call_id, philox_keys(G.seed_lo, G.seed_hi), w);
    const float2 n01 = box_muller(w[0], w[1]), n23 = box_muller(w[2], w[3]);
    F.x += G.sigma * n01.x;
    F.y += G.sigma * n01.y;
    F.z += G.sigma * n23.x;
    F.w += G.sigma * n23.y;
    return F;
}

__device__ __forceinline__ float4 game_dual_row(const GameArgs& G, uint32_t i0, uint32_t k, uint32_t call_id)
{
    return game_noisy_row(G, game_operator_row(G, i0), i0, k, call_id);
}

// t^q for a small positive integer q (the same q in every lane).
__device__ __forceinline__ double pow_int(double t, uint32_t q)
{
    double r = 1.0;
    for (; q; q >>= 1) {
        if (q & 1u) r *= t;
        t *= t;
    }
    return r;
}

// s^(1/q) for s >= 1 in binary64: a single-precision guess, then Newton steps on x^q = s (each one
// squares the error, so three reach the last bits from a guess good to 1e-6).
__device__ __forceinline__ double root_int(double s, uint32_t q)
{
    double x = (double)__builtin_amdgcn_exp2f(__builtin_amdgcn_logf((float)s) / (float)q);   // v_exp_f32, v_log_f32: base 2
    for (int it = 0; it < 3; ++it) {
        const double xq1 = pow_int(x, q - 1u);
        x -= (xq1 * x - s) / ((double)q * xq1);
    }
    return x;
}

// A load through the scalar cache, of what an earlier launch wrote and this one only reads: no vector
// registers, and no wait on the vector loads in flight.
__device__ __forceinline__ uint32_t scalar_load(const void* p)
{
    return *reinterpret_cast<const __attribute__((address_space(4))) uint32_t*>(reinterpret_cast<uintptr_t>(p));
}

// LDS accesses by byte address.  A pointer derived from the dynamic LDS array carries the array's
// base as a late-bound addend that the compiler adds again on every access; an address computed once
// as an integer does not.
__device__ __forceinline__ uint32_t lds_address(const void* p)
{
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

typedef uint32_t lds_u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t lds_load_u32(uint32_t addr)
{
    return *(const __attribute__((address_space(3))) uint32_t*)(uintptr_t)addr;
}

__device__ __forceinline__ uint2 lds_load_u2(uint32_t addr)
{
    const lds_u32x2 r = *(const __attribute__((address_space(3))) lds_u32x2*)(uintptr_t)addr;
    return make_uint2(r.x, r.y);
}

__device__ __forceinline__ uint4 lds_load_u4(uint32_t addr)
{
    const lds_u32x4 r = *(const __attribute__((address_space(3))) lds_u32x4*)(uintptr_t)addr;
    return make_uint4(r.x, r.y, r.z, r.w);
}

__device__ __forceinline__ void raise_error(Scalars* sc, unsigned int bit)
{
    atomicOr(&sc->err, bit);
}

}  // namespace qgx
