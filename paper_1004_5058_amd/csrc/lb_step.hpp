// Device code shared by the step kernels (lb_kernels.hip: any tau; lb_unit.hip:
// tau = 1): storage formats, raw buffer access, the populations of one site,
// the pseudo-potential, wave sums and the order of the tiles.  Internal to the
// HIP library.
#pragma once
#include "lb_device.hpp"
#include "lb_kernels.hpp"
#include <type_traits>

namespace lbk {

// ---------------------------------------------------------------- storage --

// Every format stores the deviation d_is = f_is - w_i rho_ref_s of a population
// from the rest equilibrium at the lattice's reference densities; arithmetic
// is FP64 for FP64 storage and FP32 otherwise.  fast_psi: the pseudo-potential
// from the hardware 2^x instead of expm1 (see dpsi).
struct StF64 { using S = double;   using C = double; static constexpr bool fast_psi = false; };
struct StF32 { using S = float;    using C = float;  static constexpr bool fast_psi = false; };
struct StF16 { using S = _Float16; using C = float;  static constexpr bool fast_psi = true; };
struct StBF16 { using S = __bf16;  using C = float;  static constexpr bool fast_psi = true; };
// The moment form (tau = 1), FP32 and FP64.
struct MomF32 { using S = float;  using C = float;  static constexpr bool fast_psi = true; };
struct MomF64 { using S = double; using C = double; static constexpr bool fast_psi = false; };

template <class C> struct V4;
template <> struct V4<float> { using T = float4; };
template <> struct V4<double> { using T = double4; };

// Raw buffer access.  A block addresses each species' plane stack through a
// buffer resource: the per-lane column byte offset is the VGPR offset and the
// uniform (direction, row) byte offset is the SGPR offset, so the 18 loads and
// 18 stores of a row need no 64-bit address arithmetic.
using rsrc_t = __amdgpu_buffer_rsrc_t;
constexpr int RSRC_WORD3 = 0x00020000;

__device__ __forceinline__ rsrc_t make_rsrc(const void* p, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, RSRC_WORD3);
}

template <class S> __device__ __forceinline__ S bload(rsrc_t r, unsigned voff, unsigned soff);
template <> __device__ __forceinline__ float bload<float>(rsrc_t r, unsigned voff, unsigned soff)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, (int)soff, 0));
}
template <> __device__ __forceinline__ double bload<double>(rsrc_t r, unsigned voff, unsigned soff)
{
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(double, (u2)__builtin_amdgcn_raw_buffer_load_b64(r, voff, (int)soff, 0));
}
template <> __device__ __forceinline__ _Float16 bload<_Float16>(rsrc_t r, unsigned voff, unsigned soff)
{
    return __builtin_bit_cast(_Float16, __builtin_amdgcn_raw_buffer_load_b16(r, voff, (int)soff, 0));
}
template <> __device__ __forceinline__ __bf16 bload<__bf16>(rsrc_t r, unsigned voff, unsigned soff)
{
    return __builtin_bit_cast(__bf16, __builtin_amdgcn_raw_buffer_load_b16(r, voff, (int)soff, 0));
}

// Buffer store of one value; CP is the instruction's cache policy (0: default,
// CP_NT: non-temporal).
constexpr int CP_NT = 2;
template <class S, int CP = 0> __device__ __forceinline__ void bstore(S v, rsrc_t r, unsigned voff, unsigned soff)
{
    if constexpr (std::is_same<S, float>::value) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, voff, (int)soff, CP);
    } else if constexpr (std::is_same<S, double>::value) {
        typedef unsigned u2 __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), r, voff, (int)soff, CP);
    } else {
        static_assert(sizeof(S) == 2, "2-, 4- and 8-byte values");
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, v), r, voff, (int)soff, CP);
    }
}

// Load / store one deviation, converting between the storage and the
// arithmetic type (round to nearest even on the way down).  The SGPR offset is
// uniform by construction; readfirstlane states it, so a store under a
// divergent branch does not become a per-lane loop.
template <class P>
__device__ __forceinline__ typename P::C ld(rsrc_t r, unsigned voff, unsigned soff)
{
    return (typename P::C)bload<typename P::S>(r, voff, __builtin_amdgcn_readfirstlane(soff));
}

template <class P>
__device__ __forceinline__ void st(rsrc_t r, unsigned voff, unsigned soff, typename P::C v)
{
    bstore<typename P::S>((typename P::S)v, r, voff, (unsigned)__builtin_amdgcn_readfirstlane((int)soff));
}
template <class P, int CP = 0>
__device__ __forceinline__ void st_s(rsrc_t r, unsigned voff, unsigned soff, typename P::S v)
{
    bstore<typename P::S, CP>(v, r, voff, (unsigned)__builtin_amdgcn_readfirstlane((int)soff));
}

// A value of the arithmetic type, rounded to the storage format on its own:
// the value is first rounded to the arithmetic type, so the compiler cannot
// fuse the conversion into the multiply-add that produced it (for FP16 that
// fusion, v_fma_mixlo_f16, rounds once and can differ in the last bit; which
// stores it fuses would otherwise depend on the code around them).
template <class S, class C>
__device__ __forceinline__ S to_store(C x)
{
    if constexpr (std::is_same<S, C>::value) {
        return x;
    } else {
        asm("" : "+v"(x));
        return (S)x;
    }
}

// Two values of the arithmetic type rounded to the storage format on their own
// (FP16 as to_store, BF16 as the plain conversion).  16-bit storage from FP32:
// one packed conversion, which rounds each half as the single conversion does.
template <class S, class C>
__device__ __forceinline__ void to_store2(C a, C b, S& sa, S& sb)
{
    if constexpr (sizeof(S) == 2 && std::is_same<C, float>::value) {
        typedef float f2 __attribute__((ext_vector_type(2)));
        typedef S s2 __attribute__((ext_vector_type(2)));
        if constexpr (std::is_same<S, _Float16>::value) {
            asm("" : "+v"(a));
            asm("" : "+v"(b));
        }
        const s2 h = __builtin_convertvector((f2){a, b}, s2);
        sa = h.x;
        sb = h.y;
    } else {
        sa = to_store<S>(a);
        sb = to_store<S>(b);
    }
}

// The 18 populations of one site held in registers between the row load and
// the collision: the arithmetic type for 32/64-bit storage; for 16-bit storage
// the raw values, two per VGPR (d16 loads fill the low and high halves), and
// converted when read.  Besides single values a row gives the sums the
// collision needs, in one fixed order (left to right): the species densities
// (dens), the momentum (mom), the deviation f_q - x of one population from a
// value (dev), and the post-collision value f_q - w t in the storage format,
// rounded from its FP32 value (post).
template <class P, bool PACK = (sizeof(typename P::S) == 2)> struct Row;

// The sums in the arithmetic type, through the row's operator[].
template <class R, class C>
__device__ __forceinline__ void row_dens(const R& f, C& da, C& db)
{
    da = f[0];
    db = f[9];
#pragma unroll
    for (int q = 1; q < 9; ++q) { da += f[q]; db += f[9 + q]; }
}
template <class R, class C>
__device__ __forceinline__ void row_mom(const R& f, C& jx, C& jy)
{
    jx = (f[1] - f[3] + f[5] - f[6] - f[7] + f[8]) + (f[10] - f[12] + f[14] - f[15] - f[16] + f[17]);
    jy = (f[2] - f[4] + f[5] + f[6] - f[7] - f[8]) + (f[11] - f[13] + f[14] + f[15] - f[16] - f[17]);
}

// FP16 halves enter FP32 sums through the mixed-precision multiply-add
// v_fma_mix_f32 (an operand may be the low or high FP16 half of a VGPR): the
// widening is exact and a*1 + c rounds once, so each step equals the FP32 add
// of the converted value bit for bit, without the conversion instruction.
// mix_acc: x + s h, mix_pair: a + s b, mix_dev: h - x (s = +1 or -1; h, a, b
// the halves H, HA, HB of the packed pairs; a single value in a register of its
// own is half 0).
template <int H, bool NEG, class T>
__device__ __forceinline__ float mix_acc(T p, float x)
{
    float r;
    if constexpr (NEG && H)
        asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(p), "v"(x));
    else if constexpr (NEG)
        asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(p), "v"(x));
    else if constexpr (H)
        asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(p), "v"(x));
    else
        asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(p), "v"(x));
    return r;
}
template <int HA, int HB, bool NEG, class T>
__device__ __forceinline__ float mix_pair(T a, T b)
{
    float r;
    if constexpr (NEG)
        asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[%c3,0,%c4] op_sel_hi:[1,0,1]"
            : "=v"(r) : "v"(b), "v"(a), "n"(HB), "n"(HA));
    else
        asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[%c3,0,%c4] op_sel_hi:[1,0,1]"
            : "=v"(r) : "v"(b), "v"(a), "n"(HB), "n"(HA));
    return r;
}
template <int H>
__device__ __forceinline__ float mix_dev(unsigned p, float x)
{
    float r;
    if constexpr (H)
        asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(p), "v"(x));
    else
        asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(p), "v"(x));
    return r;
}

template <class P> struct Row<P, false> {
    using C = typename P::C;
    C v[18];
    __device__ __forceinline__ C operator[](int q) const { return v[q]; }
    __device__ __forceinline__ void dens(C& da, C& db) const { row_dens(*this, da, db); }
    __device__ __forceinline__ void mom(C& jx, C& jy) const { row_mom(*this, jx, jy); }
    __device__ __forceinline__ C dev(int q, C x) const { return v[q] - x; }
    __device__ __forceinline__ C post(int q, C w, C t) const { return v[q] - w * t; }   // S = C
    // f_QA + f_QB (NEG: f_QA - f_QB) and x + f_Q (NEG: x - f_Q)
    template <int QA, int QB, bool NEG = false> __device__ __forceinline__ C two() const
    {
        return NEG ? v[QA] - v[QB] : v[QA] + v[QB];
    }
    template <int Q, bool NEG = false> __device__ __forceinline__ C more(C x) const
    {
        return NEG ? x - v[Q] : x + v[Q];
    }
    // the 18 post-collision values of a site (species A's nine, then B's)
    __device__ __forceinline__ void set(const C (&a)[9], const C (&b)[9])
    {
#pragma unroll
        for (int i = 0; i < 9; ++i) { v[i] = a[i]; v[9 + i] = b[i]; }
    }
    // Planes are stored shifted in x by c_ix: population q of the lane's node
    // sits one column left (c_ix = +1: vl), in place (vc) or one column right
    // (c_ix = -1: vr).  so: uniform SGPR byte offset; v*: per-lane byte offsets.
    __device__ __forceinline__ void load(rsrc_t r0, rsrc_t r1, unsigned vl, unsigned vc, unsigned vr, unsigned so,
                                         unsigned pbytes)
    {
#pragma unroll
        for (int q = 0; q < 18; ++q) {
            const int cx = CX[q % 9];
            v[q] = ld<P>(q < 9 ? r0 : r1, cx > 0 ? vl : (cx < 0 ? vr : vc), so + (q % 9) * pbytes);
        }
    }
};

template <class P> struct Row<P, true> {
    using S = typename P::S;
    typedef S S2 __attribute__((ext_vector_type(2)));
    S2 v[9];
    static constexpr bool MIX = std::is_same<S, _Float16>::value;
    __device__ __forceinline__ float operator[](int q) const
    {
        return (float)((q & 1) ? v[q >> 1].y : v[q >> 1].x);
    }
    template <int Q> __device__ __forceinline__ unsigned u() const { return __builtin_bit_cast(unsigned, v[Q >> 1]); }
    template <int Q, bool NEG> __device__ __forceinline__ float acc(float x) const
    {
        return mix_acc<Q & 1, NEG>(u<Q>(), x);
    }
    template <int QA, int QB, bool NEG> __device__ __forceinline__ float pair() const
    {
        return mix_pair<QA & 1, QB & 1, NEG>(u<QA>(), u<QB>());
    }
    __device__ __forceinline__ void dens(float& da, float& db) const
    {
        if constexpr (MIX) {
            da = acc<8, false>(acc<7, false>(acc<6, false>(acc<5, false>(
                acc<4, false>(acc<3, false>(acc<2, false>(pair<0, 1, false>())))))));
            db = acc<17, false>(acc<16, false>(acc<15, false>(acc<14, false>(
                acc<13, false>(acc<12, false>(acc<11, false>(pair<9, 10, false>())))))));
        } else {
            row_dens(*this, da, db);
        }
    }
    __device__ __forceinline__ void mom(float& jx, float& jy) const
    {
        if constexpr (MIX) {
            const float ax = acc<8, false>(acc<7, true>(acc<6, true>(acc<5, false>(pair<1, 3, true>()))));
            const float bx = acc<17, false>(acc<16, true>(acc<15, true>(acc<14, false>(pair<10, 12, true>()))));
            const float ay = acc<8, true>(acc<7, true>(acc<6, false>(acc<5, false>(pair<2, 4, true>()))));
            const float by = acc<17, true>(acc<16, true>(acc<15, false>(acc<14, false>(pair<11, 13, true>()))));
            jx = ax + bx;
            jy = ay + by;
        } else {
            row_mom(*this, jx, jy);
        }
    }
    __device__ __forceinline__ float dev(int q, float x) const
    {
        if constexpr (MIX) {
            const unsigned p = __builtin_bit_cast(unsigned, v[q >> 1]);
            return (q & 1) ? mix_dev<1>(p, x) : mix_dev<0>(p, x);
        } else {
            return (*this)[q] - x;
        }
    }
    // the FP32 value rounded to the storage format (FP16 through to_store:
    // the compiler would otherwise fuse the conversion into the multiply-add
    // at some stores and not at others; BF16 has no such fusion)
    __device__ __forceinline__ S post(int q, float w, float t) const
    {
        if constexpr (MIX) return to_store<S>((*this)[q] - w * t);
        else return (S)((*this)[q] - w * t);
    }
    __device__ __forceinline__ void load(rsrc_t r0, rsrc_t r1, unsigned vl, unsigned vc, unsigned vr, unsigned so,
                                         unsigned pbytes)
    {
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            const int q0 = 2 * k, q1 = 2 * k + 1;
            const int c0 = CX[q0 % 9], c1 = CX[q1 % 9];
            v[k].x = bload<S>(q0 < 9 ? r0 : r1, c0 > 0 ? vl : (c0 < 0 ? vr : vc),
                              (unsigned)__builtin_amdgcn_readfirstlane((int)(so + (q0 % 9) * pbytes)));
            v[k].y = bload<S>(q1 < 9 ? r0 : r1, c1 > 0 ? vl : (c1 < 0 ? vr : vc),
                              (unsigned)__builtin_amdgcn_readfirstlane((int)(so + (q1 % 9) * pbytes)));
        }
    }
};

// Deviation of the pseudo-potential from its value at the reference density:
// psi(rho_ref + d) - psi(rho_ref) = -E expm1(-d/rho0), E = rho0 exp(-rho_ref/rho0),
// to the library's 1 ulp.  (A polynomial of 15 operations for its 25 ran 4096^2 FP32 in
// pairs 3 % faster; it was off by up to 1.5 ulp and gave NaN at infinities.)
__host__ __device__ __forceinline__ float dpsi_of(float d, float e, float inv_rho0)
{
    return -e * expm1f(-d * inv_rho0);
}
__device__ __forceinline__ double dpsi_of(double d, double e, double inv_rho0)
{
    return -e * expm1(-d * inv_rho0);
}
// The same deviation as E (1 - 2^(-d log2(e) / rho0)) with the hardware
// base-2 exponential (one transcendental and two multiply-adds instead of the
// ~24 instructions of expm1f).  Its absolute error is a few 1e-8 of E: far
// below the storage rounding of the 16-bit forms, about one FP32 rounding of
// the populations per step in the FP32 moment form.  The forms whose step is
// bound by arithmetic use it (fast_psi); FP32 and FP64 population storage
// keep expm1.
template <class P>
__device__ __forceinline__ typename P::C dpsi(typename P::C d, typename P::C e, typename P::C inv_rho0)
{
    if constexpr (P::fast_psi) {
        const float t = __builtin_amdgcn_exp2f(d * (-1.4426950408889634f * inv_rho0));
        return e - e * t;
    } else {
        return dpsi_of(d, e, inv_rho0);
    }
}

// Reciprocal: the hardware approximation (<= 1 ulp) in FP32, exact division in FP64.
__device__ __forceinline__ float rcp(float v) { return __builtin_amdgcn_rcpf(v); }
__device__ __forceinline__ double rcp(double v) { return 1.0 / v; }

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// A 32-bit lane move by DPP control CTRL applied to both halves of an FP64
// value (all 64 lanes active).
template <int CTRL>
__device__ __forceinline__ double dpp_move(double x)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
    const unsigned lo = __builtin_amdgcn_update_dpp(0u, (unsigned)b, CTRL, 0xF, 0xF, false);
    const unsigned hi = __builtin_amdgcn_update_dpp(0u, (unsigned)(b >> 32), CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// The wave-wide sums of two vectors at once (FP64, all 64 lanes active),
// without the LDS crossbar: the sum of d0 ends in lanes 0..31, of d1 in lanes
// 32..63.  The gfx950 row swap v_permlane32_swap exchanges the upper half of
// d0 with the lower half of d1, so one addition does the lane-distance-32
// step of both; v_permlane16_swap then pairs 16-lane rows; the rest is the
// xor butterfly over lane distances 1 and 2 (DPP quad permutations), then 4
// and 8 (the half-row and row mirrors: after the first steps every lane of a
// quad, then of an 8-lane group, holds the same value, so the mirror's
// partner holds what the xor partner holds).  About half the work of two
// separate wave sums.
__device__ __forceinline__ double wave_sum2_dpp(double d0, double d1)
{
    auto lo = [](double x) { return (unsigned)__builtin_bit_cast(unsigned long long, x); };
    auto hi = [](double x) { return (unsigned)(__builtin_bit_cast(unsigned long long, x) >> 32); };
    auto mk = [](unsigned l, unsigned h) { return __builtin_bit_cast(double, ((unsigned long long)h << 32) | l); };
    // first result: d0's lower half, then d1's lower half moved up; second:
    // d0's upper half moved down, then d1's upper half
    const auto l32 = __builtin_amdgcn_permlane32_swap(lo(d0), lo(d1), false, false);
    const auto h32 = __builtin_amdgcn_permlane32_swap(hi(d0), hi(d1), false, false);
    double v = mk(l32[0], h32[0]) + mk(l32[1], h32[1]);
    // with both operands v: the first result holds, in odd rows, the even row
    // below; the second, in even rows, the odd row above
    const auto l16 = __builtin_amdgcn_permlane16_swap(lo(v), lo(v), false, false);
    const auto h16 = __builtin_amdgcn_permlane16_swap(hi(v), hi(v), false, false);
    const bool odd = (__lane_id() >> 4) & 1;
    v += odd ? mk(l16[0], h16[0]) : mk(l16[1], h16[1]);
    v += dpp_move<0xB1>(v);    // quad_perm [1,0,3,2]: lane l^1
    v += dpp_move<0x4E>(v);    // quad_perm [2,3,0,1]: lane l^2
    v += dpp_move<0x141>(v);   // row_half_mirror: the other quad of the 8-lane group
    v += dpp_move<0x140>(v);   // row_mirror: the other 8-lane group of the 16-lane row
    return v;
}

// Work item l of a lattice with n tiles -> its tile.  Blocks go to the eight XCDs
// in turn (block b to XCD b mod 8), so items l, l + 8, l + 16, ... run on one XCD:
// they map to a band of contiguous tiles (numbered strip-fastest), so neighbouring
// tiles, which share halo rows and columns, share an XCD's L2.  A band has n / 8
// tiles, the first n mod 8 bands one more; the lattices' items follow each other
// without gaps, so a batch spreads over the XCDs to within one tile.  (Padding items
// that ended each lattice on a multiple of 8 took turns in the hand-out to the
// compute units: 252 tiles and 12 such items on 256 units left some with two tiles
// and ran 196 us against 118 for 216 taller tiles, three 2048 x 1024 FP32 lattices.)
__device__ __forceinline__ int xcd_tile(int l, int n)
{
    const int x = l & 7, q = n >> 3, r = n & 7;
    return x * q + (x < r ? x : r) + (l >> 3);
}

template <class P>
__device__ __forceinline__ int map_row(int r, int ny, int walls)
{
    if (walls) {
        if (r < 0) r = -1 - r;
        else if (r >= ny) r = 2 * ny - 1 - r;
    } else {
        r %= ny;
        if (r < 0) r += ny;
    }
    return r;
}

// ------------------------------------------------------------------ step ---

template <class C> struct V2;
template <> struct V2<float> { using T = float2; };
template <> struct V2<double> { using T = double2; };

// Workgroup barrier that orders LDS only: this wave's LDS reads and writes
// complete (lgkmcnt 0), then s_barrier.  Global loads issued before it stay in
// flight (the row prefetch), and so do direct-to-LDS halo loads: only the wave
// that issued those reads their data, behind its own vmcnt wait.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);   // gfx9 encoding: lgkmcnt(0), vmcnt/expcnt unchanged
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}
}  // namespace lbk
