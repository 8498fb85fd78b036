// psm_kernels.hip -- gfx950 kernels of the PSM-LBM hot path.
//
// Method: Kemmler et al., arXiv 2303.11811.
//   Sec. 2.1   D3Q19 SRT collision with forcing, eqs. (1)-(8)
//   Sec. 2.3   PSM collision, solid operator, particle velocity at the cell
//              centre, hydrodynamic force and torque, eqs. (17)-(22)
//   Sec. 2.3.2 linear-approximation solid fraction, eqs. (25)-(27)
//   Sec. 3.1   GPU time step: mapping -> PSM kernel -> force reduction
//
// Storage is pull-scheme: grid[p] holds the post-collision PDFs of the last
// step at their source cell, so a cell gathers f_q(x,t) = grid[p][q][x - c_q]
// (eq. 2 read backwards), collides, and writes grid[p^1][q][x] aligned.
// The paper's separate mapping / setU / redF kernels are fused into the
// stream-collide launch: each workgroup stages its tile's sphere candidates in
// LDS, maps solid fractions in registers, evaluates U_p(x) (eq. 20) on the fly
// and sums the per-sphere force/torque of its tile deterministically; the
// launch of the next step adds them per sphere.
#include "psm_internal.h"

#include <algorithm>
#include <mutex>

namespace psm {

// ---------------------------------------------------------------------------
// PDF access of the step kernel through buffer resources. A resource covers
// one z-plane of a grid (raw bytes, fewer than 2^31); every load or store
// takes the cell's byte offset inside the plane per lane and the run of its
// direction (q * 64 values) as a scalar offset, so that no per-access 64-bit
// address arithmetic runs on the vector ALU.
typedef __amdgpu_buffer_rsrc_t Rsrc;
typedef unsigned int u32x2 __attribute__((__vector_size__(8)));
constexpr int RSRC_WORD3 = 0x00020000;   // raw 32-bit data format, no swizzle

// Cache policy of the PDF streams (compile-time switches, measured by the
// tuning sweeps): nontemporal stores / loads bypass cache retention. The step
// kernel's KEEP instances store without it (grids that fit the caches), its
// STREAM instances also load so what no other wave reads.
#ifndef PSM_NT_STORE
#define PSM_NT_STORE 1
#endif
#ifndef PSM_NT_LOAD
#define PSM_NT_LOAD 0
#endif
constexpr int LD_AUX = PSM_NT_LOAD ? 2 : 0;
constexpr int ST_AUX = PSM_NT_STORE ? 2 : 0;

#ifndef PSM_BUFFER_IO
#define PSM_BUFFER_IO 1
#endif
#if PSM_BUFFER_IO
__device__ __forceinline__ Rsrc plane_rsrc(const void* base, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, RSRC_WORD3);
}
#define PSM_LD(B, T, r, vo, so, aux) __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_##B(r, vo, so, aux))
#define PSM_ST(B, U, v, r, vo, so, aux) __builtin_amdgcn_raw_buffer_store_##B(__builtin_bit_cast(U, v), r, vo, so, aux)
#else
// plain global accesses from the plane's base address (compile-time alternative)
typedef const char* RsrcPtr;
#define Rsrc RsrcPtr
__device__ __forceinline__ Rsrc plane_rsrc(const void* base, unsigned) { return (const char*)base; }
#define GLB __attribute__((address_space(1)))
#define PSM_LD(B, T, r, vo, so, aux) (*(const GLB T*)((r) + (so) + (vo)))
#define PSM_ST(B, U, v, r, vo, so, aux) __builtin_nontemporal_store(v, (GLB decltype(v)*)((r) + (so) + (vo)))
#endif

// ---------------------------------------------------------------------------
// Storage traits: FP64 stores f; the deviation forms store d = f - w_q
// (FP16 as scale * d) and compute in FP32.
struct St64 {
    using T = double;
    using R = double;
    static constexpr bool DEV = false;
    static constexpr bool SCALED = false;
    template <int AUX = LD_AUX> __device__ static R ld(Rsrc r, unsigned vo, int so) { return PSM_LD(b64, double, r, vo, so, AUX); }
    template <int AUX = ST_AUX> __device__ static void st(Rsrc r, unsigned vo, int so, R v) {
        PSM_ST(b64, u32x2, v, r, vo, so, AUX);
    }
    __device__ static double to_f64(T v, float) { return v; }
    __device__ static T from_f64(double v, float) { return v; }
};
struct St32 {
    using T = float;
    using R = float;
    static constexpr bool DEV = true;
    static constexpr bool SCALED = false;
    template <int AUX = LD_AUX> __device__ static R ld(Rsrc r, unsigned vo, int so) { return PSM_LD(b32, float, r, vo, so, AUX); }
    template <int AUX = ST_AUX> __device__ static void st(Rsrc r, unsigned vo, int so, R v) {
        PSM_ST(b32, unsigned int, v, r, vo, so, AUX);
    }
    __device__ static double to_f64(T v, float) { return (double)v; }
    __device__ static T from_f64(double v, float) { return (float)v; }
};
struct St16 {
    using T = _Float16;
    using R = float;
    static constexpr bool DEV = true;
    // The step kernel works on the stored scaled deviations s d directly (the
    // scale s is folded into the collision constants), so its loads and
    // stores are bare conversions. State I/O converts with the scale.
    static constexpr bool SCALED = true;
    template <int AUX = LD_AUX> __device__ static R ld(Rsrc r, unsigned vo, int so) { return (float)PSM_LD(b16, _Float16, r, vo, so, AUX); }
    template <int AUX = ST_AUX> __device__ static void st(Rsrc r, unsigned vo, int so, R v) {
        const _Float16 h = (_Float16)v;
        PSM_ST(b16, unsigned short, h, r, vo, so, AUX);
    }
    // scale is a power of two: multiplication by it and by 1/scale is exact
    __device__ static double to_f64(T v, float inv) { return (double)((float)v * inv); }
    // (rounded once: not by way of FP32)
    __device__ static T from_f64(double v, float scale) { return (_Float16)(v * (double)scale); }
};

// The box constant of the collision's precision R: the FP64 value or its
// FP32 copy (both set by the host).
template <class R> __device__ __forceinline__ R pick(double d, float f);
template <> __device__ __forceinline__ double pick<double>(double d, float) { return d; }
template <> __device__ __forceinline__ float pick<float>(double, float f) { return f; }

__device__ __forceinline__ float fmar(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmar(double a, double b, double c) { return __builtin_fma(a, b, c); }

// n / d for 0 <= n < 2^31 by the multiplier and shift of udiv_magic: scalar
// instructions, where a division goes through the vector ALU.
__device__ __forceinline__ int udiv(int n, unsigned mul, unsigned shift) {
    return mul ? (int)(__umulhi(mul, (unsigned)n) >> shift) : n;
}

__device__ inline double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// ---------------------------------------------------------------------------
// Cross-lane moves on the vector ALU. DPP forms stay inside a row of 16
// lanes: quad permutations, the mirror inside each half row (lane i <-> 7 - i
// of its group of 8) and the rotation of a row by 8 (lane i <-> i ^ 8).
// Across rows, the gfx950 swaps exchange odd with even rows (lanes i and
// i ^ 16) and the two halves of the wave (lanes i and i ^ 32): with both
// operands the same value v, the two results are v at the lower partner and
// v at the upper partner, so their sum is the pair sum, taken in the same
// order on both lanes.
template <int CTRL> __device__ __forceinline__ float dpp_f32(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
template <int CTRL> __device__ __forceinline__ double dpp_f64(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
constexpr int DPP_QUAD_XOR1 = 0xB1;         // quad_perm [1, 0, 3, 2]
constexpr int DPP_QUAD_XOR2 = 0x4E;         // quad_perm [2, 3, 0, 1]
constexpr int DPP_ROW_HALF_MIRROR = 0x141;
constexpr int DPP_ROW_ROR8 = 0x128;

__device__ __forceinline__ float pair_sum16(float v) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float pair_sum32(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ double join(unsigned lo, unsigned hi) {
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double pair_sum16(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const auto l = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    return join(l[0], h[0]) + join(l[1], h[1]);
}
__device__ __forceinline__ double pair_sum32(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const auto l = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    return join(l[0], h[0]) + join(l[1], h[1]);
}
template <int CTRL> __device__ __forceinline__ float dppv(float v) { return dpp_f32<CTRL>(v); }
template <int CTRL> __device__ __forceinline__ double dppv(double v) { return dpp_f64<CTRL>(v); }

// Wave sums of six values at once (V = float or double). Inside each group
// of 8 lanes a butterfly splits the values (padded to 8) between exchanging
// lanes: the mirror pair by bit 2 of the lane, then quad partners by bits 1
// and 0 (7 exchanges), after which lane l holds the group's sum of value
// l & 7; three exchanges across groups (row rotation by 8, the row swap, the
// half swap) finish the sums. Lane l returns the total of value l & 7
// (values 6 and 7 are padding). The order of the additions is fixed, so the
// result is reproducible bit for bit.
template <class V>
__device__ inline V wave_sum6(const V v[6], int lane) {
    const bool b2 = lane & 4, b1 = lane & 2, b0 = lane & 1;
    V a[4], b[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const V lo = v[i], hi = i + 4 < 6 ? v[i + 4] : (V)0;
        const V keep = b2 ? hi : lo, send = b2 ? lo : hi;
        a[i] = keep + dppv<DPP_ROW_HALF_MIRROR>(send);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const V keep = b1 ? a[i + 2] : a[i], send = b1 ? a[i] : a[i + 2];
        b[i] = keep + dppv<DPP_QUAD_XOR2>(send);
    }
    const V keep = b0 ? b[1] : b[0], send = b0 ? b[0] : b[1];
    V d = keep + dppv<DPP_QUAD_XOR1>(send);
    d += dppv<DPP_ROW_ROR8>(d);
    d = pair_sum16(d);
    return pair_sum32(d);
}

// Uniform (wave-invariant) data is read through the constant address space so
// that it lands in scalar registers.
#define PSM_CONST __attribute__((address_space(4)))
template <class T> __device__ __forceinline__ const PSM_CONST T* cptr(const T* p) {
    return (const PSM_CONST T*)p;
}

// ---------------------------------------------------------------------------
// Lattice products of direction Q with only its nonzero terms (D3Q19
// components are 0 or +-1; at most two are nonzero), in x, y, z order.
template <int C, class R> __device__ __forceinline__ R cterm(R v) { return C > 0 ? v : -v; }
template <class R, int Q> __device__ __forceinline__ R cdot(R x, R y, R z) {
    constexpr int a = CX[Q], b = CY[Q], c = CZ[Q];
    if constexpr (a != 0 && b != 0) return cterm<a>(x) + cterm<b>(y);
    else if constexpr (a != 0 && c != 0) return cterm<a>(x) + cterm<c>(z);
    else if constexpr (b != 0 && c != 0) return cterm<b>(y) + cterm<c>(z);
    else if constexpr (a != 0) return cterm<a>(x);
    else if constexpr (b != 0) return cterm<b>(y);
    else if constexpr (c != 0) return cterm<c>(z);
    else return (R)0;
}
// c.M.c for a symmetric M given as the diagonal (Mxx, Myy, Mzz) and the
// doubled off-diagonal terms (2 Mxy, 2 Mxz, 2 Myz).
template <class R, int Q>
__device__ __forceinline__ R cmc(R Mxx, R Myy, R Mzz, R Mxy2, R Mxz2, R Myz2) {
    constexpr int a = CX[Q], b = CY[Q], c = CZ[Q];
    if constexpr (a != 0 && b != 0) return (a * b > 0) ? (Mxx + Myy) + Mxy2 : (Mxx + Myy) - Mxy2;
    else if constexpr (a != 0 && c != 0) return (a * c > 0) ? (Mxx + Mzz) + Mxz2 : (Mxx + Mzz) - Mxz2;
    else if constexpr (b != 0 && c != 0) return (b * c > 0) ? (Myy + Mzz) + Myz2 : (Myy + Mzz) - Myz2;
    else if constexpr (a != 0) return Mxx;
    else if constexpr (b != 0) return Myy;
    else return Mzz;
}

// Per weight class W (axis or diagonal) of a cell: the terms of the SRT
// update with forcing (eqs. 3, 5, 8) that do not depend on the direction.
//   E_q(U) = W (base + k45 (c.U)^2) + 3 W (c.U) = s + a,  E_qbar(U) = s - a,
//   F_q = fa + fs (c.U) - pu,  F_qbar = -fa + fs (c.U) - pu,  base = rho - k15 U.U
template <class R>
struct WClass {
    R Wb;      // W base (per cell)
    R owb_pu;  // omega W base - pu (per cell)
    R Wk;      // W k45 (box constant)
    R W3;      // 3 W
    R owk;     // omega W k45 (box constant)
    R ow3;     // 3 omega W (box constant)
};

// One inverse pair (q, q+1) of the plain update f~ = f + omega (E - f) + F:
//   f~_q = (1 - omega) f_q + P + A,  f~_qbar = (1 - omega) f_qbar + P - A,
//   P = omega s + fs (c.U) - pu,  A = omega a + fa.
template <class R, int Q>
__device__ __forceinline__ void pair_fluid(R& fq, R& fb, R cu, const WClass<R>& w, R fa, R fs, R om1) {
    const R P = fmar(fs, cu, fmar(w.owk, cu * cu, w.owb_pu));
    const R A = fmar(w.ow3, cu, fa);
    fq = fmar(om1, fq, P + A);
    fb = fmar(om1, fb, P - A);
}

// The same pair under PSM (eqs. 17-19):
//   f~_q = f_q + (1-B) t_q + B (f_qbar - E_qbar(U) - f_q) + sum_s B_s E_q(V_s),
//   t_q = omega (E_q(U) - f_q) + F_q,
// with the slot sum folded into ten cell scalars:
//   sum_s B_s E_q(V_s) = W (A0 + k45 c.M.c) + 3 W c.P,
//   A0 = sum_s B_s (rho - k15 V_s.V_s), M = sum_s B_s V_s V_s^T, P = sum_s B_s V_s.
// Collected by parity in c_q, with alpha = 1 - (1-B) omega - B, beta = (1-B) omega - B
// and gamma = (1-B) omega + B (per cell):
//   f~_q    = alpha f_q + B f_qbar + Sym + Anti,  f~_qbar = alpha f_qbar + B f_q + Sym - Anti,
//   Sym  = [beta W base - (1-B) pu + W A0] + beta W k45 (c.U)^2 + (1-B) fs (c.U) + W k45 c.M.c,
//   Anti = gamma 3 W (c.U) + (1-B) fa + 3 W c.P,
// where the bracket (C1), beta W k45 (C2) and gamma 3 W (C3) are per weight class.
template <class R, int Q>
__device__ __forceinline__ void pair_psm(R& fq, R& fb, R cu, R C1, R C2, R C3, R Wk, R W3, R ofs, R ofa, R alpha,
                                         R Bt, R cM, R cP) {
    const R Sym = fmar(C2, cu * cu, fmar(ofs, cu, fmar(Wk, cM, C1)));
    const R Anti = fmar(C3, cu, fmar(W3, cP, ofa));
    const R nq = fmar(alpha, fq, fmar(Bt, fb, Sym + Anti));
    const R nb = fmar(alpha, fb, fmar(Bt, fq, Sym - Anti));
    fq = nq;
    fb = nb;
}

// Lever arm d = x - x_p (minimum image, taken in FP64) and particle velocity
// at the cell centre (eq. 20) in FP64 (FP64 storage).
__device__ __forceinline__ void slot_geometry64(int c, double cxc, double cyc, double czc, double Lx, double hLx,
                                                double Ly, double hLy, double Lz, double hLz, const double* px,
                                                const double* py, const double* pz, const double* ux,
                                                const double* uy, const double* uz, const double* ox,
                                                const double* oy, const double* oz, double& dx, double& dy,
                                                double& dz, double& Vx, double& Vy, double& Vz) {
    dx = min_image(cxc - px[c], Lx, hLx);
    dy = min_image(cyc - py[c], Ly, hLy);
    dz = min_image(czc - pz[c], Lz, hLz);
    Vx = ux[c] + (oy[c] * dz - oz[c] * dy);
    Vy = uy[c] + (oz[c] * dx - ox[c] * dz);
    Vz = uz[c] + (ox[c] * dy - oy[c] * dx);
}

// Minimum image in FP32 of a displacement that is within a few box lengths.
__device__ __forceinline__ float wrap32(float t, float L, float invL) { return fmar(-L, __builtin_rintf(t * invL), t); }

// Waves per SIMD the register budget of the step kernel is cut for: 3 for
// FP64 storage (168 VGPRs), 4 for the deviation forms (128 VGPRs), 5 for FP16
// (96 VGPRs) without sampling and filter, which would spill there: its vector
// ALU is busy two thirds of the time and hides more with more waves (256^3
// 284 -> 272 us, 384^3 870 -> 857 us). FP32 spills at 5 waves (512^3 3.67 ->
// 5.42 ms). Sampling keeps 16 squares beside the rest: at 4 waves 16 to 33
// registers of the deviation forms went to scratch memory, so it takes 3 (4^3
// points, FP32 256^3 896 -> 552 us, 128^3 119 -> 79, 32^3 11.2 -> 9.8; FP16 256^3
// 475 -> 459, 32^3 11.0 -> 9.9, 128^3 70.8 -> 71.0).
#ifndef PSM_WAVES_F64
#define PSM_WAVES_F64 3
#endif
#ifndef PSM_WAVES_DEV
#define PSM_WAVES_DEV 4
#endif
#ifndef PSM_WAVES_F16
#define PSM_WAVES_F16 5
#endif
#ifndef PSM_WAVES_MAP
#define PSM_WAVES_MAP 3
#endif
// Pull order of the step kernel (measured per storage form): the FP32 form
// pulls the next cell's values while it works on the current one; FP64 issues
// each cell's pulls before its mapping (not with the candidate filter, whose
// registers that would spill); FP16 pulls after the mapping (earlier or ahead
// was slower there). Contexts that sample pull after the mapping: its squares
// take the registers (FP64 128^3 141 -> 134 us).
#ifndef PSM_PREFETCH_F32
#define PSM_PREFETCH_F32 1
#endif
#ifndef PSM_PREFETCH_F16
#define PSM_PREFETCH_F16 0
#endif
#ifndef PSM_EARLY_PULLS_F64
#define PSM_EARLY_PULLS_F64 1
#endif
#ifndef PSM_EARLY_PULLS_F16
#define PSM_EARLY_PULLS_F16 0
#endif

// pull of the 19 values of one cell from the source planes z (rz), z-1 (rm)
// and z+1 (rp); direction q lies q * QB bytes into a block. The nine directions
// without an x component, whose lines no other wave reads, are loaded with
// cache policy AUX0.
#define PSM_LOAD19(F, rz, rm, rp, AUX0)                         \
    do {                                                        \
        F[0] = S::template ld<AUX0>(rz, o00, 0 * QB);           \
        F[1] = S::ld(rz, om0, 1 * QB);                          \
        F[2] = S::ld(rz, op0, 2 * QB);                          \
        F[3] = S::template ld<AUX0>(rz, o0m, 3 * QB);           \
        F[4] = S::template ld<AUX0>(rz, o0p, 4 * QB);           \
        F[5] = S::template ld<AUX0>(rm, o00, 5 * QB);           \
        F[6] = S::template ld<AUX0>(rp, o00, 6 * QB);           \
        F[7] = S::ld(rz, omm, 7 * QB);                          \
        F[8] = S::ld(rz, opp, 8 * QB);                          \
        F[9] = S::ld(rz, omp, 9 * QB);                          \
        F[10] = S::ld(rz, opm, 10 * QB);                        \
        F[11] = S::ld(rm, om0, 11 * QB);                        \
        F[12] = S::ld(rp, op0, 12 * QB);                        \
        F[13] = S::ld(rp, om0, 13 * QB);                        \
        F[14] = S::ld(rm, op0, 14 * QB);                        \
        F[15] = S::template ld<AUX0>(rm, o0m, 15 * QB);         \
        F[16] = S::template ld<AUX0>(rp, o0p, 16 * QB);         \
        F[17] = S::template ld<AUX0>(rp, o0m, 17 * QB);         \
        F[18] = S::template ld<AUX0>(rm, o0p, 18 * QB);         \
    } while (0)

__device__ inline void box_tiles(const BoxDev& bx, const TileShape& ts, double x, double y, double z, double r,
                                 AxisTiles& ax, AxisTiles& ay, AxisTiles& az) {
    int lo, hi;
    aabb_cells(x, r, lo, hi);
    ax = axis_tiles(lo, hi, bx.nx, ts.tx, bx.ntx);
    aabb_cells(y, r, lo, hi);
    ay = axis_tiles(lo, hi, bx.ny, ts.ty, bx.nty);
    aabb_cells(z, r, lo, hi);
    az = axis_tiles(lo, hi, bx.nz, ts.tz, bx.ntz);
}

// Force and torque of global sphere p from its tile partials, for the whole
// wave: lane l takes tiles l, l + 64, ... of the bounding box in a fixed order,
// then a fixed butterfly adds the lanes (the same bits on every lane).
__device__ __forceinline__ void reduce_sphere(const BoxDev& bx, const TileShape& ts, const Particles& P,
                                              const double* partial, int p, int lane, double acc[6]) {
#pragma unroll
    for (int c = 0; c < 6; ++c) acc[c] = 0.0;
    const int lp = p - bx.part_base;
    if (lp < bx.np) {
        AxisTiles ax, ay, az;
        box_tiles(bx, ts, P.x[p], P.y[p], P.z[p], P.r[p], ax, ay, az);
        const int ntot = ax.count() * ay.count() * az.count();
        // the sphere's slots: one run per tile of its bounding box, in that order
        const double* pp = partial + (((long long)bx.pbase + (long long)lp * bx.pstride) << ts.zshift) * 6;
        for (int k = lane; k < ntot << ts.zshift; k += 64) {
#pragma unroll
            for (int c = 0; c < 6; ++c) acc[c] += pp[(long long)k * 6 + c];
        }
    }
#pragma unroll
    for (int c = 0; c < 6; ++c) acc[c] = wave_sum(acc[c]);
}

// Byte offset of a cell inside a z-plane (direction 0): its block of 64 cells
// is NQ runs long. In-plane cells are below 2^24 (a plane holds fewer than
// 2^31 bytes in FP64), so the products are 24-bit ones.
template <class T> __device__ __forceinline__ unsigned cell_offset(int x, int y, int pitch) {
    const unsigned c = (unsigned)x + __umul24((unsigned)pitch, (unsigned)y);
    return __umul24(c & ~(unsigned)(BLK - 1), (NQ - 1) * (unsigned)sizeof(T)) + c * (unsigned)sizeof(T);
}

// The step kernel's arguments, read anew at each use of this function: held in
// scalar registers from the start of the kernel they are spilled lane by
// lane to vector registers and back (130 vector instructions per wave).
__device__ __forceinline__ const PSM_CONST StepParams* step_args() {
    const PSM_CONST StepParams* p = (const PSM_CONST StepParams*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}
__device__ __forceinline__ Particles particles(const PSM_CONST StepParams* a) {
    return Particles{a->P.x, a->P.y, a->P.z, a->P.r, a->P.fr, a->P.ux, a->P.uy, a->P.uz,
                     a->P.ox, a->P.oy, a->P.oz, a->P.acc, a->P.fprev, a->P.prev_ok};
}

// Bound by memory where the grids exceed the last-level cache: a copy with the
// same tiles, pulls and stores takes as long (512^3 FP64 7.05 ms a step, copy
// 7.05, at 5.8 of the 6.25 TB/s of a plain copy; FP32 3.66, FP16 2.00 against
// 1.92, its vector ALU busy two thirds of the time). In the cache by the latency
// of staging, pulls and mapping in sequence (FP64 64^3 18 us, copy 13), and below
// by that of one cell (32^3 7.7 us). Two or three workgroups per CU instead of
// three to five leave FP64 and FP32 unchanged there, FP16 slows by 4 and 20 %.
template <class S, int MAP, bool FILT, bool WALL, int CACHE>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(
    !S::DEV ? PSM_WAVES_F64 : (MAP != 0 ? PSM_WAVES_MAP : (S::SCALED && !FILT ? PSM_WAVES_F16 : PSM_WAVES_DEV)), 8))) void k_psm_step(
    StepParams) {
    using R = typename S::R;
    using T = typename S::T;
    const PSM_CONST StepParams* ka = step_args();

    __shared__ double s_px[MAXC], s_py[MAXC], s_pz[MAXC], s_pr[MAXC], s_pfr[MAXC];
    __shared__ double s_ux[MAXC], s_uy[MAXC], s_uz[MAXC], s_ox[MAXC], s_oy[MAXC], s_oz[MAXC];
    // FP32 copies: centre relative to the tile's reference point (minimum image), the
    // squared reach of the overlap test with a rounding margin, and (for the
    // deviation forms) the velocities
    __shared__ float s_qx[MAXC], s_qy[MAXC], s_qz[MAXC], s_lim2[MAXC], s_rf[MAXC], s_frf[MAXC];
    __shared__ float s_uf[6][MAXC];
    __shared__ int s_pid[MAXC], s_slot[MAXC];
    __shared__ double s_acc[NWAVE][6][MAXC];
    __shared__ unsigned long long s_cmask[NWAVE][TZ_MAX];

    const int tid = threadIdx.x;
    const int TX = ka->tx, TY = ka->ty, TZ = ka->depth;
    const int wave = tid >> 6, lane = tid & 63;

    if ((int)blockIdx.x >= ka->grid) {
        // the force reduction of the step before (k_spheres reduces the last
        // step of a call): in a launch of its own it takes 4.5 us behind every
        // step, a third of a 32^3 step. A wave per sphere the context has room
        // for: 8 of 10^6 set, 256^3 FP64, 1587 us a step, 1588 with launches of
        // its own; those are ahead only where 10^5 are set (1234 / 1197 us,
        // FP32 684 / 673)
        const int p = (blockIdx.x - ka->grid) * NWAVE + wave;
        if (p >= ka->P_total) return;
        double acc[6];
        const TileShape ts{TX, TY, ka->tz, 0, 0, 0, ka->zshift};
        const Particles P = particles(ka);
        reduce_sphere(ka->boxes[ka->part_box[p]], ts, P, ka->partial_prev, p, lane, acc);
        if (lane == 0) {
#pragma unroll
            for (int c = 0; c < 6; ++c) P.acc[6LL * p + c] = acc[c];
        }
        return;
    }

    // XCD-aware persistent schedule: workgroup b runs on die b % 8; each die
    // walks one contiguous eighth of the tile list so that x-neighbouring
    // tiles (which share the cache lines of the shifted pulls) meet in the
    // same L2.
    const int G = ka->grid;
    const int xcd = blockIdx.x % NXCD;
    const int gx8 = (G - xcd + NXCD - 1) / NXCD;
    const int m = blockIdx.x / NXCD;
    const int t_begin = (int)(((long long)ka->T_total * xcd) / NXCD);
    const int t_end = (int)(((long long)ka->T_total * (xcd + 1)) / NXCD);

    // Tile order: with a queue (persistent grid), the workgroups of a die take
    // the next run of tiles of its eighth from that die's counter as they finish
    // one; otherwise workgroup m of a die takes tiles m, m + gx8, ...
    __shared__ int s_next;
    int* const queue = ka->queue;
    int t = t_begin + m;
    if (queue) {
        if (tid == 0) s_next = t_begin + (atomicAdd(queue + xcd, 1) << ka->run);
        __syncthreads();
        t = __builtin_amdgcn_readfirstlane(s_next);   // uniform: everything of the tile stays scalar
    }
    while (t < t_end) {
        ka = step_args();
        // part t of the tiles: 1 << zs of them along z share a tile and its list,
        // in the order that tiles of their own depth would have
        const int zs = ka->zshift;
        int b = 0;
        if (ka->nbox > 1) {
            const PSM_CONST int* tb = cptr(ka->box_tile_base);
            int lo = 0, hi = ka->nbox - 1;
            while (lo < hi) {
                int mid = (lo + hi + 1) >> 1;
                if (tb[mid] << zs <= t) lo = mid; else hi = mid - 1;
            }
            b = lo;
        }
        const PSM_CONST BoxDev& bx = cptr(ka->boxes)[b];
        const int nx = bx.nx, ny = bx.ny, nz = bx.nz;
        // MAP = 1 instantiates the sampling path for contexts in which any box
        // samples; each box still uses its own mapping
        const bool lin_map = MAP == 0 || bx.mapping == 0;
        const int ntx = bx.ntx, nty = bx.nty;
        const int lt = t - (bx.tile_base << zs);
        const int lr = udiv(lt, bx.div_ntx[0], bx.div_ntx[1]);   // row of tiles
        const int tcx = lt - lr * ntx;
        const int tcz = udiv(lr, bx.div_nty[0], bx.div_nty[1]);
        const int tcy = lr - tcz * nty;
        const int tile = bx.tile_base + tcx + ntx * (tcy + nty * (tcz >> zs));
        const int listed = cptr(ka->tile_cnt)[tile], lcap = ka->list_cap, cap = lcap < 0 ? -lcap : lcap;
        const int nc = listed < cap ? listed : cap;   // at most MAXC
        const int2* ent = ka->tile_ent + (lcap < 0 ? (long long)cptr(ka->tile_cnt)[(ka->T_total >> zs) + tile]
                                                   : (long long)tile * cap);
        const double Lx = bx.L[0], Ly = bx.L[1], Lz = bx.L[2];
        const double hLx = bx.halfL[0], hLy = bx.halfL[1], hLz = bx.halfL[2];
        const int RZ = ka->ref_z, zb = tcz * TZ & ~(RZ - 1);

        if (nc > 0) {
            for (int c = tid; c < nc; c += WG) {
                const int2 e = ent[c];
                const int p = e.x;
                s_pid[c] = p;
                s_slot[c] = (e.y << zs) + (tcz & ((1 << zs) - 1));
                const double px = ka->P.x[p], py = ka->P.y[p], pz = ka->P.z[p], pr = ka->P.r[p], pfr = ka->P.fr[p];
                s_px[c] = px; s_py[c] = py; s_pz[c] = pz;
                s_pr[c] = pr; s_pfr[c] = pfr;
                const double u[6] = {ka->P.ux[p], ka->P.uy[p], ka->P.uz[p], ka->P.ox[p], ka->P.oy[p], ka->P.oz[p]};
                if constexpr (S::DEV) {
                    // reference point of the FP32 geometry in cell coordinates: the
                    // tile's centre, in z that of the block of ref_z planes it lies in
                    const double tmx = tcx * TX + 0.5 * TX, tmy = tcy * TY + 0.5 * TY, tmz = zb + 0.5 * RZ;
                    s_qx[c] = (float)min_image(px - tmx, Lx, hLx);
                    s_qy[c] = (float)min_image(py - tmy, Ly, hLy);
                    s_qz[c] = (float)min_image(pz - tmz, Lz, hLz);
                    const double lim = pr + (lin_map ? pfr : bx.reach) + bx.margin32;
                    s_lim2[c] = (float)(lim * lim);
                    s_rf[c] = (float)pr;
                    s_frf[c] = (float)pfr;
#pragma unroll
                    for (int k = 0; k < 6; ++k) s_uf[k][c] = (float)u[k];
                } else {
                    s_ux[c] = u[0]; s_uy[c] = u[1]; s_uz[c] = u[2];
                    s_ox[c] = u[3]; s_oy[c] = u[4]; s_oz[c] = u[5];
                }
            }
            for (int i = tid; i < NWAVE * 6 * MAXC; i += WG) (&s_acc[0][0][0])[i] = 0.0;
            // a list cut short: the results are not valid from here on, whatever
            // the lists of later steps hold
            if (listed > cap && tid == 0) atomicOr(step_args()->flags, FLAG_LIST_CUT);
        }
        __syncthreads();

        ka = step_args();
        // the thread's column in the tile (TX is a power of two), taken from the
        // thread id again for every tile: held across the staging it is spilled
        int tl = tid;
        asm volatile("" : "+v"(tl));
        const int lx = tl & (TX - 1), ly = tl >> __builtin_ctz(TX);
        const int x = tcx * TX + lx;
        const int y = tcy * TY + ly;
        const bool lane_ok = (x < nx) && (y < ny);
        const int xs = lane_ok ? x : 0, ys = lane_ok ? y : 0;
        const int xm = xs == 0 ? nx - 1 : xs - 1, xp = xs == nx - 1 ? 0 : xs + 1;
        const int ym = ys == 0 ? ny - 1 : ys - 1, yp = ys == ny - 1 ? 0 : ys + 1;
        // byte offsets inside a z-plane of the nine (x, y) source columns;
        // they do not depend on z (a plane holds fewer than 2^31 bytes)
        const int pitch = bx.pitch;
        auto inplane = [pitch](int xx, int yy) -> unsigned { return cell_offset<T>(xx, yy, pitch); };
        // lanes next to a resting side wall (x = 0, nx - 1; y = 0, ny - 1): bits 0-3
        const int edge = !WALL || !lane_ok || !bx.walls_xy ? 0
                         : (((bx.walls_xy & 1) && xs == 0) ? 1 : 0) | (((bx.walls_xy & 1) && xs == nx - 1) ? 2 : 0) |
                               (((bx.walls_xy & 2) && ys == 0) ? 4 : 0) | (((bx.walls_xy & 2) && ys == ny - 1) ? 8 : 0);
        const bool edge_wave = WALL && __ballot(edge != 0) != 0ull;
        const unsigned o00 = inplane(xs, ys), om0 = inplane(xm, ys), op0 = inplane(xp, ys);
        const unsigned o0m = inplane(xs, ym), o0p = inplane(xs, yp);
        const unsigned omm = inplane(xm, ym), opp = inplane(xp, yp), omp = inplane(xm, yp), opm = inplane(xp, ym);
        const long long pbytes = bx.plane_elems * (long long)sizeof(T);
        const unsigned pb32 = (unsigned)pbytes;
        const char* src = (const char*)bx.grid[ka->parity];
        const char* dst = (const char*)bx.grid[ka->parity ^ 1];
        // scaled storage (FP16): the kernel works on s d; the quadratic terms
        // carry 1/s and every particle velocity is multiplied by s
        const R sc = S::SCALED ? (R)ka->h_scale : (R)1;
        const double cxc = xs + 0.5, cyc = ys + 0.5;
        // this cell's centre relative to the reference point (FP32, exact)
        const float rx = (float)(lx + 0.5 - 0.5 * TX), ry = (float)(ly + 0.5 - 0.5 * TY);
        const float Lxf = (float)Lx, Lyf = (float)Ly, Lzf = (float)Lz;
        const float iLx = 1.0f / Lxf, iLy = 1.0f / Lyf, iLz = 1.0f / Lzf;
        // Candidate filter: bit c of s_cmask[wave][k] is set if candidate c
        // can reach a cell of this wave at the tile's k-th z: the distance from
        // the sphere centre to the rectangle of the wave's cell centres (lanes
        // past the box edge only enlarge it) is below r + f(r), or r + the
        // sampling reach, plus a margin that covers the FP32 rounding of the
        // test. Other candidates give zero fraction to all of those cells.
        if (FILT && nc > 0) {
            float xy2 = 0.0f, pz = 0.0f, lim2 = -1.0f;
            if (lane < nc) {
                const int wwx = TX < 64 ? TX : 64, wwy = TX < 64 ? 64 / TX : 1;
                const int wx0 = tcx * TX + (64 * wave) % TX, wy0 = tcy * TY + (64 * wave) / TX;
                double ex = fabs(min_image(wx0 + 0.5 * wwx - s_px[lane], bx.L[0], bx.halfL[0])) - 0.5 * (wwx - 1);
                double ey = fabs(min_image(wy0 + 0.5 * wwy - s_py[lane], bx.L[1], bx.halfL[1])) - 0.5 * (wwy - 1);
                ex = ex > 0.0 ? ex : 0.0;
                ey = ey > 0.0 ? ey : 0.0;
                xy2 = (float)(ex * ex + ey * ey);
                pz = (float)s_pz[lane];
                const double lim = s_pr[lane] + (lin_map ? s_pfr[lane] : bx.reach) + 0.05;
                lim2 = (float)(lim * lim);
            }
            const float fnz = (float)nz;
            for (int k = 0; k < TZ; ++k) {
                float ez = (float)(tcz * TZ + k) + 0.5f - pz;
                ez = ez >= 0.5f * fnz ? ez - fnz : (ez < -0.5f * fnz ? ez + fnz : ez);
                const unsigned long long m = __ballot(xy2 + ez * ez < lim2);
                if (lane == 0) s_cmask[wave][k] = m;
            }
        }

        constexpr int QB = BLK * (int)sizeof(T);

        // Latency hiding: PREF pulls the next cell's 19 values (one cell up in
        // z) while the current one is mapped and collided; EARLY issues the
        // current cell's pulls before its mapping.
        constexpr bool PREF = S::DEV && !FILT && MAP == 0 && (S::SCALED ? PSM_PREFETCH_F16 : PSM_PREFETCH_F32);
        constexpr bool EARLY = !PREF && !FILT && MAP == 0 && (S::DEV ? (S::SCALED && PSM_EARLY_PULLS_F16) : PSM_EARLY_PULLS_F64);
        constexpr int LINE_AUX = CACHE == STREAM ? 2 : LD_AUX;
        R fn[NQ];
        if constexpr (PREF) {
            const int z0 = tcz * TZ;
            if (lane_ok && z0 < nz) {
                const int zm0 = z0 == 0 ? nz - 1 : z0 - 1, zp0 = z0 == nz - 1 ? 0 : z0 + 1;
                const Rsrc a = plane_rsrc(src + z0 * pbytes, pb32), am = plane_rsrc(src + zm0 * pbytes, pb32),
                           ap = plane_rsrc(src + zp0 * pbytes, pb32);
                PSM_LOAD19(fn, a, am, ap, LINE_AUX);
            }
        }

        for (int k = 0; k < TZ; ++k) {
            const int z = tcz * TZ + k;
            if (z >= nz) break;
            const double czc = z + 0.5;
            const float rz = (float)(z - zb + 0.5 - 0.5 * RZ);
            const int zm = z == 0 ? nz - 1 : z - 1, zp = z == nz - 1 ? 0 : z + 1;
            // buffer resources of the source planes z, z-1, z+1 and the
            // destination plane z
            const Rsrc sz = plane_rsrc(src + z * pbytes, pb32);
            const Rsrc sm = plane_rsrc(src + zm * pbytes, pb32);
            const Rsrc sp = plane_rsrc(src + zp * pbytes, pb32);
            const Rsrc dz_ = plane_rsrc(dst + z * pbytes, pb32);

            // 2a. pull: f_q(x) = grid[q][x - c_q] (eq. 2 read backwards)
            R f[NQ];
            if constexpr (PREF) {
#pragma unroll
                for (int q = 0; q < NQ; ++q) f[q] = fn[q];
                const int z1 = z + 1;
                if (lane_ok && k + 1 < TZ && z1 < nz) {
                    // planes z + 1 (own), z (below) and z + 2 (above, periodic)
                    const Rsrc a2 = plane_rsrc(src + (z1 == nz - 1 ? 0 : z1 + 1) * pbytes, pb32);
                    PSM_LOAD19(fn, sp, sz, a2, LINE_AUX);
                }
            } else if constexpr (EARLY) {
                if (lane_ok) PSM_LOAD19(f, sz, sm, sp, LINE_AUX);
            }

            // 1. solid fractions of this cell from the staged candidates (Sec. 2.3.2);
            // with the filter, only the candidates that can reach this wave at this z.
            // The fraction is FP64, bit for bit that of the read-out path, except
            // that the FP16 form takes the linear approximation in FP32.
            int c0 = -1, c1 = -1;
            double B0 = 0.0, B1 = 0.0;
            int dropped = 0;   // overlaps beyond the two slots at this cell
#define PSM_MAP_ONE(c)                                                                                       \
    do {                                                                                                    \
        bool near_ = true;                                                                                  \
        if constexpr (S::DEV) {                                                                             \
            const float tx_ = wrap32(rx - s_qx[c], Lxf, iLx);                                               \
            const float ty_ = wrap32(ry - s_qy[c], Lyf, iLy);                                               \
            const float tz_ = wrap32(rz - s_qz[c], Lzf, iLz);                                               \
            const float d2_ = fmar(tz_, tz_, fmar(ty_, ty_, tx_ * tx_));                                    \
            near_ = d2_ <= s_lim2[c];                                                                       \
            if (S::SCALED && near_ && lin_map) {                                                            \
                /* FP16 storage: linear approximation of eq. (26) in FP32 (its error, about */              \
                /* 1e-6 of a cell, is far below the FP16 rounding of the stored values) */                  \
                const float eps_ = s_frf[c] - (__builtin_amdgcn_sqrtf(d2_) - s_rf[c]);                       \
                if (eps_ > 0.0f) slots_insert(sl, c, s_pid[c], (double)(eps_ < 1.0f ? eps_ : 1.0f));         \
                near_ = false;                                                                              \
            }                                                                                               \
        }                                                                                                   \
        if (near_) {                                                                                        \
            double dx = min_image(cxc - s_px[c], Lx, hLx);                                                  \
            double dy = min_image(cyc - s_py[c], Ly, hLy);                                                  \
            double dz = min_image(czc - s_pz[c], Lz, hLz);                                                  \
            double B = lin_map ? overlap_linear(dx, dy, dz, s_pr[c], s_pfr[c])                              \
                               : overlap_subsample(dx, dy, dz, s_pr[c], bx.nsub, bx.sub_off, bx.reach);     \
            if (B > 0.0) slots_insert(sl, c, s_pid[c], B);                                                  \
        }                                                                                                   \
    } while (0)
            if constexpr (FILT) {
                unsigned long long cm = nc > 0 ? s_cmask[wave][k] : 0ull;
                // wave-uniform: keep the mask and its loop in scalar registers (the
                // builtin returns an int: its sign must not reach the upper half)
                cm = ((unsigned long long)__builtin_amdgcn_readfirstlane((unsigned)(cm >> 32)) << 32) |
                     (unsigned)__builtin_amdgcn_readfirstlane((unsigned)cm);
                if (cm != 0ull) {
                    Slots sl;
                    slots_init(sl);
                    if (lane_ok) {
                        while (cm != 0ull) {
                            const int c = __ffsll((long long)cm) - 1;
                            cm &= cm - 1ull;
                            PSM_MAP_ONE(c);
                        }
                        slots_finish(sl);
                    }
                    c0 = sl.c0; c1 = sl.c1; B0 = sl.B0; B1 = sl.B1; dropped = sl.dropped;
                }
            } else if (nc > 0) {
                Slots sl;
                slots_init(sl);
                if (lane_ok) {
                    for (int c = 0; c < nc; ++c) PSM_MAP_ONE(c);
                    slots_finish(sl);
                }
                c0 = sl.c0; c1 = sl.c1; B0 = sl.B0; B1 = sl.B1; dropped = sl.dropped;
            }
#undef PSM_MAP_ONE
            const bool psm_wave = __ballot(c0 >= 0) != 0ull;
            // a third overlap is dropped (the two strongest slots stay) and flagged
            // once per wave; the host reports it in strict-slot mode
            if (psm_wave && __ballot(dropped != 0) != 0ull && lane == 0) atomicOr(step_args()->flags, FLAG_SLOT_OVERFLOW);

            const R omega = pick<R>(bx.omega, bx.omega_f);
            const R om1 = pick<R>(bx.om1, bx.om1_f);
            const R gx = pick<R>(bx.g[0], bx.g_f[0]), gy = pick<R>(bx.g[1], bx.g_f[1]),
                    gz = pick<R>(bx.g[2], bx.g_f[2]);
            const R k15 = pick<R>(bx.k15, bx.k15_f);
            const R k45 = pick<R>(bx.k45, bx.k45_f);

            // 2b. boundaries of the pulled values
            R hx = 0, hy = 0, hz = 0;   // 2 j - U, for the force of eq. (21)
            if (lane_ok) {
                // through a face (first and last z plane of a box with walls):
                // the population this cell sent against it last step, by the
                // face rule; computed before the pulls so that its
                // temporaries are not live beside them (uniform branches)
                const bool face_plane = WALL && bx.walls && (z == 0 || z == nz - 1);
                R fb[5] = {0, 0, 0, 0, 0};
                if (face_plane) {
                    const int w = z == 0 ? 0 : 1;
                    // entering directions through this face and their opposites
                    constexpr int in0[5] = {5, 11, 14, 15, 18}, in1[5] = {6, 12, 13, 16, 17};
                    if (bx.face_type[w] == FACE_VELOCITY) {
                        const R ws = S::SCALED ? sc : (R)1;
#pragma unroll
                        for (int i = 0; i < 5; ++i) {
                            const int q = w == 0 ? in0[i] : in1[i];
                            fb[i] = S::ld(sz, o00, inv_dir(q) * QB) + ws * (R)bx.bw[w][q];
                        }
                    } else {
                        // anti-bounce-back with the cell's post-collision velocity
                        // (its own 19 slots); deviation units carry rho_w - 1
                        R ux = 0, uy = 0, uz = 0;
#pragma unroll
                        for (int q = 1; q < NQ; ++q) {
                            const R v = S::ld(sz, o00, q * QB);
                            ux += (R)CX[q] * v; uy += (R)CY[q] * v; uz += (R)CZ[q] * v;
                        }
                        const R rw = S::DEV ? (R)(bx.face_rho[w] - 1.0) * sc : (R)bx.face_rho[w];
                        const R uu = k15 * (ux * ux + uy * uy + uz * uz);
#pragma unroll
                        for (int i = 0; i < 5; ++i) {
                            const int q = w == 0 ? in0[i] : in1[i];
                            const R cu = (R)CX[q] * ux + (R)CY[q] * uy + (R)CZ[q] * uz;
                            fb[i] = (R)(2.0 * wq(q)) * (rw + k45 * (cu * cu) - uu) - S::ld(sz, o00, inv_dir(q) * QB);
                        }
                    }
                }
                if constexpr (!PREF && !EARLY) PSM_LOAD19(f, sz, sm, sp, LINE_AUX);
                if (face_plane) {
                    if (z == 0) {
                        f[5] = fb[0]; f[11] = fb[1]; f[14] = fb[2]; f[15] = fb[3]; f[18] = fb[4];
                    } else {
                        f[6] = fb[0]; f[12] = fb[1]; f[13] = fb[2]; f[16] = fb[3]; f[17] = fb[4];
                    }
                }
                if (edge_wave && edge) {
                    // resting side walls (they win over a z face): a population
                    // pulled from behind a wall is the one this cell sent
                    // against it last step
#pragma unroll
                    for (int q = 1; q < NQ; ++q) {
                        const bool hit = (CX[q] == 1 && (edge & 1)) || (CX[q] == -1 && (edge & 2)) ||
                                         (CY[q] == 1 && (edge & 4)) || (CY[q] == -1 && (edge & 8));
                        if (hit) f[q] = S::ld(sz, o00, inv_dir(q) * QB);
                    }
                }

                // 3. moments, eqs. (6)-(7), accumulated from the sum and the
                // difference of each inverse pair (q, q+1), q = 2k-1 with c_q =
                // +x, +y, +z, (1,1,0), (1,-1,0), (1,0,1), (1,0,-1), (0,1,1),
                // (0,1,-1) for k = 1..9; U carries the f/2 shift
                R rho = f[0], jx, jy, jz;
                {
                    R d;
                    rho += f[1] + f[2]; jx = f[1] - f[2];
                    rho += f[3] + f[4]; jy = f[3] - f[4];
                    rho += f[5] + f[6]; jz = f[5] - f[6];
                    rho += f[7] + f[8]; d = f[7] - f[8]; jx += d; jy += d;
                    rho += f[9] + f[10]; d = f[9] - f[10]; jx += d; jy -= d;
                    rho += f[11] + f[12]; d = f[11] - f[12]; jx += d; jz += d;
                    rho += f[13] + f[14]; d = f[13] - f[14]; jx += d; jz -= d;
                    rho += f[15] + f[16]; d = f[15] - f[16]; jy += d; jz += d;
                    rho += f[17] + f[18]; d = f[17] - f[18]; jy += d; jz -= d;
                }
                const R half = (R)0.5;
                const R Ux = fmar(half, sc * gx, jx), Uy = fmar(half, sc * gy, jy), Uz = fmar(half, sc * gz, jz);
                const R uu = fmar(Uz, Uz, fmar(Uy, Uy, Ux * Ux));
                const R base = fmar(-k15, uu, rho);
                const R Ug3 = (R)3.0 * fmar(Uz, gz, fmar(Uy, gy, Ux * gx));
                const R pu0 = pick<R>(bx.pw[0], bx.pw_f[0]) * Ug3;
                WClass<R> w1, w2;
                {
                    constexpr R W1r = (R)W1, W2r = (R)W2;
                    w1.Wb = W1r * base; w2.Wb = W2r * base;
                    w1.W3 = (R)3 * W1r; w2.W3 = (R)3 * W2r;
                    w1.Wk = pick<R>(bx.wk[1], bx.wk_f[1]); w2.Wk = pick<R>(bx.wk[2], bx.wk_f[2]);
                    w1.owk = pick<R>(bx.owk[1], bx.owk_f[1]); w2.owk = pick<R>(bx.owk[2], bx.owk_f[2]);
                    w1.ow3 = pick<R>(bx.ow3[1], bx.ow3_f[1]); w2.ow3 = pick<R>(bx.ow3[2], bx.ow3_f[2]);
                    w1.owb_pu = fmar(omega, w1.Wb, -pick<R>(bx.pw[1], bx.pw_f[1]) * Ug3);
                    w2.owb_pu = fmar(omega, w2.Wb, -pick<R>(bx.pw[2], bx.pw_f[2]) * Ug3);
                }
#define PSM_FA(Q) pick<R>(S::SCALED ? bx.fa_scaled[Q / 2] : bx.fa[Q / 2], S::SCALED ? bx.fa_scaled_f[Q / 2] : bx.fa_f[Q / 2])
#define PSM_FS(Q) pick<R>(bx.fs[Q / 2], bx.fs_f[Q / 2])
#define PSM_STORE(Q) S::template st<CACHE == KEEP ? 0 : ST_AUX>(dz_, o00, (Q) * QB, f[Q])

                // 4. collision; each pair is stored as soon as it is final
                if (!psm_wave) {
                    f[0] = fmar(om1, f[0], fmar(omega * (R)W0, base, -pu0));
                    PSM_STORE(0);
#define PSM_PAIR(Q)                                                                                 \
    pair_fluid<R, Q>(f[Q], f[Q + 1], cdot<R, Q>(Ux, Uy, Uz), Q < 7 ? w1 : w2, PSM_FA(Q), PSM_FS(Q), om1); \
    PSM_STORE(Q);                                                                                   \
    PSM_STORE(Q + 1)
                    PSM_PAIR(1); PSM_PAIR(3); PSM_PAIR(5); PSM_PAIR(7); PSM_PAIR(9);
                    PSM_PAIR(11); PSM_PAIR(13); PSM_PAIR(15); PSM_PAIR(17);
#undef PSM_PAIR
                } else {
                    hx = (R)2 * jx - Ux; hy = (R)2 * jy - Uy; hz = (R)2 * jz - Uz;
                    // slot terms with U_p(x) of eq. (20) (times the storage scale)
                    // (a wave with a slot somewhere: lanes without one add nothing)
                    R Bt = 0, A0 = 0, Mxx = 0, Myy = 0, Mzz = 0, Mxy = 0, Mxz = 0, Myz = 0, Px = 0, Py = 0, Pz = 0;
#pragma unroll
                    for (int sl = 0; sl < 2; ++sl) {
                        const int c = sl == 0 ? c0 : c1;
                        if (c < 0) continue;   // slot 1 is only filled after slot 0
                        R Vx, Vy, Vz;
                        if constexpr (S::DEV) {
                            // lever arm from the FP32 tile-relative centre
                            const float dx = wrap32(rx - s_qx[c], Lxf, iLx);
                            const float dy = wrap32(ry - s_qy[c], Lyf, iLy);
                            const float dz = wrap32(rz - s_qz[c], Lzf, iLz);
                            Vx = sc * (s_uf[0][c] + (s_uf[4][c] * dz - s_uf[5][c] * dy));
                            Vy = sc * (s_uf[1][c] + (s_uf[5][c] * dx - s_uf[3][c] * dz));
                            Vz = sc * (s_uf[2][c] + (s_uf[3][c] * dy - s_uf[4][c] * dx));
                        } else {
                            double dx, dy, dz;
                            slot_geometry64(c, cxc, cyc, czc, Lx, hLx, Ly, hLy, Lz, hLz, s_px, s_py, s_pz, s_ux,
                                            s_uy, s_uz, s_ox, s_oy, s_oz, dx, dy, dz, Vx, Vy, Vz);
                        }
                        const R Bs = (R)(sl == 0 ? B0 : B1);
                        const R qx = Bs * Vx, qy = Bs * Vy, qz = Bs * Vz;
                        const R a0 = Bs * fmar(-k15, fmar(Vz, Vz, fmar(Vy, Vy, Vx * Vx)), rho);
                        if (sl == 0) {
                            Bt = Bs; A0 = a0; Px = qx; Py = qy; Pz = qz;
                            Mxx = qx * Vx; Myy = qy * Vy; Mzz = qz * Vz;
                            Mxy = qx * Vy; Mxz = qx * Vz; Myz = qy * Vz;
                        } else {
                            Bt = Bt + Bs; A0 = A0 + a0;
                            Px = Px + qx; Py = Py + qy; Pz = Pz + qz;
                            Mxx = fmar(qx, Vx, Mxx); Myy = fmar(qy, Vy, Myy); Mzz = fmar(qz, Vz, Mzz);
                            Mxy = fmar(qx, Vy, Mxy); Mxz = fmar(qx, Vz, Mxz); Myz = fmar(qy, Vz, Myz);
                        }
                    }
                    const R omB = (R)1 - Bt;
                    const R Mxy2 = Mxy + Mxy, Mxz2 = Mxz + Mxz, Myz2 = Myz + Myz;
                    const R omw = omB * omega;
                    const R alpha = ((R)1 - Bt) - omw, beta = omw - Bt, gamma = omw + Bt;
                    const R pu1 = pick<R>(bx.pw[1], bx.pw_f[1]) * Ug3, pu2 = pick<R>(bx.pw[2], bx.pw_f[2]) * Ug3;
                    const R C11 = fmar(beta, w1.Wb, fmar(-omB, pu1, (R)W1 * A0));
                    const R C12 = fmar(beta, w2.Wb, fmar(-omB, pu2, (R)W2 * A0));
                    const R C21 = beta * w1.Wk, C22 = beta * w2.Wk;
                    const R C31 = gamma * w1.W3, C32 = gamma * w2.W3;
                    // rest population: c = 0, qbar = q
                    f[0] = fmar(alpha + Bt, f[0], fmar(beta * (R)W0, base, fmar(-omB, pu0, (R)W0 * A0)));
                    PSM_STORE(0);
#define PSM_PAIR(Q)                                                                                              \
    pair_psm<R, Q>(f[Q], f[Q + 1], cdot<R, Q>(Ux, Uy, Uz), Q < 7 ? C11 : C12, Q < 7 ? C21 : C22, Q < 7 ? C31 : C32, \
                   Q < 7 ? w1.Wk : w2.Wk, Q < 7 ? w1.W3 : w2.W3, omB * PSM_FS(Q), omB * PSM_FA(Q), alpha, Bt,        \
                   cmc<R, Q>(Mxx, Myy, Mzz, Mxy2, Mxz2, Myz2), cdot<R, Q>(Px, Py, Pz));                             \
    PSM_STORE(Q);                                                                                                \
    PSM_STORE(Q + 1)
                    PSM_PAIR(1); PSM_PAIR(3); PSM_PAIR(5); PSM_PAIR(7); PSM_PAIR(9);
                    PSM_PAIR(11); PSM_PAIR(13); PSM_PAIR(15); PSM_PAIR(17);
#undef PSM_PAIR
                }
#undef PSM_STORE
#undef PSM_FA
#undef PSM_FS
            }

            // 5. force and torque of eqs. (21)-(22): sum_q C^solid_{q,s} c_qbar
            // = 2 j - U - U_p(x) per slot (first moment of eq. 19); per-sphere
            // wave sums accumulated per wave in LDS in FP64 in a fixed order.
            // The deviation forms compute each cell's share and the wave sum in
            // FP32 (the collision's precision); FP64 storage does both in FP64.
            if (psm_wave) {
                int pend0 = lane_ok ? c0 : -1, pend1 = lane_ok ? c1 : -1;
                while (true) {
                    unsigned long long live = __ballot(pend0 >= 0 || pend1 >= 0);
                    if (live == 0ull) break;
                    int leader = __ffsll((long long)live) - 1;
                    int mine = pend0 >= 0 ? pend0 : pend1;
                    // the leader's candidate, read into a scalar register
                    const int c = __builtin_amdgcn_readlane(mine, leader);
                    double Bs = 0.0;
                    if (pend0 == c) { Bs = B0; pend0 = -1; }
                    else if (pend1 == c) { Bs = B1; pend1 = -1; }
                    R v[6] = {0, 0, 0, 0, 0, 0};
                    if (Bs != 0.0) {
                        R dx, dy, dz, Vx, Vy, Vz;
                        if constexpr (S::DEV) {
                            dx = wrap32(rx - s_qx[c], Lxf, iLx);
                            dy = wrap32(ry - s_qy[c], Lyf, iLy);
                            dz = wrap32(rz - s_qz[c], Lzf, iLz);
                            Vx = sc * (s_uf[0][c] + (s_uf[4][c] * dz - s_uf[5][c] * dy));
                            Vy = sc * (s_uf[1][c] + (s_uf[5][c] * dx - s_uf[3][c] * dz));
                            Vz = sc * (s_uf[2][c] + (s_uf[3][c] * dy - s_uf[4][c] * dx));
                        } else {
                            slot_geometry64(c, cxc, cyc, czc, Lx, hLx, Ly, hLy, Lz, hLz, s_px, s_py, s_pz, s_ux,
                                            s_uy, s_uz, s_ox, s_oy, s_oz, dx, dy, dz, Vx, Vy, Vz);
                        }
                        const R Bh = (R)(S::SCALED ? Bs * (double)step_args()->h_inv : Bs);
                        const R fx = Bh * (hx - Vx), fy = Bh * (hy - Vy), fz = Bh * (hz - Vz);
                        v[0] = fx;
                        v[1] = fy;
                        v[2] = fz;
                        v[3] = dy * fz - dz * fy;
                        v[4] = dz * fx - dx * fz;
                        v[5] = dx * fy - dy * fx;
                    }
                    const R sum = wave_sum6<R>(v, lane);
                    if (lane < 6) s_acc[wave][lane][c] += (double)sum;
                }
            }
        }

        __syncthreads();
        if (nc > 0) {
            double* const partial = step_args()->partial;
            for (int i = tid; i < nc * 6; i += WG) {
                int c = i / 6, k6 = i - 6 * c;
                double s = 0.0;
#pragma unroll
                for (int w = 0; w < NWAVE; ++w) s += s_acc[w][k6][c];
                partial[(long long)s_slot[c] * 6 + k6] = s;
            }
        }
        __syncthreads();
        // every thread has read s_next before the barriers of this tile
        if (queue) {
            const int run = step_args()->run;
            ++t;
            if (((t - t_begin) & ((1 << run) - 1)) == 0) {
                if (tid == 0) s_next = t_begin + (atomicAdd(queue + xcd, 1) << run);
                __syncthreads();
                t = __builtin_amdgcn_readfirstlane(s_next);
            }
        } else {
            t += gx8;
        }
    }
}

// ---------------------------------------------------------------------------
// Work per sphere, one 64-wide wave each:
//   UPLOAD  the spheres of one box first take new columns from pinned host
//           staging (lane c reads column c), before their tiles are found.
//   REDUCE  force and torque of the last step (reduce_sphere; earlier steps of
//           one call are reduced inside the next step's launch where the
//           context has two sets of partials).
//   SCHEME  sphere update (Sec. 2.2.2) for collision-free spheres:
//           m = rho_p (4/3) pi r^3, I = (2/5) m r^2; the total force is the
//           hydrodynamic force of the last step plus m times the box's
//           external acceleration, the torque is the hydrodynamic torque.
//             Euler:  x += dt U;  U += dt F/m;  Om += dt T/I.
//             Verlet (eqs. 15-16), once after each fluid step: complete the
//             velocity with the previous and the new force (skipped until a
//             previous force exists), then advance the position with the new one.
//           Positions are wrapped into [0, L) along periodic axes; along an
//           axis with walls a centre leaving [r + 1, L - r - 1] is mirrored
//           back and its velocity component reversed (elastic contact keeping
//           the mapping's one-cell gap). No fused multiply-add, so that the
//           update is reproducible bit for bit; every lane computes it.
//   BIN     tile lists (the paper's sub-block particle lists): the lanes walk
//           the tiles of the (new) bounding box and append the sphere to each.
// Latency bound: a few dependent loads and an atomic per wave, a few us in
// all, so what counts is the number of launches. Lists of a fixed capacity
// are built in one launch (counting, scanning and filling compact lists took
// seven of 2-5 us each), and psm_run does all three parts in one: 9 launches
// beside the step kernel became 1.
template <bool REDUCE, int SCHEME, bool BIN, bool UPLOAD = false>
__global__ __launch_bounds__(256) void k_spheres(SphereParams sp, UploadParams up = UploadParams{}) {
#pragma clang fp contract(off)
    if (BIN) {
        // the counts of the lists being replaced, for the build after this one
        const int i0 = blockIdx.x * 256 + threadIdx.x;
        for (int i = i0; i < sp.T_total; i += gridDim.x * 256) sp.cnt_old[i] = 0;
        if (i0 == 0) *sp.over_old = 0;
    }
    const int lane = threadIdx.x & 63;
    const int p = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (REDUCE && sp.host_acc && blockIdx.x == 0 && threadIdx.x < ERR_WORDS)
        ((int*)(sp.host_acc + 6LL * sp.P_total))[threadIdx.x] = sp.err[threadIdx.x];
    if (p >= sp.P_total) return;   // whole wave leaves together
    const BoxDev& bx = sp.boxes[sp.part_box[p]];
    const int lp = p - bx.part_base;
    bool there = lp < bx.np;
    const long long slot0 = (long long)bx.pbase + (long long)lp * bx.pstride;
    double pos[3] = {sp.P.x[p], sp.P.y[p], sp.P.z[p]};
    double r = sp.P.r[p];
    if (UPLOAD && up.part_base == bx.part_base) {
        there = lp < up.n;
        double v = 0.0;
        if (there && lane < up.ncols) {
            v = up.src[(long long)lane * up.m + lp];
            up.table[(up.first + lane) * up.pitch + lp] = v;
        }
        for (int a = 0; a < 3; ++a) pos[a] = __shfl(v, a, 64);   // an upload with lists starts at x
        if (up.ncols > 3) r = __shfl(v, 3, 64);
        if (lane == 0) {
            if (up.prev_ok) up.prev_ok[lp] = 0;
            if (up.np && lp == 0) *up.np = up.n;
        }
    }
    double acc[6];
    if (REDUCE) {
        reduce_sphere(bx, sp.ts, sp.P, sp.partial, p, lane, acc);
        if (lane == 0) {
#pragma unroll
            for (int c = 0; c < 6; ++c) sp.P.acc[6LL * p + c] = acc[c];
        }
        if (sp.host_acc) {
            // lanes 0-5: one 48-B store to the host
            double v = acc[0];
#pragma unroll
            for (int c = 1; c < 6; ++c) v = lane == c ? acc[c] : v;
            if (lane < 6) sp.host_acc[6LL * p + lane] = v;
        }
    }
    if (!there) return;
    if (SCHEME != SCHEME_NONE) {
        if (!REDUCE) {
#pragma unroll
            for (int c = 0; c < 6; ++c) acc[c] = sp.P.acc[6LL * p + c];
        }
        const double pi = 3.14159265358979323846;
        const double dt = sp.dt;
        const double m = bx.rho_p * (4.0 / 3.0) * pi * r * r * r;
        const double inertia = 0.4 * m * r * r;
        double* dpos[3] = {sp.P.x, sp.P.y, sp.P.z};
        double* dvel[3] = {sp.P.ux, sp.P.uy, sp.P.uz};
        double* dang[3] = {sp.P.ox, sp.P.oy, sp.P.oz};
        double* fp = sp.P.fprev + 6LL * p;
        const bool prev = SCHEME == SCHEME_VERLET && sp.P.prev_ok[p] != 0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const double F = acc[a] + m * bx.accel[a];
            const double T = acc[3 + a];
            double x = pos[a], U = dvel[a][p], W = dang[a][p];
            if (SCHEME == SCHEME_EULER) {
                x = x + dt * U;
                U = U + dt * F / m;
                W = W + dt * T / inertia;
            } else {
                if (prev) {
                    U = U + dt / (2.0 * m) * (fp[a] + F);
                    W = W + dt / (2.0 * inertia) * (fp[3 + a] + T);
                }
                x = x + (dt * U + dt * dt / (2.0 * m) * F);
                if (lane == 0) {
                    fp[a] = F;
                    fp[3 + a] = T;
                }
            }
            const double L = bx.L[a];
            const bool walled = a == 2 ? bx.walls != 0 : (bx.walls_xy & (1 << a)) != 0;
            if (walled) {
                // elastic contact one cell before the walls: mirror the centre back
                // into [r + 1, L - r - 1] and reverse the normal velocity
                const double lo = r + 1.0, hi = L - r - 1.0;
                if (x < lo) { x = 2.0 * lo - x; U = -U; }
                else if (x > hi) { x = 2.0 * hi - x; U = -U; }
            } else {
                double w = x - L * floor(x / L);
                if (w >= L) w -= L;
                if (w < 0.0) w = 0.0;
                x = w;
            }
            pos[a] = x;
            if (lane == 0) {
                dpos[a][p] = x;
                dvel[a][p] = U;
                dang[a][p] = W;
            }
        }
        if (SCHEME == SCHEME_VERLET && lane == 0) sp.P.prev_ok[p] = 1;
    }
    if (BIN) {
        AxisTiles ax, ay, az;
        box_tiles(bx, sp.ts, pos[0], pos[1], pos[2], r, ax, ay, az);
        const int nxt = ax.count(), nyt = ay.count(), nzt = az.count();
        const int ntot = nxt * nyt * nzt;
        for (int k = lane; k < ntot; k += 64) {
            const int kx = k % nxt, ky = (k / nxt) % nyt, kz = k / (nxt * nyt);
            const int t = bx.tile_base + ax.at(kx) + bx.ntx * (ay.at(ky) + bx.nty * az.at(kz));
            const int at = atomicAdd(&sp.cnt[t], 1);
            if (sp.count_only) continue;
            if (at < sp.list_cap) {
                sp.ent[(sp.off ? (long long)sp.off[t] : (long long)t * sp.list_cap) + at] = make_int2(p, (int)(slot0 + k));
            } else {
                // a list holds at most MAXC spheres: the excess is dropped and reported
                atomicMax(sp.over, at + 1);
                for (int c = 0; c < 6 << sp.ts.zshift; ++c) {
                    sp.partial[((slot0 + k) << sp.ts.zshift) * 6 + c] = 0.0;
                    sp.partial_next[((slot0 + k) << sp.ts.zshift) * 6 + c] = 0.0;
                }
            }
        }
    }
}

// Compact lists: the first entry of each tile's list from the counts, which
// start again from zero for the fill; off[T], zero on entry, counts the entries
// given out. Which run of entries a tile gets does not matter.
__global__ __launch_bounds__(256) void k_list_offsets(int* cnt, int* off, int T, int list_cap) {
    const int t = blockIdx.x * 256 + threadIdx.x, lane = threadIdx.x & 63;
    const int n = t < T ? min(cnt[t], list_cap) : 0;
    int sum = n;   // of the lanes up to this one
    for (int d = 1; d < 64; d <<= 1) {
        const int below = __shfl_up(sum, d, 64);
        sum += lane >= d ? below : 0;
    }
    int base = 0;
    if (lane == 63 && sum > 0) base = atomicAdd(off + T, sum);
    base = __shfl(base, 63, 64);
    if (t < T) {
        off[t] = base + sum - n;
        cnt[t] = 0;
    }
}

// Sphere-table columns from pinned host staging, one value per thread
// (coalesced reads over the host link).
__global__ __launch_bounds__(256) void k_upload(UploadParams up) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i < (long long)up.ncols * up.n) {
        const int c = (int)(i / up.n), lp = (int)(i - (long long)c * up.n);
        up.table[(up.first + c) * up.pitch + lp] = up.src[(long long)c * up.m + lp];
    }
    if (up.prev_ok && i < up.m) up.prev_ok[i] = 0;
    if (up.np && i == 0) *up.np = up.n;
}

// Sphere data and the error words to pinned host memory: one launch where a
// copy per range and one for the words took 10-20 us.
__global__ __launch_bounds__(256) void k_download(DownloadParams dp) {
    const long long stride = (long long)gridDim.x * 256;
    const long long i0 = (long long)blockIdx.x * 256 + threadIdx.x;
    double* dst = dp.dst;
    for (int g = 0; g < 2; ++g) {
        const long long total = dp.n * dp.ncols[g];
        for (long long i = i0; i < total; i += stride) {
            const long long c = i / dp.n;
            dst[i] = dp.src[g][c * dp.pitch[g] + (i - c * dp.n)];
        }
        dst += total;
    }
    if (i0 < ERR_WORDS) dp.err_dst[i0] = dp.err[i0];
}

__global__ void k_fill_int(int* a, long long n, int v) {
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    long long stride = (long long)gridDim.x * blockDim.x;
    for (; i < n; i += stride) a[i] = v;
}

// ---------------------------------------------------------------------------
// State I/O. Canonical f(x,t) = grid[q][x - c_q] (pull storage).

// Face crossed by a neighbour at z-index zz: -1 none (inside or periodic), 0 bottom, 1 top.
__device__ inline int face_of(const BoxDev& bx, int zz) {
    return !bx.walls ? -1 : (zz < 0 ? 0 : (zz >= bx.nz ? 1 : -1));
}

// True if the neighbour at (xx, yy) lies behind a resting side wall.
__device__ inline bool behind_side_wall(const BoxDev& bx, int xx, int yy) {
    return ((bx.walls_xy & 1) && (xx < 0 || xx >= bx.nx)) || ((bx.walls_xy & 2) && (yy < 0 || yy >= bx.ny));
}

// Post-collision velocity of a cell from its own 19 stored slots (slot q of
// cell x holds the value it sent in direction q), in S::to_f64 units.
template <class S>
__device__ inline void slot_velocity(const BoxDev& bx, const typename S::T* g, int x, int y, int z, float inv,
                                     double u[3]) {
    u[0] = u[1] = u[2] = 0.0;
    for (int q = 1; q < NQ; ++q) {
        double v = S::to_f64(g[pdf_index(bx, q, x, y, z)], inv);
        u[0] += v * CX[q]; u[1] += v * CY[q]; u[2] += v * CZ[q];
    }
}

// Anti-bounce-back: the population entering in direction q through a
// pressure face, from the one sent in direction inv_dir(q) (s_opp), the face
// density term rho (minus 1 in deviation units) and the cell's velocity u.
__device__ inline double abb_value(int q, double s_opp, double rho, const double u[3]) {
    double cu = CX[q] * u[0] + CY[q] * u[1] + CZ[q] * u[2];
    double uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    return -s_opp + 2.0 * wq(q) * (rho + 4.5 * cu * cu - 1.5 * uu);
}

// Canonical f_q(x, t) of cell (x, y, z) from the stored (pulled) layout, in
// the units of S::to_f64 (the deviation for the deviation forms): the value
// streamed from x - c_q, or, through a face, the face rule applied to the
// population the cell sent against it (direction inv_dir(q)).
template <class S>
__device__ inline double pull_value(const BoxDev& bx, const typename S::T* g, int q, int x, int y, int z, float inv) {
    if (behind_side_wall(bx, x - CX[q], y - CY[q]))   // resting side wall: bounce-back
        return S::to_f64(g[pdf_index(bx, inv_dir(q), x, y, z)], inv);
    int zs = z - CZ[q];
    int w = face_of(bx, zs);
    if (w >= 0) {
        double so = S::to_f64(g[pdf_index(bx, inv_dir(q), x, y, z)], inv);
        if (bx.face_type[w] == FACE_PRESSURE) {
            double u[3];
            slot_velocity<S>(bx, g, x, y, z, inv, u);
            return abb_value(q, so, S::DEV ? bx.face_rho[w] - 1.0 : bx.face_rho[w], u);
        }
        return so + bx.bw[w][q];
    }
    int xs = x - CX[q], ys = y - CY[q];
    xs = xs < 0 ? xs + bx.nx : (xs >= bx.nx ? xs - bx.nx : xs);
    ys = ys < 0 ? ys + bx.ny : (ys >= bx.ny ? ys - bx.ny : ys);
    zs = zs < 0 ? zs + bx.nz : (zs >= bx.nz ? zs - bx.nz : zs);
    return S::to_f64(g[pdf_index(bx, q, xs, ys, zs)], inv);
}

// Inverse of pull_value for the 19 slots of cell (x, y, z): given the
// canonical field through canon(dir, cell) (FP64, full f), the slot values
// that pulling turns back into it. A slot whose reader is inside (or across
// a periodic boundary) holds the reader's value; a slot sent against a
// velocity face holds the cell's own opposite value minus the wall term; the
// slots sent against a pressure face solve the anti-bounce-back rule, whose
// velocity depends on all 19 slots, by fixed-point iteration (the
// dependence is quadratic in the velocity, so a few sweeps reach round-off).
template <class S, class Canon>
__device__ inline void store_cell_slots(const BoxDev& bx, typename S::T* g, int x, int y, int z, float scale,
                                        Canon canon) {
    const long long self = x + (long long)bx.nx * (y + (long long)bx.ny * z);
    double sl[NQ];
    int pface = -1;
    for (int q = 0; q < NQ; ++q) {
        int zd = z + CZ[q];
        int w = face_of(bx, zd);
        if (behind_side_wall(bx, x + CX[q], y + CY[q])) {
            sl[q] = canon(inv_dir(q), self);
        } else if (w < 0) {
            int xd = x + CX[q], yd = y + CY[q];
            xd = xd < 0 ? xd + bx.nx : (xd >= bx.nx ? xd - bx.nx : xd);
            yd = yd < 0 ? yd + bx.ny : (yd >= bx.ny ? yd - bx.ny : yd);
            zd = zd < 0 ? zd + bx.nz : (zd >= bx.nz ? zd - bx.nz : zd);
            sl[q] = canon(q, xd + (long long)bx.nx * (yd + (long long)bx.ny * zd));
        } else if (bx.face_type[w] == FACE_VELOCITY) {
            sl[q] = canon(inv_dir(q), self) - bx.bw[w][inv_dir(q)];
        } else {
            sl[q] = -canon(inv_dir(q), self) + 2.0 * wq(q) * bx.face_rho[w];
            pface = w;
        }
    }
    if (pface >= 0) {
        for (int it = 0; it < 12; ++it) {
            double u[3] = {0.0, 0.0, 0.0};
            for (int q = 1; q < NQ; ++q) {
                u[0] += sl[q] * CX[q]; u[1] += sl[q] * CY[q]; u[2] += sl[q] * CZ[q];
            }
            for (int q = 0; q < NQ; ++q)
                if (face_of(bx, z + CZ[q]) == pface && !behind_side_wall(bx, x + CX[q], y + CY[q]))
                    sl[q] = abb_value(q, canon(inv_dir(q), self), bx.face_rho[pface], u);
        }
    }
    for (int q = 0; q < NQ; ++q) {
        double v = S::DEV ? sl[q] - wq(q) : sl[q];
        g[pdf_index(bx, q, x, y, z)] = S::from_f64(v, scale);
    }
}

// Tiles of the state I/O kernels: 256 cells of one z-plane, rows of 16 to 64,
// one cell per thread, walked like the step's tiles (each die takes a
// contiguous eighth, so that the lines two x-neighbouring tiles share in a
// shifted access meet in one L2; psm_get_pdfs has a walk of its own). HBM bound.
// With an index division per cell, 64-bit addresses and boundary rules for every
// value these kernels moved 1.3-5 TB/s, now 5.2-6.5 like the step's own pattern
// (us at 256^3):
//   read-out of rho and u  FP64 904 -> 588, FP32 769 -> 333, FP16 746 -> 209
//   set_pdfs               FP64 1210 -> 924, FP32 990 -> 697, FP16 990 -> 593
// Cells next to a wall or face are left to the general kernels after them (which
// take a small box alone).
struct RowGrid {
    int shift;            // rows of 1 << shift cells
    int nbx, nby, T;
    unsigned div_x[2], div_y[2];
};

static RowGrid row_grid(const BoxDev& bx) {
    RowGrid g;
    g.shift = bx.nx <= 16 ? 4 : (bx.nx <= 32 ? 5 : 6);
    g.nbx = (bx.nx + (1 << g.shift) - 1) >> g.shift;
    const int rows = 256 >> g.shift;
    g.nby = (bx.ny + rows - 1) / rows;
    g.T = g.nbx * g.nby * bx.nz;
    udiv_magic(g.nbx, g.div_x);
    udiv_magic(g.nby, g.div_y);
    return g;
}

static unsigned row_blocks(const RowGrid& g) { return (unsigned)(g.T + NXCD - 1) / NXCD * NXCD; }

// The cell of this thread; false past the end of the tiles or of the box.
__device__ __forceinline__ bool row_cell(const RowGrid& g, const BoxDev& bx, int& x, int& y, int& z) {
    const int xcd = blockIdx.x % NXCD, m = blockIdx.x / NXCD;
    const int t = (int)(((long long)g.T * xcd) / NXCD) + m;
    if (t >= (int)(((long long)g.T * (xcd + 1)) / NXCD)) return false;
    const int r = udiv(t, g.div_x[0], g.div_x[1]);
    z = udiv(r, g.div_y[0], g.div_y[1]);
    const int tid = threadIdx.x;
    x = ((t - r * g.nbx) << g.shift) + (tid & ((1 << g.shift) - 1));
    y = (r - z * g.nby) * (256 >> g.shift) + (tid >> g.shift);
    return x < bx.nx && y < bx.ny;
}

// The cell of this thread where a kernel writes 19 canonical values per cell: 256
// cells of a plane in index order, as they lie in the field, whatever its row
// length; rows cut into tiles leave partial lines to several workgroups. LINES
// (every direction of the field starts at a 128-byte line): nontemporal
// stores, and the dies share consecutive blocks, which keeps the 19 streams
// close together; else ordinary stores, whose partial lines meet in the L2 of a
// die that takes a contiguous eighth. psm_get_pdfs, us, tiles / index order with
// either, FP64: 256^3 928 / 885 / 969, 97 x 92 x 184 130 / 90 / 106,
// 109 x 272 x 40 83 / 57 / 80; not at lines 581 x 455 x 143 3146 / 2578 / 2326,
// 332 x 134 x 547 1828 / 1440 / 1439; FP32 581 x 455 x 143 2666 / 2150 / 1770.
// Blocks start at lines of the field also where planes do not (74 x 131 x 696
// FP64 428 -> 390 us, FP32 362 -> 299).
struct IndexGrid {
    int nb, T;            // blocks per plane, and in all
    unsigned div_nb[2], div_nx[2];
};

static IndexGrid index_grid(const BoxDev& bx) {
    IndexGrid g;
    g.nb = (bx.nx * bx.ny + (bx.nx * bx.ny % 16 ? 15 : 0) + 255) / 256;
    g.T = g.nb * bx.nz;
    udiv_magic(g.nb, g.div_nb);
    udiv_magic(bx.nx, g.div_nx);
    return g;
}

// A value of a field that is read out.
template <bool LINES, class V> __device__ __forceinline__ void put(V* p, V v) {
    if constexpr (LINES) __builtin_nontemporal_store(v, p);
    else *p = v;
}

template <bool LINES>
__device__ __forceinline__ bool index_cell(const IndexGrid& g, const BoxDev& bx, int& x, int& y, int& z) {
    const int xcd = blockIdx.x % NXCD;
    const int t = LINES ? (int)blockIdx.x : (int)(((long long)g.T * xcd) / NXCD) + (int)blockIdx.x / NXCD;
    if (t >= (LINES ? g.T : (int)(((long long)g.T * (xcd + 1)) / NXCD))) return false;
    z = udiv(t, g.div_nb[0], g.div_nb[1]);
    // blocks start at whole lines of the field also where planes do not
    const int plane = bx.nx * bx.ny, i = (t - z * g.nb) * 256 + (int)threadIdx.x - ((z & 15) * (plane & 15) & 15);
    if (i < 0 || i >= plane) return false;
    y = udiv(i, g.div_nx[0], g.div_nx[1]);
    x = i - y * bx.nx;
    return true;
}

// True for the cells whose values a wall or face enters.
__device__ __forceinline__ bool at_wall(const BoxDev& bx, int x, int y, int z) {
    return (bx.walls && (z == 0 || z == bx.nz - 1)) || ((bx.walls_xy & 1) && (x == 0 || x == bx.nx - 1)) ||
           ((bx.walls_xy & 2) && (y == 0 || y == bx.ny - 1));
}
static bool has_walls(const BoxDev& bx) { return bx.walls || bx.walls_xy; }

// A box with walls of at most so many cells: its general kernel alone, see wall_cell().
static bool general_alone(const BoxDev& bx, int cells) { return has_walls(bx) && bx.N <= cells; }
static bool general_set_pdfs(const BoxDev& bx, int storage) { return general_alone(bx, storage == 2 ? 1 << 19 : 1 << 20); }
static bool general_equilibrium(const BoxDev& bx, int storage) {
    return general_alone(bx, storage == 0 && (bx.walls_xy & 1) ? 1 << 20 : 1 << 19);
}
static bool general_macroscopic(const BoxDev& bx) { return general_alone(bx, 3 << 17); }
static bool general_get_pdfs(const BoxDev& bx, int storage) {
    return general_alone(bx, 5 << 18) || ((bx.walls_xy & 1) && (storage == 0 || (bx.N > 3 << 20 && bx.nx < 224)));
}

// Number of those cells, and cell i of them: the two z planes, then of the
// planes between the two rows at y, then of the rows between the two ends. The
// kernels over them launch one thread for each (500 x 200 x 800 with walls on
// all sides, fields of its 1.3 M such cells: a thread per cell of the box 1113
// us, these about 200; psm_get_macroscopic 3861 / 2947).
__host__ __device__ inline long long wall_cells(const BoxDev& bx) {
    const long long nzi = bx.nz - (bx.walls ? 2 : 0), nyi = bx.ny - ((bx.walls_xy & 2) ? 2 : 0);
    return (bx.walls ? 2LL * bx.nx * bx.ny : 0) + ((bx.walls_xy & 2) ? 2 * nzi * bx.nx : 0) +
           ((bx.walls_xy & 1) ? 2 * nzi * nyi : 0);
}
// ALL: every cell of the box instead, in index order, where one launch of a
// general kernel takes less than two (all / the two, us: 8 x 15 x 89 between z
// walls psm_get_pdfs 8 / 12; 64^3 between walls on all sides FP64 psm_get_pdfs 17 /
// 30, psm_set_pdfs 18 / 31, psm_get_macroscopic 16 / 24, psm_set_equilibrium 22 /
// 32; 96^3 FP64 51 / 62, 57 / 63, 43 / 39, 65 / 68, FP16 37 / 49, 55 / 48, 46 / 30, 63 /
// 56), and where psm_get_pdfs would write the ends of rows at x walls apart from
// the rows, each a line of its own for every direction: in FP64 (124 x 194 x 974
// 1404 / 1992, 256^3 999 / 1133), in the deviation forms where the rows are short
// and the field exceeds the caches (FP32 124 x 194 x 974 1314 / 1631, 203 x 385 x 144
// 612 / 759; but 128^3 119 / 100, 500 x 200 x 400 2029 / 1897). Walls within the
// kernels of the interior instead: FP32 psm_get_macroscopic of 128^3 between x
// walls 94 against 54, between z walls 40 against 45.
template <bool ALL>
__device__ __forceinline__ bool wall_cell(const BoxDev& bx, int& x, int& y, int& z) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (ALL ? (long long)bx.N : wall_cells(bx))) return false;
    unsigned k = (unsigned)i;   // cells of a box are counted in int
    const unsigned nx = bx.nx, plane = nx * bx.ny;
    if (ALL) {
        z = k / plane;
        k -= z * plane;
        y = k / nx;
        x = k - y * nx;
        return true;
    }
    if (bx.walls) {
        if (k < 2 * plane) {
            z = k < plane ? 0 : bx.nz - 1;
            k -= k < plane ? 0 : plane;
            y = k / nx;
            x = k - y * nx;
            return true;
        }
        k -= 2 * plane;
    }
    const int z0 = bx.walls ? 1 : 0, nzi = bx.nz - 2 * z0, y0 = (bx.walls_xy & 2) ? 1 : 0;
    if (y0) {
        if (k < 2 * nx * nzi) {
            const unsigned row = k / nx;
            x = k - row * nx;
            z = z0 + (row >> 1);
            y = row & 1 ? bx.ny - 1 : 0;
            return true;
        }
        k -= 2 * nx * nzi;
    }
    const unsigned nyi = bx.ny - 2 * y0, row = k >> 1;
    x = k & 1 ? bx.nx - 1 : 0;
    z = z0 + row / nyi;
    y = y0 + row % nyi;
    return true;
}

// The 19 stored values that stream into cell (x, y, z) of a periodic box (or
// away from walls), in the units of S::ld.
template <class S>
__device__ __forceinline__ void pull19(const BoxDev& bx, int parity, int x, int y, int z, typename S::R f[NQ]) {
    using T = typename S::T;
    constexpr int QB = BLK * (int)sizeof(T);
    const int xm = x == 0 ? bx.nx - 1 : x - 1, xp = x == bx.nx - 1 ? 0 : x + 1;
    const int ym = y == 0 ? bx.ny - 1 : y - 1, yp = y == bx.ny - 1 ? 0 : y + 1;
    const int zm = z == 0 ? bx.nz - 1 : z - 1, zp = z == bx.nz - 1 ? 0 : z + 1;
    const int pitch = bx.pitch;
    auto inplane = [pitch](int xx, int yy) -> unsigned { return cell_offset<T>(xx, yy, pitch); };
    const unsigned o00 = inplane(x, y), om0 = inplane(xm, y), op0 = inplane(xp, y);
    const unsigned o0m = inplane(x, ym), o0p = inplane(x, yp);
    const unsigned omm = inplane(xm, ym), opp = inplane(xp, yp), omp = inplane(xm, yp), opm = inplane(xp, ym);
    const long long pbytes = bx.plane_elems * (long long)sizeof(T);
    const char* src = (const char*)bx.grid[parity];
    const Rsrc rz = plane_rsrc(src + z * pbytes, (unsigned)pbytes);
    const Rsrc rm = plane_rsrc(src + zm * pbytes, (unsigned)pbytes);
    const Rsrc rp = plane_rsrc(src + zp * pbytes, (unsigned)pbytes);
    PSM_LOAD19(f, rz, rm, rp, LD_AUX);
}

// FP32 value of v rounded to odd: rounding it on to FP16 gives the nearest FP16
// value of v itself (FP32 has more than two bits beyond FP16's). The direct
// conversion is about 25 instructions.
__device__ __forceinline__ float to_odd(double v) {
    const float f = (float)v;
    const double e = (double)f;
    unsigned b = __float_as_uint(f);
    if (e != v) b = (fabs(e) > fabs(v) ? b - 1 : b) | 1u;   // towards zero, last bit set
    return __uint_as_float(b);
}

// Store the 19 slots sl (full FP64 values) of cell (x, y, z).
template <class S>
__device__ __forceinline__ void store19(const BoxDev& bx, int parity, int x, int y, int z, float scale,
                                        const double sl[NQ]) {
    using T = typename S::T;
    constexpr int QB = BLK * (int)sizeof(T);
    const unsigned o = cell_offset<T>(x, y, bx.pitch);
    const long long pbytes = bx.plane_elems * (long long)sizeof(T);
    const Rsrc d = plane_rsrc((const char*)bx.grid[parity] + z * pbytes, (unsigned)pbytes);
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        double v = sl[q];
        if constexpr (S::DEV) {
            // not fused with the product an equilibrium ends in
#pragma clang fp contract(off)
            v = v - wq(q);
        }
        if constexpr (S::SCALED) S::st(d, o, q * QB, to_odd(v * (double)scale));
        else S::st(d, o, q * QB, (typename S::R)v);
    }
}

// Neighbour x + c_q (periodic): plane and in-plane index of a canonical field.
struct Around {
    int z[3];            // z - 1, z, z + 1
    unsigned xy[3][3];   // [dy + 1][dx + 1]
    __device__ Around(const BoxDev& bx, int x, int y, int z0) {
        z[0] = z0 == 0 ? bx.nz - 1 : z0 - 1;
        z[1] = z0;
        z[2] = z0 == bx.nz - 1 ? 0 : z0 + 1;
        const int xs[3] = {x == 0 ? bx.nx - 1 : x - 1, x, x == bx.nx - 1 ? 0 : x + 1};
        const int ys[3] = {y == 0 ? bx.ny - 1 : y - 1, y, y == bx.ny - 1 ? 0 : y + 1};
#pragma unroll
        for (int b = 0; b < 3; ++b)
#pragma unroll
            for (int a = 0; a < 3; ++a) xy[b][a] = (unsigned)(xs[a] + bx.nx * ys[b]);
    }
};

// E_d(rho, u) of eq. (5)
__device__ __forceinline__ double equilibrium(int d, double r, double vx, double vy, double vz) {
    double cv = CX[d] * vx + CY[d] * vy + CZ[d] * vz;
    double vv = vx * vx + vy * vy + vz * vz;
    return wq(d) * (r + 3.0 * cv + 4.5 * cv * cv - 1.5 * vv);
}

template <class S>
__global__ __launch_bounds__(256) void k_set_pdfs(BoxDev bx, RowGrid rg, int parity, const double* __restrict__ f,
                                                  float scale) {
    int x, y, z;
    if (!row_cell(rg, bx, x, y, z) || at_wall(bx, x, y, z)) return;
    const Around n(bx, x, y, z);
    const long long plane = (long long)bx.nx * bx.ny;
    double sl[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
        sl[q] = (f + (long long)q * bx.N + n.z[CZ[q] + 1] * plane)[n.xy[CY[q] + 1][CX[q] + 1]];
    store19<S>(bx, parity, x, y, z, scale, sl);
}

// Slot q of a cell holds the equilibrium of its neighbour x + c_q, so a tile
// keeps density and velocity of three planes with a rim of one cell in LDS
// while it marches up z: 6 global loads per cell instead of 76, which left the
// kernel waiting for them (256^3: FP64 1115 -> 603 us, FP32 874 -> 402, FP16
// 882 -> 377). LDS reads and FP64 arithmetic bound the FP16 form.
template <class S, int SHIFT>
__global__ __launch_bounds__(256) void k_set_equilibrium(BoxDev bx, RowGrid rg, int depth, int parity,
                                                         const double* __restrict__ rho,
                                                         const double* __restrict__ u, float scale) {
    constexpr int W = 1 << SHIFT, H = 256 >> SHIFT, W2 = W + 2, H2 = H + 2, CELLS = W2 * H2;
    constexpr int PER = (CELLS + 255) / 256;
    __shared__ double2 s_rx[3][CELLS], s_yz[3][CELLS];   // (rho, u_x), (u_y, u_z)
    const int tid = threadIdx.x;
    const int r = udiv(blockIdx.x, rg.div_x[0], rg.div_x[1]);
    const int tz = udiv(r, rg.div_y[0], rg.div_y[1]);
    const int x0 = (blockIdx.x - r * rg.nbx) << SHIFT, y0 = (r - tz * rg.nby) * H;
    const int nx = bx.nx, ny = bx.ny, nz = bx.nz;
    const int z0 = tz * depth, z1 = min(z0 + depth, nz);
    const long long plane = (long long)nx * ny, N = bx.N;
    // the cells of the rimmed tile this thread loads: in-plane index, -1 past the box
    int at[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = tid + 256 * k, cy = i / W2, cx = i - cy * W2;
        int gx = x0 - 1 + cx, gy = y0 - 1 + cy;
        const bool in = i < CELLS && gx <= nx && gy <= ny;
        gx = gx < 0 ? nx - 1 : (gx == nx ? 0 : gx);
        gy = gy < 0 ? ny - 1 : (gy == ny ? 0 : gy);
        at[k] = in ? gx + nx * gy : -1;
    }
    double2 rx[PER], yz[PER];
    auto load = [&](int z) {
        const long long p = (z < 0 ? nz - 1 : (z >= nz ? 0 : z)) * plane;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            if (at[k] < 0) continue;
            rx[k] = make_double2(rho ? (rho + p)[at[k]] : 1.0, (u + p)[at[k]]);
            yz[k] = make_double2((u + N + p)[at[k]], (u + 2 * N + p)[at[k]]);
        }
    };
    auto keep = [&](int slot) {
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            if (at[k] < 0) continue;
            s_rx[slot][tid + 256 * k] = rx[k];
            s_yz[slot][tid + 256 * k] = yz[k];
        }
    };
    const int lx = tid & (W - 1), ly = tid >> SHIFT;
    const int x = x0 + lx, y = y0 + ly;
    const int c0 = (ly + 1) * W2 + lx + 1;
    int lo = 0, mid = 1, hi = 2;   // LDS planes of z - 1, z, z + 1
    load(z0 - 1);
    keep(lo);
    load(z0);
    keep(mid);
    load(z0 + 1);
    for (int z = z0; z < z1; ++z) {
        keep(hi);
        __syncthreads();
        if (z + 1 < z1) load(z + 2);
        if (x < nx && y < ny && !at_wall(bx, x, y, z)) {
            double sl[NQ];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int pl = CZ[q] < 0 ? lo : (CZ[q] > 0 ? hi : mid);
                const int c = c0 + CX[q] + W2 * CY[q];
                const double2 a = s_rx[pl][c], b = s_yz[pl][c];
                sl[q] = equilibrium(q, a.x, a.y, b.x, b.y);
            }
            store19<S>(bx, parity, x, y, z, scale, sl);
        }
        __syncthreads();
        const int t = lo;
        lo = mid; mid = hi; hi = t;
    }
}

// The cells at walls and faces, or with ALL every cell.
template <class S, bool ALL>
__global__ void k_set_pdfs_wall(BoxDev bx, int parity, const double* __restrict__ f, float scale) {
    int x, y, z;
    if (!wall_cell<ALL>(bx, x, y, z)) return;
    typename S::T* g = (typename S::T*)bx.grid[parity];
    const long long N = bx.N;
    store_cell_slots<S>(bx, g, x, y, z, scale, [&](int d, long long c) { return f[(long long)d * N + c]; });
}

template <class S, bool ALL>
__global__ void k_set_equilibrium_wall(BoxDev bx, int parity, const double* __restrict__ rho,
                                       const double* __restrict__ u, float scale) {
    int x, y, z;
    if (!wall_cell<ALL>(bx, x, y, z)) return;
    typename S::T* g = (typename S::T*)bx.grid[parity];
    const long long N = bx.N;
    store_cell_slots<S>(bx, g, x, y, z, scale, [&](int d, long long c) {
        return equilibrium(d, rho ? rho[c] : 1.0, u[c], u[N + c], u[2 * N + c]);
    });
}

// Canonical value of a pulled one (units of S::ld).
template <class S> __device__ __forceinline__ double canonical(typename S::R v, int q, float inv) {
    const double d = S::SCALED ? (double)((float)v * inv) : (double)v;
    return S::DEV ? d + wq(q) : d;
}

template <class S, bool LINES>
__global__ __launch_bounds__(256) void k_get_pdfs(BoxDev bx, IndexGrid ig, int parity, double* __restrict__ f,
                                                  float inv) {
    int x, y, z;
    if (!index_cell<LINES>(ig, bx, x, y, z) || at_wall(bx, x, y, z)) return;
    typename S::R v[NQ];
    pull19<S>(bx, parity, x, y, z, v);
    const unsigned i = (unsigned)(x + bx.nx * y);
    const long long p = (long long)z * bx.nx * bx.ny;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        put<LINES>((f + (long long)q * bx.N + p) + i, canonical<S>(v[q], q, inv));
    }
}

template <class S, bool ALL>
__global__ void k_get_pdfs_wall(BoxDev bx, int parity, double* __restrict__ f, float inv) {
    int x, y, z;
    if (!wall_cell<ALL>(bx, x, y, z)) return;
    const long long n = (long long)z * bx.nx * bx.ny + bx.nx * y + x;
    const typename S::T* g = (const typename S::T*)bx.grid[parity];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        double v = pull_value<S>(bx, g, q, x, y, z, inv);
        if (S::DEV) v += wq(q);
        f[(long long)q * bx.N + n] = v;
    }
}

template <class S>
__global__ void k_get_pdfs_at(BoxDev bx, int parity, const int* __restrict__ cells, int ncells,
                              double* __restrict__ out, float inv, int* __restrict__ flags) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ncells) return;
    long long n = cells[i];
    if (n < 0 || n >= bx.N) {
        // an index outside the box reads nothing: NaN out, flag for the host
        for (int q = 0; q < NQ; ++q) out[(long long)q * ncells + i] = __builtin_nan("");
        atomicOr(flags, FLAG_BAD_CELL);
        return;
    }
    int x = n % bx.nx, y = (n / bx.nx) % bx.ny, z = n / ((long long)bx.nx * bx.ny);
    const typename S::T* g = (const typename S::T*)bx.grid[parity];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        double v = pull_value<S>(bx, g, q, x, y, z, inv);
        if (S::DEV) v += wq(q);
        out[(long long)q * ncells + i] = v;
    }
}

// Density and velocity of one cell from its canonical values, in direction
// order. The terms of zero velocity components are added too: they carry a
// NaN or infinity of any population into every component.
template <class Value>
__device__ __forceinline__ void write_fields(const BoxDev& bx, long long n, double* __restrict__ rho,
                                             double* __restrict__ u, Value value) {
    double r = 0, j[3] = {0, 0, 0};
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const double v = value(q);
        r += v;
        j[0] += v * CX[q]; j[1] += v * CY[q]; j[2] += v * CZ[q];
    }
    __builtin_nontemporal_store(r, rho + n);
#pragma unroll
    for (int a = 0; a < 3; ++a) __builtin_nontemporal_store(j[a] + 0.5 * bx.g[a], u + a * (long long)bx.N + n);
}

template <class S>
__global__ __launch_bounds__(256) void k_macroscopic(BoxDev bx, RowGrid rg, int parity, double* __restrict__ rho,
                                                     double* __restrict__ u, float inv) {
    int x, y, z;
    if (!row_cell(rg, bx, x, y, z) || at_wall(bx, x, y, z)) return;
    typename S::R f[NQ];
    pull19<S>(bx, parity, x, y, z, f);
    write_fields(bx, x + bx.nx * (y + (long long)bx.ny * z), rho, u, [&](int q) { return canonical<S>(f[q], q, inv); });
}

template <class S, bool ALL>
__global__ void k_macroscopic_wall(BoxDev bx, int parity, double* __restrict__ rho, double* __restrict__ u,
                                   float inv) {
    int x, y, z;
    if (!wall_cell<ALL>(bx, x, y, z)) return;
    const long long n = (long long)z * bx.nx * bx.ny + bx.nx * y + x;
    const typename S::T* g = (const typename S::T*)bx.grid[parity];
    write_fields(bx, n, rho, u, [&](int q) {
        const double v = pull_value<S>(bx, g, q, x, y, z, inv);
        return S::DEV ? v + wq(q) : v;
    });
}

// Dense two-slot solid fractions of one box (read-out, or with B null the
// overflow count alone), through the same candidate lists and mapping
// function as the step kernel: a workgroup per plane of a tile, the spheres
// staged in LDS. Fewer than three spheres cannot overflow a cell. Bound by the
// writes (24 B per cell) or the mapping. SAMPLE: boxes that sample; the registers
// of the sampling would halve the waves of the others (256^3 FP64 at 10 % solid
// 206 us, 142 without them, and 136 with a plane per workgroup; 64^3 and depth 16
// at 10 % 77, now 9.6). LINES: rows are whole lines (16 cells), stored past the
// caches. Else tiles leave partial lines to their neighbours in x: the tiles of a
// row run on one die, whose L2 puts the lines together (581 x 455 x 143 without
// spheres 391 us with nontemporal stores and a row over all dies, 171 so).
template <bool LINES, bool SAMPLE>
__global__ __launch_bounds__(WG) void k_map_dense(BoxDev bx, Particles P, const int* __restrict__ tile_cnt,
                                                  const int* __restrict__ tile_off,
                                                  const int2* __restrict__ tile_ent, int list_cap, TileShape ts,
                                                  double* __restrict__ B, int* __restrict__ pid,
                                                  unsigned long long* dropped) {
    __shared__ double s_x[MAXC], s_y[MAXC], s_z[MAXC], s_r[MAXC], s_fr[MAXC];
    __shared__ int s_p[MAXC];
    int lt = blockIdx.x;
    if (!LINES) {
        const int m = lt / NXCD, r = udiv(m, bx.div_ntx[0], bx.div_ntx[1]);   // r * NXCD + die: row of tiles
        lt = (r * NXCD + lt % NXCD) * bx.ntx + m - r * bx.ntx;
        if (lt >= bx.ntx * bx.nty * bx.ntz) return;
    }
    const int t = bx.tile_base + lt;
    const int nc = tile_cnt[t] < list_cap ? tile_cnt[t] : list_cap;
    if (!B && nc < 3) return;
    const int tid = threadIdx.x;
    if (tid < nc) {
        const int p = tile_ent[(tile_off ? (long long)tile_off[t] : (long long)t * list_cap) + tid].x;
        s_p[tid] = p;
        s_x[tid] = P.x[p]; s_y[tid] = P.y[p]; s_z[tid] = P.z[p];
        s_r[tid] = P.r[p]; s_fr[tid] = P.fr[p];
    }
    __syncthreads();
    const int tr = udiv(lt, bx.div_ntx[0], bx.div_ntx[1]);
    const int tcz = udiv(tr, bx.div_nty[0], bx.div_nty[1]);
    const int x = (lt - tr * bx.ntx) * ts.tx + (tid & (ts.tx - 1));
    const int y = (tr - tcz * bx.nty) * ts.ty + (tid >> __builtin_ctz(ts.tx));
    const int z = tcz * ts.tz + (int)blockIdx.y;
    if (x >= bx.nx || y >= bx.ny || z >= bx.nz) return;
    Slots sl;
    slots_init(sl);
    for (int c = 0; c < nc; ++c) {
        const double dx = min_image((x + 0.5) - s_x[c], bx.L[0], bx.halfL[0]);
        const double dy = min_image((y + 0.5) - s_y[c], bx.L[1], bx.halfL[1]);
        const double dz = min_image((z + 0.5) - s_z[c], bx.L[2], bx.halfL[2]);
        const double b = !SAMPLE ? overlap_linear(dx, dy, dz, s_r[c], s_fr[c])
                                 : overlap_subsample(dx, dy, dz, s_r[c], bx.nsub, bx.sub_off, bx.reach);
        if (b > 0.0) slots_insert(sl, s_p[c], s_p[c], b);
    }
    slots_finish(sl);
    const long long n = x + bx.nx * (y + (long long)bx.ny * z);
    if (B) {
        put<LINES>(B + n, sl.c0 >= 0 ? sl.B0 : 0.0);
        put<LINES>(B + bx.N + n, sl.c1 >= 0 ? sl.B1 : 0.0);
        put<LINES>(pid + n, sl.c0 >= 0 ? sl.c0 - bx.part_base : -1);
        put<LINES>(pid + bx.N + n, sl.c1 >= 0 ? sl.c1 - bx.part_base : -1);
    }
    if (sl.dropped) atomicAdd(dropped, (unsigned long long)sl.dropped);
}

// Sum of 4 doubles per thread over the block, in a fixed tree; lane c < 4
// holds component c.
__device__ inline double block_sum4(const double v[4], double (*sh)[256]) {
    const int tid = threadIdx.x;
    for (int k = 0; k < 4; ++k) sh[k][tid] = v[k];
    __syncthreads();
    for (int d = 128; d > 0; d >>= 1) {
        if (tid < d)
            for (int k = 0; k < 4; ++k) sh[k][tid] += sh[k][tid + d];
        __syncthreads();
    }
    return sh[tid & 3][0];
}

// FP64 mass and momentum of the stored state (each slot is one f_q(x,t)):
// per-block partial sums, then one block adds them in a fixed order. A wave
// takes one 64-cell storage block at a time: 19 aligned loads in flight, no
// index division per cell. A call of psm_get_stats, 256^3: FP64 754 -> 493 us,
// FP32 963 -> 271, FP16 940 -> 168; 32^3: 150 -> 26 (the final sum over the
// blocks was serial: 125 us).
template <class S, bool WALL>
__global__ __launch_bounds__(256) void k_stats_partial(BoxDev bx, unsigned div0, unsigned div1, unsigned pit0,
                                                       unsigned pit1, int parity, float inv,
                                                       double* __restrict__ part) {
    using T = typename S::T;
    __shared__ double sh[4][256];
    const T* g = (const T*)bx.grid[parity];
    const int lane = threadIdx.x & 63;
    double m = 0, px = 0, py = 0, pz = 0;
    const long long nblk = (long long)bx.pblk * bx.nz;
    for (long long b = (long long)blockIdx.x * 4 + (threadIdx.x >> 6); b < nblk; b += (long long)gridDim.x * 4) {
        const int z = udiv((int)b, div0, div1);
        const int s = ((int)b - z * bx.pblk) * BLK + lane;
        const int y = udiv(s, pit0, pit1), x = s - y * bx.pitch;
        if (x >= bx.nx || y >= bx.ny) continue;   // padding is never written
        const T* c = g + b * (NQ * BLK) + lane;
        T raw[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) raw[q] = c[q * BLK];
        const bool wall = WALL && at_wall(bx, x, y, z);
        double uc[3] = {0.0, 0.0, 0.0};
        if (wall) slot_velocity<S>(bx, g, x, y, z, inv, uc);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            double v = S::to_f64(raw[q], inv);
            int d = q;
            if (wall) {
                // across a wall or face: the cell's own f_opp(q) by its rule
                const int w = face_of(bx, z + CZ[q]);
                if (behind_side_wall(bx, x + CX[q], y + CY[q])) {
                    d = inv_dir(q);
                } else if (w >= 0) {
                    d = inv_dir(q);
                    v = bx.face_type[w] == FACE_PRESSURE
                            ? abb_value(d, v, S::DEV ? bx.face_rho[w] - 1.0 : bx.face_rho[w], uc)
                            : v + bx.bw[w][d];
                }
            }
            if (S::DEV) v += wq(q);
            m += v;
            px += v * CX[d]; py += v * CY[d]; pz += v * CZ[d];
        }
    }
    const double v[4] = {m, px, py, pz};
    const double sum = block_sum4(v, sh);
    if (threadIdx.x < 4) part[blockIdx.x * 4 + threadIdx.x] = sum;
}

__global__ __launch_bounds__(256) void k_stats_final(const double* part, int nblk, double* out) {
    __shared__ double sh[4][256];
    double v[4] = {0, 0, 0, 0};
    for (int b = threadIdx.x; b < nblk; b += 256)
        for (int k = 0; k < 4; ++k) v[k] += part[b * 4 + k];
    const double sum = block_sum4(v, sh);
    if (threadIdx.x < 4) out[threadIdx.x] = sum;
}

// Plain streaming copy (bandwidth reference): one-shot grid, each thread
// moves one 16-byte vector (of the copy forms measured, the fastest).
__global__ __launch_bounds__(256) void k_stream_copy(const double2* __restrict__ a, double2* __restrict__ b,
                                                     long long n) {
    long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i < n) b[i] = a[i];
}

// ---------------------------------------------------------------------------
// FP64 totals of a canonical field without a context or a workspace, for
// callers that cannot allocate device memory. The per-block partial sums go
// to a library-owned array (one copy per GPU, alive until the process ends):
// block b sums cells [b * per, (b + 1) * per), each thread every 256th of
// them in cell order, then a fixed tree in LDS; one more kernel adds the
// blocks in a fixed order. Every partial slot a call reads was written by the
// same call, so nothing needs clearing; calls that overlap on one GPU
// (different streams) race on the array. Cells per block grow only once the
// array's 4096 blocks are used up (at 64 cells per thread 128^3 cells were 128
// blocks: 510 -> 68 us; 256^3 776 -> 442).
constexpr int NOALLOC_BLOCKS = 4096;
constexpr long long NOALLOC_CELLS_PER_BLOCK = 256LL * 64;   // the most
static __device__ __align__(256) double scratch[NOALLOC_BLOCKS * 4];

__global__ __launch_bounds__(256) void k_field_stats_partial(const double* __restrict__ f, long long N, int per,
                                                             double* __restrict__ part) {
    __shared__ double s[4][256];
    double m = 0.0, px = 0.0, py = 0.0, pz = 0.0;
    const long long c0 = (long long)blockIdx.x * per;
    const long long c1 = c0 + per < N ? c0 + per : N;
    for (long long n = c0 + threadIdx.x; n < c1; n += 256) {
        double v[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) v[q] = f[(long long)q * N + n];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            m += v[q];
            px += v[q] * CX[q]; py += v[q] * CY[q]; pz += v[q] * CZ[q];
        }
    }
    const double v[4] = {m, px, py, pz};
    const double sum = block_sum4(v, s);
    if (threadIdx.x < 4) part[blockIdx.x * 4 + threadIdx.x] = sum;
}

// Device address of `scratch` on each GPU, looked up once per device with
// that device current (the array's name is only a host-side stand-in).
static double* g_scratch_dev[64];
static std::mutex g_scratch_mu;

static hipError_t scratch_of_current_device(double** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_dev[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_dev[dev] = (double*)p;
    }
    *out = g_scratch_dev[dev];
    return hipSuccess;
}

long long noalloc_max_cells() { return NOALLOC_BLOCKS * NOALLOC_CELLS_PER_BLOCK; }

hipError_t launch_field_stats_noalloc(const double* f, long long N, double* out, hipStream_t st) {
    double* part = nullptr;
    hipError_t e = scratch_of_current_device(&part);
    if (e != hipSuccess) return e;
    if (N > noalloc_max_cells()) return hipErrorInvalidValue;
    const int per = 256 * (int)std::max(1LL, (N + 256LL * NOALLOC_BLOCKS - 1) / (256LL * NOALLOC_BLOCKS));
    const int nblk = (int)((N + per - 1) / per);
    if (nblk > 0) hipLaunchKernelGGL(k_field_stats_partial, dim3(nblk), dim3(256), 0, st, f, N, per, part);
    hipLaunchKernelGGL(k_stats_final, dim3(1), dim3(256), 0, st, part, nblk, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Launchers (called by the engine).

static inline unsigned blocks_for(long long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

// ---------------------------------------------------------------------------
// Bandwidth reference for the step's access pattern: the tile walk, pulls and
// stores of k_psm_step with no arithmetic. SHIFT pulls each direction from
// x - c_q on the source planes z, z -+ 1 as the step does; otherwise every
// direction comes from the cell itself. Values are stored unchanged at the
// cell in the other grid (the source grid is not written).
template <class S, bool SHIFT>
__global__ __launch_bounds__(WG) void k_pattern_copy(StepParams kp) {
    using R = typename S::R;
    using T = typename S::T;
    const int tid = threadIdx.x;
    const int TX = kp.tx, TY = kp.ty, TZ = kp.depth, zs = kp.zshift;
    const int lx = tid % TX, ly = tid / TX;
    const int G = gridDim.x;
    const int xcd = blockIdx.x % NXCD;
    const int gx8 = (G - xcd + NXCD - 1) / NXCD;
    const int t_begin = (int)(((long long)kp.T_total * xcd) / NXCD);
    const int t_end = (int)(((long long)kp.T_total * (xcd + 1)) / NXCD);
    const PSM_CONST BoxDev* boxes = cptr(kp.boxes);
    for (int t = t_begin + (int)blockIdx.x / NXCD; t < t_end; t += gx8) {
        int b = 0;
        if (kp.nbox > 1) {
            const PSM_CONST int* tb = cptr(kp.box_tile_base);
            int lo = 0, hi = kp.nbox - 1;
            while (lo < hi) {
                int mid = (lo + hi + 1) >> 1;
                if (tb[mid] << zs <= t) lo = mid; else hi = mid - 1;
            }
            b = lo;
        }
        const PSM_CONST BoxDev& bx = boxes[b];
        const int nx = bx.nx, ny = bx.ny, nz = bx.nz;
        const int lt = t - (bx.tile_base << zs);
        const int tcx = lt % bx.ntx, tcy = (lt / bx.ntx) % bx.nty, tcz = lt / (bx.ntx * bx.nty);
        const int x = tcx * TX + lx, y = tcy * TY + ly;
        if (x >= nx || y >= ny) continue;
        const int xm = x == 0 ? nx - 1 : x - 1, xp = x == nx - 1 ? 0 : x + 1;
        const int ym = y == 0 ? ny - 1 : y - 1, yp = y == ny - 1 ? 0 : y + 1;
        const int pitch = bx.pitch;
        auto inplane = [pitch](int xx, int yy) -> unsigned {
            int c = xx + pitch * yy;
            return (unsigned)(((c / BLK) * (NQ * BLK) + (c % BLK)) * (int)sizeof(T));
        };
        const unsigned o00 = inplane(x, y);
        const unsigned om0 = SHIFT ? inplane(xm, y) : o00, op0 = SHIFT ? inplane(xp, y) : o00;
        const unsigned o0m = SHIFT ? inplane(x, ym) : o00, o0p = SHIFT ? inplane(x, yp) : o00;
        const unsigned omm = SHIFT ? inplane(xm, ym) : o00, opp = SHIFT ? inplane(xp, yp) : o00;
        const unsigned omp = SHIFT ? inplane(xm, yp) : o00, opm = SHIFT ? inplane(xp, ym) : o00;
        const long long pbytes = bx.plane_elems * (long long)sizeof(T);
        const unsigned pb32 = (unsigned)pbytes;
        const char* src = (const char*)bx.grid[kp.parity];
        const char* dst = (const char*)bx.grid[kp.parity ^ 1];
        constexpr int QB = BLK * (int)sizeof(T);
        for (int k = 0; k < TZ; ++k) {
            const int z = tcz * TZ + k;
            if (z >= nz) break;
            const int zm = z == 0 ? nz - 1 : z - 1, zp = z == nz - 1 ? 0 : z + 1;
            const Rsrc sz = plane_rsrc(src + z * pbytes, pb32);
            const Rsrc sm = SHIFT ? plane_rsrc(src + zm * pbytes, pb32) : sz;
            const Rsrc sp = SHIFT ? plane_rsrc(src + zp * pbytes, pb32) : sz;
            const Rsrc dz_ = plane_rsrc(dst + z * pbytes, pb32);
            R f[NQ];
            PSM_LOAD19(f, sz, sm, sp, LD_AUX);
#pragma unroll
            for (int q = 0; q < NQ; ++q) S::st(dz_, o00, q * QB, f[q]);
        }
    }
}

hipError_t launch_pattern_copy(int storage, bool shifted, const StepParams& kp, hipStream_t st) {
    const void* k;
    switch (storage) {
        case 0: k = shifted ? (const void*)k_pattern_copy<St64, true> : (const void*)k_pattern_copy<St64, false>; break;
        case 1: k = shifted ? (const void*)k_pattern_copy<St32, true> : (const void*)k_pattern_copy<St32, false>; break;
        default: k = shifted ? (const void*)k_pattern_copy<St16, true> : (const void*)k_pattern_copy<St16, false>;
    }
    void* args[] = {(void*)&kp};
    return hipLaunchKernel(k, dim3(kp.grid), dim3(WG), args, 0, st);
}

// The step kernel instance for (storage, MAP, FILT, WALL, CACHE): storage
// psm_storage; MAP 1 if any box samples and the context has room for spheres,
// else 0 (the linear approximation); FILT the per-wave candidate filter; WALL if
// any box has walls or faces; CACHE the load and store form (cache_form). The
// filter, which no context starts with, is built for MIXED grids alone: KEEP and
// STREAM were measured without it.
template <int MAP, bool FILT, bool WALL, int CACHE>
static const void* step_kernel_of(int storage) {
    switch (storage) {
        case 0: return (const void*)k_psm_step<St64, MAP, FILT, WALL, CACHE>;
        case 1: return (const void*)k_psm_step<St32, MAP, FILT, WALL, CACHE>;
        default: return (const void*)k_psm_step<St16, MAP, FILT, WALL, CACHE>;
    }
}

template <bool WALL>
static const void* step_kernel_walls(int storage, const StepForm& f) {
    if (f.filter) return f.map ? step_kernel_of<1, true, WALL, MIXED>(storage) : step_kernel_of<0, true, WALL, MIXED>(storage);
    if (f.cache == KEEP) return f.map ? step_kernel_of<1, false, WALL, KEEP>(storage) : step_kernel_of<0, false, WALL, KEEP>(storage);
    if (f.cache == STREAM) return f.map ? step_kernel_of<1, false, WALL, STREAM>(storage) : step_kernel_of<0, false, WALL, STREAM>(storage);
    return f.map ? step_kernel_of<1, false, WALL, MIXED>(storage) : step_kernel_of<0, false, WALL, MIXED>(storage);
}

static const void* step_kernel(int storage, const StepForm& f) {
    return f.walls ? step_kernel_walls<true>(storage, f) : step_kernel_walls<false>(storage, f);
}

hipError_t launch_step(int storage, const StepForm& form, const StepParams& kp, hipStream_t st) {
    void* args[] = {(void*)&kp};
    const unsigned reduce = kp.partial_prev ? blocks_for(kp.P_total, NWAVE) : 0u;
    return hipLaunchKernel(step_kernel(storage, form), dim3(kp.grid + reduce), dim3(WG), args, 0, st);
}

int step_blocks_per_cu(int storage, const StepForm& form) {
    int nb = 0;
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, step_kernel(storage, form), WG, 0);
    return nb > 0 ? nb : 1;
}

// Blocks of 4 spheres, and at least enough to clear the old counts beside them.
template <bool REDUCE, int SCHEME, bool BIN, bool UPLOAD = false>
static hipError_t launch_spheres_of(const SphereParams& sp, hipStream_t st, const UploadParams& up = UploadParams{}) {
    unsigned nb = blocks_for(sp.P_total, 4);
    if (BIN) {
        const unsigned clear = blocks_for(sp.T_total, 1024);
        nb = std::max(nb, std::min(clear, 1024u));
    }
    hipLaunchKernelGGL((k_spheres<REDUCE, SCHEME, BIN, UPLOAD>), dim3(nb), dim3(256), 0, st, sp, up);
    return hipGetLastError();
}

hipError_t launch_spheres(bool reduce, int scheme, bool bin, const SphereParams& sp, hipStream_t st) {
    if (sp.P_total == 0) return hipSuccess;
    if (reduce) {
        if (!bin) return launch_spheres_of<true, SCHEME_NONE, false>(sp, st);
        return scheme == SCHEME_EULER ? launch_spheres_of<true, SCHEME_EULER, true>(sp, st)
                                      : launch_spheres_of<true, SCHEME_VERLET, true>(sp, st);
    }
    switch (scheme) {
        case SCHEME_EULER: return launch_spheres_of<false, SCHEME_EULER, true>(sp, st);
        case SCHEME_VERLET: return launch_spheres_of<false, SCHEME_VERLET, true>(sp, st);
        default: return launch_spheres_of<false, SCHEME_NONE, true>(sp, st);
    }
}

hipError_t launch_list_offsets(int* cnt, int* off, int T, int list_cap, hipStream_t st) {
    hipLaunchKernelGGL(k_list_offsets, dim3(blocks_for(T, 256)), dim3(256), 0, st, cnt, off, T, list_cap);
    return hipGetLastError();
}

hipError_t launch_upload_bin(const SphereParams& sp, const UploadParams& up, hipStream_t st) {
    return launch_spheres_of<false, SCHEME_NONE, true, true>(sp, st, up);
}

hipError_t launch_upload(const UploadParams& up, hipStream_t st) {
    const long long n = std::max({(long long)up.ncols * up.n, up.prev_ok ? (long long)up.m : 0LL, 1LL});
    hipLaunchKernelGGL(k_upload, dim3(blocks_for(n, 256)), dim3(256), 0, st, up);
    return hipGetLastError();
}

hipError_t launch_download(const DownloadParams& dp, hipStream_t st) {
    const long long n = std::max(dp.n * std::max(dp.ncols[0], dp.ncols[1]), 1LL);
    hipLaunchKernelGGL(k_download, dim3(std::min(blocks_for(n, 256), 4096u)), dim3(256), 0, st, dp);
    return hipGetLastError();
}

#define PSM_BY_STORAGE(CALL)                \
    switch (storage) {                      \
        case 0: { using S = St64; CALL; } break; \
        case 1: { using S = St32; CALL; } break; \
        default: { using S = St16; CALL; }       \
    }

hipError_t launch_set_pdfs(int storage, const BoxDev& bx, int parity, const double* f, float scale,
                           hipStream_t st) {
    if (general_set_pdfs(bx, storage)) {
        PSM_BY_STORAGE(hipLaunchKernelGGL((k_set_pdfs_wall<S, true>), dim3(blocks_for(bx.N, 256)), dim3(256), 0, st,
                                          bx, parity, f, scale));
        return hipGetLastError();
    }
    const RowGrid rg = row_grid(bx);
    PSM_BY_STORAGE(hipLaunchKernelGGL(k_set_pdfs<S>, dim3(row_blocks(rg)), dim3(256), 0, st, bx, rg, parity, f, scale));
    if (has_walls(bx))
        PSM_BY_STORAGE(hipLaunchKernelGGL((k_set_pdfs_wall<S, false>), dim3(blocks_for(wall_cells(bx), 256)), dim3(256), 0, st,
                                          bx, parity, f, scale));
    return hipGetLastError();
}

hipError_t launch_set_equilibrium(int storage, const BoxDev& bx, int parity, const double* rho, const double* u,
                                  float scale, hipStream_t st) {
    if (general_equilibrium(bx, storage)) {
        PSM_BY_STORAGE(hipLaunchKernelGGL((k_set_equilibrium_wall<S, true>), dim3(blocks_for(bx.N, 256)), dim3(256), 0,
                                          st, bx, parity, rho, u, scale));
        return hipGetLastError();
    }
    const RowGrid rg = row_grid(bx);
    // 16 planes per tile read 18; fewer while that leaves CUs idle
    int depth = 16;
    while (depth > 1 && (long long)rg.nbx * rg.nby * ((bx.nz + depth - 1) / depth) < 1024) depth /= 2;
    const dim3 grid(rg.nbx * rg.nby * ((bx.nz + depth - 1) / depth));
    switch (rg.shift) {
        case 4: PSM_BY_STORAGE(hipLaunchKernelGGL((k_set_equilibrium<S, 4>), grid, dim3(256), 0, st, bx, rg, depth, parity, rho, u, scale)); break;
        case 5: PSM_BY_STORAGE(hipLaunchKernelGGL((k_set_equilibrium<S, 5>), grid, dim3(256), 0, st, bx, rg, depth, parity, rho, u, scale)); break;
        default: PSM_BY_STORAGE(hipLaunchKernelGGL((k_set_equilibrium<S, 6>), grid, dim3(256), 0, st, bx, rg, depth, parity, rho, u, scale));
    }
    if (has_walls(bx))
        PSM_BY_STORAGE(hipLaunchKernelGGL((k_set_equilibrium_wall<S, false>), dim3(blocks_for(wall_cells(bx), 256)), dim3(256), 0, st,
                                          bx, parity, rho, u, scale));
    return hipGetLastError();
}

hipError_t launch_get_pdfs(int storage, const BoxDev& bx, int parity, double* f, float inv, hipStream_t st) {
    if (general_get_pdfs(bx, storage)) {
        PSM_BY_STORAGE(hipLaunchKernelGGL((k_get_pdfs_wall<S, true>), dim3(blocks_for(bx.N, 256)), dim3(256), 0, st,
                                          bx, parity, f, inv));
        return hipGetLastError();
    }
    const IndexGrid ig = index_grid(bx);
    const dim3 grid((unsigned)(ig.T + NXCD - 1) / NXCD * NXCD);
    if (bx.N % 16 == 0 && ((uintptr_t)f & 127) == 0)
        PSM_BY_STORAGE(hipLaunchKernelGGL((k_get_pdfs<S, true>), grid, dim3(256), 0, st, bx, ig, parity, f, inv))
    else
        PSM_BY_STORAGE(hipLaunchKernelGGL((k_get_pdfs<S, false>), grid, dim3(256), 0, st, bx, ig, parity, f, inv))
    if (has_walls(bx))
        PSM_BY_STORAGE(hipLaunchKernelGGL((k_get_pdfs_wall<S, false>), dim3(blocks_for(wall_cells(bx), 256)), dim3(256), 0, st,
                                          bx, parity, f, inv));
    return hipGetLastError();
}

hipError_t launch_get_pdfs_at(int storage, const BoxDev& bx, int parity, const int* cells, int ncells, double* out,
                              float inv, int* flags, hipStream_t st) {
    unsigned g = blocks_for(ncells, 256);
    switch (storage) {
        case 0: hipLaunchKernelGGL(k_get_pdfs_at<St64>, dim3(g), dim3(256), 0, st, bx, parity, cells, ncells, out, inv, flags); break;
        case 1: hipLaunchKernelGGL(k_get_pdfs_at<St32>, dim3(g), dim3(256), 0, st, bx, parity, cells, ncells, out, inv, flags); break;
        default: hipLaunchKernelGGL(k_get_pdfs_at<St16>, dim3(g), dim3(256), 0, st, bx, parity, cells, ncells, out, inv, flags); break;
    }
    return hipGetLastError();
}

hipError_t launch_macroscopic(int storage, const BoxDev& bx, int parity, double* rho, double* u, float inv,
                              hipStream_t st) {
    if (general_macroscopic(bx)) {
        PSM_BY_STORAGE(hipLaunchKernelGGL((k_macroscopic_wall<S, true>), dim3(blocks_for(bx.N, 256)), dim3(256), 0, st,
                                          bx, parity, rho, u, inv));
        return hipGetLastError();
    }
    const RowGrid rg = row_grid(bx);
    PSM_BY_STORAGE(hipLaunchKernelGGL(k_macroscopic<S>, dim3(row_blocks(rg)), dim3(256), 0, st, bx, rg, parity, rho, u,
                                      inv));
    if (has_walls(bx))
        PSM_BY_STORAGE(hipLaunchKernelGGL((k_macroscopic_wall<S, false>), dim3(blocks_for(wall_cells(bx), 256)), dim3(256), 0, st,
                                          bx, parity, rho, u, inv));
    return hipGetLastError();
}

hipError_t launch_map_dense(const BoxDev& bx, const Particles& P, const int* tile_cnt, const int* tile_off,
                            const int2* tile_ent, int list_cap, TileShape ts, double* B, int* pid,
                            unsigned long long* dropped, hipStream_t st) {
    const int rows = bx.nty * bx.ntz;
    const bool lines = bx.nx % 16 == 0;
    const dim3 grid((lines ? rows : (rows + NXCD - 1) / NXCD * NXCD) * bx.ntx, ts.tz);
    const auto k = bx.mapping == 0 ? (lines ? k_map_dense<true, false> : k_map_dense<false, false>)
                                   : (lines ? k_map_dense<true, true> : k_map_dense<false, true>);
    hipLaunchKernelGGL(k, grid, dim3(WG), 0, st, bx, P, tile_cnt, tile_off, tile_ent, list_cap, ts, B, pid, dropped);
    return hipGetLastError();
}

int stats_blocks() { return 2048; }

hipError_t launch_stats(int storage, const BoxDev& bx, int parity, float inv, double* part, double* out,
                        hipStream_t st) {
    // a wave per storage block while there are enough blocks of work for all
    const long long work = ((long long)bx.pblk * bx.nz + 3) / 4;
    const int nb = (int)std::min<long long>(stats_blocks(), work);
    unsigned dz[2], dp[2];
    udiv_magic(bx.pblk, dz);
    udiv_magic(bx.pitch, dp);
    if (has_walls(bx))
        PSM_BY_STORAGE(hipLaunchKernelGGL((k_stats_partial<S, true>), dim3(nb), dim3(256), 0, st, bx, dz[0], dz[1], dp[0],
                                          dp[1], parity, inv, part))
    else
        PSM_BY_STORAGE(hipLaunchKernelGGL((k_stats_partial<S, false>), dim3(nb), dim3(256), 0, st, bx, dz[0], dz[1],
                                          dp[0], dp[1], parity, inv, part))
    hipLaunchKernelGGL(k_stats_final, dim3(1), dim3(256), 0, st, part, nb, out);
    return hipGetLastError();
}

hipError_t launch_fill_int(int* a, long long n, int v, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    unsigned nb = blocks_for(n, 256);
    hipLaunchKernelGGL(k_fill_int, dim3(nb > 4096 ? 4096 : nb), dim3(256), 0, st, a, n, v);
    return hipGetLastError();
}

hipError_t launch_stream_copy(const void* src, void* dst, size_t bytes, hipStream_t st) {
    long long n = (long long)(bytes / 16);
    long long blocks = (n + 255) / 256;
    if (blocks == 0) return hipSuccess;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_stream_copy, dim3((unsigned)blocks), dim3(256), 0, st, (const double2*)src, (double2*)dst,
                       n);
    return hipGetLastError();
}

}  // namespace psm
