// The per-ray pipeline of sec. 3 in two kernels.  Integration (k_box*): emission (3.1), then the index grid
// (3.2, eqs. 3-6).  Finish (k_finish*): aperture and thick lens (3.3, eq. 7), sensor hit and erf-integrated
// Gaussian spot (3.4, eq. 8), deposited as Q32.32 integers with 64-bit atomics.
//
// Precision layout.  The integration inside the box runs in the template type F (float by
// default).  Positions are kept cell-local: an integer cell index plus a fraction of the cell
// (summed in FP64, see rkn_step), so the rounding of a position is relative to the cell size
// rather than to the metres of the scene.  The direction vector T = n dR/ds is kept as its value at the box entry (T_ref,
// constant) plus the accumulated change dT, so the small increments (A + 4B + C)/6 are summed
// into a small number.  Emission, the box entry, the lens and the sensor run in FP64: they cost a
// few hundred operations per ray against a few hundred thousand in the integration loop.
#include "pbr_internal.h"

namespace pbr {
namespace {

constexpr double kTwoPi = 6.283185307179586476925286766559;

// SplitMix64 (Steele, Lea & Flood, OOPSLA 2014) evaluated at counter k: output number k of the
// generator seeded with `seed`.
__device__ __forceinline__ uint64_t splitmix64_at(uint64_t seed, uint64_t k)
{
    uint64_t z = seed + (k + 1ull) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Checked builds: the access that the caller is about to make is in range if ok; a failed test
// is counted in the CNT_BAD_ACCESS slot, and the caller then clamps the index into its buffer or
// skips the access.  Regular builds return true and compile the test and its fix-up out.
__device__ __forceinline__ bool access_ok(const TraceParams &P, bool ok)
{
#if PBR_CHECKED
    if (!ok && P.counters)
        __hip_atomic_fetch_add(P.counters + CNT_BAD_ACCESS, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return ok;
#else
    (void)P;
    (void)ok;
    return true;
#endif
}

// A stage-point coordinate x (cell units, relative to the ray's cell) split into the whole cells it
// lies ahead, floor(x), and the fraction x - floor(x) inside that cell.  For float two instructions
// (v_cvt_flr_i32_f32 saturates out-of-range values; v_fract_f32 keeps the fraction below 1).
template <typename F> __device__ __forceinline__ int split_cell(F x, F &t);
template <> __device__ __forceinline__ int split_cell<float>(float x, float &t)
{
    int o;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(o) : "v"(x));
    t = __builtin_amdgcn_fractf(x);
    return o;
}
template <> __device__ __forceinline__ int split_cell<double>(double x, double &t)
{
    const double o = floor(x);
    t = x - o;
    return (int)o;
}

// The coefficients (cell layout) or corner values (node layout) of one cell, the ray's base cell,
// held in registers.  A ray's position is kept as the integer base cell and a fraction relative to
// it; a stage point whose fractions all lie in [0, 1) is sampled from the registers as it is, and
// only a point outside moves the base to its cell (enter_cell).
template <typename V> struct CellRecord {
    V c[kCellFloat4];
};
using CellCache = CellRecord<float4>;

// FP64 integration through per-cell records keeps them widened: a record serves about four samples of a
// wave, and a conversion issues at the rate of an FP64 multiply-add (4.3 cycles per wave), of which
// a sample takes 28 next to 32 conversions.
using CellCache64 = CellRecord<double4>;
template <typename F, int NODES> struct CacheOf { using type = CellCache; };
template <> struct CacheOf<double, 0> { using type = CellCache64; };

// Node layout: the eight corners (n - 1, grad n) of cell ic, in the order 000, 100, 010, 001, 110,
// 101, 011, 111 (x, y, z offsets), loaded into the cache.  They are interpolated as they are (see
// sample_field): steps in the fine grids this layout serves cross a cell every one or two
// samples, so a per-gather transform into polynomial coefficients would cost more than it saves.
// d: ic minus the cached cell.  A move of one cell towards +z, the way the light travels, keeps the four
// corners of the shared face and loads the other four: half the gather traffic on most crossings.  Every
// other move loads all eight: with a branch for each of the six faces the few lanes that move sideways
// cost their wave a pass of loads and copies per face (BOS pair 4.84 -> 4.57 ms, 512^3 shock 48.3 -> 45.5,
// and 11 registers fewer).
__device__ __forceinline__ void gather_nodes(const TraceParams &P, const int ic[3], const int d[3], CellCache &cc)
{
    const size_t sy = (size_t)P.nx, sz = (size_t)P.nx * (size_t)P.ny;
    {   // Every gathering lane wants the same cell (about a quarter of the gathers on the Tomo-PIV
        // image, a wave's rays travelling together): its eight corners through the scalar cache,
        // which takes them off the texture-data path, the bound of this kernel on fine grids.
        const int u0 = __builtin_amdgcn_readfirstlane(ic[0]), u1 = __builtin_amdgcn_readfirstlane(ic[1]),
                  u2 = __builtin_amdgcn_readfirstlane(ic[2]);
        const bool same = (ic[0] == u0) & (ic[1] == u1) & (ic[2] == u2);
        if (__builtin_amdgcn_ballot_w64(!same) == 0ull) {
            typedef __attribute__((address_space(4))) const float cfloat;  // constant: scalar loads
            cfloat *s = (cfloat *)(P.cells + (size_t)u2 * sz + (size_t)u1 * sy + (size_t)u0);
            auto at = [&](size_t o) { return make_float4(s[4 * o], s[4 * o + 1], s[4 * o + 2], s[4 * o + 3]); };
            float4 *c = cc.c;
            c[0] = at(0); c[1] = at(1); c[2] = at(sy); c[3] = at(sz);
            c[4] = at(sy + 1); c[5] = at(sz + 1); c[6] = at(sz + sy); c[7] = at(sz + sy + 1);
            return;
        }
    }
    const float4 *b = P.cells + (size_t)ic[2] * sz + (size_t)ic[1] * sy + (size_t)ic[0];
    float4 *c = cc.c;
    if (d[0] == 0 && d[1] == 0 && d[2] == 1) {
        c[0] = c[3]; c[1] = c[5]; c[2] = c[6]; c[4] = c[7];
        asm volatile("");  // keeps the branches apart (no merged stores through selected addresses)
    } else {
        c[0] = b[0]; c[1] = b[1]; c[2] = b[sy]; c[4] = b[sy + 1];
    }
    c[3] = b[sz]; c[5] = b[sz + 1]; c[6] = b[sz + sy]; c[7] = b[sz + sy + 1];
}

// The same gather with every load issued last: the kept corners are shifted one axis at a time
// (z, then x, then y, so a diagonal move keeps what it can), and each corner the new cell still
// lacks is loaded by one instruction masked to the lanes that lack it.  The cache ends up with the
// same eight values.  It issues 37% fewer load instructions on the Tomo-PIV image but moves the
// same bytes, which is what the texture-data path spends its time on, and costs more vector and
// scalar instructions; what it does save is registers, so the kernels that also hold FP64 steps
// (mixed precision, calibration) use it: four waves per SIMD instead of three.
__device__ __forceinline__ void gather_nodes_deferred(const TraceParams &P, const int ic[3], const int d[3],
                                                      CellCache &cc)
{
    const size_t sy = (size_t)P.nx, sz = (size_t)P.nx * (size_t)P.ny;
    const float4 *b = P.cells + (size_t)ic[2] * sz + (size_t)ic[1] * sy + (size_t)ic[0];
    float4 *c = cc.c;
    const int dx = d[0], dy = d[1], dz = d[2];
    const bool near = (unsigned)(dx + 1) <= 2u && (unsigned)(dy + 1) <= 2u && (unsigned)(dz + 1) <= 2u;
    // corners of the new cell that the cached cell does not hold: slot bits of the x = 1 corners
    // (1, 4, 5, 7), the x = 0 corners (0, 2, 3, 6), likewise for y and z
    unsigned need = 0xFFu;
    if (near) {
        need = (dx == 1 ? 0xB2u : dx == -1 ? 0x4Du : 0u) | (dy == 1 ? 0xD4u : dy == -1 ? 0x2Bu : 0u) |
               (dz == 1 ? 0xE8u : dz == -1 ? 0x17u : 0u);
        // shift the kept corners into place, one axis at a time (register copies only: every load
        // is issued at the end, so no copy waits on one)
        if (dz == 1) {
            c[0] = c[3]; c[1] = c[5]; c[2] = c[6]; c[4] = c[7];
            asm volatile("");  // keeps mirrored branches apart (no merged stores through selected addresses)
        } else if (dz == -1) {
            c[3] = c[0]; c[5] = c[1]; c[6] = c[2]; c[7] = c[4];
        }
        if (dx == 1) {
            c[0] = c[1]; c[2] = c[4]; c[3] = c[5]; c[6] = c[7];
            asm volatile("");
        } else if (dx == -1) {
            c[1] = c[0]; c[4] = c[2]; c[5] = c[3]; c[7] = c[6];
        }
        if (dy == 1) {
            c[0] = c[2]; c[1] = c[4]; c[3] = c[6]; c[5] = c[7];
            asm volatile("");
        } else if (dy == -1) {
            c[2] = c[0]; c[4] = c[1]; c[6] = c[3]; c[7] = c[5];
        }
    }
    if (need & 0x01u) c[0] = b[0];
    if (need & 0x02u) c[1] = b[1];
    if (need & 0x04u) c[2] = b[sy];
    if (need & 0x08u) c[3] = b[sz];
    if (need & 0x10u) c[4] = b[sy + 1];
    if (need & 0x20u) c[5] = b[sz + 1];
    if (need & 0x40u) c[6] = b[sz + sy];
    if (need & 0x80u) c[7] = b[sz + sy + 1];
}

// Loads cell ic into the cache; d: ic minus the cached cell (any large value when nothing is
// cached).  NODES: 0 per-cell records, 1 and 2 the node layout (its two gathers).
template <int NODES>
__device__ __forceinline__ void gather_cell(const TraceParams &P, const int ic[3], const int d[3], CellCache &cc)
{
    if (NODES == 2) gather_nodes_deferred(P, ic, d, cc);
    else if (NODES) gather_nodes(P, ic, d, cc);
    else {
        const int key = (ic[2] * (P.ny - 1) + ic[1]) * (P.nx - 1) + ic[0];
        const float4 *p = P.cells + (size_t)key * kCellFloat4;
#pragma unroll
        for (int m = 0; m < kCellFloat4; ++m) cc.c[m] = p[m];
    }
}

template <int NODES>
__device__ __forceinline__ void gather_cell(const TraceParams &P, const int ic[3], const int d[3], CellCache64 &cc)
{
    static_assert(NODES == 0, "widened records are per cell");
    CellCache t;
    gather_cell<0>(P, ic, d, t);
#pragma unroll
    for (int k = 0; k < kCellFloat4; ++k) {
        cc.c[k] = double4{(double)t.c[k].x, (double)t.c[k].y, (double)t.c[k].z, (double)t.c[k].w};
        // widened here, once per record, and not at each use
        asm volatile("" : "+v"(cc.c[k].x), "+v"(cc.c[k].y), "+v"(cc.c[k].z), "+v"(cc.c[k].w));
    }
}

// The first cell of a ray (c inside the grid).
template <int NODES, typename C>
__device__ __forceinline__ void first_cell(const TraceParams &P, int c[3], C &cc)
{
    if (PBR_CHECKED && !access_ok(P, (unsigned)c[0] <= (unsigned)(P.nx - 2) && (unsigned)c[1] <= (unsigned)(P.ny - 2) &&
                                         (unsigned)c[2] <= (unsigned)(P.nz - 2))) {
        c[0] = min(max(c[0], 0), P.nx - 2);
        c[1] = min(max(c[1], 0), P.ny - 2);
        c[2] = min(max(c[2], 0), P.nz - 2);
    }
    const int far[3] = {1 << 20, 0, 0};
    gather_cell<NODES>(P, c, far, cc);
}

// One word per fraction that orders like it for values >= 0 and is large for negative ones and NaN,
// and its value at 1: x lies in [0, 1) exactly if unit_word(x) < unit_one.
__device__ __forceinline__ unsigned unit_word(float x) { return __float_as_uint(x); }
__device__ __forceinline__ unsigned unit_word(double x) { return (unsigned)__double2hiint(x); }
template <typename F> struct UnitOne { static constexpr unsigned value = 0x3F800000u; };
template <> struct UnitOne<double> { static constexpr unsigned value = 0x3FF00000u; };

// A point q (relative to the base cell c) outside the base cell: the base moves to the cell that
// holds the point (its record is gathered, the ray's own position fd, f becomes relative to it) and
// q becomes the fraction inside that cell.  The index is clamped to the grid, which keeps every
// gather in bounds whatever the values.  EDGE: the point may lie outside the box; it is then moved
// onto it.
template <typename F, bool EDGE, int NODES, typename C>
__device__ __forceinline__ void enter_cell(const TraceParams &P, C &cc, int c[3], double fd[3], F f[3], F q[3])
{
    const int nmax[3] = {P.nx - 2, P.ny - 2, P.nz - 2};
    int ic[3], d[3];
    bool off = false;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        // NaN becomes finite first where the point is not known to be (fmax/fmin return the number)
        const F x = EDGE ? fmin(fmax(q[a], (F)(-1.0e6)), (F)(1.0e6)) : q[a];
        d[a] = split_cell<F>(x, q[a]);
        ic[a] = c[a] + d[a];
        off = off | ((unsigned)ic[a] > (unsigned)nmax[a]);
    }
    if (__builtin_expect(off, 0)) {  // outside the grid, or on an upper face (fraction 1 of the last cell)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int i = min(max(ic[a], 0), nmax[a]);
            if (EDGE) q[a] = ic[a] < 0 ? (F)0 : q[a];
            q[a] = ic[a] > nmax[a] ? (F)1 : q[a];
            ic[a] = i;
            d[a] = i - c[a];
        }
    }
    if ((d[0] | d[1] | d[2]) != 0) {
        if (PBR_CHECKED && !access_ok(P, (unsigned)ic[0] <= (unsigned)nmax[0] && (unsigned)ic[1] <= (unsigned)nmax[1] &&
                                             (unsigned)ic[2] <= (unsigned)nmax[2])) {
#pragma unroll
            for (int a = 0; a < 3; ++a) ic[a] = min(max(ic[a], 0), nmax[a]);
        }
        gather_cell<NODES>(P, ic, d, cc);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            c[a] = ic[a];
            fd[a] -= (double)d[a];
            f[a] = (F)fd[a];
        }
    }
}

// Trilinear interpolation of (n - 1, grad n) at fractions w of the cached cell.  Returns n - 1, writes
// G = grad n (D = n G, eq. 6, is formed by the caller).
template <typename F, int NODES, typename C>
__device__ __forceinline__ F interpolate(const C &cc, const F w[3], F G[3])
{
    const F x = w[0], y = w[1], z = w[2];
    F v[4];
    if (NODES) {
        // seven linear interpolations per quantity from the corners: along x on the four edges,
        // then y, then z
#define PBR_LERP(a, b, t) ((a) + (t) * ((b) - (a)))
#define PBR_TRI(ch, out)                                                                   \
    {                                                                                      \
        const F e00 = PBR_LERP((F)cc.c[0].ch, (F)cc.c[1].ch, x);                           \
        const F e10 = PBR_LERP((F)cc.c[2].ch, (F)cc.c[4].ch, x);                           \
        const F e01 = PBR_LERP((F)cc.c[3].ch, (F)cc.c[5].ch, x);                           \
        const F e11 = PBR_LERP((F)cc.c[6].ch, (F)cc.c[7].ch, x);                           \
        out = PBR_LERP(PBR_LERP(e00, e10, y), PBR_LERP(e01, e11, y), z);                   \
    }
        PBR_TRI(x, v[0]);
        PBR_TRI(y, v[1]);
        PBR_TRI(z, v[2]);
        PBR_TRI(w, v[3]);
#undef PBR_TRI
#undef PBR_LERP
    } else {
        // the cell's polynomial c0 + x c1 + y c2 + z c3 + xy c4 + xz c5 + yz c6 + xyz c7, Horner form
#define PBR_TRI(ch, out)                                                                   \
    {                                                                                      \
        const F t1 = (F)cc.c[4].ch + z * (F)cc.c[7].ch;                                    \
        const F t2 = (F)cc.c[1].ch + y * t1 + z * (F)cc.c[5].ch;                           \
        const F t3 = (F)cc.c[2].ch + z * (F)cc.c[6].ch;                                    \
        out = (F)cc.c[0].ch + z * (F)cc.c[3].ch + y * t3 + x * t2;                         \
    }
        PBR_TRI(x, v[0]);
        PBR_TRI(y, v[1]);
        PBR_TRI(z, v[2]);
        PBR_TRI(w, v[3]);
#undef PBR_TRI
    }
    G[0] = v[1];
    G[1] = v[2];
    G[2] = v[3];
    return v[0];
}

// The field at the point q relative to the base cell (fractions anywhere): see enter_cell and
// interpolate.  Whether the point has left the base cell is one maximum and one compare over all
// three axes, where finding its cell from scratch takes five slow instructions per axis.
template <typename F, bool EDGE, int NODES, typename C>
__device__ __forceinline__ F sample_field(const TraceParams &P, C &cc, int c[3], double fd[3], F f[3], F q[3],
                                          F G[3])
{
    const unsigned m = max(max(unit_word(q[0]), unit_word(q[1])), unit_word(q[2]));
    if (m >= UnitOne<F>::value) enter_cell<F, EDGE, NODES>(P, cc, c, fd, f, q);
    if (sizeof(F) == sizeof(double) && NODES == 2) {
#pragma unroll
        for (int k = 0; k < kCellFloat4; ++k)
            asm volatile("" : "+v"(cc.c[k].x), "+v"(cc.c[k].y), "+v"(cc.c[k].z), "+v"(cc.c[k].w));
    }
    return interpolate<F, NODES>(cc, q, G);
}

// Margin (cells) that the steps of a run keep from every face they move towards.
constexpr float kFaceMargin = 1.0e-3f;

// Per-launch constants of the integration loop.  The direction of a ray is carried as V = Vr + dV, the
// value at the entry plus the accumulated change, in the units of the kernel's field layout:
//   node layout  V = T, with D = n grad n as the acceleration; a step's increment is g (T + ...), g = h / spacing
//   cell layout  V = W = h T / spacing (cells per step), with (h^2 / spacing) D as the acceleration: g and h
//                drop out of the sums, and an increment takes one rounding instead of three
// Both are eqs. 3 and 5 with g, h, h / 4, h / 2 and h / 6 below.  In FP32 the rounding of the increment is
// the same at every step of a straight path and makes up most of the error of a hit (512^3 shock: up to 1e-5 px
// in T, half that in W).  The node layout keeps T: its images are the ones of 1e8 rays and more, where one ray
// in 1e9 within 1e-6 px of the sensor's border decides a pixel there (with W, two of eight images of 2e8 rays
// gained or lost a ray against the increments in T, 5e-3 of the rms pixel; an image took 1.4% less).
template <typename F> struct StepGeom {
    F s[3];                 // cells: h^2 / spacing
    F g[3], gh[3];          // per unit of V in a full step: cells, half of them
    F hstep, h4, h2, h6;    // the step, a quarter, half, sixth of it
    F reuse;                // see rkn_step
    int last[3];            // n - 1 per axis (the upper face, in cells)
};

template <typename F, int NODES> __device__ __forceinline__ StepGeom<F> step_geom(const TraceParams &P)
{
    constexpr bool f32 = sizeof(F) == sizeof(float);
    StepGeom<F> sg;
    const int nn[3] = {P.nx, P.ny, P.nz};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        sg.last[a] = nn[a] - 1;
        if (NODES) {  // FP32: the constants the host rounded once (uniform: scalar registers)
            sg.g[a] = f32 ? (F)P.g32[a] : (F)P.step_cell[a];
            sg.gh[a] = f32 ? (F)P.gh32[a] : (F)(0.5 * P.step_cell[a]);
            continue;
        }
        sg.g[a] = (F)1;
        sg.gh[a] = (F)0.5;
        sg.s[a] = (F)P.step2_cell[a];
        // an FP32 operation with a scalar-register operand issues at half the rate of one on vector
        // registers alone (4.4 against 2.7 cycles per wave measured): the constants of every sample
        // stay in vector registers
        if (f32) asm("" : "+v"(sg.s[a]));
    }
    sg.hstep = !NODES ? (F)1 : f32 ? (F)P.h32 : (F)P.h;
    sg.h4 = NODES && f32 ? (F)P.h4_32 : (F)0.25 * sg.hstep;
    sg.h2 = NODES && f32 ? (F)P.h2_32 : (F)0.5 * sg.hstep;
    sg.h6 = NODES && f32 ? (F)P.h6_32 : sg.hstep * ((F)1 / (F)6);
    sg.reuse = NODES ? (F)P.reuse32 : (F)(6.0f * kReuse);
    return sg;
}

// The acceleration at the end point of the step before, when that step's last sample serves for it (see
// rkn_step).
// D is D_C of the step before in any case (zero before the first step); cached: the base cell's
// record is loaded.
template <typename F> struct StageCarry {
    F D[3] = {(F)0, (F)0, (F)0};
    bool have = false, cached = false;
};

// One step of eqs. 3 and 5 of length lam * h in the parameter t (dR/dt = T, dT/dt = D), in
// cell units (written here with V = T; see StepGeom).  The position fd (relative to the base cell) is
// accumulated in FP64: its increment is nearly the same every step, so FP32 rounding of the running sum
// would err the same way every step and grow linearly with the step count.  Stage points are formed
// in F, from f = (F)fd.
// With D_A, D_B, D_C the values of D = n grad n at the three stage points, so that eq. 5's
// A = h D_A, B = h D_B, C = h D_C, the sums are regrouped without forming A, B, C:
//   stage B point  R + (h/2) (T + (h/4) D_A)        (= R + h (T/2 + A/8))
//   stage C point  R + h (T + (h/2) D_B)            (= R + h (T + B/2))
//   R'             R + h (T + (h/6) (D_A + 2 D_B))  (= R + h (T + (A + 2B)/6))
//   T'             T + (h/6) (D_A + 4 D_B + D_C)    (= T + (A + 4B + C)/6)
// A partial step (lam = 1) and a full step form the same constants and give the same bits.
// EDGE: points of the step may lie outside the box (see enter_cell).
// The stage C point and R' differ by g h (D_B - D_A) / 6.  In FP32, where that is at most kReuse cells on
// every axis (|D_B - D_A| <= sg.reuse), D_C is also the next step's D_A, which saves a third of the
// samples: nearly all of them in fields as smooth as the turbulence, all but those within the shock in
// the shock's.  The kernel is bound by VALU issue, where a sample costs 34 instructions and this test five.
template <typename F, bool FULL, bool EDGE, int NODES, typename C>
__device__ __forceinline__ void rkn_step(const TraceParams &P, C &cc, int c[3], double fd[3], F f[3],
                                         const F Vr[3], F dV[3], StageCarry<F> &carry, const StepGeom<F> &sg, F lam)
{
    const F hh = FULL ? sg.hstep : lam * sg.hstep;
    const F h4 = FULL ? sg.h4 : (F)0.25 * hh, h2 = FULL ? sg.h2 : (F)0.5 * hh;
    const F h6 = FULL ? sg.h6 : hh * ((F)1 / (F)6);
    F V[3], DA[3], DB[3], G[3], q[3], step[3], sum[3], dn;
    auto sample = [&] { dn = sample_field<F, EDGE, NODES>(P, cc, c, fd, f, q, G); };
    // the acceleration at the sampled point
    auto accel = [&](int a) { return (NODES ? (F)1 + dn : sg.s[a] + sg.s[a] * dn) * G[a]; };
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        V[a] = Vr[a] + dV[a];
        DA[a] = carry.D[a];
    }
    if (sizeof(F) == sizeof(double) || !carry.have) {
#pragma unroll
        for (int a = 0; a < 3; ++a) q[a] = f[a];
        sample();
#pragma unroll
        for (int a = 0; a < 3; ++a) DA[a] = accel(a);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const F gh = FULL ? sg.gh[a] : (F)0.5 * (lam * sg.g[a]);
        q[a] = f[a] + gh * (V[a] + h4 * DA[a]);
    }
    sample();
    // D_A and D_B only through their sums from here on
    F e = (F)0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const F gg = FULL ? sg.g[a] : lam * sg.g[a];
        DB[a] = accel(a);
        q[a] = f[a] + gg * (V[a] + h2 * DB[a]);
        if (sizeof(F) == sizeof(float)) e = fmax(e, fabs(DB[a] - DA[a]));
        step[a] = gg * (V[a] + h6 * (DA[a] + (F)2 * DB[a]));
        sum[a] = DA[a] + (F)4 * DB[a];
    }
    sample();
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        fd[a] += (double)step[a];
        f[a] = (F)fd[a];
        dV[a] = dV[a] + h6 * (accel(a) + sum[a]);
        carry.D[a] = accel(a);
    }
    carry.have = sizeof(F) == sizeof(float) && e <= sg.reuse;
}

template <typename T> __device__ __forceinline__ T pick3(const T v[3], int k)
{
    return k == 0 ? v[0] : (k == 1 ? v[1] : v[2]);
}

// Full steps (at most kRunSteps) the ray can take before any point of a step comes within kFaceMargin
// cells of a face the ray may move towards; 0: the exit rule decides.  No component of T changes by
// more than P.bend32 in kRunSteps steps (a bound on |D| from the range of the density), so the
// path of the run lies between the straight lines of T - bend and T + bend; the stage points lie
// between the same lines.  A field steep enough to leave no step within that bound is tried with the
// bound for one step.
template <typename F>
__device__ __forceinline__ int run_budget(const TraceParams &P, const StepGeom<F> &sg, const int c[3], const double fd[3],
                                          const F Vr[3], const F dV[3], int steps)
{
    float W[3], lo[3], hi[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        W[a] = (float)(sg.g[a] * (Vr[a] + dV[a]));
        lo[a] = ((float)c[a] + (float)fd[a]) - kFaceMargin;
        hi[a] = ((float)(sg.last[a] - c[a]) - (float)fd[a]) - kFaceMargin;
    }
    // a direction that is not a number (or far beyond the grid in one step) takes the exit rule
    if (!(fabsf(W[0]) + fabsf(W[1]) + fabsf(W[2]) < 1.0e6f)) return 0;
    auto reach = [&](float bend) {
        float k = (float)kRunSteps;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float b = P.g32[a] * bend, up = W[a] + b, dn = b - W[a];
            if (up > 0.0f) k = fminf(k, hi[a] * __builtin_amdgcn_rcpf(up));
            if (dn > 0.0f) k = fminf(k, lo[a] * __builtin_amdgcn_rcpf(dn));
        }
        return (int)floorf(k * 0.99999f);
    };
    int k = reach(P.bend32);
    if (k < 1) k = min(reach(P.bend32 * (1.0f / (float)kRunSteps)), 1);
    return min(k, P.max_steps + 1 - steps);
}

// Exit rule: before each step find the smallest straight-line step fraction lam at which the ray
// reaches a face it moves towards; if lam <= 1 take one step of lam (when lam > 0), then move
// straight along the new T onto that face.  (Per-axis values are selected with pick3 / unrolled
// loops: no dynamically indexed arrays.)
enum : int { STEP_GO = 0, STEP_EXIT = 1, STEP_LIMIT = 2 };

// Word of the map of uniform gas (launch_skip_map) for the brick of a position; p: the position in cells, b:
// the brick.
__device__ __forceinline__ unsigned skip_word(const TraceParams &P, const int c[3], const double fd[3], const int last[3],
                                              double p[3], int b[3])
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        p[a] = (double)c[a] + fd[a];
        b[a] = min(max((int)floor(p[a]), 0), last[a] - 1) / kBrick;
    }
    if (PBR_CHECKED && !access_ok(P, b[0] < P.nbx && b[1] < P.nby && b[2] < P.nbz)) return 0u;
    return P.skip[((size_t)b[2] * P.nby + b[1]) * P.nbx + b[0]];
}

// Steps through uniform gas worth leaving the wave for (short of the box's face): a lane that jumps ahead no longer
// crosses cells with its neighbours, and its jump costs the wave a stretch's look.  15,000 rays past a narrow
// bump in 100^3 nodes (527 us when every step was taken): 562 us with jumps of any length, 516 from 32 steps on,
// 425 from 64, 423 from 128; 1e7 rays beside a 256^3 shock 3.66 ms with any, 3.74 from 32, 64 or 128 steps on.
constexpr int kSkipSteps = 2 * kRunSteps;

// Ray in gas of uniform index.  P.skip holds per brick (kBrick^3 cells) two boxes of bricks without a
// gradient at any of their nodes (see launch_skip_map): the cube around it that reaches the nearest
// gradient, and the column of 3 x 3 bricks from it on towards +z.  Within such a box D is exactly zero
// at every sample and the steps are straight and equal, so all that end inside the box are taken at
// once, and if it reaches the box face that the ray heads for, the partial step and the move onto the
// face too: the same number of steps.  Cell layout: the same line, without the rounding of each step's
// increment.  Node layout: each step by the increment that rkn_step rounds (see StepGeom), except where
// the whole field is uniform: nothing bends a ray there, and it keeps its line to the last bit.
// Called at the start of a stretch where the last sample of the ray was zero (or none has been taken): once per run
// of steps, like its neighbours with something to integrate.  Looks every four steps made the rays of a wave
// wait for runs of unequal length (5e5 rays beside a 353^3 shock 1.36 ms, now 0.54, 1.07 when every step was
// taken; 2e8 rays beside the 512^3 one 36.9 and 30.8).  Returns STEP_EXIT when the ray left the box.
// Regions of ambient gas around a flow, the reference render of a BOS pair and the whole volume on
// either side of a shock are of this kind: the 512^3 shock image took 21.7 ms per 1.7e7 rays stepping through
// them (98% of its steps), now 1.63.  The columns matter beside a shock along z, where the cubes are small.
template <typename F, int NODES>
__device__ __forceinline__ int skip_uniform(const TraceParams &P, int c[3], double fd[3], const F Vr[3], const F dV[3],
                                            StageCarry<F> &carry, const StepGeom<F> &sg, int &steps)
{
    const int *last = sg.last;
    int b[3];
    double p[3];
    unsigned word = skip_word(P, c, fd, last, p, b);
    if (skip_distance(word) == 0) return STEP_GO;
    const bool rounded = NODES && P.bend32 != 0.0f;
    double W[3];  // cells per step
#pragma unroll
    for (int a = 0; a < 3; ++a)
        W[a] = rounded ? (double)(sg.g[a] * (Vr[a] + dV[a]))
                       : (NODES ? P.step_cell[a] : 1.0) * ((double)Vr[a] + (double)dV[a]);
    if (!(fabs(W[0]) + fabs(W[1]) + fabs(W[2]) < 1.0e6)) return STEP_GO;
    const double iW[3] = {1.0 / W[0], 1.0 / W[1], 1.0 / W[2]};
    for (;;) {
        const int d = skip_distance(word);
        // bricks the box extends beyond the ray's own: the column where it reaches further ahead
        const int run = W[2] > 0.0 ? skip_run(word) : 0;
        const int side = run > d ? 1 : d - 1, ahead = run > d ? run - 1 : d - 1;
        double s = 3.0e38, end = 0.0;
        int ax = -1;
        bool face = false;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            if (W[a] == 0.0) continue;
            const bool u = W[a] > 0.0;
            const int e = u ? min((b[a] + 1 + (a == 2 ? ahead : side)) * kBrick, last[a]) : max((b[a] - side) * kBrick, 0);
            const double l = fmax(((double)e - p[a]) * iW[a], 0.0);
            if (l < s) {
                s = l;
                ax = a;
                end = (double)e;
                face = e == (u ? last[a] : 0);
            }
        }
        if (ax < 0 || !(s < (double)(P.max_steps - steps))) return STEP_GO;
        // full steps while a whole one stays inside; at a face also the partial step onto it
        const int m = face ? (int)ceil(s) : (int)floor(s * (1.0 - 1.0e-12));
        if (!face && m < kSkipSteps) return STEP_GO;
        steps += m;
        double l = face ? s : (double)m;
        if (rounded && face) {  // the whole steps, then as the exit rule goes: a step of the rounded fraction, the rest
            const double whole = (double)max(m - 1, 0);
#pragma unroll
            for (int a = 0; a < 3; ++a) p[a] += whole * W[a];
            const F lam = (F)(end - pick3<double>(p, ax)) / (F)pick3<double>(W, ax);
#pragma unroll
            for (int a = 0; a < 3; ++a) p[a] += (double)(lam * sg.g[a] * (Vr[a] + dV[a]));
            l = (end - pick3<double>(p, ax)) * pick3<double>(iW, ax);
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const double q = face && a == ax ? end : p[a] + l * W[a];
            c[a] = min(max((int)floor(q), 0), last[a] - 1);
            fd[a] = q - (double)c[a];
        }
        carry.cached = false;
        if (face) return STEP_EXIT;
        word = skip_word(P, c, fd, last, p, b);
        if (skip_distance(word) == 0) return STEP_GO;
    }
}

// One stretch of the integration: a run of full steps that stay clear of the faces (run_budget), or,
// where the straight line of the next full step reaches a face, the partial step of fraction lam
// and, if the ray still heads out, the straight move onto that face.  Returns STEP_EXIT when the
// ray left the box, STEP_LIMIT when it ran out of steps, STEP_GO otherwise.
// step.inside(f): a full step without the edge extension; step.edge(f, lam): a step of fraction lam
// with it (a full step there, at fraction 1, gives the same bits as the inside one wherever both
// apply).
// The test of the faces costs about 50 instructions, as much as a fifth of a step; testing once per
// run of up to kRunSteps = 32 instead of before every step leaves it below 1% of the time, and longer
// runs let lanes that end a run early wait longer for their wave.
template <typename F, int NODES, typename Step, typename C>
__device__ __forceinline__ int trace_stretch(const TraceParams &P, C &cc, int c[3], double fd[3], const F Vr[3],
                                             const F dV[3], StageCarry<F> &carry, const StepGeom<F> &sg, int &steps,
                                             Step &step)
{
    const bool calm = (carry.D[0] == (F)0) & (carry.D[1] == (F)0) & (carry.D[2] == (F)0);
    if (calm && P.skip && skip_uniform<F, NODES>(P, c, fd, Vr, dV, carry, sg, steps) == STEP_EXIT) return STEP_EXIT;
    if (!carry.cached) {
        first_cell<NODES>(P, c, cc);
        carry.cached = true;
    }
    int k = run_budget<F>(P, sg, c, fd, Vr, dV, steps);
    F f[3] = {(F)fd[0], (F)fd[1], (F)fd[2]};
    if (k > 0) {
        steps += k;
        do step.inside(f);
        while (--k > 0);
        return steps > P.max_steps ? STEP_LIMIT : STEP_GO;
    }
    const int *last = sg.last;
    F lam = (F)3.0e38;
    int ax = -1;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const F v = sg.g[a] * (Vr[a] + dV[a]);
        F l = (F)3.0e38;
        if (v > (F)0) l = (F)((double)(last[a] - c[a]) - fd[a]) / v;
        else if (v < (F)0) l = (F)((double)(-c[a]) - fd[a]) / v;
        if (l < lam) { lam = l; ax = a; }
    }
    const bool hit = ax >= 0 && lam <= (F)1;
    const bool up = hit && (pick3<F>(Vr, ax) + pick3<F>(dV, ax)) > (F)0;
    // one call site for both the partial step and the edge-extended full step
    if (!hit || lam > (F)0) {
        step.edge(f, hit ? lam : (F)1);
        ++steps;
    }
    if (!hit) return steps > P.max_steps ? STEP_LIMIT : STEP_GO;
    const F Vn[3] = {Vr[0] + dV[0], Vr[1] + dV[1], Vr[2] + dV[2]};
    const F Va = pick3<F>(Vn, ax);
    if (up ? (Va > (F)0) : (Va < (F)0)) {
        const int la = pick3<int>(last, ax);
        const double target = up ? (double)la : 0.0;
        const double l2 = (target - ((double)pick3<int>(c, ax) + pick3<double>(fd, ax))) /
                          ((double)pick3<F>(sg.g, ax) * (double)Va);
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            if (b == ax) {
                c[b] = up ? la - 1 : 0;
                fd[b] = up ? 1.0 : 0.0;
            } else {
                fd[b] += l2 * (double)sg.g[b] * (double)Vn[b];
            }
        }
        return STEP_EXIT;
    }
    return steps > P.max_steps ? STEP_LIMIT : STEP_GO;  // turned back within the last step
}

// The steps of one precision throughout.
template <typename F, int NODES, typename C> struct PlainStep {
    const TraceParams &P;
    C &cc;
    int *c;
    double *fd;
    const F *Vr;
    F *dV;
    StageCarry<F> &carry;
    const StepGeom<F> &sg;
    __device__ __forceinline__ void inside(F f[3])
    {
        rkn_step<F, true, false, NODES>(P, cc, c, fd, f, Vr, dV, carry, sg, (F)1);
    }
    __device__ __forceinline__ void edge(F f[3], F lam)
    {
        rkn_step<F, false, true, NODES>(P, cc, c, fd, f, Vr, dV, carry, sg, lam);
    }
};

template <typename F, int NODES = 0, typename C>
__device__ __forceinline__ int trace_run(const TraceParams &P, C &cc, int c[3], double fd[3], const F Vr[3],
                                         F dV[3], StageCarry<F> &carry, const StepGeom<F> &sg, int &steps)
{
    PlainStep<F, NODES, C> step{P, cc, c, fd, Vr, dV, carry, sg};
    return trace_stretch<F, NODES>(P, cc, c, fd, Vr, dV, carry, sg, steps, step);
}

// Integrate from the cell-local state until the ray leaves the box (see
// trace_stretch).  Returns the number of steps; sets *limited when max_steps is exceeded.
template <typename F, int NODES = 0, typename C>
__device__ __forceinline__ int trace_box(const TraceParams &P, C &cc, int c[3], double fd[3],
                                         const F Vr[3], F dV[3], bool *limited)
{
    const StepGeom<F> sg = step_geom<F, NODES>(P);
    StageCarry<F> carry;
    int steps = 0;
    for (;;) {
        const int r = trace_run<F, NODES>(P, cc, c, fd, Vr, dV, carry, sg, steps);
        if (r != STEP_GO) {
            *limited = r == STEP_LIMIT;
            return steps;
        }
    }
}

// Ray-sphere intersection on the cap around the vertex.  Vertex at lens-frame z = zv, signed
// radius Rs (centre at zv + Rs), ir = 1 / Rs.  H: hit point, N: unit normal facing -z near the axis.
__device__ __forceinline__ bool cap_hit(const double Pp[3], const double u[3], double zv,
                                        double Rs, double ir, double H[3], double N[3])
{
    #pragma clang fp contract(off)
    const double qx = Pp[0], qy = Pp[1], qz = Pp[2] - zv;
    const double b = qx * u[0] + qy * u[1] + qz * u[2] - Rs * u[2];
    const double cc = qx * qx + qy * qy + qz * qz - 2.0 * Rs * qz;
    const double disc = b * b - cc;
    if (!(disc >= 0.0)) return false;
    const double sq = sqrt(disc);
    const double den = b >= 0.0 ? -(b + sq) : -(b - sq);
    if (den == 0.0) return false;
    const double s = cc / den;  // the smaller root: the cap near the vertex
    H[0] = Pp[0] + s * u[0];
    H[1] = Pp[1] + s * u[1];
    H[2] = Pp[2] + s * u[2];
    N[0] = H[0] * ir;
    N[1] = H[1] * ir;
    N[2] = (H[2] - zv - Rs) * ir;
    return true;
}

// Snell's law (eq. 7) in vector form, eta = n1 / n2; false on total internal reflection.
__device__ __forceinline__ bool snell(const double u[3], const double N[3], double eta, double out[3])
{
    #pragma clang fp contract(off)
    const double ci = -(u[0] * N[0] + u[1] * N[1] + u[2] * N[2]);
    const double k = 1.0 - eta * eta * (1.0 - ci * ci);
    if (k < 0.0) return false;
    const double m = eta * ci - sqrt(k);
    out[0] = eta * u[0] + m * N[0];
    out[1] = eta * u[1] + m * N[1];
    out[2] = eta * u[2] + m * N[2];
    return true;
}

// Aperture, both lens surfaces and the sensor plane (lens frame: z from the front vertex).
__device__ __forceinline__ int optics_to_sensor(const TraceParams &P, const double R[3], const double u[3],
                                double *xpx, double *ypx)
{
    #pragma clang fp contract(off)
    if (!(u[2] > 0.0)) return PBR_RAY_MISSED;
    const double s = (P.z_lens - R[2]) / u[2];
    double A[3] = {R[0] + s * u[0], R[1] + s * u[1], 0.0};
    if (A[0] * A[0] + A[1] * A[1] > P.a * P.a) return PBR_RAY_BLOCKED_APERTURE;
    double H1[3], N[3], v[3], w[3], H2[3];
    if (!cap_hit(A, u, 0.0, P.R, P.inv_R, H1, N)) return PBR_RAY_BLOCKED_LENS;
    if (H1[0] * H1[0] + H1[1] * H1[1] > P.clear * P.clear) return PBR_RAY_BLOCKED_LENS;
    if (!snell(u, N, P.eta_in, v)) return PBR_RAY_TIR;
    if (!cap_hit(H1, v, P.t, -P.R, -P.inv_R, H2, N)) return PBR_RAY_BLOCKED_LENS;
    if (H2[0] * H2[0] + H2[1] * H2[1] > P.clear * P.clear) return PBR_RAY_BLOCKED_LENS;
    if (!snell(v, N, P.eta_out, w)) return PBR_RAY_TIR;
    if (!(w[2] > 0.0)) return PBR_RAY_MISSED;
    const double s2 = (P.z_sensor - P.z_lens - H2[2]) / w[2];
    *xpx = (H2[0] + s2 * w[0]) * P.inv_pitch + 0.5 * (double)P.W;
    *ypx = (H2[1] + s2 * w[1]) * P.inv_pitch + 0.5 * (double)P.H;
    return PBR_RAY_DEPOSITED;
}

__device__ __forceinline__ void atomic_add_u64(unsigned long long *p, unsigned long long v)
{
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------------------------------ general optical chain (sec. 3.3)

// First intersection at s > 1e-12 along P + s u with the sphere of signed radius Rs whose vertex
// is (cx, cy, zv), on the half of the sphere facing its vertex; Rs = 0: the plane z = zv.  Writes
// the hit and the geometric normal (H - C) / Rs ((0, 0, -1) for a plane).
__device__ __forceinline__ bool chain_hit(const double P[3], const double u[3], double cx, double cy, double zv,
                                          double Rs, double H[3], double N[3])
{
    #pragma clang fp contract(off)
    const double eps = 1e-12;
    if (Rs == 0.0) {
        if (u[2] == 0.0) return false;
        const double s = (zv - P[2]) / u[2];
        if (!(s > eps)) return false;
        H[0] = P[0] + s * u[0];
        H[1] = P[1] + s * u[1];
        H[2] = zv;
        N[0] = 0.0; N[1] = 0.0; N[2] = -1.0;
        return true;
    }
    const double C[3] = {cx, cy, zv + Rs};
    const double d[3] = {P[0] - C[0], P[1] - C[1], P[2] - C[2]};
    const double b = d[0] * u[0] + d[1] * u[1] + d[2] * u[2];
    const double c = d[0] * d[0] + d[1] * d[1] + d[2] * d[2] - Rs * Rs;
    const double disc = b * b - c;
    if (disc < 0.0) return false;
    const double sq = sqrt(disc);
    const double q = -(b + (b >= 0.0 ? sq : -sq));  // roots q and c / q without cancellation
    const double ra = q, rb = q != 0.0 ? c / q : q;
    const double r1 = fmin(ra, rb), r2 = fmax(ra, rb);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const double s = k ? r2 : r1;
        if (!(s > eps)) continue;
        const double h[3] = {P[0] + s * u[0], P[1] + s * u[1], P[2] + s * u[2]};
        if ((h[2] - C[2]) * Rs > 0.0) continue;  // the far half of the sphere
#pragma unroll
        for (int a = 0; a < 3; ++a) { H[a] = h[a]; N[a] = (h[a] - C[a]) / Rs; }
        return true;
    }
    return false;
}

// The ray from R along unit u through the chain's surfaces in order, then onto the sensor plane
// (refraction by eq. 7 with total internal reflection, reflection about the local normal, stops
// and rims blocking; a lenslet array refracts at the cap of the lenslet whose cell the ray meets).
__device__ int chain_to_sensor(const TraceParams &P, const double R[3], const double u0[3], double *xpx,
                               double *ypx)
{
    #pragma clang fp contract(off)
    const pbr_optical_chain &ch = *P.chain;
    double X[3] = {R[0], R[1], R[2]}, u[3] = {u0[0], u0[1], u0[2]};
    double n_cur = P.n_inf;
    for (int k = 0; k < ch.n_surfaces; ++k) {
        const pbr_surface f = ch.s[k];
        const bool stop = f.type == PBR_SURF_APERTURE;
        const int blocked = stop ? PBR_RAY_BLOCKED_APERTURE : PBR_RAY_BLOCKED_LENS;
        double cx = 0.0, cy = 0.0, H[3], N[3];
        if (f.type == PBR_SURF_LENSLETS) {  // the lenslet whose square cell the ray enters
            if (!chain_hit(X, u, 0.0, 0.0, f.z, 0.0, H, N)) return PBR_RAY_BLOCKED_LENS;
            cx = f.pitch * floor(H[0] / f.pitch + 0.5);
            cy = f.pitch * floor(H[1] / f.pitch + 0.5);
        }
        if (!chain_hit(X, u, cx, cy, f.z, stop ? 0.0 : f.radius, H, N)) return blocked;
        if (H[0] * H[0] + H[1] * H[1] > f.clear * f.clear) return blocked;
        if (f.type == PBR_SURF_LENSLETS && (fabs(H[0] - cx) > 0.5 * f.pitch || fabs(H[1] - cy) > 0.5 * f.pitch))
            return PBR_RAY_BLOCKED_LENS;
        if (u[0] * N[0] + u[1] * N[1] + u[2] * N[2] > 0.0) { N[0] = -N[0]; N[1] = -N[1]; N[2] = -N[2]; }
        if (f.type == PBR_SURF_MIRROR) {
            const double dn = u[0] * N[0] + u[1] * N[1] + u[2] * N[2];
#pragma unroll
            for (int a = 0; a < 3; ++a) u[a] = u[a] - 2.0 * dn * N[a];
        } else if (!stop) {
            const double n_next = f.n_after > 0.0 ? f.n_after : P.n_inf;
            double v[3];
            if (!snell(u, N, n_cur / n_next, v)) return PBR_RAY_TIR;
            const double vl = sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
#pragma unroll
            for (int a = 0; a < 3; ++a) u[a] = v[a] / vl;
            n_cur = n_next;
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) X[a] = H[a];
    }
    if (u[2] == 0.0) return PBR_RAY_MISSED;
    const double s = (P.z_sensor - X[2]) / u[2];
    if (!(s > 0.0)) return PBR_RAY_MISSED;
    *xpx = (X[0] + s * u[0]) * P.inv_pitch + 0.5 * (double)P.W;
    *ypx = (X[1] + s * u[1]) * P.inv_pitch + 0.5 * (double)P.H;
    return PBR_RAY_DEPOSITED;
}

// ------------------------------------------------------------------ kernel 1: emission, entry

// sec. 3.1: ray j of source s aims at the aperture point (a sqrt(u1) cos 2 pi u2,
// a sqrt(u1) sin 2 pi u2) of the front-vertex plane; (u1, u2) are the two 24-bit fields of
// SplitMix64 output number (s << 32 | j).  The ray goes straight to the box (slab test) and its
// state is written cell-local; a ray that never enters keeps its world position and direction.
// Source position S and unit direction u of ray j of source s as it leaves its source.
__device__ __forceinline__ void initial_direction(const TraceParams &P, int64_t s, int32_t j, double S[3], double u[3])
{
    #pragma clang fp contract(off)
    if (PBR_CHECKED && !access_ok(P, s >= 0 && s < P.n_src)) s = s < 0 ? 0 : P.n_src - 1;
    const float4 sv = P.src[s];
    S[0] = (double)sv.x;
    S[1] = (double)sv.y;
    S[2] = (double)sv.z;
    const uint64_t hsh = splitmix64_at(P.seed, ((uint64_t)s << 32) | (uint64_t)(uint32_t)j);
    const double u1 = (double)(hsh >> 40) * (1.0 / 16777216.0);
    const double u2 = (double)((hsh >> 16) & 0xFFFFFFull) * (1.0 / 16777216.0);
    const double rr = P.a * sqrt(u1);
    double sn, cs;
    sincospi(2.0 * u2, &sn, &cs);
    u[0] = rr * cs - S[0];
    u[1] = rr * sn - S[1];
    u[2] = P.z_lens - S[2];
    const double il = rsqrt(u[0] * u[0] + u[1] * u[1] + u[2] * u[2]);
    u[0] *= il; u[1] *= il; u[2] *= il;
}

// Mie factor of a ray leaving its source along u (sec. 3.1): the intensity table at the
// scattering angle acos(u . laser), linear between its nodes theta_k = k pi / (mie_n - 1).
__device__ __forceinline__ double mie_weight(const TraceParams &P, const double u[3])
{
    #pragma clang fp contract(off)
    double c = u[0] * P.laser[0] + u[1] * P.laser[1] + u[2] * P.laser[2];
    c = fmin(fmax(c, -1.0), 1.0);
    const double t = acos(c) / 3.14159265358979323846 * (double)(P.mie_n - 1);
    int i = min((int)floor(t), P.mie_n - 2);
    if (PBR_CHECKED && !access_ok(P, i >= 0)) i = 0;
    const double f = t - (double)i;
    return P.mie[i] * (1.0 - f) + P.mie[i + 1] * f;
}

// A ray: source s, ray j of it, and the run k of the processing order it belongs to (the positions
// k * rays_per_src ... of one source).
struct RayKey {
    int64_t s;
    int32_t j;
    uint32_t k;
};

// n / rays_per_src by multiplication (Granlund & Montgomery, PLDI 1994, fig. 4.1).  Positions fit 32 bits:
// no accumulation and no training set takes 2^32 rays or more.
__device__ __forceinline__ uint32_t run_of(const TraceParams &P, uint32_t n)
{
    const uint32_t t = __umulhi(P.div_magic, n);
    return (t + ((n - t) >> P.div_sh1)) >> P.div_sh2;
}

// Key of the ray at position q of the processing order.  With a source order, position q is ray
// q mod rays_per_src of source order[q / rays_per_src] (clamped into range), and the key is that
// ray's position without the order: everything the ray is (random numbers, weight, record index,
// per-source sums) follows from the key, so the order changes nothing but the schedule.
__device__ __forceinline__ RayKey ray_key(const TraceParams &P, int64_t q)
{
    RayKey r;
    r.k = run_of(P, (uint32_t)q);
    r.j = (int32_t)((uint32_t)q - r.k * (uint32_t)P.rays_per_src);
    r.s = r.k;
    if (!P.order) return r;
    if (PBR_CHECKED && !access_ok(P, (int64_t)r.k < P.n_src)) return r;
    const int64_t s = P.order[r.k];
    if (PBR_CHECKED) access_ok(P, s >= 0 && s < P.n_src);  // an entry that is no source index is counted
    r.s = s < 0 ? 0 : (s >= P.n_src ? P.n_src - 1 : s);
    return r;
}

__device__ __forceinline__ void emit_ray(const TraceParams &P, const RayKey &key, RayState &r)
{
    // FP64 set-up and optics: no contracted multiply-adds, so every kernel that inlines this
    // (single-image and batched paths) computes the same bits
    #pragma clang fp contract(off)
    double S[3], u[3];
    initial_direction(P, key.s, key.j, S, u);
    double Rw[3] = {S[0], S[1], S[2]};
    bool inside = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) inside = inside && S[a] >= P.lo[a] && S[a] <= P.hi[a];
    bool entered = inside;
    int eax = -1;
    if (!inside) {
        double tn = -1.0e308, tf = 1.0e308;
        bool ok = true;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            if (u[a] != 0.0) {
                const double iu = 1.0 / u[a], t1 = (P.lo[a] - S[a]) * iu, t2 = (P.hi[a] - S[a]) * iu;
                const double nr = t1 < t2 ? t1 : t2, fr = t1 < t2 ? t2 : t1;
                if (nr > tn) { tn = nr; eax = a; }
                if (fr < tf) tf = fr;
            } else if (S[a] < P.lo[a] || S[a] > P.hi[a]) {
                ok = false;
            }
        }
        if (ok && eax >= 0 && tn <= tf && tn >= 0.0) {
            entered = true;
#pragma unroll
            for (int a = 0; a < 3; ++a) Rw[a] = S[a] + tn * u[a];
        }
    }
    if (!entered) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            r.fd[a] = Rw[a];
            r.Tr[a] = (float)u[a];
            r.dT[a] = (float)(u[a] - (double)r.Tr[a]);  // direction kept as a float hi/lo pair
            r.c[a] = 0;
        }
        r.info = 0;
        return;
    }
    const int nn[3] = {P.nx, P.ny, P.nz};
    float f[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double p = (Rw[a] - P.origin[a]) * P.inv_spacing[a];
        if (a == eax) p = u[a] > 0.0 ? 0.0 : (double)(nn[a] - 1);
        p = p < 0.0 ? 0.0 : p;
        p = p > (double)(nn[a] - 1) ? (double)(nn[a] - 1) : p;
        int ci = (int)floor(p);
        ci = ci > nn[a] - 2 ? nn[a] - 2 : ci;
        r.c[a] = ci;
        r.fd[a] = p - (double)ci;
        f[a] = (float)r.fd[a];
    }
    // inside: T = n dR/ds = n u (eq. 4), n interpolated at the entry point
    CellCache cc;
    float G0[3], n0;
    if (P.node_layout) {
        first_cell<2>(P, r.c, cc);
        n0 = 1.0f + interpolate<float, 2>(cc, f, G0);
    } else {
        first_cell<0>(P, r.c, cc);
        n0 = 1.0f + interpolate<float, 0>(cc, f, G0);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {  // T0 as a float hi/lo pair: no rounding of the entry direction
        const double T0 = (double)n0 * u[a];
        r.Tr[a] = (float)T0;
        r.dT[a] = (float)(T0 - (double)r.Tr[a]);
    }
    r.info = RS_ENTERED;
}

// States in memory: groups of 64 rays, each as four planes of 16 bytes per ray, so that a wave's load or
// store instruction covers 1 KB in one piece; the last group of the n states is as much smaller as they
// are fewer.  With each ray's 64 bytes together every instruction touched 64 separate lines: 512^3 shock,
// 2e8 rays, 42.1 -> 39.2 ms, BOS pair 4.57 -> 4.39.
constexpr int64_t kWholeGroups = (int64_t)1 << 62;  // number of states of an array without a smaller last group
__device__ __forceinline__ int64_t state_slot(int64_t i, int64_t n, int &stride)
{
    stride = (i >> 6) == (n >> 6) ? (int)(n & 63) : 64;
    return (i >> 6) * 256 + (i & 63);
}
__device__ __forceinline__ RayState load_state(const RayState *st, int64_t i, int64_t n)
{
    int k;
    const uint4 *q = (const uint4 *)st + state_slot(i, n, k);
    const uint4 v[4] = {q[0], q[k], q[2 * k], q[3 * k]};
    RayState r;
    __builtin_memcpy(&r, v, sizeof r);
    return r;
}
__device__ __forceinline__ void store_state(RayState *st, int64_t i, int64_t n, const RayState &r)
{
    int k;
    uint4 *q = (uint4 *)st + state_slot(i, n, k);
    uint4 v[4];
    __builtin_memcpy(v, &r, sizeof r);
    q[0] = v[0];
    q[k] = v[1];
    q[2 * k] = v[2];
    q[3 * k] = v[3];
}

// Emission on its own, for what reads the states before the integration (the surrogate) or takes them from a
// queue (lane refill).
__global__ void __launch_bounds__(256) k_emit(TraceParams P, RayState *__restrict__ st, int64_t first,
                                              int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    RayState r;
    emit_ray(P, ray_key(P, first + i), r);
    store_state(st, i, n, r);
}

// ------------------------------------------------------------------ kernel 2: the ray equation

// V of a state as the integration carries it (see StepGeom): a float hi/lo pair in FP32 (about 48
// significant bits, no rounding of the entry direction; its low part starts the accumulated change), one
// double in FP64.
template <int NODES>
__device__ __forceinline__ void load_direction(const TraceParams &P, const RayState &r, float Vr[3], float dV[3])
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double V = (NODES ? 1.0 : P.step_cell[a]) * ((double)r.Tr[a] + (double)r.dT[a]);
        Vr[a] = NODES ? r.Tr[a] : (float)V;
        dV[a] = NODES ? r.dT[a] : (float)(V - (double)Vr[a]);
    }
}
template <int NODES>
__device__ __forceinline__ void load_direction(const TraceParams &P, const RayState &r, double Vr[3], double dV[3])
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        Vr[a] = (NODES ? 1.0 : P.step_cell[a]) * ((double)r.Tr[a] + (double)r.dT[a]);
        dV[a] = 0.0;
    }
}
// T back from V, as a float hi/lo pair.
template <typename F, int NODES>
__device__ __forceinline__ void store_direction(const TraceParams &P, RayState &r, const F Vr[3], const F dV[3])
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double T = ((double)Vr[a] + (double)dV[a]) * (NODES ? 1.0 : P.cell_step[a]);
        r.Tr[a] = (float)T;
        r.dT[a] = (float)(T - (double)r.Tr[a]);
    }
}

template <typename F, int NODES = 0>
__device__ __forceinline__ void box_ray(const TraceParams &P, RayState &r)
{
    F Vr[3], dV[3];
    load_direction<NODES>(P, r, Vr, dV);
    typename CacheOf<F, NODES>::type cc;
    bool limited = false;
    const int steps = trace_box<F, NODES>(P, cc, r.c, r.fd, Vr, dV, &limited);
    store_direction<F, NODES>(P, r, Vr, dV);
    r.info = RS_ENTERED | (limited ? RS_LIMITED : 0) | (steps << RS_STEP_SHIFT);
}

// Ray i = k, or i = list[k] for k < *count when a list is given (the rays the surrogate left to
// the tracer, packed densely so that waves are not held by a few scattered rays).
__device__ __forceinline__ bool box_index(int64_t n, const int *__restrict__ list,
                                          const unsigned long long *__restrict__ count, int64_t *i)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (list) {
        const unsigned long long m = *count;
        if ((unsigned long long)k >= m) return false;
        *i = list[k];
        return true;
    }
    *i = k;
    return k < n;
}

// State of ray i at the start of the integration: emitted here (ray first + i of the image), or read where
// another kernel has emitted it (first < 0).  False: the ray has no path through the box; one
// emitted here is stored as it is.  Emitting here takes 64 bytes a ray written and read again and a
// launch off the image: 512^3 shock, 2e8 rays, 39.2 -> 36.5 ms; BOS pair 4.39 -> 4.27 ms; a preview of 2000
// rays 238 -> 232 us.
__device__ __forceinline__ bool start_state(const TraceParams &P, RayState *__restrict__ st, int64_t i, int64_t n,
                                            int64_t first, RayState &r)
{
    if (first < 0) {
        r = load_state(st, i, n);
        return (r.info & (RS_ENTERED | RS_SURR)) == RS_ENTERED;
    }
    emit_ray(P, ray_key(P, first + i), r);
    if (r.info & RS_ENTERED) return true;
    store_state(st, i, n, r);
    return false;
}

template <typename F, int NODES = 0>
__device__ __forceinline__ void box_body(const TraceParams &P, RayState *__restrict__ st, int64_t n,
                                         const int *__restrict__ list, const unsigned long long *__restrict__ count,
                                         int64_t first)
{
    int64_t i;
    if (!box_index(n, list, count, &i)) return;
    RayState r;
    if (!start_state(P, st, i, n, first, r)) return;
    box_ray<F, NODES>(P, r);
    store_state(st, i, n, r);
}

// FP32 integration: 96 VGPRs, five waves per SIMD.  NODES: field stored per node (the corner gather
// needs more registers: four waves per SIMD).
// Bound by VALU issue (about 140 instructions per wave-step, half of wave-steps moving some lane to a new
// cell) with the L2 misses of those moves behind it; four waves per SIMD with nothing spilled are 3% slower
// on the turbulence below.  A render of 5e6 rays through the 128^3 turbulence takes 14.2 ms, 22.6 when
// every stage point's cell was found from scratch and every step took three samples (203
// instructions); 5.2e6 rays through the 257^2 x 81 slice (node layout, BOS pair) 4.29 against 11.3 ms.
template <bool NODES = false>
__global__ void __launch_bounds__(256, NODES ? 4 : 5) k_box32(TraceParams P, RayState *__restrict__ st, int64_t n,
                                                  const int *__restrict__ list,
                                                  const unsigned long long *__restrict__ count, int64_t first)
{
    box_body<float, NODES>(P, st, n, list, count, first);
}

// FP64 integration, bound by VALU issue (every FP64 operation 4.3 cycles per wave).  With the records
// widened on arrival 145 VGPRs and three waves per SIMD: 500,300 rays through the 64^3 turbulence 2.57 ms
// a render, 3.17 with the conversions at each sample (a quarter of the instructions, 172 VGPRs).
template <bool NODES = false>
__global__ void __launch_bounds__(256, 3) k_box64(TraceParams P, RayState *__restrict__ st, int64_t n,
                                               const int *__restrict__ list,
                                               const unsigned long long *__restrict__ count, int64_t first)
{
    box_body<double, NODES>(P, st, n, list, count, first);
}

// Persistent FP32 integration with lane refill: a fixed grid of waves (five per SIMD) takes rays
// from one queue; a lane whose ray has left the box takes the next one at once, one atomic per
// wave for all lanes that need a ray, so that short and long paths do not leave lanes idle until
// the longest ray of a wave is done.  Same per-ray arithmetic as k_box32 (bit-identical states).
// *queue must be zero at launch; every wave leaves once the queue is drained and its lanes idle.
__global__ void __launch_bounds__(256, 5) k_box32_refill(TraceParams P, RayState *__restrict__ st, int64_t n,
                                                         const int *__restrict__ list,
                                                         const unsigned long long *__restrict__ count,
                                                         unsigned long long *__restrict__ queue)
{
    if (P.node_layout) return;  // cell records only (the host never launches it otherwise)
    const int lane = threadIdx.x & 63;
    const unsigned long long total = list ? *count : (unsigned long long)n;
    const StepGeom<float> sg = step_geom<float, 0>(P);
    int64_t i = -1;  // this lane's ray, -1: none
    RayState r;
    float Vr[3], dV[3];
    CellCache cc;
    StageCarry<float> carry;
    int steps = 0;
    bool drained = false;  // the queue had nothing left for this wave
    for (;;) {
        const bool need = i < 0;
        const unsigned long long want = __ballot(need);
        if (want && !drained) {
            unsigned long long base = 0;
            if (lane == 0) base = atomicAdd(queue, (unsigned long long)__popcll(want));
            base = __shfl(base, 0);
            if (base + (unsigned long long)__popcll(want) >= total) drained = true;
            if (need) {
                const unsigned long long k = base + __popcll(want & ((1ull << lane) - 1ull));
                if (k < total) {
                    const int64_t j = list ? (int64_t)list[k] : (int64_t)k;
                    r = load_state(st, j, n);
                    if ((r.info & (RS_ENTERED | RS_SURR)) == RS_ENTERED) {
                        i = j;
                        load_direction<0>(P, r, Vr, dV);
                        carry = StageCarry<float>();
                        steps = 0;
                    }
                }
            }
            continue;  // lanes that drew a ray with nothing to integrate draw again
        }
        if (__ballot(i >= 0) == 0) break;  // queue drained and no lane busy
        if (i >= 0) {
            const int res = trace_run<float>(P, cc, r.c, r.fd, Vr, dV, carry, sg, steps);
            if (res != STEP_GO) {
                store_direction<float, 0>(P, r, Vr, dV);
                r.info = RS_ENTERED | (res == STEP_LIMIT ? RS_LIMITED : 0) | (steps << RS_STEP_SHIFT);
                store_state(st, i, n, r);
                i = -1;
            }
        }
    }
}

// ------------------------------------------------------------------ mixed precision

// FP64 flag of the brick holding cell c (cell clamped onto the grid).
__device__ __forceinline__ bool brick_is_fp64(const TraceParams &P, const int c[3])
{
    const int bx = min(max(c[0], 0), P.nx - 2) / kBrick;
    const int by = min(max(c[1], 0), P.ny - 2) / kBrick;
    const int bz = min(max(c[2], 0), P.nz - 2) / kBrick;
    if (PBR_CHECKED && !access_ok(P, bx < P.nbx && by < P.nby && bz < P.nbz)) return true;
    return P.brick_fp64[((size_t)bz * P.nby + by) * P.nbx + bx] != 0;
}

// Steps whose precision is chosen one by one from the brick of the ray's current cell: FP64 from the
// FP32 state (V = Vr + dV carried in double through the step, then split again into a float hi/lo
// pair), or FP32.
template <int NODES> struct MixedStep {
    const TraceParams &P;
    CellCache &cc;
    int *c;
    double *fd;
    float *Vr, *dV;
    StageCarry<float> &carry;
    const StepGeom<float> &sg;
    int &n64;
    template <bool FULL, bool EDGE> __device__ __forceinline__ void take(float f[3], float lam)
    {
        const int cell[3] = {c[0] + (int)floorf(f[0]), c[1] + (int)floorf(f[1]), c[2] + (int)floorf(f[2])};
        if (!brick_is_fp64(P, cell)) {
            rkn_step<float, FULL, EDGE, NODES>(P, cc, c, fd, f, Vr, dV, carry, sg, lam);
            return;
        }
        const StepGeom<double> sg64 = step_geom<double, NODES>(P);
        StageCarry<double> none;
        double V64[3], d64[3] = {0.0, 0.0, 0.0}, f64[3] = {fd[0], fd[1], fd[2]};
#pragma unroll
        for (int a = 0; a < 3; ++a) V64[a] = (double)Vr[a] + (double)dV[a];
        rkn_step<double, FULL, EDGE, NODES>(P, cc, c, fd, f64, V64, d64, none, sg64, (double)lam);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const double V = V64[a] + d64[a];
            Vr[a] = (float)V;
            dV[a] = (float)(V - (double)Vr[a]);
            f[a] = (float)fd[a];
            carry.D[a] = (float)none.D[a];
        }
        carry.have = false;
        ++n64;
    }
    __device__ __forceinline__ void inside(float f[3]) { take<true, false>(f, 1.0f); }
    __device__ __forceinline__ void edge(float f[3], float lam) { take<false, true>(f, lam); }
};

// trace_box<float> with the step precision chosen per step.
template <int NODES>
__device__ __forceinline__ int trace_box_mixed(const TraceParams &P, CellCache &cc, int c[3], double fd[3],
                                               float Vr[3], float dV[3], bool *limited, int *n64)
{
    const StepGeom<float> sg = step_geom<float, NODES>(P);
    StageCarry<float> carry;
    MixedStep<NODES> step{P, cc, c, fd, Vr, dV, carry, sg, *n64};
    int steps = 0;
    for (;;) {
        const int r = trace_stretch<float, NODES>(P, cc, c, fd, Vr, dV, carry, sg, steps, step);
        if (r != STEP_GO) {
            *limited = r == STEP_LIMIT;
            return steps;
        }
    }
}

// Waves per SIMD: three with per-cell records (168 VGPRs, the records' conversions kept across samples) are
// faster than two (169) by 13% where every step is FP64 (500,300 rays, 64^3 turbulence, 4.72 -> 4.09 ms a render)
// and by 14% where few are (2.5e6 rays, 128^3 shock, 1.19 -> 1.02), and than four with the conversions at each
// sample (4.47, 1.03).
template <bool NODES>
__global__ void __launch_bounds__(256, NODES ? 4 : 3) k_box_mixed(TraceParams P, RayState *__restrict__ st, int64_t n,
                                                   const int *__restrict__ list,
                                                   const unsigned long long *__restrict__ count, int64_t first)
{
    __shared__ unsigned long long s64;
    if (threadIdx.x == 0) s64 = 0ull;
    __syncthreads();
    int64_t i;
    const bool live = box_index(n, list, count, &i);
    int n64 = 0;
    if (live) {
        RayState r;
        if (start_state(P, st, i, n, first, r)) {
            float Vr[3], dV[3];
            load_direction<NODES>(P, r, Vr, dV);
            CellCache cc;
            bool limited = false;
            const int steps = trace_box_mixed<NODES ? 2 : 0>(P, cc, r.c, r.fd, Vr, dV, &limited, &n64);
            store_direction<float, NODES>(P, r, Vr, dV);
            r.info = RS_ENTERED | (limited ? RS_LIMITED : 0) | (steps << RS_STEP_SHIFT);
            store_state(st, i, n, r);
        }
    }
    if (n64) atomicAdd(&s64, (unsigned long long)n64);
    __syncthreads();
    if (threadIdx.x == 0 && s64) atomic_add_u64(P.counters + CNT_STEPS64, s64);
}

// Calibration of the precision policy: each block samples one brick.  Sample ray k starts at a
// uniform point of the brick, aimed at a uniform point of the aperture, and is integrated over
// n_steps full steps in FP32 and in FP64 from the same state.  The two results are compared where
// they matter on the sensor: the apparent source point on the focused plane, times |M| / pitch.
template <bool NODES>
__global__ void __launch_bounds__(256) k_calibrate(TraceParams P, const int *__restrict__ bricks,
                                                   int n_steps, uint64_t seed, double z_focus,
                                                   double px_per_m, float *__restrict__ err)
{
    __shared__ unsigned s_err;
    if (threadIdx.x == 0) s_err = 0u;
    __syncthreads();
    const int b = bricks[blockIdx.x];
    const int bb[3] = {b % P.nbx, (b / P.nbx) % P.nby, b / (P.nbx * P.nby)};
    const int nn[3] = {P.nx, P.ny, P.nz};
    const uint64_t h1 = splitmix64_at(seed, ((uint64_t)(uint32_t)b << 32) | (2u * threadIdx.x));
    const uint64_t h2 = splitmix64_at(seed, ((uint64_t)(uint32_t)b << 32) | (2u * threadIdx.x + 1u));
    const double uu[5] = {(double)(h1 >> 40) * (1.0 / 16777216.0), (double)((h1 >> 16) & 0xFFFFFFull) * (1.0 / 16777216.0),
                          (double)(h2 >> 40) * (1.0 / 16777216.0), (double)((h2 >> 16) & 0xFFFFFFull) * (1.0 / 16777216.0),
                          (double)(h1 & 0xFFFFull) * (1.0 / 65536.0)};
    int c[3];
    double fd[3], X[3];
    float f[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double p = (double)(bb[a] * kBrick) + (double)kBrick * uu[a];
        p = p > (double)(nn[a] - 1) ? (double)(nn[a] - 1) : p;
        int ci = (int)floor(p);
        ci = ci > nn[a] - 2 ? nn[a] - 2 : ci;
        c[a] = ci;
        fd[a] = p - (double)ci;
        f[a] = (float)fd[a];
        X[a] = P.origin[a] + p * P.spacing[a];
    }
    const double rr = P.a * sqrt(uu[3]);
    double sn, cs;
    sincos(kTwoPi * uu[4], &sn, &cs);
    double u[3] = {rr * cs - X[0], rr * sn - X[1], P.z_lens - X[2]};
    const double il = 1.0 / sqrt(u[0] * u[0] + u[1] * u[1] + u[2] * u[2]);
#pragma unroll
    for (int a = 0; a < 3; ++a) u[a] *= il;
    constexpr int L = NODES ? 2 : 0;
    CellCache cc;
    float G0[3];
    first_cell<L>(P, c, cc);
    const float n0 = 1.0f + interpolate<float, L>(cc, f, G0);
    // FP32
    int c32[3] = {c[0], c[1], c[2]};
    double fd32[3] = {fd[0], fd[1], fd[2]};
    RayState r0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double T0 = (double)n0 * u[a];
        r0.Tr[a] = (float)T0;
        r0.dT[a] = (float)(T0 - (double)r0.Tr[a]);
    }
    float Vr[3], dV[3];
    load_direction<L>(P, r0, Vr, dV);
    const StepGeom<float> sg = step_geom<float, L>(P);
    StageCarry<float> a32;
    for (int k = 0; k < n_steps; ++k) rkn_step<float, true, true, L>(P, cc, c32, fd32, f, Vr, dV, a32, sg, 1.0f);
    // FP64
    int c64[3] = {c[0], c[1], c[2]};
    double fd64[3] = {fd[0], fd[1], fd[2]};
    double V64[3], d64[3] = {0.0, 0.0, 0.0};
    const StepGeom<double> sg64 = step_geom<double, L>(P);
#pragma unroll
    for (int a = 0; a < 3; ++a) V64[a] = (L ? 1.0 : P.step_cell[a]) * ((double)n0 * u[a]);
    first_cell<L>(P, c64, cc);
    StageCarry<double> a64;
    double f64[3] = {fd64[0], fd64[1], fd64[2]};
    for (int k = 0; k < n_steps; ++k) rkn_step<double, true, true, L>(P, cc, c64, fd64, f64, V64, d64, a64, sg64, 1.0);
    double q32[2], q64[2];
    {
        double Xa[3], Xb[3], da[3], db[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            Xa[a] = P.origin[a] + ((double)c32[a] + fd32[a]) * P.spacing[a];
            Xb[a] = P.origin[a] + ((double)c64[a] + fd64[a]) * P.spacing[a];
            const double unit = L ? 1.0 : P.step_cell[a];
            da[a] = ((double)Vr[a] + (double)dV[a]) / unit;
            db[a] = (V64[a] + d64[a]) / unit;
        }
        const double ta = (Xa[2] - z_focus) / da[2], tb = (Xb[2] - z_focus) / db[2];
        q32[0] = Xa[0] - ta * da[0]; q32[1] = Xa[1] - ta * da[1];
        q64[0] = Xb[0] - tb * db[0]; q64[1] = Xb[1] - tb * db[1];
    }
    const double e = px_per_m * sqrt((q32[0] - q64[0]) * (q32[0] - q64[0]) + (q32[1] - q64[1]) * (q32[1] - q64[1]));
    const float ef = (float)e;
    if (ef > 0.0f) atomicMax(&s_err, __float_as_uint(ef));
    __syncthreads();
    if (threadIdx.x == 0) err[blockIdx.x] = __uint_as_float(s_err);
}

// ------------------------------------------------------------------ kernel 3: lens, sensor, spot

// Workgroup scope: an LDS instruction of its own.  With the scope of the global addition beside it the two
// merge into one through a pointer of either kind (a flat instruction).
__device__ __forceinline__ void lds_add_u64(unsigned long long *p, unsigned long long v)
{
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Window of the sensor whose deposits a block sums in LDS: pixels [x0, x0 + w) x [y0, y0 + h), rows
// from slot `off` on.
struct DepositWindow {
    int x0, y0, w, h, off;
};

// Spot of one ray (sec. 3.4): fractions of a Gaussian of sigma_px centred at (x, y) over the
// pixels of the (2R+1)^2 window around the hit pixel, each the product of two erf differences,
// times the source weight, rounded to Q32.32.  Pixels inside the block's LDS window are summed
// there first (integer adds, so the order does not matter); the others go straight to HBM.
template <int RF>
__device__ __forceinline__ void deposit(const TraceParams &P, double x, double y, double w,
                                        unsigned long long *tile, const DepositWindow &win)
{
    #pragma clang fp contract(off)
    const int i0 = (int)x, j0 = (int)y;
    const double inv = P.spot_inv;
    float ex[2 * RF + 2], ey[2 * RF + 2];
#pragma unroll
    for (int m = 0; m < 2 * RF + 2; ++m) {
        ex[m] = erff((float)(((double)(i0 - RF + m) - x) * inv));
        ey[m] = erff((float)(((double)(j0 - RF + m) - y) * inv));
    }
    const float wf = (float)w;
#pragma unroll
    for (int dj = 0; dj <= 2 * RF; ++dj) {
        const int jj = j0 - RF + dj;
        if (jj < 0 || jj >= P.H) continue;
        const float fy = 0.5f * (ey[dj + 1] - ey[dj]) * wf;
        const int ly = jj - win.y0;
        const int row = win.off + ly * win.w - win.x0;  // slot of the row's pixel 0 (may lie outside the tile)
#pragma unroll
        for (int di = 0; di <= 2 * RF; ++di) {
            const int ii = i0 - RF + di;
            if (ii < 0 || ii >= P.W) continue;
            const float cval = 0.5f * (ex[di + 1] - ex[di]) * fy;
            if (!(cval > 0.0f)) continue;
            // cval * 2^32 is a float exactly, so its half-even integer is too: 32 bits, or the whole light of a ray
            const float v = __builtin_rintf(cval * 4294967296.0f);
            const unsigned long long q = v < 4294967296.0f ? (unsigned long long)(unsigned)v : 1ull << 32;
            if (!q) continue;
            if ((unsigned)(ii - win.x0) < (unsigned)win.w && (unsigned)ly < (unsigned)win.h)
                lds_add_u64(tile + (row + ii), q);
            else
                atomic_add_u64(P.accum + (size_t)jj * (size_t)P.W + ii, q);
        }
    }
}

// Adds the sensor hits of this wave's deposited rays (on) into the per-source sums.  The rays of
// a source are consecutive, so the wave holds a few runs of one source index each: every run is
// summed across the wave and added by its first lane.  Integer sums (hits in units of 2^-24
// pixel): the result does not depend on the order in which rays arrive.  Wave-uniform control.
__device__ __forceinline__ void add_source_sums(const TraceParams &P, bool on, int64_t s, double xpx,
                                                double ypx)
{
    const long long qx = on ? (long long)rint(xpx * 16777216.0) : 0ll;
    const long long qy = on ? (long long)rint(ypx * 16777216.0) : 0ll;
    unsigned long long pending = __ballot(on);
    while (pending) {
        const int lead = __ffsll((unsigned long long)pending) - 1;
        const int64_t s0 = __shfl(s, lead, 64);
        const bool mine = on && s == s0;
        long long vx = mine ? qx : 0ll, vy = mine ? qy : 0ll, c = mine ? 1ll : 0ll;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            vx += __shfl_xor(vx, o, 64);
            vy += __shfl_xor(vy, o, 64);
            c += __shfl_xor(c, o, 64);
        }
        if ((int)__lane_id() == lead && (!PBR_CHECKED || access_ok(P, s0 >= 0 && s0 < P.n_src))) {
            pbr_source_sum *d = P.src_sums + s0;
            atomic_add_u64((unsigned long long *)&d->sum_x, (unsigned long long)vx);
            atomic_add_u64((unsigned long long *)&d->sum_y, (unsigned long long)vy);
            atomic_add_u64((unsigned long long *)&d->hits, (unsigned long long)c);
        }
        pending &= ~__ballot(mine);
    }
}

// Shared memory of the finish step of one block.  Deposits are summed per group of rays: a run of
// one source's rays where sources have at least kRunRays each, otherwise all rays of the block.
constexpr int kRunRays = 5, kGroups = 64;
static_assert(255 / kRunRays + 2 <= kGroups, "runs of a block");
template <int TILE>
struct FinishShared {
    unsigned long long tile[2 * TILE * TILE];
    unsigned long long cnt[CNT_SLOTS];
    int lo_x[kGroups], hi_x[kGroups], lo_y[kGroups], hi_y[kGroups];  // hit pixels of a group
    DepositWindow win[kGroups];
    int used;  // slots of the windows
};

__device__ __forceinline__ int wave_min(int v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, 64));
    return v;
}

// Lens, sensor, spot, records and counters for the rays [first + base, first + base + 256) of one
// image, whose states are base .. of the n_states at st; rays at or beyond n are padding.  All threads of the block
// take part (barriers inside).
// RFX: footprint radius fixed at compile time (1..8), or 0 to switch on P.rfp per call (batches,
// whose images differ).  A fixed radius keeps the spot arrays, and so the register count, small.
// FEAT: optional steps compiled in only where used (each costs registers): bit 0 the Mie weighting,
// bit 1 a general optical chain in place of the singlet.
// The deposit: each group's window is the bounding box of its hits widened by the footprint, so that
// every pixel of the block is summed in LDS and leaves in one global atomic.  A window fixed around
// the block's first ray left the rays of its other sources to (2R+1)^2 global atomics each, which is
// what this kernel waited for wherever sources have few rays.  5e6 rays of 100 per dot 3.25 -> 0.29 ms,
// 5.2e6 of 1000 per dot 0.87 -> 0.37, 1.7e7 of 2000 per particle 1.38 -> 0.95.  There it is bound by VALU issue
// (busy 83% of the time): 1700 instructions per 64 rays, of which FP64 optics 14%, FP32 (erf) 20% and the rest
// the integers of the deposit; its LDS additions are waited for 4% of the waves' time.
enum : int { FEAT_MIE = 1, FEAT_CHAIN = 2 };
template <int TILE, int RFX = 0, int FEAT = 0>
__device__ __forceinline__ void finish_block(const TraceParams &P, const RayState *__restrict__ st,
                                             int64_t first, int64_t base, int64_t n, int64_t n_states,
                                             FinishShared<TILE> &sh)
{
    #pragma clang fp contract(off)
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int rf = RFX > 0 ? RFX : P.rfp;
    // groups of the block: its rays' runs, counted from the run of its first ray
    const bool by_run = P.rays_per_src >= kRunRays;
    const uint32_t k0 = run_of(P, (uint32_t)(first + base));
    const int64_t last = base + blockDim.x < n ? base + blockDim.x : n;
    const int ngroups = by_run ? (int)(run_of(P, (uint32_t)(first + last - 1)) - k0) + 1 : 1;
    if ((int)threadIdx.x < ngroups) {
        sh.lo_x[threadIdx.x] = sh.lo_y[threadIdx.x] = 0x7fffffff;
        sh.hi_x[threadIdx.x] = sh.hi_y[threadIdx.x] = -1;
    }
    __syncthreads();

    const int64_t i = base + threadIdx.x;
    const bool valid = i < n;
    int status = PBR_RAY_MISSED, nsteps = 0;
    bool entered = false;
    double Rw[3] = {0, 0, 0}, dir[3] = {0, 0, 1}, xpx = 0.0, ypx = 0.0;
    if (valid) {
        const RayState r = load_state(st, i, n_states);
        entered = (r.info & RS_ENTERED) != 0;
        nsteps = entered ? (r.info >> RS_STEP_SHIFT) : 0;
        status = PBR_RAY_DEPOSITED;
        double tn2 = 0.0, T[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            Rw[a] = entered ? P.origin[a] + ((double)r.c[a] + r.fd[a]) * P.spacing[a] : r.fd[a];
            T[a] = (double)r.Tr[a] + (double)r.dT[a];
            tn2 += T[a] * T[a];
        }
        const double it = rsqrt(tn2);
#pragma unroll
        for (int a = 0; a < 3; ++a) dir[a] = T[a] * it;
        if (r.info & RS_LIMITED) status = PBR_RAY_STEP_LIMIT;
        if (status == PBR_RAY_DEPOSITED)
            status = ((FEAT & FEAT_CHAIN) && P.chain) ? chain_to_sensor(P, Rw, dir, &xpx, &ypx)
                                                      : optics_to_sensor(P, Rw, dir, &xpx, &ypx);
        if (status == PBR_RAY_DEPOSITED &&
            !(xpx >= 0.0 && ypx >= 0.0 && xpx < (double)P.W && ypx < (double)P.H))
            status = PBR_RAY_OFF_SENSOR;
    }
    const bool on = valid && status == PBR_RAY_DEPOSITED;
    RayKey key = {0, 0, k0};
    if (valid) key = ray_key(P, first + i);
    const int g = by_run ? (int)(key.k - k0) : 0;
    if (valid) {
        const int64_t rid = key.s * (int64_t)P.rays_per_src + key.j;
        if (P.record && rid >= P.rec_first) {
            const int64_t off = rid - P.rec_first;
            const int64_t k = off / P.rec_stride;
            if (k * P.rec_stride == off && k < P.rec_max) {
                pbr_ray_exit e;
                e.ray_id = rid;
                e.status = status;
                e.n_steps = nsteps;
                e.entered = entered ? 1 : 0;
                e.reserved = 0;
#pragma unroll
                for (int a = 0; a < 3; ++a) { e.vol_exit_pos[a] = Rw[a]; e.vol_exit_dir[a] = dir[a]; }
                e.sensor_px[0] = xpx;
                e.sensor_px[1] = ypx;
                P.rec[k] = e;
            }
        }
        atomicAdd(&sh.cnt[CNT_STATUS + status], 1ull);
        if (entered) atomicAdd(&sh.cnt[CNT_ENTERED], 1ull);
        atomicAdd(&sh.cnt[CNT_STEPS], (unsigned long long)nsteps);
    }
    {   // bounding boxes: a wave of one group adds its own once
        const int x = (int)xpx, y = (int)ypx, g0 = __builtin_amdgcn_readfirstlane(g);
        const unsigned long long dep = __ballot(on);
        if (dep && __ballot(on && g != g0) == 0ull) {
            const int lx = wave_min(on ? x : 0x7fffffff), ly = wave_min(on ? y : 0x7fffffff);
            const int hx = -wave_min(on ? -x : 1), hy = -wave_min(on ? -y : 1);
            if (lane == 0) {
                atomicMin(&sh.lo_x[g0], lx);
                atomicMin(&sh.lo_y[g0], ly);
                atomicMax(&sh.hi_x[g0], hx);
                atomicMax(&sh.hi_y[g0], hy);
            }
        } else if (on) {
            atomicMin(&sh.lo_x[g], x);
            atomicMin(&sh.lo_y[g], y);
            atomicMax(&sh.hi_x[g], x);
            atomicMax(&sh.hi_y[g], y);
        }
    }
    __syncthreads();
    if (wave == 0) {  // windows of the groups, one lane each, packed in group order while they fit
        DepositWindow w = {0, 0, 0, 0, 0};
        if (lane < ngroups && sh.hi_x[lane] >= 0) {
            w.x0 = max(sh.lo_x[lane] - rf, 0);
            w.y0 = max(sh.lo_y[lane] - rf, 0);
            w.w = min(sh.hi_x[lane] + rf, P.W - 1) - w.x0 + 1;
            w.h = min(sh.hi_y[lane] + rf, P.H - 1) - w.y0 + 1;
            if (w.w > TILE && (long long)w.w * w.h > 2 * TILE * TILE) {  // blurred: its middle
                w.x0 += (w.w - TILE) / 2;
                w.w = TILE;
            }
            if (w.h > TILE && (long long)w.w * w.h > 2 * TILE * TILE) {
                w.y0 += (w.h - TILE) / 2;
                w.h = TILE;
            }
        }
        const int area = w.w * w.h;
        int end = area;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(end, o, 64);
            if (lane >= o) end += t;
        }
        w.off = end - area;
        const bool fits = end <= 2 * TILE * TILE;
        if (!fits) w.w = w.h = 0;  // no room: straight to HBM
        if (lane < ngroups) sh.win[lane] = w;
        const int used = -wave_min(fits ? -end : 0);
        if (lane == 0) sh.used = used;
    }
    __syncthreads();
    for (int q = threadIdx.x; q < sh.used; q += blockDim.x) sh.tile[q] = 0ull;
    __syncthreads();
    if (P.src_sums) add_source_sums(P, on, key.s, xpx, ypx);
    if (on) {
        int64_t s = key.s;
        if (PBR_CHECKED && !access_ok(P, s >= 0 && s < P.n_src)) s = s < 0 ? 0 : P.n_src - 1;
        const float4 sv = P.src[s];
        double w = sv.w > 0.0f ? (sv.w < 1.0f ? (double)sv.w : 1.0) : 0.0;  // weights in [0, 1]
        if ((FEAT & FEAT_MIE) && P.mie) {  // the ray's Mie factor, from its direction at the source
            double S0[3], u0[3];
            initial_direction(P, key.s, key.j, S0, u0);
            w *= mie_weight(P, u0);
        }
        const DepositWindow win = sh.win[g];
        if (RFX > 0) deposit<(RFX > 0 ? RFX : 1)>(P, xpx, ypx, w, sh.tile, win);
        else switch (P.rfp) {
            case 1: deposit<1>(P, xpx, ypx, w, sh.tile, win); break;
            case 2: deposit<2>(P, xpx, ypx, w, sh.tile, win); break;
            case 3: deposit<3>(P, xpx, ypx, w, sh.tile, win); break;
            case 4: deposit<4>(P, xpx, ypx, w, sh.tile, win); break;
            case 5: deposit<5>(P, xpx, ypx, w, sh.tile, win); break;
            case 6: deposit<6>(P, xpx, ypx, w, sh.tile, win); break;
            case 7: deposit<7>(P, xpx, ypx, w, sh.tile, win); break;
            default: deposit<8>(P, xpx, ypx, w, sh.tile, win); break;
        }
    }
    __syncthreads();
    // flush the windows, one wave per group, lanes as 8 x 8 pixels: one global atomic per touched pixel
    for (int k = wave; k < ngroups; k += (int)blockDim.x / 64) {
        const DepositWindow w = sh.win[k];
        for (int y = lane >> 3; y < w.h; y += 8)
            for (int x = lane & 7; x < w.w; x += 8) {
                const unsigned long long v = sh.tile[w.off + y * w.w + x];
                if (PBR_CHECKED && v &&
                    !access_ok(P, (unsigned)(w.y0 + y) < (unsigned)P.H && (unsigned)(w.x0 + x) < (unsigned)P.W))
                    continue;
                if (v) atomic_add_u64(P.accum + (size_t)(w.y0 + y) * (size_t)P.W + (w.x0 + x), v);
            }
    }
    __syncthreads();
}

template <int TILE>
__device__ __forceinline__ void flush_counters(const TraceParams &P, FinishShared<TILE> &sh)
{
    if (threadIdx.x < CNT_STEPS + 1 && sh.cnt[threadIdx.x] != 0ull)
        atomic_add_u64(P.counters + threadIdx.x, sh.cnt[threadIdx.x]);
}

template <int TILE, int RF, int FEAT = 0>
__global__ void __launch_bounds__(256) k_finish(TraceParams P, const RayState *__restrict__ st,
                                                int64_t first, int64_t n)
{
    __shared__ FinishShared<TILE> sh;
    if (threadIdx.x < CNT_SLOTS) sh.cnt[threadIdx.x] = 0ull;
    for (int64_t base = (int64_t)blockIdx.x * blockDim.x; base < n; base += (int64_t)gridDim.x * blockDim.x)
        finish_block<TILE, RF, FEAT>(P, st, first, base, n, n, sh);
    flush_counters<TILE>(P, sh);
}

// ------------------------------------------------------------------ batches of images

// Segment of one round of a batch: rays [first_ray, first_ray + n_rays) of image `image`, whose
// states start at slot slot_base (a slot = 256 rays; segments are padded to whole slots).
__device__ __forceinline__ int find_segment(const BatchSeg *__restrict__ segs, int nseg, int64_t slot)
{
    int lo = 0, hi = nseg - 1;
    while (lo < hi) {  // last segment with slot_base <= slot
        const int mid = (lo + hi + 1) >> 1;
        if (segs[mid].slot_base <= slot) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__global__ void __launch_bounds__(256) k_emit_batch(const TraceParams *__restrict__ params,
                                                    const BatchSeg *__restrict__ segs, int nseg,
                                                    RayState *__restrict__ st)
{
    const int k = __builtin_amdgcn_readfirstlane(find_segment(segs, nseg, blockIdx.x));
    const BatchSeg sg = segs[k];
    const int64_t local = (int64_t)(blockIdx.x - sg.slot_base) * 256 + threadIdx.x;
    if (local >= sg.n_rays) return;
    RayState r;
    emit_ray(params[sg.image], ray_key(params[sg.image], sg.first_ray + local), r);
    store_state(st, (int64_t)blockIdx.x * 256 + threadIdx.x, kWholeGroups, r);
}

// Persistent integration over one round: every wave pulls the next unit of `unit_rays` rays
// (64, 128 or 256: units never straddle a slot) from a global counter until none is left.
// Segments are ordered by decreasing estimated cost, so long rays start first.  NODES: the
// images whose field is stored per node (their own counter, queue[1]; the per-cell images use
// queue[0]); each kernel passes over the other layout's units.
template <int BLOCK, bool NODES>
__global__ void __launch_bounds__(BLOCK, NODES ? 4 : 5) k_box_batch(const TraceParams *__restrict__ params,
                                                                    const BatchSeg *__restrict__ segs, int nseg,
                                                                    RayState *__restrict__ st, unsigned *queue,
                                                                    unsigned n_units, int unit_rays)
{
    const int lane = threadIdx.x & 63;
    for (;;) {
        unsigned u = 0;
        if (lane == 0) u = atomicAdd(queue + (NODES ? 1 : 0), 1u);
        u = __builtin_amdgcn_readfirstlane(__shfl(u, 0, 64));
        if (u >= n_units) break;
        const int64_t ray0 = (int64_t)u * unit_rays;  // state index of the unit's first ray
        const int k = __builtin_amdgcn_readfirstlane(find_segment(segs, nseg, ray0 >> 8));
        const BatchSeg sg = segs[k];
        const TraceParams &P = params[sg.image];
        if ((P.node_layout != 0) != NODES) continue;  // the other kernel's image
        for (int sub = 0; sub < unit_rays; sub += 64) {
            const int64_t idx = ray0 + sub + lane;
            if (idx - sg.slot_base * 256 >= sg.n_rays) continue;
            RayState r = load_state(st, idx, kWholeGroups);
            if ((r.info & (RS_ENTERED | RS_SURR)) != RS_ENTERED) continue;
            box_ray<float, NODES>(P, r);
            store_state(st, idx, kWholeGroups, r);
        }
    }
}

template <int TILE>
__global__ void __launch_bounds__(256) k_finish_batch(const TraceParams *__restrict__ params,
                                                      const BatchSeg *__restrict__ segs, int nseg,
                                                      const RayState *__restrict__ st)
{
    __shared__ FinishShared<TILE> sh;
    if (threadIdx.x < CNT_SLOTS) sh.cnt[threadIdx.x] = 0ull;
    const int k = __builtin_amdgcn_readfirstlane(find_segment(segs, nseg, blockIdx.x));
    const BatchSeg sg = segs[k];
    const TraceParams &P = params[sg.image];
    const int64_t base = (int64_t)(blockIdx.x - sg.slot_base) * 256;
    // states of this segment start at slot_base * 256; ray ids at first_ray
    finish_block<TILE>(P, st + sg.slot_base * 256, sg.first_ray, base, sg.n_rays, kWholeGroups, sh);
    flush_counters<TILE>(P, sh);
}

// ------------------------------------------------------------------ ray surrogate

// Entry point (world) and unit direction of an emitted state that entered through z = z_lo.
__device__ __forceinline__ bool entry_of(const TraceParams &P, const RayState &r, double E[3], double u[3])
{
    if (!(r.info & RS_ENTERED) || r.c[2] != 0 || r.fd[2] != 0.0) return false;
    double n2 = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        E[a] = P.origin[a] + ((double)r.c[a] + r.fd[a]) * P.spacing[a];
        u[a] = (double)r.Tr[a] + (double)r.dT[a];
        n2 += u[a] * u[a];
    }
    const double il = 1.0 / sqrt(n2);
#pragma unroll
    for (int a = 0; a < 3; ++a) u[a] *= il;
    return u[2] > 0.0;
}

__device__ __forceinline__ void surr_features(const SurrogateSpec &sp, const double E[3], const double u[3], float x[6])
{
    x[0] = (float)((2.0 * E[0] - sp.x_lo - sp.x_hi) * sp.inv_wx);
    x[1] = (float)((2.0 * E[1] - sp.y_lo - sp.y_hi) * sp.inv_wy);
    x[2] = (float)(u[0] * sp.inv_theta);
    x[3] = (float)(u[1] * sp.inv_theta);
    // the periodic encodings in single precision (inputs of an FP32 layer)
    x[4] = sinf((float)((E[0] - sp.x_lo) * sp.kx));
    x[5] = sinf((float)((E[1] - sp.y_lo) * sp.ky));
}

__device__ __forceinline__ int surr_tile(const SurrogateSpec &sp, const double E[3])
{
    int tx = (int)((E[0] - sp.x_lo) * sp.inv_wx * sp.tiles);
    int ty = (int)((E[1] - sp.y_lo) * sp.inv_wy * sp.tiles);
    tx = min(max(tx, 0), sp.tiles - 1);
    ty = min(max(ty, 0), sp.tiles - 1);
    return ty * sp.tiles + tx;
}

// Straight-line exit on z = z_hi from the entry.
__device__ __forceinline__ void straight_exit(const SurrogateSpec &sp, const double E[3], const double u[3], double Q[3])
{
    const double l = (sp.z_hi - E[2]) / u[2];
    Q[0] = E[0] + l * u[0];
    Q[1] = E[1] + l * u[1];
    Q[2] = sp.z_hi;
}

__global__ void __launch_bounds__(256) k_surr_samples(TraceParams P, SurrogateSpec sp, const RayState *__restrict__ st,
                                                      int64_t first, int64_t n, SurrogateSample *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    SurrogateSample smp;
    for (int k = 0; k < 6; ++k) smp.t[k] = 0.0f;
    smp.E[0] = smp.E[1] = 0.0; smp.u[0] = smp.u[1] = smp.u[2] = 0.0; smp.px[0] = smp.px[1] = 0.0;
    smp.tile = 0;
    smp.flags = 0;
    RayState e;
    emit_ray(P, ray_key(P, first + i), e);  // the entry state again (the trace overwrote it)
    double E[3], u[3];
    const RayState r = load_state(st, i, n);
    const bool enters = entry_of(P, e, E, u);
    if (enters) {
        smp.E[0] = E[0];
        smp.E[1] = E[1];
        smp.tile = surr_tile(sp, E);
        smp.flags = 4;
    }
    if (enters && !(r.info & RS_LIMITED) && r.c[2] == P.nz - 2 && r.fd[2] == 1.0) {
        double X[3], d[3], Q[3], n2 = 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            X[a] = P.origin[a] + ((double)r.c[a] + r.fd[a]) * P.spacing[a];
            d[a] = (double)r.Tr[a] + (double)r.dT[a];
            n2 += d[a] * d[a];
        }
        const double il = 1.0 / sqrt(n2);
#pragma unroll
        for (int a = 0; a < 3; ++a) d[a] *= il;
        straight_exit(sp, E, u, Q);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            smp.t[a] = (float)(X[a] - Q[a]);
            smp.t[3 + a] = (float)(d[a] - u[a]);
            smp.u[a] = u[a];
        }
        smp.flags |= 1;
        double xp, yp;
        if (optics_to_sensor(P, X, d, &xp, &yp) == PBR_RAY_DEPOSITED) {
            smp.px[0] = xp;
            smp.px[1] = yp;
            smp.flags |= 2;
        }
    }
    out[i] = smp;
}

// Features of every ray of the chunk in place (row i = ray i; rows of rays the network does not
// take are zero and flagged 0 in elig), and the list of the other rays that entered the box for
// the integration kernel (one atomic per wave that has any).
__global__ void __launch_bounds__(256) k_surr_features(TraceParams P, SurrogateSpec sp, const RayState *__restrict__ st,
                                                       int64_t n, float *__restrict__ x,
                                                       unsigned char *__restrict__ elig, int *__restrict__ tlist,
                                                       unsigned long long *__restrict__ tcount)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & 63;
    double E[3], u[3];
    bool ok = false, traced = false;
    if (i < n) {
        const RayState r = load_state(st, i, n);
        ok = entry_of(P, r, E, u);
        if (ok) ok = sp.tile_ok[surr_tile(sp, E)] != 0;
        traced = !ok && (r.info & RS_ENTERED);
        float f[6] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        if (ok) surr_features(sp, E, u, f);
#pragma unroll
        for (int k = 0; k < 6; ++k) x[i * 6 + k] = f[k];
        elig[i] = ok ? 1 : 0;
    }
    const unsigned long long tmask = __ballot(traced);
    if (tmask) {
        unsigned long long tbase = 0;
        if (lane == 0) tbase = atomicAdd(tcount, (unsigned long long)__popcll(tmask));
        tbase = __shfl(tbase, 0);
        if (traced) tlist[tbase + __popcll(tmask & ((1ull << lane) - 1ull))] = (int)i;
    }
}

// Predicted exit: straight exit plus the position change (on z = z_hi), direction u + change.
__device__ __forceinline__ void surr_predict(const SurrogateSpec &sp, const double E[3], const double u[3],
                                             const float *y, double X[3], double d[3])
{
    double Q[3];
    straight_exit(sp, E, u, Q);
    double n2 = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double dp = (double)y[a] * sp.t_scale[a] + sp.t_mean[a];
        const double dd = (double)y[3 + a] * sp.t_scale[3 + a] + sp.t_mean[3 + a];
        X[a] = Q[a] + dp;
        d[a] = u[a] + dd;
        n2 += d[a] * d[a];
    }
    X[2] = sp.z_hi;
    const double il = 1.0 / sqrt(n2);
#pragma unroll
    for (int a = 0; a < 3; ++a) d[a] *= il;
}

__global__ void __launch_bounds__(256) k_surr_apply(TraceParams P, SurrogateSpec sp, const float *__restrict__ y,
                                                    const unsigned char *__restrict__ elig, int64_t n,
                                                    RayState *__restrict__ st)
{
    __shared__ unsigned s_cnt;
    if (threadIdx.x == 0) s_cnt = 0u;
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n && elig[i]) {
        RayState r = load_state(st, i, n);
        double E[3], u[3], X[3], d[3];
        entry_of(P, r, E, u);
        surr_predict(sp, E, u, y + i * 6, X, d);
        const int nn[3] = {P.nx, P.ny, P.nz};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            double p = (X[a] - P.origin[a]) / P.spacing[a];
            if (a == 2) p = (double)(nn[2] - 1);
            p = p < 0.0 ? 0.0 : (p > (double)(nn[a] - 1) ? (double)(nn[a] - 1) : p);
            int ci = (int)floor(p);
            ci = ci > nn[a] - 2 ? nn[a] - 2 : ci;
            r.c[a] = ci;
            r.fd[a] = p - (double)ci;
            r.Tr[a] = (float)d[a];
            r.dT[a] = (float)(d[a] - (double)r.Tr[a]);
        }
        r.info = RS_ENTERED | RS_SURR;
        store_state(st, i, n, r);
        atomicAdd(&s_cnt, 1u);
    }
    __syncthreads();
    if (threadIdx.x == 0 && s_cnt) atomic_add_u64(P.counters + CNT_SURR, (unsigned long long)s_cnt);
}

__global__ void __launch_bounds__(256) k_surr_validate(TraceParams P, SurrogateSpec sp,
                                                       const SurrogateSample *__restrict__ smp, const float *__restrict__ y,
                                                       int64_t n, float *__restrict__ err, unsigned *__restrict__ tile_err,
                                                       unsigned *__restrict__ tile_cnt)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const SurrogateSample s = smp[i];
    float e = -1.0f;  // not compared
    if ((s.flags & 5) == 4) {
        // entered through the front face but left elsewhere: the network cannot represent it
        e = 1.0e30f;
    } else if (s.flags & 1) {
        const double E[3] = {s.E[0], s.E[1], sp.z_lo};
        double X[3], d[3], xp, yp;
        surr_predict(sp, E, s.u, y + i * 6, X, d);
        const bool dep = optics_to_sensor(P, X, d, &xp, &yp) == PBR_RAY_DEPOSITED;
        if (dep && (s.flags & 2))
            e = (float)sqrt((xp - s.px[0]) * (xp - s.px[0]) + (yp - s.px[1]) * (yp - s.px[1]));
        else if (dep != ((s.flags & 2) != 0))
            e = -2.0f;  // passes an aperture or lens rim on one side and not the other
    }
    // a rim case would add or drop a whole ray: its tile is never eligible (the tracer keeps it)
    const float te = e == -2.0f ? 1.0e30f : e;
    if (te >= 0.0f) {
        atomicMax(tile_err + s.tile, __float_as_uint(te));
        atomicAdd(tile_cnt + s.tile, 1u);
    }
    err[i] = e;
}

__global__ void __launch_bounds__(256) k_surr_gather(SurrogateSpec sp, const SurrogateSample *__restrict__ smp,
                                                     const int *__restrict__ idx, int64_t rows, float *__restrict__ x,
                                                     float *__restrict__ t, const int *__restrict__ step,
                                                     int64_t steps_per_epoch)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= rows * 6) return;
    if (step) idx += (int64_t)(*step % steps_per_epoch) * rows;
    const int64_t m = q / 6;
    const int k = (int)(q % 6);
    const SurrogateSample &s = smp[idx ? (int64_t)idx[m] : m];
    const double E[3] = {s.E[0], s.E[1], sp.z_lo};
    float f[6];
    surr_features(sp, E, s.u, f);
    x[q] = f[k];
    t[q] = (s.t[k] - sp.t_mean[k]) / sp.t_scale[k];
}

__global__ void __launch_bounds__(256) k_surr_moments(const SurrogateSample *__restrict__ smp, int64_t n,
                                                      double *__restrict__ part)
{
    __shared__ double s[kMoments][256];
    double a[kMoments];
#pragma unroll
    for (int k = 0; k < kMoments; ++k) a[k] = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const SurrogateSample &q = smp[i];
        if (!(q.flags & 1)) continue;
        a[0] += 1.0;
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const double v = q.t[k];
            a[1 + k] += v;
            a[7 + k] += v * v;
        }
        a[13] += q.u[0] * q.u[0];
        a[14] += q.u[1] * q.u[1];
    }
#pragma unroll
    for (int k = 0; k < kMoments; ++k) s[k][threadIdx.x] = a[k];
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o)
#pragma unroll
            for (int k = 0; k < kMoments; ++k) s[k][threadIdx.x] += s[k][threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x < kMoments) part[blockIdx.x * kMoments + threadIdx.x] = s[threadIdx.x][0];
}

__global__ void __launch_bounds__(256) k_surr_extract(const SurrogateSample *__restrict__ smp, int64_t n, int field,
                                                      int *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = field ? smp[i].tile : smp[i].flags;
}

}  // namespace

int launch_surr_extract(const SurrogateSample *smp, int64_t n, int field, int *out, hipStream_t s)
{
    if (n <= 0) return 0;
    hipLaunchKernelGGL(k_surr_extract, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, smp, n, field, out);
    return (int)hipGetLastError();
}

int launch_surr_samples(const TraceParams &p, const SurrogateSpec &sp, const RayState *st, int64_t first,
                        int64_t n, SurrogateSample *out, hipStream_t s)
{
    if (n <= 0) return 0;
    hipLaunchKernelGGL(k_surr_samples, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, sp, st, first, n, out);
    return (int)hipGetLastError();
}

int launch_surr_features(const TraceParams &p, const SurrogateSpec &sp, const RayState *st, int64_t n, float *x,
                         unsigned char *elig, int *tlist, unsigned long long *tcount, hipStream_t s)
{
    if (n <= 0) return 0;
    hipLaunchKernelGGL(k_surr_features, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, sp, st, n, x, elig,
                       tlist, tcount);
    return (int)hipGetLastError();
}

int launch_surr_apply(const TraceParams &p, const SurrogateSpec &sp, const float *y, const unsigned char *elig,
                      int64_t n, RayState *st, hipStream_t s)
{
    if (n <= 0) return 0;
    hipLaunchKernelGGL(k_surr_apply, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, sp, y, elig, n, st);
    return (int)hipGetLastError();
}

int launch_surr_validate(const TraceParams &p, const SurrogateSpec &sp, const SurrogateSample *smp,
                         const float *y, int64_t n, float *err, unsigned *tile_err, unsigned *tile_cnt,
                         hipStream_t s)
{
    if (n <= 0) return 0;
    hipLaunchKernelGGL(k_surr_validate, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, sp, smp, y, n, err,
                       tile_err, tile_cnt);
    return (int)hipGetLastError();
}

int launch_surr_gather(const SurrogateSpec &sp, const SurrogateSample *smp, const int *idx, int64_t rows,
                       float *x, float *t, hipStream_t s)
{
    if (rows <= 0) return 0;
    hipLaunchKernelGGL(k_surr_gather, dim3((unsigned)((rows * 6 + 255) / 256)), dim3(256), 0, s, sp, smp, idx, rows,
                       x, t, (const int *)nullptr, (int64_t)1);
    return (int)hipGetLastError();
}

int launch_surr_gather_step(const SurrogateSpec &sp, const SurrogateSample *smp, const int *perm, const int *step,
                            int64_t steps_per_epoch, int64_t rows, float *x, float *t, hipStream_t s)
{
    hipLaunchKernelGGL(k_surr_gather, dim3((unsigned)((rows * 6 + 255) / 256)), dim3(256), 0, s, sp, smp, perm, rows,
                       x, t, step, steps_per_epoch);
    return (int)hipGetLastError();
}

int launch_surr_moments(const SurrogateSample *smp, int64_t n, double *part, int *blocks, hipStream_t s)
{
    int nb = (int)((n + 255) / 256);
    nb = nb < 1024 ? (nb < 1 ? 1 : nb) : 1024;
    *blocks = nb;
    hipLaunchKernelGGL(k_surr_moments, dim3((unsigned)nb), dim3(256), 0, s, smp, n, part);
    return (int)hipGetLastError();
}

int launch_calibrate(const TraceParams &p, const int *bricks, int n_bricks, int rays_per_brick,
                     int n_steps, uint64_t seed, double z_focus, double px_per_m, float *err,
                     hipStream_t stream)
{
    if (n_bricks <= 0) return 0;
    if (p.node_layout)
        hipLaunchKernelGGL(k_calibrate<true>, dim3((unsigned)n_bricks), dim3((unsigned)rays_per_brick), 0, stream, p,
                           bricks, n_steps, seed, z_focus, px_per_m, err);
    else
        hipLaunchKernelGGL(k_calibrate<false>, dim3((unsigned)n_bricks), dim3((unsigned)rays_per_brick), 0, stream, p,
                           bricks, n_steps, seed, z_focus, px_per_m, err);
    return (int)hipGetLastError();
}

int launch_trace_chunk(const TraceParams &p, RayState *st, int64_t first, int64_t n, int prec,
                       hipStream_t stream, hipEvent_t box_begin, hipEvent_t box_end, const ChunkHook *hook,
                       bool deposit, bool refill)
{
    if (n <= 0) return 0;
    const unsigned blocks = (unsigned)((n + 255) / 256);
    // the integration kernels emit their own rays, unless something else reads the states first or the
    // kernel takes them from a queue
    const bool own = !hook && !(refill && prec == PREC_FP32);
    const int64_t from = own ? first : -1;
    int e = 0;
    if (!own) {
        hipLaunchKernelGGL(k_emit, dim3(blocks), dim3(256), 0, stream, p, st, first, n);
        if ((e = (int)hipGetLastError())) return e;
    }
    TraceList tl{nullptr, nullptr};
    if (hook && (e = hook->run(hook->self, p, st, first, n, stream, &tl))) return e;
    if (box_begin && (e = (int)hipEventRecord(box_begin, stream))) return e;
    if (prec == PREC_FP64) {
        if (p.node_layout) hipLaunchKernelGGL(k_box64<true>, dim3(blocks), dim3(256), 0, stream, p, st, n, tl.idx, tl.count, from);
        else hipLaunchKernelGGL(k_box64<false>, dim3(blocks), dim3(256), 0, stream, p, st, n, tl.idx, tl.count, from);
    }
    else if (prec == PREC_MIXED) {
        if (p.node_layout) hipLaunchKernelGGL(k_box_mixed<true>, dim3(blocks), dim3(256), 0, stream, p, st, n, tl.idx, tl.count, from);
        else hipLaunchKernelGGL(k_box_mixed<false>, dim3(blocks), dim3(256), 0, stream, p, st, n, tl.idx, tl.count, from);
    }
    else if (refill) {
        // persistent grid: five 256-thread blocks per compute unit, fewer for small chunks
        int dev = 0, ncu = 256;
        if (hipGetDevice(&dev) == hipSuccess)
            (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
        const unsigned pblocks = (unsigned)ncu * 5u < blocks ? (unsigned)ncu * 5u : blocks;
        if ((e = launch_clear_u64(p.counters + CNT_QUEUE, 1, stream))) return e;
        hipLaunchKernelGGL(k_box32_refill, dim3(pblocks), dim3(256), 0, stream, p, st, n, tl.idx, tl.count,
                           p.counters + CNT_QUEUE);
    } else if (p.node_layout)
        hipLaunchKernelGGL(k_box32<true>, dim3(blocks), dim3(256), 0, stream, p, st, n, tl.idx, tl.count, from);
    else
        hipLaunchKernelGGL(k_box32<false>, dim3(blocks), dim3(256), 0, stream, p, st, n, tl.idx, tl.count, from);
    e = (int)hipGetLastError();
    if (e) return e;
    if (box_end && (e = (int)hipEventRecord(box_end, stream))) return e;
    if (!deposit) return 0;
    unsigned fblocks = blocks < 4096u ? blocks : 4096u;
    const RayState *cst = st;
    const int feat = (p.mie ? FEAT_MIE : 0) | (p.chain ? FEAT_CHAIN : 0);
    if (feat) {
        // spot radii of 1-3 pixels cover focused particles; wider spots take the run-time radius
        const int rf = p.rfp <= 3 ? p.rfp : 0;
#define PBR_FINISH_FEAT(F)                                                                                          \
        switch (rf) {                                                                                               \
            case 1: hipLaunchKernelGGL((k_finish<kTile, 1, F>), dim3(fblocks), dim3(256), 0, stream, p, cst, first, n); break; \
            case 2: hipLaunchKernelGGL((k_finish<kTile, 2, F>), dim3(fblocks), dim3(256), 0, stream, p, cst, first, n); break; \
            case 3: hipLaunchKernelGGL((k_finish<kTile, 3, F>), dim3(fblocks), dim3(256), 0, stream, p, cst, first, n); break; \
            default: hipLaunchKernelGGL((k_finish<kTile, 0, F>), dim3(fblocks), dim3(256), 0, stream, p, cst, first, n); break; \
        }
        if (feat == FEAT_MIE) { PBR_FINISH_FEAT(FEAT_MIE) }
        else if (feat == FEAT_CHAIN) { PBR_FINISH_FEAT(FEAT_CHAIN) }
        else { PBR_FINISH_FEAT(FEAT_MIE | FEAT_CHAIN) }
#undef PBR_FINISH_FEAT
    }
    else switch (p.rfp) {
        case 1: hipLaunchKernelGGL((k_finish<kTile, 1>), dim3(fblocks), dim3(256), 0, stream, p, cst, first, n); break;
        case 2: hipLaunchKernelGGL((k_finish<kTile, 2>), dim3(fblocks), dim3(256), 0, stream, p, cst, first, n); break;
        case 3: hipLaunchKernelGGL((k_finish<kTile, 3>), dim3(fblocks), dim3(256), 0, stream, p, cst, first, n); break;
        case 4: hipLaunchKernelGGL((k_finish<kTile, 4>), dim3(fblocks), dim3(256), 0, stream, p, cst, first, n); break;
        case 5: hipLaunchKernelGGL((k_finish<kTile, 5>), dim3(fblocks), dim3(256), 0, stream, p, cst, first, n); break;
        case 6: hipLaunchKernelGGL((k_finish<kTile, 6>), dim3(fblocks), dim3(256), 0, stream, p, cst, first, n); break;
        case 7: hipLaunchKernelGGL((k_finish<kTile, 7>), dim3(fblocks), dim3(256), 0, stream, p, cst, first, n); break;
        default: hipLaunchKernelGGL((k_finish<kTile, 8>), dim3(fblocks), dim3(256), 0, stream, p, cst, first, n); break;
    }
    return (int)hipGetLastError();
}

int launch_batch_round(const TraceParams *params, const BatchSeg *segs, int nseg, int64_t n_slots,
                       RayState *st, unsigned *queue, const BatchConfig &cfg, int n_cu, hipStream_t stream,
                       bool cells, bool nodes)
{
    if (n_slots <= 0) return 0;
    int e = launch_clear_u64((unsigned long long *)queue, 1, stream);  // both counters
    if (e) return e;
    hipLaunchKernelGGL(k_emit_batch, dim3((unsigned)n_slots), dim3(256), 0, stream, params, segs, nseg, st);
    if ((e = (int)hipGetLastError())) return e;
    const unsigned n_units = (unsigned)(n_slots * 256 / cfg.unit_rays);
    // a persistent grid per field layout present in the round: five waves per SIMD for the
    // per-cell kernel, four for the node kernel (its register budget)
    const unsigned w_cells = (unsigned)n_cu * 4u * 5u, w_nodes = (unsigned)n_cu * 4u * 4u;
    if (cells) {
        if (cfg.box_block == 64)
            hipLaunchKernelGGL((k_box_batch<64, false>), dim3(w_cells), dim3(64), 0, stream, params, segs, nseg, st,
                               queue, n_units, cfg.unit_rays);
        else
            hipLaunchKernelGGL((k_box_batch<256, false>), dim3(w_cells / 4u), dim3(256), 0, stream, params, segs,
                               nseg, st, queue, n_units, cfg.unit_rays);
        if ((e = (int)hipGetLastError())) return e;
    }
    if (nodes) {
        if (cfg.box_block == 64)
            hipLaunchKernelGGL((k_box_batch<64, true>), dim3(w_nodes), dim3(64), 0, stream, params, segs, nseg, st,
                               queue, n_units, cfg.unit_rays);
        else
            hipLaunchKernelGGL((k_box_batch<256, true>), dim3(w_nodes / 4u), dim3(256), 0, stream, params, segs,
                               nseg, st, queue, n_units, cfg.unit_rays);
        if ((e = (int)hipGetLastError())) return e;
    }
    if (cfg.tile == 16)
        hipLaunchKernelGGL(k_finish_batch<16>, dim3((unsigned)n_slots), dim3(256), 0, stream, params, segs, nseg,
                           (const RayState *)st);
    else
        hipLaunchKernelGGL(k_finish_batch<32>, dim3((unsigned)n_slots), dim3(256), 0, stream, params, segs, nseg,
                           (const RayState *)st);
    return (int)hipGetLastError();
}

}  // namespace pbr
