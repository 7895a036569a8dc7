// sweep_dev.h -- device helpers of the REGC trial kernels (pair terms, wave
// reductions, slab access, the energy change of a trial), included by the
// sampling kernels.  Each including file is compiled once per precision
// (-DREGC_FP64 or -DREGC_FP32); the helpers then live in namespace
// regc::fp64 or regc::fp32 with Real = double or float.
#pragma once
#include "regc_dev.h"
#include "philox_dev.h"

namespace regc {

// Each compilation gets its own namespace: the kernels are templates
// with the same names in both precisions, and one symbol per precision must reach
// the code-object registry.
#if defined(REGC_FP64)
#define REGC_PREC fp64
#elif defined(REGC_FP32)
#define REGC_PREC fp32
#else
#error "compile with -DREGC_FP64 or -DREGC_FP32"
#endif

namespace REGC_PREC {
#if defined(REGC_FP64)
typedef double Real;
struct alignas(32) Real4 { double x, y, z, w; };
#else
typedef float Real;
struct alignas(16) Real4 { float x, y, z, w; };
#endif

struct Box {
    Real lx, ly;
};

// |d| of the nearest periodic image of d, up to its sign: min(|d|, L - |d|), for |d| <= 1.5 L
// (gas particles lie in the cell, slab atoms at most half a cell outside).  Only its square
// is used, so the sign is left out: three operations instead of four with a rounded
// quotient (FP32) and of eight with two compares (FP64, the same value bit for bit).
__device__ __forceinline__ Real min_image_abs(Real d, Real L)
{
#if defined(REGC_FP64)
    const double a = __builtin_fabs(d);
    return __builtin_fmin(a, L - a);
#else
    const float a = __builtin_fabsf(d);
    return __builtin_fminf(a, L - a);
#endif
}

// XFIRST (FP32): which square the fused sum starts from, x^2 instead of y^2.
template <bool XFIRST = false>
__device__ __forceinline__ Real dist2(const Box &b, Real px, Real py, Real pz, const Real4 &q)
{
    const Real dx = min_image_abs(px - q.x, b.lx);
    const Real dy = min_image_abs(py - q.y, b.ly);
    const Real dz = pz - q.z;
#if defined(REGC_FP64)
    return dx * dx + dy * dy + dz * dz;
#else
    return __builtin_fmaf(dz, dz, XFIRST ? __builtin_fmaf(dy, dy, dx * dx) : __builtin_fmaf(dx, dx, dy * dy));
#endif
}

struct Pair {
    Real sig2, eps4, shift, rc2, hc2;
};

// truncated-shifted LJ 12-6 at squared distance r2 (r2 < rc2 is the caller's business)
__device__ __forceinline__ Real lj_inside(Real r2, Real sig2, Real eps4, Real shift)
{
#if defined(REGC_FP64)
    // the quotient sig2 / r2 by the steps of an IEEE division without the rescaling of
    // extreme exponents, which no squared distance of a gas region needs (two Newton
    // steps, one residual: the same bits as the division)
    double y = __builtin_amdgcn_rcp(r2);
    y = __builtin_fma(__builtin_fma(-r2, y, 1.0), y, y);
    y = __builtin_fma(__builtin_fma(-r2, y, 1.0), y, y);
    const double q = sig2 * y;
    const double s2 = __builtin_fma(__builtin_fma(-r2, q, sig2), y, q);
    const double s6 = s2 * s2 * s2;
    return eps4 * (s6 * s6 - s6) - shift;
#else
    const float s2 = sig2 * __builtin_amdgcn_rcpf(r2);
    const float s6 = s2 * (s2 * s2);
    return __builtin_fmaf(eps4, __builtin_fmaf(s6, s6, -s6), -shift);
#endif
}

__device__ __forceinline__ Real lj(Real r2, const Pair &p)
{
    const Real v = lj_inside(r2, p.sig2, p.eps4, p.shift);
    return r2 < p.rc2 ? v : Real(0);
}

// Wave-wide sum with DPP (quad permutes, row mirrors, row broadcasts); wave_sum63: the
// total in lane 63 only, wave_sum: read back as a wave-uniform value.  The order of
// the additions is fixed, so the result is deterministic.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_f32(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK, 0xF, false));
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_f64(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROW_MASK, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROW_MASK, 0xF, false);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ float wave_sum63(float v)
{
    v += dpp_f32<0xB1, 0xF>(v);    // quad_perm [1,0,3,2]
    v += dpp_f32<0x4E, 0xF>(v);    // quad_perm [2,3,0,1]
    v += dpp_f32<0x141, 0xF>(v);   // row_half_mirror
    v += dpp_f32<0x140, 0xF>(v);   // row_mirror
    v += dpp_f32<0x142, 0xA>(v);   // row_bcast:15 into rows 1, 3
    v += dpp_f32<0x143, 0xC>(v);   // row_bcast:31 into rows 2, 3
    return v;
}

__device__ __forceinline__ float wave_sum(float v)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wave_sum63(v)), 63));
}

__device__ __forceinline__ double wave_sum63(double v)
{
    v += dpp_f64<0xB1, 0xF>(v);
    v += dpp_f64<0x4E, 0xF>(v);
    v += dpp_f64<0x141, 0xF>(v);
    v += dpp_f64<0x140, 0xF>(v);
    v += dpp_f64<0x142, 0xA>(v);
    v += dpp_f64<0x143, 0xC>(v);
    return v;
}

__device__ __forceinline__ double wave_sum(double x)
{
    const double v = wave_sum63(x);
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), 63);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), 63);
    return __hiloint2double(hi, lo);
}

// Sum over each quad of lanes (4 lanes), the total in every lane of the quad.
__device__ __forceinline__ float quad_sum(float v)
{
    v += dpp_f32<0xB1, 0xF>(v);    // quad_perm [1,0,3,2]
    v += dpp_f32<0x4E, 0xF>(v);    // quad_perm [2,3,0,1]
    return v;
}

__device__ __forceinline__ double quad_sum(double v)
{
    v += dpp_f64<0xB1, 0xF>(v);
    v += dpp_f64<0x4E, 0xF>(v);
    return v;
}

// Sum over aligned groups of G lanes (16, 32 or 64), the total in every lane of the
// group; the order of the additions is fixed (DPP within rows of 16, then across rows).
template <int G>
__device__ __forceinline__ float group_sum(float v)
{
    v += dpp_f32<0xB1, 0xF>(v);    // quad_perm [1,0,3,2]
    v += dpp_f32<0x4E, 0xF>(v);    // quad_perm [2,3,0,1]
    v += dpp_f32<0x141, 0xF>(v);   // row_half_mirror
    v += dpp_f32<0x140, 0xF>(v);   // row_mirror: every lane holds its row's sum
    if (G >= 32) v += __shfl_xor(v, 16);
    if (G >= 64) v += __shfl_xor(v, 32);
    return v;
}

template <int G>
__device__ __forceinline__ double group_sum(double v)
{
    v += dpp_f64<0xB1, 0xF>(v);
    v += dpp_f64<0x4E, 0xF>(v);
    v += dpp_f64<0x141, 0xF>(v);
    v += dpp_f64<0x140, 0xF>(v);
    if (G >= 32) v += __shfl_xor(v, 16);
    if (G >= 64) v += __shfl_xor(v, 32);
    return v;
}

// A condition that every lane of the wave holds alike, as a wave-uniform value: the
// branch on it is a scalar branch.
__device__ __forceinline__ bool uniform(bool c)
{
    return __ballot(c) != 0ull;
}

// A value that every lane of the wave holds alike, moved to a scalar register.
__device__ __forceinline__ int scalar(int v) { return __builtin_amdgcn_readfirstlane(v); }

// The lane's bit of a wave-uniform mask (no instruction: the mask is used as it is).
__device__ __forceinline__ bool lane_in(uint64_t mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); }

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Keep a wave-uniform constant in a VGPR: the hot loop has more uniform values
// than SGPRs, and VALU operands read from VGPRs cost no scalar-register spills.
template <typename T>
__device__ __forceinline__ T in_vgpr(T x)
{
    asm volatile("" : "+v"(x));
    return x;
}

__device__ __forceinline__ uint32_t bcast(uint32_t v, int lane)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}

__device__ __forceinline__ double bcast(double v, int lane)
{
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ float bcast(float v, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

__device__ __forceinline__ Real bcast_real(Real v, int lane) { return bcast(v, lane); }

// What a wave with a new pair inside the hard core sends in the place of its sum: a NaN whose
// bits no arithmetic makes.
#if defined(REGC_FP64)
__device__ __forceinline__ double core_mark() { return __hiloint2double(0x7FF8C0DE, 0); }
__device__ __forceinline__ bool is_core_mark(double v) { return __double2hiint(v) == 0x7FF8C0DE; }
#else
__device__ __forceinline__ float core_mark() { return __int_as_float(0x7FC0C0DE); }
__device__ __forceinline__ bool is_core_mark(float v) { return __float_as_int(v) == 0x7FC0C0DE; }
#endif

// Slab access: all atoms, or the 3x3 block of x-y columns around a column
// (periodic in x and y; column ids row-major, y outer).
//  kSlabAll   every packed entry (a slab too narrow for columns);
//  kSlabHalo  the LDS copy has one more column on every side, the periodic images of
//             the columns at the other end with their coordinates unchanged (distances
//             take the nearest image), so the three columns of each row of a block are
//             consecutive and an entry's index is a per-lane constant plus the block's
//             first entry.  Deriving it with periodic wraps took about 30 issue slots per
//             64 candidates, as much as a candidate's pair term;
//  kSlabWrap  no halo, indices by periodic wrap: for a slab whose halo does not fit LDS.

struct SlabView {
    const Real4 *atoms;
    int len;                  // entries a trial scans: all, or 9 * cap
    int mode, ncx, ncy, cap;
    int row;                  // columns per row of the LDS copy (ncx, or ncx + 2 with the halo)
    float inv_cap;
    Real inv_cw_x, inv_cw_y;
    Real top_plus_rc;
};

// MODE: the launch's slab access where its kernel is made for one (kSlabAny: the class's).
template <int MODE = kSlabAny>
__device__ __forceinline__ SlabView slab_view(const ClassDev &C, const SweepArgs &a, const Real4 *atoms)
{
    SlabView sv;
    sv.atoms = atoms;
    sv.mode = MODE != kSlabAny ? MODE : !C.bins ? kSlabAll : (a.slab_halo ? kSlabHalo : kSlabWrap);
    sv.len = C.bins ? 9 * C.cap : C.slab_len;
    sv.ncx = C.ncx; sv.ncy = C.ncy; sv.cap = C.cap;
    sv.row = sv.mode == kSlabHalo ? C.ncx + 2 : C.ncx;
    sv.inv_cap = C.bins ? 1.0f / (float)C.cap : 0.f;
    sv.inv_cw_x = (Real)C.inv_cw_x; sv.inv_cw_y = (Real)C.inv_cw_y;
    sv.top_plus_rc = (Real)(C.slab_top + sqrt(a.pot.rc2));
    return sv;
}

// The class slab into LDS by `threads` threads, with its halo when the launch has one.
__device__ __forceinline__ void load_slab(const ClassDev &C, const SweepArgs &a, Real4 *slab, int tid, int threads)
{
    const bool halo = C.bins && a.slab_halo;
    const int row = C.ncx + 2, len = halo ? row * (C.ncy + 2) * C.cap : C.slab_len;
    for (int k = tid; k < len; k += threads) {
        int from = k;
        if (halo) {
            const int col = k / C.cap, ey = col / row, ex = col - ey * row;
            const int cx = ex == 0 ? C.ncx - 1 : (ex > C.ncx ? 0 : ex - 1);
            const int cy = ey == 0 ? C.ncy - 1 : (ey > C.ncy ? 0 : ey - 1);
            from = (cy * C.ncx + cx) * C.cap + (k - col * C.cap);
        }
#if defined(REGC_FP64)
        const double *src = a.slab4 + 4 * (size_t)(C.slab_off + from);
#else
        const float *src = a.slab4f + 4 * (size_t)(C.slab_off + from);
#endif
        Real4 v;
        v.x = src[0]; v.y = src[1]; v.z = src[2]; v.w = 0;
        slab[k] = v;
    }
}

// Column (cx, cy) of a position, clamped to the grid.
__device__ __forceinline__ void column_of(const SlabView &sv, Real x, Real y, int &cx, int &cy)
{
    cx = min(max((int)(x * sv.inv_cw_x), 0), sv.ncx - 1);
    cy = min(max((int)(y * sv.inv_cw_y), 0), sv.ncy - 1);
}

// Periodic neighbour c + d (d in -1..1) of a column index in [0, nc): as an
// unsigned value, -1 wraps to the largest integer and min() picks nc - 1, and
// nc becomes 0 the same way.
__device__ __forceinline__ uint32_t wrap_col(int c, int d, int nc)
{
    uint32_t u = (uint32_t)(c + d);
    u = min(u, u + (uint32_t)nc);
    return min(u, u - (uint32_t)nc);
}

// First entry of the 3x3 block around column (cx, cy) of the halo layout, and the entry
// kk (0 <= kk < 9 cap) of a block relative to it: the three columns of a row are
// consecutive, the rows sv.row columns apart.
__device__ __forceinline__ int block_first(const SlabView &sv, int cx, int cy)
{
    return (int)__umul24(__umul24((uint32_t)cy, (uint32_t)sv.row) + (uint32_t)cx, (uint32_t)sv.cap);
}

__device__ __forceinline__ int block_offset(const SlabView &sv, int kk)
{
    const int skip = (sv.row - 3) * sv.cap;
    return kk + (kk >= 3 * sv.cap ? skip : 0) + (kk >= 6 * sv.cap ? skip : 0);
}

// Slab entry kk (0 <= kk < 9 cap) of the 3x3 column block around column (cx, cy):
// slot kk % cap of the block's column sp = kk / cap, sp = 3 (dy + 1) + (dx + 1).
__device__ __forceinline__ int block_entry(const SlabView &sv, int cx, int cy, int kk)
{
    if (sv.mode == kSlabHalo) return block_first(sv, cx, cy) + block_offset(sv, kk);
    const int sp = (int)(((float)kk + 0.5f) * sv.inv_cap);
    const int q = (sp * 11) >> 5;   // sp / 3 for sp in 0..8
    const uint32_t ux = wrap_col(cx, sp - 3 * q - 1, sv.ncx);
    const uint32_t uy = wrap_col(cy, q - 1, sv.ncy);
    return (int)((uy * (uint32_t)sv.ncx + ux) * (uint32_t)sv.cap) + (kk - sp * sv.cap);
}

// This wave's part (wave `part` of SPLIT) of the walker's total energy: every gas
// pair once and every gas atom against the slab entries that can lie within the
// cutoff (its column block, or all entries when unbinned), pair terms in Real,
// per-lane sums in FP64.  Returns the wave-uniform partial sum.
template <int SPLIT>
__device__ double full_energy_part(const Real4 *gas, int n, const SlabView &sv, const Box &b, const Pair &gg,
                                   const Pair &gs, int lane, int part)
{
    double acc = 0.0;
    const int total = sv.len;
    for (int i = 0; i < n; ++i) {
        const Real4 p = gas[i];
        for (int j = i + 1 + part * kWave + lane; j < n; j += SPLIT * kWave)
            acc += (double)lj(dist2(b, p.x, p.y, p.z, gas[j]), gg);
        if (p.z < sv.top_plus_rc) {
            int cx = 0, cy = 0;
            if (sv.mode != kSlabAll) column_of(sv, p.x, p.y, cx, cy);
            for (int k = part * kWave + lane; k < total; k += SPLIT * kWave) {
                const int idx = sv.mode != kSlabAll ? block_entry(sv, cx, cy, k) : k;
                acc += (double)lj(dist2(b, p.x, p.y, p.z, sv.atoms[idx]), gs);
            }
        }
    }
    return wave_sum(acc);
}

// Appends the lanes' values whose predicate holds to an LDS queue (wave-wide
// compaction): each lane's slot is the number of set predicate bits below it.
__device__ __forceinline__ void push(Real *queue, int &count, bool pred, Real value)
{
    const uint64_t mask = __ballot(pred);
    const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
    if (pred) queue[count + (int)below] = value;
    count += __popcll(mask);
}

// One candidate atom g per lane (mask m: the lanes that hold one): pair terms of the
// new position p (NEW, added) and of the old position q (OLD, subtracted).  The masks
// are wave-uniform: they are combined, and the pairs inside the cutoff counted, on the
// scalar unit.  What a masked lane read is not used.  CULL queues the in-cutoff squared
// distances (old ones negated) instead of evaluating them.
template <bool NEW, bool OLD, bool CULL, bool XFIRST = false>
__device__ __forceinline__ void candidate(const Box &b, const Pair &pp, uint64_t m, const Real4 &g, Real px, Real py,
                                          Real pz, Real qx, Real qy, Real qz, Real &acc, uint64_t &core,
                                          uint32_t &useful, Real *queue, int &count)
{
    if (NEW) {
        const Real r2 = dist2<XFIRST>(b, px, py, pz, g);
        const uint64_t in = __ballot(r2 < pp.rc2) & m;
        core |= __ballot(r2 < pp.hc2) & m;
        if (CULL) {
            push(queue, count, lane_in(in), r2);
        } else {
            const Real v = lj_inside(r2, pp.sig2, pp.eps4, pp.shift);
            useful += (uint32_t)__popcll(in);
            acc += lane_in(in) ? v : Real(0);
        }
    }
    if (OLD) {
        const Real r2 = dist2(b, qx, qy, qz, g);
        const uint64_t in = __ballot(r2 < pp.rc2) & m;
        if (CULL) {
            push(queue, count, lane_in(in), -r2);
        } else {
            const Real v = lj_inside(r2, pp.sig2, pp.eps4, pp.shift);
            useful += (uint32_t)__popcll(in);
            acc -= lane_in(in) ? v : Real(0);
        }
    }
}

// The lane's slab candidates of a wave's first two blocks of 64: their place in the
// scan (halo layout: relative to the block's first entry) and the lanes that hold one.
struct SlabLane {
    int off[2];
    uint64_t ok[2];
};

template <int SPLIT>
__device__ __forceinline__ SlabLane slab_lane(const SlabView &sv, int lane, int part)
{
    SlabLane s;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int k = (part + u * SPLIT) * kWave + lane;
        s.ok[u] = __ballot(k < sv.len);
        const int kk = k < sv.len ? k : 0;
        s.off[u] = in_vgpr(sv.mode == kSlabHalo ? block_offset(sv, kk) : kk);
    }
    return s;
}

// This wave's part of the energy change of a trial: sum over the other gas atoms
// (all j < n except `skip`) and over the slab candidates of phi(|p - r|) (NEW)
// minus phi(|q - r|) (OLD).  The wave with index `part` of SPLIT takes every
// SPLIT-th block of 64 candidates.  n and skip are wave-uniform; lanes past n read
// LDS entries that their mask leaves out (the layouts keep 64 entries readable after
// the gas atoms).  Returns the lane's sum; `core` gets the lanes whose new position
// lies inside a hard core, `useful` the count of pairs inside the cutoff, `near`
// whether the slab was scanned.  PRE: `pre` holds the wave's first block (one wave per walker: its first two), read by the caller.
template <bool NEW, bool OLD, int SPLIT, bool CULL, bool PRE = false>
__device__ __forceinline__ Real lane_delta(const Real4 *gas, int n, int skip, const SlabView &sv, const SlabLane &sl,
                                           const Box &b, const Pair &gg, const Pair &gs, int lane, int part, Real px,
                                           Real py, Real pz, Real qx, Real qy, Real qz, Real *qgas, Real *qslab,
                                           uint64_t &core, uint32_t &useful, bool &near, const Real4 *pre = nullptr)
{
    constexpr int STEP = SPLIT * kWave;
    Real acc = 0;
    int ng = 0, ns = 0;
    // (one wave per walker, the two blocks read ahead: the squared distances of the new
    // position are summed from x^2, as they were before the trial loop was laid out anew,
    // so that FP32 trajectories stay the same bit for bit)
    constexpr bool XF = PRE && SPLIT == 1;
    auto gas_mask = [&](int j0) {
        const int j = j0 + lane;
        uint64_t m = __ballot(j < n);
        if (OLD) m &= __ballot(j != skip);      // (an insertion leaves no particle out)
        return m;
    };
    auto gas_block = [&](const Real4 &g, int j0) {
        candidate<NEW, OLD, CULL>(b, gg, gas_mask(j0), g, px, py, pz, qx, qy, qz, acc, core, useful, qgas, ng);
    };
    // two blocks per step where a wave has two left: both reads before their terms
    const Real4 *gl = gas + lane;
    int j0 = part * kWave;
    if (PRE && j0 < n) {
        candidate<NEW, OLD, CULL, XF>(b, gg, gas_mask(j0), pre[0], px, py, pz, qx, qy, qz, acc, core, useful, qgas, ng);
        j0 += STEP;
        if (SPLIT == 1 && j0 < n) {
            candidate<NEW, OLD, CULL, XF>(b, gg, gas_mask(j0), pre[1], px, py, pz, qx, qy, qz, acc, core, useful, qgas,
                                          ng);
            j0 += STEP;
        }
    }
    for (; j0 + STEP < n; j0 += 2 * STEP) {
        const Real4 ga = gl[j0], gb = gl[j0 + STEP];
        gas_block(ga, j0);
        gas_block(gb, j0 + STEP);
    }
    if (j0 < n) gas_block(gl[j0], j0);

    const Real zmin = (NEW && OLD) ? (pz < qz ? pz : qz) : (NEW ? pz : qz);
    near = uniform(zmin < sv.top_plus_rc);
    if (near) {
        // (all entries in one list: the column is 0 and its first entry 0)
        int cx, cy;
        column_of(sv, OLD ? qx : px, OLD ? qy : py, cx, cy);
        const Real4 *sa = sv.atoms + block_first(sv, cx, cy);
        auto slab_block = [&](int off, uint64_t ok) {
            const Real4 g = sv.mode == kSlabWrap ? sv.atoms[block_entry(sv, cx, cy, off)] : sa[off];
            candidate<NEW, OLD, CULL>(b, gs, ok, g, px, py, pz, qx, qy, qz, acc, core, useful, qslab, ns);
        };
        int k0 = part * kWave;
        if (k0 < sv.len) slab_block(sl.off[0], sl.ok[0]);
        k0 += STEP;
        if (k0 < sv.len) {
            slab_block(sl.off[1], sl.ok[1]);
            for (k0 += STEP; k0 < sv.len; k0 += STEP) {
                const int k = k0 + lane, kk = k < sv.len ? k : 0;
                slab_block(sv.mode == kSlabHalo ? block_offset(sv, kk) : kk, __ballot(k < sv.len));
            }
        }
    }
    if (CULL) {
        useful += (uint32_t)(ng + ns);
        wave_sync();
        // LJ terms of the queued pairs: gas pairs, then slab pairs, in one lane space
        const int nq = ng + ns;
        for (int k0 = 0; k0 < nq; k0 += kWave) {
            const int k = k0 + lane;
            if (k < nq) {
                const bool is_gas = k < ng;
                const Real v = is_gas ? qgas[k] : qslab[k - ng];
                const Real r2 = v < Real(0) ? -v : v;
                const Real phi = lj_inside(r2, is_gas ? gg.sig2 : gs.sig2, is_gas ? gg.eps4 : gs.eps4,
                                           is_gas ? gg.shift : gs.shift);
                acc += v < Real(0) ? -phi : phi;
            }
        }
    }
    return acc;
}

}  // namespace fp64 / fp32
}  // namespace regc
