// Wave-level primitives and constants shared by the clipping passes.
#pragma once

#include <type_traits>

#include "vd_internal.h"

namespace vd {
namespace {

// node queue of the 64-vertex pass: kQueue0 entries, the first 64 in
// registers (one per lane), the rest in LDS and touched only when the queue
// is that long.  With one entry per vertex slot (64), cells of far-reaching
// power cells and of sparse regions next to dense ones filled the queue long
// before their vertex slots and went to the slower second pass.
constexpr int kQueue0 = 256;

constexpr float kU = 5.9604645e-08f;  // FP32 unit roundoff 2^-24
constexpr double kU64 = 1.1102230246251565e-16;

// The launch arguments seen through a pointer the compiler cannot keep
// constant: the fields used once per cell (outputs, lists, counters) are then
// loaded where they are used instead of being held in scalar registers
// across the hot loops, which otherwise run out of them and spill.  Every
// clip kernel takes its ClipArgs as the first kernel argument.
using KArgs = const __attribute__((address_space(4))) ClipArgs;
__device__ __forceinline__ KArgs* cold_args() {
    KArgs* p = (KArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

enum ClipResult { kNone = 0, kChanged = 1, kEmptied = 2, kOverflow = 3, kRestart = 4 };

__device__ __forceinline__ uint32_t lane_id() { return __lane_id(); }
__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }
__device__ __forceinline__ uint32_t mbcnt(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
__device__ __forceinline__ int popc(uint64_t m) { return __popcll(m); }
__device__ __forceinline__ int lowest(uint64_t m) { return __builtin_ctzll(m); }
__device__ __forceinline__ float rdl(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ uint32_t rdl(uint32_t v, int l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); }
__device__ __forceinline__ int rdl(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ __forceinline__ float uni(float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); }
__device__ __forceinline__ uint32_t uni(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ uint64_t uni(uint64_t v) {
    return (uint64_t)uni((uint32_t)v) | ((uint64_t)uni((uint32_t)(v >> 32)) << 32);
}
// Wave reductions by DPP lane moves (no LDS round trip): within quads
// (quad_perm [1,0,3,2] and [2,3,0,1]), across half-rows and rows
// (row_half_mirror, row_mirror), then row 0 into 1 and 2 into 3
// (row_bcast:15) and rows 0-1 into 2-3 (row_bcast:31); lane 63 holds the
// result, which is returned to every lane.  All 64 lanes must be active.
// dpp: lanes of rows the move does not write get `keep` (the identity of
// the sum it feeds).
template <int kCtrl, int kRows>
__device__ __forceinline__ int dpp(int keep, int v) {
    return __builtin_amdgcn_update_dpp(keep, v, kCtrl, kRows, 0xF, false);
}
// A move within rows (every lane reads a lane of its own row, so all reads
// are valid): the compiler can fold it into the operation that uses it.
template <int kCtrl>
__device__ __forceinline__ int dpp_row(int v) {
    return __builtin_amdgcn_mov_dpp(v, kCtrl, 0xF, 0xF, true);
}
// The two row broadcasts write only rows 1, 3 and then 2, 3; what the
// other rows then hold never reaches lane 63, so they need no defined value.
template <int kCtrl, int kRows>
__device__ __forceinline__ int dpp_bcast(int v) {
    return __builtin_amdgcn_mov_dpp(v, kCtrl, kRows, 0xF, false);
}
template <typename Op>
__device__ __forceinline__ int wave_reduce_i(int v, Op op) {
    v = op(v, dpp_row<0xB1>(v));
    v = op(v, dpp_row<0x4E>(v));
    v = op(v, dpp_row<0x141>(v));
    v = op(v, dpp_row<0x140>(v));
    v = op(v, dpp_bcast<0x142, 0xA>(v));
    v = op(v, dpp_bcast<0x143, 0xC>(v));
    return __builtin_amdgcn_readlane(v, 63);
}
// Float min and max reduce as integers: the bits of a float with the
// magnitude bits of negative values flipped order like the values (NaN is
// never reduced), so each step is one integer min or max on a lane move,
// with no float canonicalisation between the steps.
__device__ __forceinline__ int ford(float f) {
    const int i = __float_as_int(f);
    return i ^ ((i >> 31) & 0x7FFFFFFF);
}
__device__ __forceinline__ float unford(int k) { return __int_as_float(k ^ ((k >> 31) & 0x7FFFFFFF)); }
// Maximum of two non-negative floats (their bits order like integers).
__device__ __forceinline__ float pmax(float a, float b) {
    return __int_as_float(max(__float_as_int(a), __float_as_int(b)));
}
__device__ __forceinline__ float wmin(float v) {
    return unford(wave_reduce_i(ford(v), [](int a, int b) { return min(a, b); }));
}
__device__ __forceinline__ float wmax(float v) {
    return unford(wave_reduce_i(ford(v), [](int a, int b) { return max(a, b); }));
}
__device__ __forceinline__ uint32_t wsum_u(uint32_t v) {
    return (uint32_t)wave_reduce_i((int)v, [](int a, int b) { return (int)((uint32_t)a + (uint32_t)b); });
}
// Sum over this lane and the lower ones (row_shr:1, 2, 4, 8, then the row
// broadcasts).
__device__ __forceinline__ uint32_t wscan_u(uint32_t v) {
    v += (uint32_t)dpp<0x111, 0xF>(0, (int)v);
    v += (uint32_t)dpp<0x112, 0xF>(0, (int)v);
    v += (uint32_t)dpp<0x114, 0xF>(0, (int)v);
    v += (uint32_t)dpp<0x118, 0xF>(0, (int)v);
    v += (uint32_t)dpp<0x142, 0xA>(0, (int)v);
    v += (uint32_t)dpp<0x143, 0xC>(0, (int)v);
    return v;
}
template <int kCtrl, int kRows>
__device__ __forceinline__ double dpp64(double v) {
    const int lo = dpp<kCtrl, kRows>(0, __double2loint(v));
    const int hi = dpp<kCtrl, kRows>(0, __double2hiint(v));
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wsum64(double v) {
    v += dpp64<0xB1, 0xF>(v);
    v += dpp64<0x4E, 0xF>(v);
    v += dpp64<0x141, 0xF>(v);
    v += dpp64<0x140, 0xF>(v);
    v += dpp64<0x142, 0xA>(v);
    v += dpp64<0x143, 0xC>(v);
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), 63);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), 63);
    return __hiloint2double(hi, lo);
}


// Orders this wave's accesses to its per-cell arrays, so that what one lane
// wrote before is seen by every lane after: in LDS, or for the arena tier in
// global memory.  Other waves need a barrier as well.
template <bool kLds>
__device__ __forceinline__ void wave_sync() {
    if constexpr (kLds) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    }
}

// Hands out the cells of a pass to its workers (a wave, or a group of waves
// that share one cell), one at a time.  The cells are split into kWorkRanges
// contiguous (Morton-ordered) ranges, one per XCD: the workers of workgroup b
// take cells of range b % 8 first, so that neighbouring cells, which walk the
// same nodes and sites, share one L2, then help the other ranges.
//
// A worker's first cell is fixed by its number, so a pass with fewer cells
// than workers claims nothing; after that each range has a counter, on a cache
// line of its own, and a worker whose range is used up reads all eight
// counters at once before it claims elsewhere.  Additions to one line go
// through one after the other, about 20 ns each over the whole device: with
// the eight counters side by side and a try at each by every worker in the
// end, 10k cells took 600 to 800 us of which the cells were 250, and a pass
// over a single large cell took 280 us.
constexpr uint32_t kNoCell = 0xFFFFFFFFu;
template <uint32_t kPerBlock>  // workers per workgroup
struct Work {
    uint32_t count;  // cells of the pass
    uint32_t stage;  // 0: first cell, 1: own range, 2: the others

    __device__ __forceinline__ explicit Work(uint32_t n) : count(n), stage(0) {}
    __device__ __forceinline__ uint32_t start(uint32_t q) const { return (uint32_t)((uint64_t)count * q / kWorkRanges); }
    // cells of range q, and those given out by number
    __device__ __forceinline__ uint32_t cells(uint32_t q) const { return start(q + 1) - start(q); }
    __device__ __forceinline__ uint32_t workers(uint32_t q) const {
        return (gridDim.x + kWorkRanges - 1 - q) / kWorkRanges * kPerBlock;
    }
    // Up to `want` cells on from the place of this worker's range: the first,
    // and how many (none when the range is used up).
    __device__ __forceinline__ uint32_t more(uint32_t want, uint32_t* got) {
        const uint32_t range = blockIdx.x % kWorkRanges, given = workers(range), all = cells(range);
        *got = 0;
        if (stage != 1 || given >= all) return 0;
        uint32_t c = 0;
        if (lane_id() == 0) c = atomicAdd(&cold_args()->work_counter[range * kCounterStride], want);
        c = uni(c) + given;
        if (c < all) *got = min(want, all - c);
        return start(range) + c;
    }
    // The next cell, or kNoCell; called by one whole wave, the worker-th of
    // its workgroup.  The counter of range q is at work_counter[q * kCounterStride].
    __device__ __forceinline__ uint32_t next(uint32_t worker) {
        const uint32_t range = blockIdx.x % kWorkRanges;
        uint32_t ln = lane_id();
        asm volatile("" : "+v"(ln));  // nothing of this is kept through the cells
        if (stage == 0) {
            stage = 1;
            const uint32_t number = blockIdx.x / kWorkRanges * kPerBlock + worker;
            if (number < cells(range)) return start(range) + number;
        }
        uint32_t* const counter = cold_args()->work_counter;
        if (stage == 1) {
            const uint32_t given = workers(range), all = cells(range);
            if (given < all) {
                uint32_t c = 0;
                if (ln == 0) c = atomicAdd(&counter[range * kCounterStride], 1u);
                c = uni(c) + given;
                if (c < all) return start(range) + c;
            }
            stage = 2;
        }
        for (;;) {
            // lane q: are there cells left in range q?  Counters only grow, so
            // a failed claim is not repeated and the loop ends.
            const uint32_t q = ln % kWorkRanges, given = workers(q), all = cells(q);
            bool left = given < all;
            if (ballot(left) == 0) return kNoCell;
            if (left)
                left = __hip_atomic_load(&counter[q * kCounterStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <
                       all - given;
            const uint32_t m = (uint32_t)ballot(left) & 0xFFu;
            if (m == 0) return kNoCell;
            const uint32_t turned = ((m | (m << 8)) >> range) & 0xFFu;  // the next range after the own one first
            const uint32_t pick = (range + (uint32_t)__builtin_ctz(turned)) % kWorkRanges;
            uint32_t c = 0;
            if (ln == 0) c = atomicAdd(&counter[pick * kCounterStride], 1u);
            c = uni(c) + workers(pick);
            if (c < cells(pick)) return start(pick) + c;
        }
    }
};

// ---------------------------------------------------------------- arithmetic
// What decides signs, orders candidates and makes the outputs, for every
// clipping pass.  The passes have to agree to the last bit (a cell may be
// begun in one and finished in another, and which of the two 64-vertex kernels
// builds a cell must not show).  No rounding of what decides is left to the
// compiler: in the FP32 functions products and sums are fused where fma is
// written and nowhere else.  The FP64 ones make outputs only, or signs that
// are held against a bound far above their rounding.

// Intersection of the planes h (a, b), P and Q by Cramer's rule, in FP32.
struct Solve32 {
    float y0, y1, y2, inv;
    float t0, t1, t2;  // absolute sums of the minors, for the error scale
    __device__ __forceinline__ Solve32(float4 P, float4 Q, float ax, float ay, float az, float b) {
#pragma clang fp contract(off)
        // a_P cross a_Q, a_Q cross a_h, a_h cross a_P
        const float n00 = fmaf(P.y, Q.z, -(P.z * Q.y)), n01 = fmaf(P.z, Q.x, -(P.x * Q.z)),
                    n02 = fmaf(P.x, Q.y, -(P.y * Q.x));
        const float n10 = fmaf(Q.y, az, -(Q.z * ay)), n11 = fmaf(Q.z, ax, -(Q.x * az)),
                    n12 = fmaf(Q.x, ay, -(Q.y * ax));
        const float n20 = fmaf(ay, P.z, -(az * P.y)), n21 = fmaf(az, P.x, -(ax * P.z)),
                    n22 = fmaf(ax, P.y, -(ay * P.x));
        const float det = fmaf(ax, n00, fmaf(ay, n01, az * n02));
        // hardware reciprocal (1 ulp): the FP32 position only decides signs,
        // within the error scale; outputs are recomputed in FP64
        inv = __builtin_amdgcn_rcpf(det);
        y0 = fmaf(Q.w, n20, fmaf(b, n00, P.w * n10)) * inv;
        y1 = fmaf(Q.w, n21, fmaf(b, n01, P.w * n11)) * inv;
        y2 = fmaf(Q.w, n22, fmaf(b, n02, P.w * n12)) * inv;
        t0 = fabsf(n00) + fabsf(n01) + fabsf(n02);
        t1 = fabsf(n10) + fabsf(n11) + fabsf(n12);
        t2 = fabsf(n20) + fabsf(n21) + fabsf(n22);
    }
    // Error scale of the vertex; sbh, sbp, sbq: sizes of the terms of b.
    __device__ __forceinline__ float scale(float sbh, float sbp, float sbq) const {
#pragma clang fp contract(off)
        const float t = fmaf(t2, sbq, fmaf(sbh, t0, sbp * t1));
        return fabsf(y2) + (fabsf(y1) + fmaf(fabsf(inv), t, fabsf(y0)));
    }
};
// A side test of size below this is doubtful: an1 the absolute sum of the
// plane's normal, sb the size of the terms of its b, e the vertex's error scale.
__device__ __forceinline__ float doubt(float an1, float e, float sb) {
#pragma clang fp contract(off)
    return 64.f * kU * fmaf(an1, e, sb);
}
// Some point of the cell's AABB may be beyond the plane; c its corner farthest
// along a, a2 = |a|^2, dw the difference of the weights.
__device__ __forceinline__ bool reaches(float ax, float ay, float az, float b, float cx, float cy, float cz, float a2,
                                        float dw) {
#pragma clang fp contract(off)
    const float mm = fmaf(ax, cx, fmaf(ay, cy, az * cz));
    const float terms = fabsf(ax * cx) + fabsf(ay * cy) + fabsf(az * cz) + a2 + fabsf(dw);
    return mm > fmaf(-8.f * kU, terms, b);
}
// A vertex at squared distance d2 from a box (r2 from the site) might be cut
// by a site of it: d2 - wm < r2 - pw, with a margin for rounding.
template <bool kW>
__device__ __forceinline__ bool ball_test(float d2, float r2, float wm, float pw) {
#pragma clang fp contract(off)
    if constexpr (kW) return (d2 - wm) - (r2 - pw) <= 16.f * kU * (d2 + (r2 + fabsf(pw)) + fabsf(wm));
    else return d2 - r2 <= 16.f * kU * (d2 + r2);
}
// Least plane distance of any site in a box at distance d (the farthest point
// at dfar, read where dw > 0 and the tighter bound is asked for), dw = w_i less
// the largest weight in it; made safe against the rounding of its terms.
template <typename Far>
__device__ __forceinline__ float least_plane(float d, float dw, bool tight, Far dfar) {
#pragma clang fp contract(off)
    float lb, err;
    if (dw > 0.f && tight) {
        // every site j in the box has b_j / |a_j| >= f(|a_j|) with
        // f(t) = t/2 + dw/(2t), and |a_j| lies between the box's nearest
        // and farthest distances: the bound is f at sqrt(dw) clamped to
        // that range (the paper's bound keeps only dw < 0 and is d/2 here)
        const float dc = fminf(fmaxf(__builtin_amdgcn_sqrtf(dw), d), dfar());
        if (dc > 0.f) {
            lb = fmaf(0.5f, dc, 0.5f * dw * __builtin_amdgcn_rcpf(dc));
            err = lb;
        } else {
            lb = 0.5f * d;
            err = 0.5f * d;
        }
    } else if (dw >= 0.f) {
        lb = 0.5f * d;
        err = 0.5f * d;
    } else if (d > 0.f) {
        const float q = 0.5f * dw * __builtin_amdgcn_rcpf(d);
        lb = fmaf(0.5f, d, q);
        err = fmaf(0.5f, d, -q);
    } else {
        lb = -INFINITY;
        err = 0.f;
    }
    return fmaf(-16.f * kU, err, lb);
}

// A plane in FP64.
struct P64 {
    double a0, a1, a2, b;
};
// Intersection of three FP64 planes: y = n / det.
struct Meet64 {
    double bc0, bc1, bc2, ca0, ca1, ca2, ab0, ab1, ab2, det;
    __device__ __forceinline__ Meet64(const P64& A, const P64& B, const P64& C) {
        bc0 = B.a1 * C.a2 - B.a2 * C.a1; bc1 = B.a2 * C.a0 - B.a0 * C.a2; bc2 = B.a0 * C.a1 - B.a1 * C.a0;
        ca0 = C.a1 * A.a2 - C.a2 * A.a1; ca1 = C.a2 * A.a0 - C.a0 * A.a2; ca2 = C.a0 * A.a1 - C.a1 * A.a0;
        ab0 = A.a1 * B.a2 - A.a2 * B.a1; ab1 = A.a2 * B.a0 - A.a0 * B.a2; ab2 = A.a0 * B.a1 - A.a1 * B.a0;
        det = fma(A.a2, bc2, fma(A.a0, bc0, A.a1 * bc1));
    }
    __device__ __forceinline__ void numerator(const P64& A, const P64& B, const P64& C, double* n) const {
        n[0] = fma(C.b, ab0, fma(B.b, ca0, A.b * bc0));
        n[1] = fma(C.b, ab1, fma(B.b, ca1, A.b * bc1));
        n[2] = fma(C.b, ab2, fma(B.b, ca2, A.b * bc2));
    }
};
// Sums over the tetrahedra (reference, Q, P, N): six times the volume and 24
// times the moments, relative to the reference.
struct Fan64 {
    double vol6 = 0.0, mx = 0.0, my = 0.0, mz = 0.0;
    __device__ __forceinline__ void add(double Qx, double Qy, double Qz, double Px, double Py, double Pz, double Nx,
                                        double Ny, double Nz) {
        const double cx = Py * Nz - Pz * Ny, cy = Pz * Nx - Px * Nz, cz = Px * Ny - Py * Nx;
        const double det = fma(Qz, cz, fma(Qx, cx, Qy * cy));
        vol6 += det;
        mx = fma(det, Qx + Px + Nx, mx);
        my = fma(det, Qy + Py + Ny, my);
        mz = fma(det, Qz + Pz + Nz, mz);
    }
};
// One coordinate of the centroid; inv = 1 / (4 vol6).
__device__ __forceinline__ float centroid_of(float p, double ref, double m, double inv) {
    return (float)fma(m, inv, (double)p + ref);
}

// queue capacity of the pass of vertex capacity cap
constexpr int queue_cap(int cap) { return cap < kQueue0 ? kQueue0 : cap; }

}  // namespace
}  // namespace vd
