// Backward pass: gradients of cell volumes, centroids and vertex positions
// with respect to site positions and weights, through the combinatorics of
// the last build (its staged cell records are the checkpoint; nothing is
// re-clipped).
//
// In the frame of site p_i a cell is {y : a_f . y <= b_f} (paper Sec. 3,
// Eq. 1: a_f = p_j - p_i, b_f = (|a_f|^2 + w_i - w_j) / 2 for the plane of
// site j; a box face has a_f = +-e_k).  Moving plane f by (da_f, db_f) moves
// the points y of its facet along the outward normal by
// (db_f - da_f . y) / |a_f|, so with A_f, Y_f and S_f = int_F y y^T dA the
// area, centroid and second moment of facet f:
//     dV = sum_f (A_f db_f - A_f Y_f . da_f) / |a_f|
//     dm = sum_f (A_f Y_f db_f - S_f da_f) / |a_f|,   m = int_C y dV,
// and c = p_i + m / V.  A vertex is x = p_i + M^-1 b (rows of M: the normals
// of its three planes), so a gradient g on x gives d/db = M^-T g and
// d/da_k = -(M^-T g)_k y.  The plane parameters then carry the gradient to
// the sites: da_f = dp_j - dp_i, db_f = a_f . da_f + (dw_i - dw_j) / 2, or
// db_f = -a_f . dp_i for a box face.
//
// Layout: a group of lanes per cell, by the pass that built it: half a wave up
// to 64 vertices, a wave up to 128, a block above (the lists of the build name
// the cells of the last two).  Lanes over facets put the FP64 planes into LDS,
// lanes over vertices solve each vertex once from them, lanes over facets walk
// their rings over the solved vertices; one walk gives the facet integrals,
// from them V and m, then the gradient of each plane.  (Solving a vertex from
// scattered loads wherever a ring met it, in two walks, was six solves a
// vertex: 935 us at 50k sites, this 140.)  The share a cell sends to neighbour
// j goes to the place of its facet in j's row (found by a binary search of
// the row), so that each site sums what stands in its own row (deterministic).
// Shares stay in FP64 until that sum: around thin cells (tight clusters) the
// shares of two neighbouring cells are many orders of magnitude larger than
// the site gradient they cancel to.
// A facet whose neighbour does not list the cell back (possible only on
// configurations FP32 cannot decide) is added with an atomic instead.
// When the box is the sites' own bounding box its faces move with the
// extreme sites (b = p_i,k - min_j p_j,k for a lower face, max_j p_j,k - p_i,k
// for an upper one): the sum over all cells of dL/db of each face goes to the
// site on that face with the lowest index, summed in a fixed order.
#include <mutex>

#include "vd_wave.h"

// Shares of thin cells cancel down to their last bits, so a gradient there
// depends on every rounding and on the order of every sum.  Neither is left
// to the compiler: products and sums are fused where it is written (fma) and
// nowhere else, and the sums over facets run in the order of one wave with
// facet f in lane f % 64, whatever the size of the group.
#pragma clang fp contract(off)

namespace vd {
namespace {

// Vertices of a cell of the block class kept in LDS (104 KB declared, with
// vertex gradients 130 KB; the compiler puts arrays of the threads into what
// is left, 156 and 136 KB in all); a larger one solves its vertices where a
// ring meets them.
constexpr int kBwdBlockCap = 2048;
constexpr int kBwdBlockCapVert = 1536;

struct CellRec {
    const float4* V;
    const uint64_t* T64;
    const int32_t* C;
    const uint16_t* FS;
    const uint16_t* FV;
};

__device__ inline CellRec record_of(const BwdArgs& a, uint32_t k) {
    const uint32_t loc = a.loc[k], tier = loc >> 30;
    const Stage st = tier == 0 ? a.stage[0] : (tier == 1 ? a.stage[1] : (tier == 2 ? a.stage[2] : a.stage[3]));
    const int64_t slot = loc & 0x3FFFFFFFu;
    const int64_t cap = st.cap;
    CellRec r;
    r.V = st.vert + slot * cap;
    r.T64 = st.tri64 ? st.tri64 + slot * cap : nullptr;
    r.C = st.code + slot * cap;
    r.FS = st.fsize + slot * cap;
    r.FV = st.fv + slot * 3 * cap;
    return r;
}

__device__ inline void ranks_of(const CellRec& r, uint32_t u, uint32_t* t) {
    if (r.T64) {
        const uint64_t x = r.T64[u];
        t[0] = (uint32_t)(x & 0x1FFFFFu);
        t[1] = (uint32_t)((x >> 21) & 0x1FFFFFu);
        t[2] = (uint32_t)((x >> 42) & 0x1FFFFFu);
    } else {
        const uint32_t x = __float_as_uint(r.V[u].w);
        t[0] = x & 1023u;
        t[1] = (x >> 10) & 1023u;
        t[2] = (x >> 20) & 1023u;
    }
}

struct Site {
    double p[3];
    double w;
};

// u0 v0 + u1 v1 + u2 v2, by the product that is rounded on its own (the first
// of three in the determinants, the second elsewhere).
__device__ inline double dot1(const double* u, const double* v) {
    return fma(u[2], v[2], fma(u[1], v[1], u[0] * v[0]));
}
__device__ inline double dot(const double* u, const double* v) {
    return fma(u[2], v[2], fma(u[0], v[0], u[1] * v[1]));
}
__device__ inline void cross(const double* u, const double* v, double* o) {
    o[0] = fma(u[1], v[2], -(u[2] * v[1]));
    o[1] = fma(u[2], v[0], -(u[0] * v[2]));
    o[2] = fma(u[0], v[1], -(u[1] * v[0]));
}

// Plane of facet code `code` in the frame of site s, FP64 from the FP32 inputs.
__device__ inline void plane_of(const BwdArgs& a, const Site& s, int32_t code, double* n, double* b) {
    if (code >= 0) {
        const float4 q = a.pts[a.inv[code]];
        n[0] = (double)q.x - s.p[0];
        n[1] = (double)q.y - s.p[1];
        n[2] = (double)q.z - s.p[2];
        *b = 0.5 * ((s.w - (double)q.w) + dot(n, n));
    } else {
        const int c = -code - 1, ax = c >> 1, side = c & 1;
        n[0] = n[1] = n[2] = 0.0;
        n[ax] = side ? 1.0 : -1.0;
        *b = side ? ((double)a.bbox[3 + ax] - s.p[ax]) : (s.p[ax] - (double)a.bbox[ax]);
    }
}

// A vertex of the cell: its position num * inv (frame of the site, inv the
// reciprocal of det, zero if that is), the cofactors of the rows of M (so that
// M^-T g = (c_k . g) / det), and its ranks.
struct Vtx {
    double num[3], inv;
    double c[3][3];
    double det;
    uint32_t t[3];
};

// from its planes (a, b), in the order of its ranks
__device__ inline void vertex_from(const double* p0, const double* p1, const double* p2, Vtx* v) {
    cross(p1, p2, v->c[0]);
    cross(p2, p0, v->c[1]);
    cross(p0, p1, v->c[2]);
    v->det = dot1(p0, v->c[0]);
    v->inv = v->det != 0.0 ? 1.0 / v->det : 0.0;
    for (int q = 0; q < 3; ++q) v->num[q] = fma(p2[3], v->c[2][q], fma(p0[3], v->c[0][q], p1[3] * v->c[1][q]));
}

// from the input, where the planes are not at hand
__device__ inline void vertex(const BwdArgs& a, const Site& s, const CellRec& r, uint32_t u, Vtx* v) {
    ranks_of(r, u, v->t);
    double p[3][4];
    for (int k = 0; k < 3; ++k) plane_of(a, s, r.C[v->t[k]], p[k], &p[k][3]);
    vertex_from(p[0], p[1], p[2], v);
}

// Value of lane ^ kMask.
template <int kMask>
__device__ inline double lane_xor(double x) {
    if constexpr (kMask == 1 || kMask == 2) {
        return dpp64<(kMask == 1 ? 0xB1 : 0x4E), 0xF>(x);  // within quads
    } else if constexpr (kMask < 32) {
        const int lo = __builtin_amdgcn_ds_swizzle(__double2loint(x), 0x1F | (kMask << 10));
        const int hi = __builtin_amdgcn_ds_swizzle(__double2hiint(x), 0x1F | (kMask << 10));
        return __hiloint2double(hi, lo);
    } else {
        return __shfl_xor(x, kMask);
    }
}
// Sums over the facets of a cell: every lane adds what its facets give, in
// rounds of GS facets; total() is the sum in every lane of the group, all lanes
// of the wave (of the block: red, 256 * N doubles of LDS) taking part.
template <int GS, int N>
struct FacetSum {
    double v[N];
    __device__ void init() {
        for (int k = 0; k < N; ++k) v[k] = 0.0;
    }
    // after each round: the round's sums of this lane
    __device__ void add(const double* x, bool first, double* red) {
        if constexpr (GS <= 64) {
            for (int k = 0; k < N; ++k) v[k] = first ? x[k] : v[k] + x[k];
        } else {
            __syncthreads();
            for (int k = 0; k < N; ++k) red[k * GS + threadIdx.x] = x[k];
            __syncthreads();
            for (int w = 0; w < GS / 64; ++w)
                for (int k = 0; k < N; ++k) {
                    const double t = red[k * GS + w * 64 + (threadIdx.x & 63)];
                    v[k] = first && w == 0 ? t : v[k] + t;
                }
        }
    }
    __device__ void total() {
        for (int k = 0; k < N; ++k) {
            double x = v[k];
            if constexpr (GS > 32) x += lane_xor<32>(x);
            x += lane_xor<16>(x);
            x += lane_xor<8>(x);
            x += lane_xor<4>(x);
            x += lane_xor<2>(x);
            x += lane_xor<1>(x);
            v[k] = x;
        }
    }
};
// Inclusive sum over the lanes of a group up to this one, and the group's total.
template <int GS>
__device__ inline uint32_t gscan(uint32_t v, uint32_t* total, uint32_t* red) {
    const int ln = threadIdx.x & (GS < 64 ? GS - 1 : 63);
    uint32_t x = v;
    for (int o = 1; o < (GS < 64 ? GS : 64); o <<= 1) {
        const uint32_t y = __shfl_up(x, o, GS < 64 ? GS : 64);
        if (ln >= o) x += y;
    }
    if constexpr (GS <= 64) {
        *total = __shfl(x, GS - 1, GS);
    } else {
        __syncthreads();
        if (ln == 63) red[threadIdx.x >> 6] = x;
        __syncthreads();
        uint32_t t = 0;
        for (int w = 0; w < GS / 64; ++w) {
            if (w < (int)(threadIdx.x >> 6)) x += red[w];
            t += red[w];
        }
        *total = t;
    }
    return x;
}
template <int GS>
__device__ inline void gsync() {
    if constexpr (GS > 64) __syncthreads();
    else wave_sync<true>();
}

// Is `who` among the neighbours of cell j (original ids)?  Binary search of
// the ascending site codes at the end of j's facet list.
__device__ inline int64_t find_facet(const BwdArgs& a, uint32_t j, int32_t who) {
    const CellRec r = record_of(a, a.inv[j]);
    const int F = (int)a.cnt_f[j], nn = (int)a.cnt_n[j];
    int lo = F - nn, hi = F - 1;
    while (lo <= hi) {
        const int mid = (lo + hi) >> 1;
        const int32_t c = r.C[mid];
        if (c == who) return mid;
        if (c < who) lo = mid + 1;
        else hi = mid - 1;
    }
    return -1;
}

// LDS of a group: planes and vertices of a cell of up to CAPF facets and CAPV
// vertices; with vertex gradients also M^-T g of each vertex and its facets.
template <int CAPV, int CAPF, bool kVert>
struct BwdMem {
    double pl[CAPF][4];  // a, b
    double v[CAPV][4];   // num, inv
    double gk[kVert ? CAPV : 1][3];
    uint16_t t[kVert ? CAPV : 1][4];  // ranks; [3]: 1 if det is zero
};

// What the walk of a facet's ring gives: area, centroid and second moment
// integrals, and dL/da_f, dL/db_f from the vertices.  A1 and AY1, which V and m
// are made of, take the last vertex of each triangle unrounded (num * inv
// fused into the edge and the sum), A and AY take it rounded.
struct Facet {
    double n[3], b, D, A1, AY1[3], A, AY[3], S[6], dA[3], dB, g[3];
};

// The cells of one size class: kTier 0 all sites (Morton order), 1 and 2 the
// cells named in list.
template <int GS, int CAPV, int CAPF, bool kVert, int kTier>
__global__ __launch_bounds__(256, (kTier < 2 ? 3 : 1)) void k_bwd_cells(BwdArgs a, const uint32_t* __restrict__ list,
                                                                        int64_t count) {
    constexpr int kGroups = 256 / GS;
    using Mem = BwdMem<CAPV, CAPF, kVert>;
    __shared__ Mem mem[kGroups];
    __shared__ double red[GS > 64 ? 4 * 256 : 1];
    __shared__ uint32_t redu[4];
    static_assert(sizeof(mem) + sizeof(red) + sizeof(redu) <= 160 * 1024 / (kTier < 2 ? 3 : 1),
                  "the groups of a block must fit the LDS of a CU, three blocks of the smaller classes");
    const int ln = threadIdx.x % GS, grp = threadIdx.x / GS;
    Mem& M = mem[grp];
    // every group of a wave takes the same number of turns (the sums over
    // lanes need the whole wave)
    for (int64_t it0 = (int64_t)blockIdx.x * kGroups; it0 < count; it0 += (int64_t)gridDim.x * kGroups) {
        const int64_t it = it0 + grp;
        bool on = it < count;
        const uint32_t k = on ? (kTier ? list[it] : (uint32_t)it) : 0u;
        const int64_t i = a.order[k];
        const float4 ps = a.pts[k];
        if (kTier == 0 && a.moving_box && on && ln < 6) {
            // the lowest original index of a site on each face of the sites' box
            // (the box is their FP32 minimum and maximum, so some site equals each face)
            const float v = ln < 2 ? ps.x : (ln < 4 ? ps.y : ps.z);
            if (v == a.bbox[(ln & 1) ? 3 + (ln >> 1) : (ln >> 1)]) atomicMin(&a.box_arg[ln], (uint32_t)i);
        }
        const uint32_t tier = a.loc[k] >> 30;
        on = on && (kTier == 0 ? tier == 0 : (kTier == 1 ? tier == 1 : tier >= 2));
        double gc[3] = {0.0, 0.0, 0.0};
        double gv = 0.0;
        int nv = 0, F = 0;
        if (on) {
            if (a.g_cen)
                for (int q = 0; q < 3; ++q) gc[q] = (double)a.g_cen[3 * i + q];
            gv = a.g_vol ? (double)a.g_vol[i] : 0.0;
            nv = (int)a.cnt_v[i];
            F = (int)a.cnt_f[i];
            // empty cell: V = 0 and c = p_i
            if (nv == 0 && ln == 0) a.gself[i] = make_double4(gc[0], gc[1], gc[2], 0.0);
        }
        Site s;
        s.p[0] = ps.x; s.p[1] = ps.y; s.p[2] = ps.z;
        s.w = ps.w;
        const CellRec r = record_of(a, k);
        // the register passes hold at most CAPV vertices and planes
        const bool cached = kTier < 2 || (nv <= CAPV && F <= CAPF);
        const float* gvert = kVert ? a.g_vert + 3 * a.off_v[i] : nullptr;
        gsync<GS>();  // the group is done with the previous cell
        if (cached)
            for (int f = ln; f < F; f += GS) {
                double n[3], b;
                plane_of(a, s, r.C[f], n, &b);
                M.pl[f][0] = n[0]; M.pl[f][1] = n[1]; M.pl[f][2] = n[2];
                M.pl[f][3] = b;
            }
        gsync<GS>();
        // every vertex once, with vertex gradients also its share of each of its
        // planes (M^-T g)
        if (cached)
            for (int u = ln; u < nv; u += GS) {
                Vtx v;
                ranks_of(r, (uint32_t)u, v.t);
                vertex_from(M.pl[v.t[0]], M.pl[v.t[1]], M.pl[v.t[2]], &v);
                for (int q = 0; q < 3; ++q) M.v[u][q] = v.num[q];
                M.v[u][3] = v.inv;
                if constexpr (kVert) {
                    const double g[3] = {(double)gvert[3 * u], (double)gvert[3 * u + 1], (double)gvert[3 * u + 2]};
                    for (int q = 0; q < 3; ++q) {
                        M.gk[u][q] = v.det == 0.0 ? 0.0 : dot(v.c[q], g) / v.det;
                        M.t[u][q] = (uint16_t)v.t[q];
                    }
                    M.t[u][3] = v.det == 0.0 ? 1 : 0;
                }
            }
        gsync<GS>();
        // the walk of facet f's ring
        auto walk = [&](int f, uint32_t base, uint32_t sz, Facet& o) {
            if (cached) {
                for (int q = 0; q < 3; ++q) o.n[q] = M.pl[f][q];
                o.b = M.pl[f][3];
            } else {
                plane_of(a, s, r.C[f], o.n, &o.b);
            }
            o.D = sqrt(dot(o.n, o.n));
            const double nh[3] = {o.n[0] / o.D, o.n[1] / o.D, o.n[2] / o.D};
            o.A = o.A1 = o.dB = 0.0;
            for (int q = 0; q < 3; ++q) o.AY[q] = o.AY1[q] = o.dA[q] = o.g[q] = 0.0;
            for (int q = 0; q < 6; ++q) o.S[q] = 0.0;
            // a vertex of the ring: num and inv, the position y, and its part of
            // the gradient: its share of plane f, and the direct term dx/dp_i = I
            // once per vertex (with its lowest facet)
            auto take = [&](uint32_t u, double* num, double* inv, double* y) {
                double gk = 0.0;
                bool flat = true;
                uint32_t t[3];
                if (cached) {
                    for (int q = 0; q < 3; ++q) num[q] = M.v[u][q];
                    *inv = M.v[u][3];
                    if constexpr (kVert) {
                        for (int q = 0; q < 3; ++q) t[q] = M.t[u][q];
                        gk = t[0] == (uint32_t)f ? M.gk[u][0] : (t[1] == (uint32_t)f ? M.gk[u][1] : M.gk[u][2]);
                        flat = M.t[u][3] != 0;
                    }
                } else {
                    Vtx v;
                    vertex(a, s, r, u, &v);
                    for (int q = 0; q < 3; ++q) num[q] = v.num[q];
                    *inv = v.inv;
                    if constexpr (kVert) {
                        const double g[3] = {(double)gvert[3 * u], (double)gvert[3 * u + 1], (double)gvert[3 * u + 2]};
                        for (int q = 0; q < 3; ++q) t[q] = v.t[q];
                        flat = v.det == 0.0;
                        const int q0 = t[0] == (uint32_t)f ? 0 : (t[1] == (uint32_t)f ? 1 : 2);
                        if (!flat) gk = dot(v.c[q0], g) / v.det;
                    }
                }
                for (int q = 0; q < 3; ++q) y[q] = num[q] * *inv;
                if constexpr (kVert) {
                    if (!flat) {
                        o.dB += gk;
                        for (int q = 0; q < 3; ++q) o.dA[q] = fma(-y[q], gk, o.dA[q]);
                        if (min(t[0], min(t[1], t[2])) == (uint32_t)f)
                            for (int q = 0; q < 3; ++q) o.g[q] += (double)gvert[3 * u + q];
                    }
                }
            };
            double num[3], inv, P0[3], P1[3], P2[3];
            take(r.FV[base], num, &inv, P0);
            take(r.FV[base + 1], num, &inv, P1);
            for (uint32_t t = 2; t < sz; ++t) {
                take(r.FV[base + t], num, &inv, P2);
                double e1[3], e2[3], cr[3], sm[3], sm1[3];
                for (int q = 0; q < 3; ++q) {
                    e1[q] = P1[q] - P0[q];
                    e2[q] = fma(num[q], inv, -P0[q]);
                    const double s01 = P0[q] + P1[q];
                    sm1[q] = fma(num[q], inv, s01);
                    sm[q] = s01 + P2[q];
                }
                cross(e1, e2, cr);
                double d = dot(cr, nh), at = 0.5 * d;
                o.A1 += at;
                for (int q = 0; q < 3; ++q) o.AY1[q] = fma(1.0 / 3.0, at * sm1[q], o.AY1[q]);
                for (int q = 0; q < 3; ++q) e2[q] = P2[q] - P0[q];
                cross(e1, e2, cr);
                d = dot(cr, nh);
                at = 0.5 * d;
                o.A += at;
                for (int q = 0; q < 3; ++q) o.AY[q] = fma(1.0 / 3.0, at * sm[q], o.AY[q]);
                // int over the triangle of y y^T = at/12 (sum_i v_i v_i^T + s s^T)
                const double h = at * (1.0 / 12.0);
                auto second = [&](int x, int y) {
                    return fma(sm[x], sm[y], fma(P2[x], P2[y], fma(P1[x], P1[y], P0[x] * P0[y])));
                };
                o.S[0] = fma(h, second(0, 0), o.S[0]);
                o.S[1] = fma(h, second(0, 1), o.S[1]);
                o.S[2] = fma(h, second(0, 2), o.S[2]);
                o.S[3] = fma(h, second(1, 1), o.S[3]);
                o.S[4] = fma(h, second(1, 2), o.S[4]);
                o.S[5] = fma(h, second(2, 2), o.S[5]);
                for (int q = 0; q < 3; ++q) P1[q] = P2[q];
            }
        };
        // the groups of a wave take the same number of rounds
        int rounds = (F + GS - 1) / GS;
        if constexpr (GS < 64) rounds = max(rounds, __shfl_xor(rounds, 32));
        Facet fa{};  // the facet of the last round walked
        FacetSum<GS, 4> vm;
        vm.init();
        uint32_t carry = 0;
        for (int q0 = 0; q0 < rounds; ++q0) {
            const int f = q0 * GS + ln;
            const uint32_t sz = f < F ? (uint32_t)r.FS[f] : 0u;
            uint32_t total;
            const uint32_t x = gscan<GS>(sz, &total, redu);
            double part[4] = {0.0, 0.0, 0.0, 0.0};
            if (f < F && sz >= 3) {
                walk(f, carry + x - sz, sz, fa);
                part[0] = fa.b * fa.A1 / (3.0 * fa.D);
                for (int q = 0; q < 3; ++q) part[1 + q] = fa.b * fa.AY1[q] / (4.0 * fa.D);
            }
            vm.add(part, q0 == 0, red);
            carry += total;
        }
        vm.total();
        // L = gv V + gc . (p_i + m / V): dL/dV and dL/dm
        const double V = vm.v[0];
        const double m[3] = {vm.v[1], vm.v[2], vm.v[3]};
        double alpha = 0.0, gam[3] = {0.0, 0.0, 0.0};
        if (V != 0.0) {
            alpha = gv - dot(gc, m) / (V * V);
            for (int q = 0; q < 3; ++q) gam[q] = gc[q] / V;
        }
        FacetSum<GS, 4> self;  // the site's own share: dp, dw
        self.init();
        carry = 0;
        for (int q0 = 0; q0 < rounds; ++q0) {
            const int f = q0 * GS + ln;
            const uint32_t sz = f < F ? (uint32_t)r.FS[f] : 0u;
            if (rounds > 1) {
                uint32_t total;
                const uint32_t x = gscan<GS>(sz, &total, redu);
                if (f < F && sz >= 3) walk(f, carry + x - sz, sz, fa);
                carry += total;
            }
            double part[4] = {0.0, 0.0, 0.0, 0.0};
            if (f < F && sz >= 3) {
                const int32_t code = r.C[f];
                // dL/db_f and dL/da_f from the cell integrals
                const double dB = fa.dB + fma(alpha, fa.A, dot(gam, fa.AY)) / fa.D;
                for (int q = 0; q < 3; ++q) part[q] = fa.g[q];
                if (code >= 0) {
                    // site plane: a = p_j - p_i, b = (|a|^2 + w_i - w_j) / 2
                    const double Sg[3] = {fma(fa.S[2], gam[2], fma(fa.S[0], gam[0], fa.S[1] * gam[1])),
                                          fma(fa.S[4], gam[2], fma(fa.S[1], gam[0], fa.S[3] * gam[1])),
                                          fma(fa.S[5], gam[2], fma(fa.S[2], gam[0], fa.S[4] * gam[1]))};
                    double gp[3];
                    for (int q = 0; q < 3; ++q) {
                        gp[q] = fma(dB, fa.n[q], fa.dA[q] - fma(alpha, fa.AY[q], Sg[q]) / fa.D);
                        part[q] -= gp[q];
                    }
                    part[3] = 0.5 * dB;
                    const double4 out = make_double4(gp[0], gp[1], gp[2], -0.5 * dB);
                    const int64_t at = find_facet(a, (uint32_t)code, (int32_t)i);
                    if (at >= 0) {
                        a.gf[a.off_f[code] + at] = out;
                    } else {
                        // not listed back: nobody writes this facet's own place
                        a.gf[a.off_f[i] + f] = make_double4(0.0, 0.0, 0.0, 0.0);
                        double* o = a.orphan + 4 * (int64_t)code;
                        atomicAdd(o, out.x);
                        atomicAdd(o + 1, out.y);
                        atomicAdd(o + 2, out.z);
                        atomicAdd(o + 3, out.w);
                    }
                } else {
                    // box face: b = +-(B_k - p_i,k), a fixed; its place in the row
                    // holds dL/db of the face
                    for (int q = 0; q < 3; ++q) part[q] -= dB * fa.n[q];
                    if (a.moving_box) a.gf[a.off_f[i] + f].x = dB;
                }
            }
            self.add(part, q0 == 0, red);
        }
        self.total();
        if (on && nv > 0 && ln == 0)
            a.gself[i] = make_double4(self.v[0] + gc[0], self.v[1] + gc[1], self.v[2] + gc[2], self.v[3]);
    }
}

// dL/db of the box faces over the cells slot, slot + nslots, ...: a cell's box
// facets stand first in its row, facet f adding to sum f of its face.
__device__ inline void box_slot(const BwdArgs& a, int64_t slot, int64_t nslots, double* sum) {
    double acc[6][6];
    for (int c = 0; c < 6; ++c)
        for (int f = 0; f < 6; ++f) acc[c][f] = 0.0;
    bool any = false;
    for (int64_t i = slot; i < a.n; i += nslots) {
        const int nbox = (int)(a.cnt_f[i] - a.cnt_n[i]);
        if (nbox == 0) continue;
        any = true;
        const CellRec r = record_of(a, a.inv[i]);
        for (int f = 0; f < nbox && f < 6; ++f) {
            const int face = -r.C[f] - 1;
            const double d = a.gf[a.off_f[i] + f].x;
#pragma unroll
            for (int c = 0; c < 6; ++c)
#pragma unroll
                for (int l = 0; l < 6; ++l)
                    if (c == face && l == f) acc[c][l] += d;
        }
    }
    for (int c = 0; c < 6; ++c)
        sum[c] = any ? ((acc[c][0] + acc[c][4]) + acc[c][2]) + ((acc[c][1] + acc[c][5]) + acc[c][3]) : 0.0;
}

__global__ __launch_bounds__(256) void k_bwd_box_part(BwdArgs a, int64_t nslots) {
    const int64_t slot = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (slot >= nslots) return;
    double s[6];
    box_slot(a, slot, nslots, s);
    for (int c = 0; c < 6; ++c) a.box_part[slot * 6 + c] = s[c];
}

// Sum over the slots, in a fixed order (one block); kDirect: the slots are
// summed here, where they are few.
template <bool kDirect>
__global__ __launch_bounds__(256) void k_bwd_box_sum(BwdArgs a, int64_t nslots) {
    __shared__ double red[6][256];
    double s[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for (int64_t w = threadIdx.x; w < nslots; w += 256) {
        double p[6];
        if (kDirect) box_slot(a, w, nslots, p);
        else
            for (int c = 0; c < 6; ++c) p[c] = a.box_part[w * 6 + c];
        for (int c = 0; c < 6; ++c) s[c] += p[c];
    }
    for (int c = 0; c < 6; ++c) red[c][threadIdx.x] = s[c];
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o)
            for (int c = 0; c < 6; ++c) red[c][threadIdx.x] += red[c][threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x < 6) a.box_sum[threadIdx.x] = red[threadIdx.x][0];
}

// Per site: its own cell's share, what its neighbours' cells put into its row
// (ascending), then the asymmetric remainder and the box faces.  Four lanes a
// site, one for each component, so that a row is read in whole lines.
__global__ __launch_bounds__(256) void k_bwd_gather(BwdArgs a) {
    const int64_t j = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 2;
    const int q = threadIdx.x & 3;
    if (j >= a.n) return;
    const int F = (int)a.cnt_f[j], nn = (int)a.cnt_n[j];
    double g = reinterpret_cast<const double*>(a.gself + j)[q];
    if (nn > 0) {
        const double* row = reinterpret_cast<const double*>(a.gf + a.off_f[j] + (F - nn)) + q;
        for (int t = 0; t < nn; ++t) g += row[4 * t];
    }
    g += a.orphan[4 * j + q];
    if (a.moving_box && q < 3)
        for (int c = 2 * q; c < 2 * q + 2; ++c)
            if (a.box_arg[c] == (uint32_t)j) g += (c & 1) ? a.box_sum[c] : -a.box_sum[c];
    if (q < 3) a.g_xyz[3 * j + q] = (float)g;
    else if (a.g_w) a.g_w[j] = (float)g;
}

// Fill of 64-bit words (clears the scratch of the allocation-free entry
// point with a kernel rather than a memset node, so that the call can be
// captured into a HIP graph).
__global__ __launch_bounds__(256) void k_fill_u64(uint64_t* dst, int64_t count, uint64_t value) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = value;
}

// Device scratch of vd_backward_noalloc: the facet shares, the per-site
// shares, the asymmetric remainders and the box-face partials of one
// backward, in one fixed array per device (set up once per device by
// bwd_scratch_init; host code uses only the address it returns).
static __device__ __align__(256) unsigned char scratch[kBwdScratchBytes];

constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices] = {};
std::mutex g_scratch_mu;

}  // namespace

hipError_t bwd_scratch_init(int device, void** ptr) {
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[device] = p;
    }
    *ptr = g_scratch_ptr[device];
    return hipSuccess;
}

hipError_t launch_fill_u64(uint64_t* dst, int64_t count, uint64_t value, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    int64_t blocks = (count + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_fill_u64, dim3((unsigned)blocks), dim3(256), 0, s, dst, count, value);
    return hipGetLastError();
}

int64_t bwd_slots(int64_t n) {
    const int64_t slots = n < 65536 ? n : 65536;
    return (slots + 3) / 4 * 4;
}

namespace {

template <bool kVert>
void launch_cells(const BwdArgs& a, hipStream_t s) {
    auto blocks = [](int64_t items, int64_t per_block, int64_t limit) {
        const int64_t b = (items + per_block - 1) / per_block;
        return dim3((unsigned)(b < limit ? b : limit));
    };
    hipLaunchKernelGGL((k_bwd_cells<32, kTierCap[0], kTierCap[0], kVert, 0>), blocks(a.n, 8, 16384), dim3(256), 0, s, a,
                       (const uint32_t*)nullptr, a.n);
    if (a.count[0] > 0)
        hipLaunchKernelGGL((k_bwd_cells<64, kTierCap[1], kTierCap[1], kVert, 1>), blocks(a.count[0], 4, 16384),
                           dim3(256), 0, s, a, a.list[0], a.count[0]);
    if (a.count[1] > 0) {
        constexpr int cap = kVert ? kBwdBlockCapVert : kBwdBlockCap;
        hipLaunchKernelGGL((k_bwd_cells<256, cap, cap / 2 + 2, kVert, 2>), blocks(a.count[1], 1, 16384), dim3(256), 0,
                           s, a, a.list[1], a.count[1]);
    }
}

}  // namespace

hipError_t launch_backward(const BwdArgs& a, hipStream_t s) {
    if (a.n < 1) return hipSuccess;
    if (a.g_vert) launch_cells<true>(a, s);
    else launch_cells<false>(a, s);
    if (a.moving_box) {
        const int64_t slots = bwd_slots(a.n);
        if (slots <= 4096) {
            hipLaunchKernelGGL(k_bwd_box_sum<true>, dim3(1), dim3(256), 0, s, a, slots);
        } else {
            hipLaunchKernelGGL(k_bwd_box_part, dim3((unsigned)((slots + 255) / 256)), dim3(256), 0, s, a, slots);
            hipLaunchKernelGGL(k_bwd_box_sum<false>, dim3(1), dim3(256), 0, s, a, slots);
        }
    }
    hipLaunchKernelGGL(k_bwd_gather, dim3((unsigned)((a.n * 4 + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace vd
