// The 64-vertex pass with the default search options (directional plus ball
// culling, best-first order, no warm start) and FP32 predicates, or, in
// mixed precision, the cells whose signs FP32 can be sure of.  It builds
// nearly every cell of a diagram, so it is written on its own: the cell
// builder of vd_clip.hip with everything those options never reach taken
// out, the same decisions in the same order (the arithmetic behind every
// decision is that of vd_wave.h in both, so both give the same cells, vertex
// order included).
//
// A cell this pass cannot finish goes elsewhere: one that outgrows 64
// vertices is handed on with its state (HandoffT) to the 128-vertex pass;
// one whose FP32 signs turn out inconsistent, or whose path to the root has
// more than 64 siblings, or in mixed precision one that meets a doubtful sign,
// goes on the retry list, which the general 64-vertex kernel builds from the
// start, with FP64 signs where needed.
//
// What bounds it: instruction issue, not memory.  One wave owns one cell
// (vertex v in lane v).  With many cells the vector unit issues in four of
// five slots; with few cells (a thousand sites are one cell per SIMD) the
// wave waits for its own code to arrive, since every instruction line is read
// for the first time.  Both ask for the same thing, fewer and smaller code:
// no FP64 re-evaluation inside the loops, one copy of the leaf and the clip,
// planes without the records that only FP64 signs read, masks of lanes kept
// as scalars (they are exec and carry masks as they are), vertex indices in
// bytes (a permute builds or changes a record in one instruction), node
// records passed on by lane moves inside the subtraction that uses them, and
// the squared length of a vertex kept beside it.  Clustered 1M sites, against
// the general pass as it was: 7600 instead of 12150 vector and 5600 instead
// of 8800 scalar instructions a cell, 15 instead of 37 KB of code, 24.8 ->
// 12.5 ms; a thousand sites 419 -> about 90 us.  Mixed precision, clustered
// 333k: 8.0 -> 4.6 ms and 0.5 for the cells left to the general pass.  The
// vector unit is then full (99% of one instruction in four cycles a SIMD) and
// the scalar unit at 73% of one a cycle a CU.
#include "vd_wave.h"

// v_writelane (the compiler has no builtin of that name): v with lane l
// replaced by the uniform value x.
extern "C" __device__ int vd_writelane(int x, int l, int v) __asm("llvm.amdgcn.writelane.i32");

namespace vd {
namespace {

__device__ __forceinline__ int wrl(int x, int l, int v) { return vd_writelane(x, l, v); }
__device__ __forceinline__ uint32_t wrl(uint32_t x, int l, uint32_t v) {
    return (uint32_t)vd_writelane((int)x, l, (int)v);
}

constexpr int kInfBits = 0x7F800000;

// m without bit l, in one scalar instruction
__device__ __forceinline__ uint64_t without(uint64_t m, int l) {
    asm("s_bitset0_b64 %0, %1" : "+s"(m) : "s"(l));
    return m;
}

// c ? a : b by value: the operator on two members selects between their
// addresses, which can leave the whole cell in scratch memory
__device__ __forceinline__ float pick(bool c, float a, float b) { return c ? a : b; }
// The lanes of a uniform mask, as a condition: the mask is the execution or
// carry mask itself, no shift per lane.
__device__ __forceinline__ bool in_mask(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
// Keeps a uniform value in a vector register: an instruction takes one
// scalar operand at most, so a second one costs a move at every use.  The
// compiler takes the value for divergent from here on: it must not reach a
// branch but through a ballot or uni().
__device__ __forceinline__ void in_vgpr(float& v) { asm("" : "+v"(v)); }
__device__ __forceinline__ uint32_t byte_of(uint32_t w, int k) { return (w >> (8 * k)) & 0xFFu; }
// Value of the even (odd) lane of each pair, for both lanes.
template <int kCtrl>
__device__ __forceinline__ float pair_move(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), kCtrl, 0xF, 0xF, true));
}
__device__ __forceinline__ float of_even(float v) { return pair_move<0xA0>(v); }  // quad_perm [0,0,2,2]
__device__ __forceinline__ float of_odd(float v) { return pair_move<0xF5>(v); }   // quad_perm [1,1,3,3]
__device__ __forceinline__ int imin_wave(int v) {
    return wave_reduce_i(v, [](int a, int b) { return min(a, b); });
}
__device__ __forceinline__ double rdl64(double v, int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                            __builtin_amdgcn_readlane(__double2loint(v), l));
}

// Per-wave LDS.  While the cell is clipped: planes, the tables through which
// the new vertices of a clip find each other, and the queue entries beyond
// the first 64.  While it is finished (the planes' codes are read first, the
// queue is empty): FP64 planes, then vertex positions in their place, and
// the facet tables.
struct ClipMem {
    float4 pl[64];      // planes: a.xyz, b (frame of the site)
    uint2 tab[64];      // .x: new vertex by its first old plane, .y: by its second (serial tag above the index)
    int32_t pcode[64];  // Morton index of the plane's site, or box code -1..-6
    float psb[64];      // size of the terms b is formed from (error scale; checked signs only)
    uint32_t sor[72];   // free slot of rank
    uint32_t edge[72];  // crossing edges by rank: kept vertex, the two planes, in bytes
    uint32_t qxe[kQueue0 - 64];
    int qxk[kQueue0 - 64];
};
struct FinalMem {
    union {
        P64 pd[64];
        struct {
            double x[64], y[64], z[64];  // by vertex number, relative to vertex 0
        } v;
    };
    uint32_t rank[64];    // plane -> facet rank
    uint32_t number[64];  // slot -> vertex number
    uint32_t tri[64];     // facet ranks of a vertex, in bytes
    uint32_t size[64];    // vertices of a facet
    uint32_t anchor[64];  // its lowest vertex
    uint8_t next[256];    // 4 v + k -> the next vertex around facet k of v, with the facet's place there
    uint32_t fv[96];      // facet rings, two 16-bit vertex numbers a word
};
union WaveMem64 {
    ClipMem c;
    FinalMem f;
};

constexpr int kWaves64 = 4;  // waves per block

#pragma clang attribute push(__attribute__((always_inline)), apply_to = function)

// kW: the sites carry weights.  kMixed: signs FP32 cannot be sure of are
// looked for, and a cell that meets one goes on the retry list (it is marked,
// and k_retries lists the marked ones).
template <bool kW, bool kMixed>
struct Cell64 {
    WaveMem64& M;
    const ClipArgs& A;
    uint32_t ln;
    uint32_t serial;
    // site
    float px, py, pz, pw;
    uint32_t self;
    // the vertex of this lane: position, its squared length, its three planes
    // and the three vertices across its edges (bytes; edge k leaves plane k)
    float y0, y1, y2, r2;
    float ev;  // error scale of the vertex (checked signs only)
    uint32_t vt, va;
    uint64_t alive;
    int np;
    // AABB of the cell and the squares of its sides (uniform, in vector
    // registers), and the vertex at each side
    float blo0, blo1, blo2, bhi0, bhi1, bhi2;
    float hx2, hy2, hz2, lx2, ly2, lz2, rmax2;
    uint32_t ext[6];
    uint64_t ext_mask;
    // queue: entry q in lane q (keys as ordered integers, infinite in the
    // lanes past the end), from 64 on in LDS
    uint32_t qe;
    int qk;
    int qn;
    // where an overflow struck
    uint32_t ov_leaf, ov_phase;
    uint64_t ov_mask;
    bool ov_ok;
    bool deep;  // the path to the root has more than 64 siblings

    __device__ Cell64(WaveMem64& m, const ClipArgs& a) : M(m), A(a), ln(lane_id()) {}
    // Ends the reach of what the compiler derives from the lane number: the
    // addresses of one phase are not kept in registers through the others.
    __device__ void new_phase() { asm volatile("" : "+v"(ln)); }
    __device__ void clear_tab() { M.c.tab[ln] = make_uint2(0u, 0u); }
    __device__ float pwv() const { if constexpr (kW) return pw; else return 0.f; }
    // queue keys order as integers; without weights they are never negative
    __device__ static int key_bits(float k) { if constexpr (kW) return ford(k); else return __float_as_int(k); }
    __device__ static float key_value(int k) { if constexpr (kW) return unford(k); else return __int_as_float(k); }
    __device__ void sync() { wave_sync<true>(); }

    // ------------------------------------------------------------ setup
    __device__ bool init(uint32_t k) {
        new_phase();
        self = k;
        const float4 s = A.pts[k];
        px = s.x; py = s.y; pz = s.z; pw = s.w;
        if (pw == -INFINITY) return false;  // coincident with a heavier site
        clear_tab();  // finishing the cell before used its memory
        serial = 0;
        const float lo0 = A.bbox[0] - px, lo1 = A.bbox[1] - py, lo2 = A.bbox[2] - pz;
        const float hi0 = A.bbox[3] - px, hi1 = A.bbox[4] - py, hi2 = A.bbox[5] - pz;
        if (ln < 6) {
            const uint32_t ax = ln >> 1;
            const bool side = (ln & 1) != 0;
            const float sg = side ? 1.f : -1.f;
            const float lo = ax == 0 ? lo0 : (ax == 1 ? lo1 : lo2), hi = ax == 0 ? hi0 : (ax == 1 ? hi1 : hi2);
            M.c.pl[ln] = make_float4(ax == 0 ? sg : 0.f, ax == 1 ? sg : 0.f, ax == 2 ? sg : 0.f, side ? hi : -lo);
            M.c.pcode[ln] = -(int)(ln + 1);
            if constexpr (kMixed) M.c.psb[ln] = fabsf(side ? hi : -lo);
        }
        alive = 0xFFull;
        {
            const uint32_t c = ln & 7;
            const uint32_t sx = c & 1, sy = (c >> 1) & 1, sz = (c >> 2) & 1;
            const uint32_t X = sx, Y = 2 + sy, Z = 4 + sz;
            const bool pos = ((sx ^ sy ^ sz) & 1) == 1;  // product of the three normal signs > 0
            const uint32_t p1 = pos ? Y : Z, p2 = pos ? Z : Y;
            vt = X | (p1 << 8) | (p2 << 16);
            va = (c ^ 1u) | ((c ^ (1u << (p1 >> 1))) << 8) | ((c ^ (1u << (p2 >> 1))) << 16);
            y0 = sx ? hi0 : lo0;
            y1 = sy ? hi1 : lo1;
            y2 = sz ? hi2 : lo2;
            r2 = fmaf(y0, y0, fmaf(y1, y1, y2 * y2));
            if constexpr (kMixed) ev = fabsf(y0) + fabsf(y1) + fabsf(y2);
        }
        np = 6;
        qn = 0;
        qk = kInfBits;
        qe = 0;
        // the box: its sides are those of the AABB, vertex 0 at the three
        // lower ones and 7 at the upper ones
        blo0 = lo0; blo1 = lo1; blo2 = lo2;
        bhi0 = hi0; bhi1 = hi1; bhi2 = hi2;
        ext[0] = 0; ext[1] = 0; ext[2] = 0;
        ext[3] = 1; ext[4] = 2; ext[5] = 4;
        derive_bounds();
        sync();
        new_phase();
        return true;
    }

    __device__ void derive_bounds() {
        in_vgpr(blo0); in_vgpr(blo1); in_vgpr(blo2);
        in_vgpr(bhi0); in_vgpr(bhi1); in_vgpr(bhi2);
        hx2 = bhi0 * bhi0; hy2 = bhi1 * bhi1; hz2 = bhi2 * bhi2;
        lx2 = blo0 * blo0; ly2 = blo1 * blo1; lz2 = blo2 * blo2;
        rmax2 = fmaxf(hx2, lx2) + fmaxf(hy2, ly2) + fmaxf(hz2, lz2);
        ext_mask = 0;
#pragma unroll
        for (int k = 0; k < 6; ++k) ext_mask |= 1ull << ext[k];
    }
    // A clip removes some vertices and adds new ones on edges it cuts, inside
    // the old cell: only the sides whose vertex it removed are reduced again.
    __device__ void bounds_after_clip(uint64_t cut_mask) {
        const bool al = in_mask(alive);
        auto low = [&](int k, float y, float& b) {
            if (!((cut_mask >> ext[k]) & 1ull)) return;
            b = unford(imin_wave(al ? ford(y) : kInfBits));
            ext[k] = (uint32_t)lowest(ballot(y == b) & alive);
        };
        auto high = [&](int k, float y, float& b) {
            if (!((cut_mask >> ext[k]) & 1ull)) return;
            b = unford(wave_reduce_i(al ? ford(y) : ford(-INFINITY), [](int p, int q) { return max(p, q); }));
            ext[k] = (uint32_t)lowest(ballot(y == b) & alive);
        };
        low(0, y0, blo0);
        low(1, y1, blo1);
        low(2, y2, blo2);
        high(3, y0, bhi0);
        high(4, y1, bhi1);
        high(5, y2, bhi2);
        derive_bounds();
    }

    // ------------------------------------------------------------ ball tests
    // Some vertex v might be cut by a site of the box: dist(v, box)^2 - wmax
    // < |v|^2 - w_i, with a margin for rounding.
    __device__ bool ball(float lx, float ly, float lz, float hx, float hy, float hz, float wm) const {
        const float dx = fmaxf(fmaxf(lx - y0, y0 - hx), 0.f);
        const float dy = fmaxf(fmaxf(ly - y1, y1 - hy), 0.f);
        const float dz = fmaxf(fmaxf(lz - y2, y2 - hz), 0.f);
        const float d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
        return ball_test<kW>(d2, r2, wm, pwv());
    }
    // of the box held by lane l
    __device__ bool ball_lane(const NodeChild& c, int l) const {
        const float lx = rdl(c.lo[0] - px, l), ly = rdl(c.lo[1] - py, l), lz = rdl(c.lo[2] - pz, l);
        const float hx = rdl(c.hi[0] - px, l), hy = rdl(c.hi[1] - py, l), hz = rdl(c.hi[2] - pz, l);
        const float wm = kW ? rdl(c.wmax, l) : 0.f;
        return (ballot(ball(lx, ly, lz, hx, hy, hz, wm)) & alive) != 0;
    }
    // of a box that every lane holds
    __device__ bool ball_all(const NodeChild& c) const {
        return (ballot(ball(c.lo[0] - px, c.lo[1] - py, c.lo[2] - pz, c.hi[0] - px, c.hi[1] - py, c.hi[2] - pz,
                            kW ? c.wmax : 0.f)) & alive) != 0;
    }

    // ------------------------------------------------------------ clip
    // The vertices of R (some, not all) are cut off by the plane held by lane
    // L of the current leaf: each edge from a kept to a removed vertex gets a
    // new vertex, and the new vertices find their neighbours around the new
    // facet through the table of their old planes.
    // cross() finds the edges, cut() does the work (returns false if the links
    // are not one cycle: the cell is then built again from the start).
    struct Cross {
        uint64_t kept, f;     // vertices kept, free places
        uint64_t m0, m1, m2;  // vertices whose first, second, third edge is crossed
        uint32_t m;           // crossing edges
    };
    __device__ Cross cross(uint64_t R) const {
        Cross c;
        c.kept = alive & ~R;
        c.f = ~alive | R;
        c.m0 = ballot(((R >> byte_of(va, 0)) & 1ull) != 0) & c.kept;
        c.m1 = ballot(((R >> byte_of(va, 1)) & 1ull) != 0) & c.kept;
        c.m2 = ballot(((R >> byte_of(va, 2)) & 1ull) != 0) & c.kept;
        c.m = (uint32_t)(popc(c.m0) + popc(c.m1) + popc(c.m2));
        return c;
    }
    __device__ bool cut(const Cross& c, int L, float cax, float cay, float caz, float cb, float csb, float ax, float ay,
                        float az, float b, float sbh, int32_t hcode) {
        const uint64_t kept = c.kept, f = c.f, m0 = c.m0, m1 = c.m1, m2 = c.m2;
        const uint32_t m = c.m;
        // crossing edges ranked by vertex, then edge; the new vertex of rank k
        // takes the free slot of rank k
        auto count_below = [](uint64_t q, uint32_t base) {
            return __builtin_amdgcn_mbcnt_hi((uint32_t)(q >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)q, base));
        };
        const uint32_t j0 = count_below(m2, count_below(m1, count_below(m0, 0u)));
        const uint32_t j1 = j0 + (in_mask(m0) ? 1u : 0u), j2 = j1 + (in_mask(m1) ? 1u : 0u);
        const uint32_t fr = count_below(f, 0u);
        const uint64_t nw = ballot(fr < m) & f;
        if (++serial >= (1u << 20)) {  // tags exhausted
            clear_tab();
            serial = 1;
        }
        const uint32_t tag = serial << 12, me = tag | ln;
        // records (vertex, t[(e+2)%3], t[(e+1)%3]): permute selectors 0 = lane
        // number, 4..6 = bytes of vt, 0x0C = zero
        if (in_mask(m0)) M.c.edge[j0] = __builtin_amdgcn_perm(vt, ln, 0x0C050600u);
        if (in_mask(m1)) M.c.edge[j1] = __builtin_amdgcn_perm(vt, ln, 0x0C060400u);
        if (in_mask(m2)) M.c.edge[j2] = __builtin_amdgcn_perm(vt, ln, 0x0C040500u);
        sync();
        // values of the lanes of nw, any in the others
        uint32_t rec = __builtin_nondeterministic_value(ln), x = __builtin_nondeterministic_value(ln),
                 y = __builtin_nondeterministic_value(ln), n1 = __builtin_nondeterministic_value(ln),
                 n2 = __builtin_nondeterministic_value(ln), own1 = __builtin_nondeterministic_value(ln),
                 own2 = __builtin_nondeterministic_value(ln);
        if (in_mask(nw)) {
            rec = M.c.edge[fr];
            x = byte_of(rec, 1);
            y = byte_of(rec, 2);
            M.c.tab[x].x = me;
            M.c.tab[y].y = me;
            M.c.sor[fr] = ln;
            sync();
            const uint2 u = M.c.tab[x], w = M.c.tab[y];
            own1 = u.x;
            own2 = w.y;
            n1 = w.x ^ tag;  // the vertex itself where the tag is this clip's
            n2 = u.y ^ tag;
        }
        // The links next (n1) and previous (n2) are inverse permutations
        // without fixed points where every entry is as written, and have to be
        // one cycle: up to five vertices they are unless two of them point at
        // each other (no cycle for six or more either).
        const uint64_t bad = (ballot(own1 != me) | ballot(own2 != me) | ballot(max(n1, n2) > 63u) |
                              (m >= 4u ? ballot(n1 == n2) : 0ull)) & nw;
        bool whole = bad == 0;
        if (m >= 6u) {  // follow the links
            const uint32_t start = (uint32_t)lowest(nw);
            uint32_t v = start, steps = 0;
            do {
                v = rdl(n1, (int)v & 63);
                ++steps;
            } while (v != start && steps <= m);
            whole = whole && steps == m;
        }
        // (a cell whose links are wrong is built again from the start: what
        // follows does no harm to it and needs no branch)
        // kept vertices point at their new neighbours
        {
            const uint32_t s0 = M.c.sor[j0], s1 = M.c.sor[j1], s2 = M.c.sor[j2];
            const uint32_t a0 = __builtin_amdgcn_perm(va, s0, 0x0C060500u);
            va = in_mask(m0) ? a0 : va;
            const uint32_t a1 = __builtin_amdgcn_perm(va, s1, 0x0C060004u);
            va = in_mask(m1) ? a1 : va;
            const uint32_t a2 = __builtin_amdgcn_perm(va, s2, 0x0C000504u);
            va = in_mask(m2) ? a2 : va;
        }
        // new vertices: planes (h, x, y), position by Cramer's rule
        const uint32_t h = (uint32_t)np;
        if (in_mask(nw)) {
            vt = (rec & 0xFFFF00u) | h;
            va = (rec & 0xFFu) | (n1 << 8) | (n2 << 16);
            const float4 P = M.c.pl[x], Q = M.c.pl[y];
            const Solve32 s(P, Q, ax, ay, az, b);
            y0 = s.y0;
            y1 = s.y1;
            y2 = s.y2;
            r2 = fmaf(y0, y0, fmaf(y1, y1, y2 * y2));
            if constexpr (kMixed) ev = s.scale(sbh, M.c.psb[x], M.c.psb[y]);
        }
        alive = kept | nw;
        if ((int)ln == L) {
            M.c.pl[h] = make_float4(cax, cay, caz, cb);
            M.c.pcode[h] = hcode;
            if constexpr (kMixed) M.c.psb[h] = csb;
        }
        np = (int)h + 1;
        sync();
        return whole;
    }

    // Drops planes no vertex uses (supplementary Sec. A, "Garbage
    // collection"): marks in the link table, which is cleared afterwards.
    __device__ void gc() {
        M.c.tab[ln] = make_uint2(0u, 0u);
        sync();
        if (in_mask(alive)) {
            M.c.tab[byte_of(vt, 0)].x = 1u;
            M.c.tab[byte_of(vt, 1)].x = 1u;
            M.c.tab[byte_of(vt, 2)].x = 1u;
        }
        sync();
        const uint64_t u = ballot((int)ln < np && M.c.tab[ln].x != 0u);
        const uint32_t dst = mbcnt(u);
        const float4 p = M.c.pl[ln];
        const int32_t c = M.c.pcode[ln];
        const float sb = kMixed ? M.c.psb[ln] : 0.f;
        sync();
        if (in_mask(u)) {
            M.c.pl[dst] = p;
            M.c.pcode[dst] = c;
            if constexpr (kMixed) M.c.psb[dst] = sb;
            M.c.tab[ln].x = dst;
        }
        sync();
        if (in_mask(alive))
            vt = M.c.tab[byte_of(vt, 0)].x | (M.c.tab[byte_of(vt, 1)].x << 8) | (M.c.tab[byte_of(vt, 2)].x << 16);
        np = popc(u);
        sync();
        M.c.tab[ln] = make_uint2(0u, 0u);
        sync();
    }

    // ------------------------------------------------------------ traversal
    // Tests one child record against the current cell (Sec. 4.2.2).
    __device__ void node_test(const NodeChild& c, float* key, bool* cull, float* delta) const {
        float blx = c.lo[0] - px, bly = c.lo[1] - py, blz = c.lo[2] - pz;
        float bhx = c.hi[0] - px, bhy = c.hi[1] - py, bhz = c.hi[2] - pz;
        float dx = fmaxf(fmaxf(blx, -bhx), 0.f), dy = fmaxf(fmaxf(bly, -bhy), 0.f), dz = fmaxf(fmaxf(blz, -bhz), 0.f);
        // hardware square roots (1 ulp), inside the bound's rounding margin
        float d = __builtin_amdgcn_sqrtf(fmaf(dx, dx, fmaf(dy, dy, dz * dz)));
        float dw = kW ? pw - c.wmax : 0.f;
        const float lbs = least_plane(d, dw, true, [&] {
            const float fx = pmax(fabsf(blx), fabsf(bhx)), fy = pmax(fabsf(bly), fabsf(bhy)),
                        fz = pmax(fabsf(blz), fabsf(bhz));
            return __builtin_amdgcn_sqrtf(fmaf(fx, fx, fmaf(fy, fy, fz * fz)));
        });
        // per axis: the far-corner square of each side the box reaches
        // (both sides: the larger one)
        const float tx = pmax(bhx >= 0.f ? hx2 : 0.f, blx < 0.f ? lx2 : 0.f);
        const float ty = pmax(bhy >= 0.f ? hy2 : 0.f, bly < 0.f ? ly2 : 0.f);
        const float tz = pmax(bhz >= 0.f ? hz2 : 0.f, blz < 0.f ? lz2 : 0.f);
        float rb = __builtin_amdgcn_sqrtf(tx + ty + tz);
        *key = lbs;
        *cull = lbs > rb * (1.f + 16.f * kU);
        *delta = lbs - rb;
    }

    __device__ void push(uint32_t e, int k) {
        if (qn < 64) {
            qe = wrl(e, qn, qe);
            qk = wrl(k, qn, qk);
        }
        if (qn >= 64) {
            if (ln == 0) {
                M.c.qxe[qn - 64] = e;
                M.c.qxk[qn - 64] = k;
            }
            sync();
        }
        ++qn;
    }

    // Removes and returns the entry of least key (the last one takes its place).
    __device__ void pop(uint32_t* e, int* k) {
        int bk = qk;
        int bs = 0;
        if (qn > 64) {
            for (int s = 1; s * 64 < qn; ++s) {
                const int idx = s * 64 + (int)ln;
                const int kk = M.c.qxk[idx - 64];
                const bool less = idx < qn && kk < bk;
                bk = less ? kk : bk;
                bs = less ? s : bs;
            }
        }
        const int m = imin_wave(bk);
        uint64_t msk = ballot(bk == m);
        msk &= qn < 64 ? (1ull << qn) - 1ull : ~0ull;
        const int L = msk ? lowest(msk) : 0;
        *k = m;
        // the last entry goes to lane L, its own lane is marked free; entries
        // in LDS: lane L is rewritten (with what it holds when the popped one
        // is in LDS itself)
        int last = qn - 1;
        *e = rdl(qe, L);
        uint32_t le = rdl(qe, last & 63);
        int lk = rdl(qk, last & 63), freed = kInfBits;
        if (qn > 64) {
            const int S = rdl(bs, L);
            le = uni(M.c.qxe[last - 64]);
            lk = (int)uni((uint32_t)M.c.qxk[last - 64]);
            if (S != 0) {
                const uint32_t ee = uni(M.c.qxe[(S - 1) * 64 + L]);
                if (ln == 0) {
                    M.c.qxe[(S - 1) * 64 + L] = le;
                    M.c.qxk[(S - 1) * 64 + L] = lk;
                }
                sync();
                le = *e;
                lk = rdl(qk, L);
                *e = ee;
            }
            last = L;
            freed = lk;
        }
        qe = wrl(le, L, qe);
        qk = wrl(lk, L, qk);
        qk = wrl(freed, last, qk);
        --qn;
    }

    // Clips by the sites of one leaf, nearest plane first.
    __device__ int leaf(uint32_t ref, uint32_t phase) {
        const uint32_t first = leaf_first(ref), nsite = leaf_count(ref);
        const uint32_t j = first + min(ln, nsite - 1u);
        const float4 q = A.pts[j];
        const float ax = q.x - px, ay = q.y - py, az = q.z - pz;
        const float a2 = fmaf(ax, ax, fmaf(ay, ay, az * az));
        const float dw = kW ? pw - q.w : 0.f;
        const float b = 0.5f * (a2 + dw);
        const uint64_t cand = ballot(ln < nsite) & ballot(j != self) & ballot(q.w != -INFINITY) & ballot(a2 > 0.f);
        const int key = key_bits(b * __builtin_amdgcn_rsqf(a2));  // orders candidates only
        // the plane misses the cell's AABB: max over the box of a.y <= b (with
        // the very slack of the general pass: a vertex may lie outside the box
        // by its rounding, so a candidate more or less could be a clip more)
        const uint64_t sx = ballot(ax >= 0.f), sy = ballot(ay >= 0.f), sz = ballot(az >= 0.f);
        auto keep = [&]() -> bool {
            const float cx = pick(in_mask(sx), bhi0, blo0), cy = pick(in_mask(sy), bhi1, blo1),
                        cz = pick(in_mask(sz), bhi2, blo2);
            return reaches(ax, ay, az, b, cx, cy, cz, a2, dw);
        };
        // for the doubtful-sign test
        const float sbl = 0.5f * (a2 + fabsf(dw)), an1 = fabsf(ax) + fabsf(ay) + fabsf(az);
        uint64_t mask = ballot(keep()) & cand;
        // Nearest plane first, equal ones by lane: each candidate counts those
        // before it (3 vector operations a candidate), and the next one is
        // found by one comparison (the least key left by a reduction over the
        // wave took 12 for each).
        uint32_t rank = 0;
        if (mask & (mask - 1ull))
            for (uint64_t u = mask; u;) {
                const int l = lowest(u);
                u = without(u, l);
                rank += rdl(key, l) < key ? 1u : 0u;
            }
        uint64_t next = 0;  // candidates of the least rank left
        // How the last clip went.  Nothing leaves the loop but the end of its
        // candidates, and no condition in it has two sides: around divergent
        // code every such way is compiled to copies of the whole cell.
        bool room = true, whole = true, gone = false;
        uint32_t edges = 0;
        uint64_t left = 0;  // the candidates not done
        for (uint32_t at = 0; mask;) {
            next &= mask;
            for (; next == 0; ++at) next = ballot(rank == at) & mask;
            const int L = lowest(next);
            mask = without(mask, L);
            const float hx = rdl(ax, L), hy = rdl(ay, L), hz = rdl(az, L), hb = rdl(b, L);
            const float sv = fmaf(hx, y0, fmaf(hy, y1, fmaf(hz, y2, -hb)));
            uint64_t R = ballot(sv > 0.f) & alive;
            float sbh = 0.f;
            if constexpr (kMixed) {
                sbh = rdl(sbl, L);
                const float beta = doubt(rdl(an1, L), ev, sbh);
                whole = (ballot(fabsf(sv) <= beta) & alive) == 0;
                mask = whole ? mask : 0ull;
                R = whole ? R : 0ull;
            }
            if (R != 0) {
                if (np >= 64) gc();
                const Cross c = cross(R);
                // no edge crosses the plane, no place for the vertices or the plane
                room = c.m - 1u < (uint32_t)popc(c.f) && np < 64;
                left = mask | (1ull << L);
                edges = c.m;
                gone = R == alive;
                mask = room ? mask : 0ull;
                if (room) {
                    whole = cut(c, L, ax, ay, az, b, sbl, hx, hy, hz, hb, sbh, (int32_t)j);
                    if ((R & ext_mask) != 0) {
                        bounds_after_clip(R);
                        mask &= ballot(keep());
                    }
                    mask = whole ? mask : 0ull;
                }
            }
        }
        if (!whole) return kRestart;
        if (room) return kNone;
        if (gone) return kEmptied;
        if (edges == 0 && np < 64) return kRestart;  // vertices cut off, but no edge crosses the plane
        ov_ok = true;  // the cell is as before this candidate
        ov_leaf = ref;
        ov_mask = left;
        ov_phase = phase;
        return kOverflow;
    }

    __device__ void load_child(uint32_t node, int s, NodeChild* c) const {
        const float4* src = reinterpret_cast<const float4*>(&A.nodes[node].c[s]);
        const float4 u = src[0], v = src[1];
        c->lo[0] = u.x; c->lo[1] = u.y; c->lo[2] = u.z; c->wmax = u.w;
        c->hi[0] = v.x; c->hi[1] = v.y; c->hi[2] = v.z; c->ref = __float_as_uint(v.w);
    }

    // Alg. 1 with the site's own leaf first (see vd_clip.hip): own leaf, the
    // siblings of its path, then the queue.  Returns kNone when done,
    // kEmptied, kOverflow or kRestart.
    __device__ int traverse() {
        ov_ok = false;
        deep = false;
        uint32_t cur = A.root;
        uint32_t path = 0;  // this lane's sibling record: (node << 1) | which child
        int ns = 0;         // siblings of the path, to be tested after the first leaf
        if (A.leaf_of != nullptr) {
            KArgs* ka = cold_args();
            const uint32_t rec = uni(ka->leaf_of[self]);
            cur = uni(A.nodes[rec >> 1].c[rec & 1].ref);
            path = rec ^ 1u;
            ns = 1;
            for (uint32_t c = rec;;) {
                const uint32_t u = uni(ka->up[c >> 1]);
                if (u == kNoParent) break;
                if (ns == 64) {  // left to the general pass
                    deep = true;
                    return kRestart;
                }
                path = wrl(u ^ 1u, ns, path);
                ++ns;
                c = u;
            }
            if ((int)ln >= ns) path = rdl(path, 0);  // lanes past the path repeat the first sibling
        }
        // every node is visited at most once in a valid tree; the bound only
        // guarantees termination if the tree were ever malformed
        int budget = (int)(4 * A.n + 1024);
        // (one way out of each loop and conditions of one side, as in leaf())
        int res = kNone;
        bool more = true;  // something may still cut the cell
        for (uint32_t phase = 0; more; phase = 1) {
            res = leaf(cur, ns > 0 ? phase : 1u);
            more = res == kNone && ns > 0;  // without siblings the root is a leaf
            NodeChild c;
            float key, delta;
            bool cull;
            if (more && phase == 0) {
                // the siblings of the path, nearest last
                load_child(path >> 1, (int)(path & 1), &c);
                node_test(c, &key, &cull, &delta);
                const int kb = key_bits(fminf(key, INFINITY));
                uint64_t live = ballot(!cull) & ballot((int)ln < ns);
                while (live) {
                    const int L = 63 - __builtin_clzll(live);
                    live = without(live, L);
                    if (ball_lane(c, L)) {
                        more = qn < kQueue0;
                        live = more ? live : 0ull;
                        if (more) push(rdl(path, L), rdl(kb, L));
                    }
                }
                res = more ? (int)kNone : (int)kOverflow;
            }
            // the next leaf: pop, then descend into the nearer children
            bool seek = more;
            while (seek) {
                more = qn != 0;
                seek = false;
                if (more) {
                    uint32_t e;
                    int k;
                    pop(&e, &k);
                    // every key left is at least this one: beyond the cell's radius nothing can cut it
                    more = ballot(key_value(k) > __builtin_amdgcn_sqrtf(rmax2) * (1.f + 16.f * kU)) == 0;
                    if (more) {
                        load_child(e >> 1, (int)(e & 1), &c);
                        node_test(c, &key, &cull, &delta);
                        bool hit = ballot(cull) == 0;
                        if (hit) hit = ball_all(c);
                        cur = uni(c.ref);
                        bool down = hit && !ref_is_leaf(cur);
                        while (down) {
                            const uint32_t node = cur;
                            load_child(node, (int)(ln & 1), &c);
                            node_test(c, &key, &cull, &delta);
                            const uint64_t cm = ballot(cull);
                            const float blx = c.lo[0] - px, bly = c.lo[1] - py, blz = c.lo[2] - pz;
                            const float bhx = c.hi[0] - px, bhy = c.hi[1] - py, bhz = c.hi[2] - pz;
                            uint64_t h0 = 0, h1 = 0;
                            if (!(cm & 1ull))
                                h0 = ballot(ball(of_even(blx), of_even(bly), of_even(blz), of_even(bhx), of_even(bhy),
                                                 of_even(bhz), kW ? of_even(c.wmax) : 0.f)) & alive;
                            if (!(cm & 2ull))
                                h1 = ballot(ball(of_odd(blx), of_odd(bly), of_odd(blz), of_odd(bhx), of_odd(bhy),
                                                 of_odd(bhz), kW ? of_odd(c.wmax) : 0.f)) & alive;
                            hit = (h0 | h1) != 0;
                            if (hit) {
                                const uint64_t closer = ballot(rdl(delta, 0) <= rdl(delta, 1));  // child 0
                                const uint64_t first = h0 == 0 ? 0ull : (h1 == 0 ? 1ull : closer);
                                const int near = first != 0 ? 0 : 1;
                                if (h0 != 0 && h1 != 0) {
                                    more = qn < kQueue0;
                                    if (more) push((node << 1) | (uint32_t)(1 - near), rdl(key_bits(fminf(key, INFINITY)), 1 - near));
                                }
                                cur = rdl(c.ref, near);
                            }
                            --budget;
                            more &= budget >= 0;
                            down = hit && more && !ref_is_leaf(cur);
                        }
                        --budget;
                        more &= budget >= 0;
                        res = more ? (int)kNone : (int)kOverflow;
                        seek = more && !hit;
                    }
                }
            }
        }
        return res;
    }

    // ------------------------------------------------------------ hand-over
    // Writes the state of a cell that overflowed, in the layout of the general
    // passes (indices of ten bits, float keys); only the header when the
    // overflow is not resumable.
    __device__ void save(HandoffT<64, kQueue0>& H) {
        auto wide = [](uint32_t w) { return byte_of(w, 0) | (byte_of(w, 1) << 10) | (byte_of(w, 2) << 20); };
        sync();
        if (ov_ok) {
            if ((int)ln < np) {
                const int32_t c = M.c.pcode[ln];
                const float4 p = M.c.pl[ln];
                const float4 site = c >= 0 ? A.pts[c] : make_float4(0.f, 0.f, 0.f, 0.f);
                H.pl[ln] = p;
                H.psite[ln] = site;
                // size of the terms of b (read by builds with checked signs only)
                const float a2 = fmaf(p.x, p.x, fmaf(p.y, p.y, p.z * p.z));
                H.psb[ln] = kMixed ? M.c.psb[ln] : c >= 0 ? 0.5f * (a2 + (kW ? fabsf(pw - site.w) : 0.f)) : fabsf(p.w);
                H.pcode[ln] = c;
            }
            H.y0[ln] = y0;
            H.y1[ln] = y1;
            H.y2[ln] = y2;
            H.ev[ln] = kMixed ? ev : 0.f;  // read by builds with checked signs only
            H.vt[ln] = wide(vt);
            H.va[ln] = wide(va);
            H.qe[ln] = qe;
            H.qk[ln] = key_value(qk);
            for (int q = 64 + (int)ln; q < qn; q += 64) {
                H.qe[q] = M.c.qxe[q - 64];
                H.qk[q] = key_value(M.c.qxk[q - 64]);
            }
            if (ln == 0) H.alive[0] = alive;
        }
        if (ln < (uint32_t)kMaxWarm) H.wsite[ln] = 0u;
        if (ln == 0) {
            H.nwarm = 0u;
            H.np = (uint32_t)np;
            H.vhi = 64u;
            H.qn = (uint32_t)qn;
            H.flags = 0u;
            H.robust = kMixed ? 1u : 0u;
            H.leaf = ov_leaf;
            H.mask = ov_mask;
            H.phase = ov_phase;
            H.skip = kNoParent;
            H.valid = ov_ok ? 1u : 0u;
        }
    }

    // ------------------------------------------------------------ output
    // Writes the cell's record: facets ordered by output code, vertices
    // renumbered in slot order and evaluated in FP64 from the input
    // coordinates.  Returns false if the structure is not a closed simple
    // polytope.
    __device__ bool finalize(uint32_t slot, uint32_t orig) {
        new_phase();
        const bool al = in_mask(alive);
        // planes in use
        M.c.tab[ln] = make_uint2(0u, 0u);
        sync();
        if (al) {
            M.c.tab[byte_of(vt, 0)].x = 1u;
            M.c.tab[byte_of(vt, 1)].x = 1u;
            M.c.tab[byte_of(vt, 2)].x = 1u;
        }
        sync();
        const uint64_t used = ballot((int)ln < np && M.c.tab[ln].x != 0u);
        const int32_t code = M.c.pcode[ln];
        sync();  // the clip tables end here
        const int F = popc(used);
        const int nv = popc(alive);
        KArgs* ka = cold_args();
        int32_t out = 0;
        if (in_mask(used)) out = code >= 0 ? (int32_t)ka->order[code] : code;
        // FP64 planes from the input coordinates
        const double qx = px, qy = py, qz = pz;
        if (in_mask(used)) {
            P64 d;
            if (code < 0) {
                const int ax = (-code - 1) >> 1;
                const bool side = ((-code - 1) & 1) != 0;
                const double sg = side ? 1.0 : -1.0;
                const double p = ax == 0 ? qx : (ax == 1 ? qy : qz);
                d.a0 = ax == 0 ? sg : 0.0;
                d.a1 = ax == 1 ? sg : 0.0;
                d.a2 = ax == 2 ? sg : 0.0;
                d.b = side ? ((double)A.bbox[3 + ax] - p) : (p - (double)A.bbox[ax]);
            } else {
                const float4 site = A.pts[code];
                d.a0 = (double)site.x - qx;
                d.a1 = (double)site.y - qy;
                d.a2 = (double)site.z - qz;
                d.b = 0.5 * (d.a0 * d.a0 + d.a1 * d.a1 + d.a2 * d.a2 + ((double)pw - (double)site.w));
            }
            M.f.pd[ln] = d;
        }
        // facet ranks: ascending output code (box faces, then sites)
        uint32_t rank = 0;
        for (uint64_t u = used; u;) {
            const int l = lowest(u);
            u = without(u, l);
            rank += rdl(out, l) < out ? 1u : 0u;
        }
        const int64_t base = (int64_t)slot * 64;
        if (in_mask(used)) ka->stage.code[base + rank] = out;
        M.f.rank[ln] = rank;
        const uint32_t v = mbcnt(alive);
        M.f.number[ln] = v;
        M.f.size[ln] = 0u;
        M.f.anchor[ln] = 0xFFFFFFFFu;
        sync();
        // every neighbour has to be a live vertex
        {
            const bool dead = ((alive >> byte_of(va, 0)) & (alive >> byte_of(va, 1)) & (alive >> byte_of(va, 2)) & 1ull) == 0;
            if (ballot(dead) & alive) return false;
        }
        double Y0 = 0.0, Y1 = 0.0, Y2 = 0.0;
        if (al) {
            const P64 P = M.f.pd[byte_of(vt, 0)], Q = M.f.pd[byte_of(vt, 1)], S = M.f.pd[byte_of(vt, 2)];
            const Meet64 y(P, Q, S);
            if (y.det != 0.0) {
                double n[3];
                y.numerator(P, Q, S, n);
                const double inv = 1.0 / y.det;
                Y0 = n[0] * inv;
                Y1 = n[1] * inv;
                Y2 = n[2] * inv;
            } else {
                Y0 = y0;
                Y1 = y1;
                Y2 = y2;
            }
        }
        sync();  // the FP64 planes are read; positions take their place
        new_phase();
        float sx = px, sy = py, sz0 = pz;
        in_vgpr(sx);
        in_vgpr(sy);
        in_vgpr(sz0);
        const int l0 = lowest(alive);
        // reference point of the tetrahedral fan: vertex 0
        const double R0 = rdl64(Y0, l0), R1 = rdl64(Y1, l0), R2 = rdl64(Y2, l0);
        const double X0 = Y0 - R0, X1 = Y1 - R1, X2 = Y2 - R2;
        uint32_t tri = 0, adj = 0;  // facet ranks and neighbour numbers, in bytes
        if (al) {
            tri = M.f.rank[byte_of(vt, 0)] | (M.f.rank[byte_of(vt, 1)] << 8) | (M.f.rank[byte_of(vt, 2)] << 16);
            adj = M.f.number[byte_of(va, 0)] | (M.f.number[byte_of(va, 1)] << 8) | (M.f.number[byte_of(va, 2)] << 16);
            M.f.v.x[v] = X0;
            M.f.v.y[v] = X1;
            M.f.v.z[v] = X2;
            M.f.tri[v] = tri;
            const uint32_t t0 = byte_of(tri, 0), t1 = byte_of(tri, 1), t2 = byte_of(tri, 2);
            const uint32_t u0 = min(t0, min(t1, t2)), u2 = max(t0, max(t1, t2)), u1 = t0 + t1 + t2 - u0 - u2;
            ka->stage.vert[base + v] = make_float4((float)((double)sx + Y0), (float)((double)sy + Y1), (float)((double)sz0 + Y2),
                                                   __uint_as_float(u0 | (u1 << 10) | (u2 << 20)));
            atomicAdd(&M.f.size[t0], 1u);
            atomicAdd(&M.f.size[t1], 1u);
            atomicAdd(&M.f.size[t2], 1u);
            atomicMin(&M.f.anchor[t0], v);
            atomicMin(&M.f.anchor[t1], v);
            atomicMin(&M.f.anchor[t2], v);
        }
        sync();
        // links of the facet rings, counter-clockwise seen from outside: from
        // vertex v around its facet k to vertex adj[(k+1)%3], with the place of
        // that facet there
        if (al) {
            auto link = [&](uint32_t w, uint32_t f) -> uint32_t {
                const uint32_t tw = M.f.tri[w];
                return 4u * w + (byte_of(tw, 0) == f ? 0u : (byte_of(tw, 1) == f ? 1u : 2u));
            };
            reinterpret_cast<uint32_t*>(M.f.next)[v] =
                link(byte_of(adj, 1), byte_of(tri, 0)) | (link(byte_of(adj, 2), byte_of(tri, 1)) << 8) |
                (link(byte_of(adj, 0), byte_of(tri, 2)) << 16);
        }
        sync();
        bool bad = false;
        {
            const uint32_t sz = M.f.size[ln], start = M.f.anchor[ln];
            uint32_t at = wscan_u(sz) - sz;
            if ((int)ln < F) {
                ka->stage.fsize[base + ln] = (uint16_t)sz;
                if (sz < 3u || start >= (uint32_t)nv) {
                    bad = true;
                } else {
                    const uint32_t ts = M.f.tri[start];
                    uint32_t he = 4u * start + (byte_of(ts, 0) == ln ? 0u : (byte_of(ts, 1) == ln ? 1u : 2u));
                    uint32_t left = sz;
                    uint16_t* ring = reinterpret_cast<uint16_t*>(M.f.fv);
                    do {
                        ring[at] = (uint16_t)(he >> 2);
                        ++at;
                        --left;
                        he = M.f.next[he];
                    } while ((he >> 2) != start && left != 0u);
                    bad = (he >> 2) != start || left != 0u;
                }
            }
        }
        if (ballot(bad)) return false;
        sync();
        // the rings (3 nv numbers) go out as whole words; the last one may
        // carry a number past the end, inside the slot
        {
            uint32_t* fv = reinterpret_cast<uint32_t*>(ka->stage.fv + base * 3);
            const int words = (3 * nv + 1) >> 1;
            if ((int)ln < words) fv[ln] = M.f.fv[ln];
            if ((int)ln + 64 < words) fv[ln + 64] = M.f.fv[ln + 64];
        }
        // volume and centroid from the tetrahedra (ref, anchor_f, v, next_f(v)),
        // in FP64 (thin cells cancel badly in FP32)
        Fan64 sum;
        if (al) {
            uint32_t f = tri, nx3 = adj >> 8 | (adj << 16);  // the facet and the next vertex around it in the low bytes
#pragma unroll 1
            for (int k = 0; k < 3; ++k, f >>= 8, nx3 >>= 8) {
                const uint32_t an = M.f.anchor[f & 0xFFu], nx = nx3 & 0xFFu;
                if (an == v || nx == an) continue;
                const double Qx = M.f.v.x[an], Qy = M.f.v.y[an], Qz = M.f.v.z[an];
                const double Nx = M.f.v.x[nx], Ny = M.f.v.y[nx], Nz = M.f.v.z[nx];
                sum.add(Qx, Qy, Qz, X0, X1, X2, Nx, Ny, Nz);
            }
        }
        if constexpr (kMixed) {
            // summed by vertex number, as the general pass does: which of the
            // two builds a cell must not show (see run_cells64)
            const int to = 4 * (int)(al ? v : (uint32_t)nv + mbcnt(~alive));
            auto turn = [&](double& x) {
                x = __hiloint2double(__builtin_amdgcn_ds_permute(to, __double2hiint(x)),
                                     __builtin_amdgcn_ds_permute(to, __double2loint(x)));
            };
            turn(sum.vol6);
            turn(sum.mx);
            turn(sum.my);
            turn(sum.mz);
        }
        const double vol6 = wsum64(sum.vol6), mx = wsum64(sum.mx), my = wsum64(sum.my), mz = wsum64(sum.mz);
        const uint32_t nbox = (uint32_t)popc(ballot(code < 0) & used);
        if (ln == 0) {
            ka->cnt_v[orig] = (uint32_t)nv;
            ka->cnt_f[orig] = (uint32_t)F;
            ka->cnt_n[orig] = (uint32_t)F - nbox;
            ka->vol[orig] = (float)(vol6 / 6.0);
            const double inv = vol6 != 0.0 ? 0.25 / vol6 : 0.0;
            ka->cen[3 * orig] = centroid_of(sx, R0, mx, inv);
            ka->cen[3 * orig + 1] = centroid_of(sy, R1, my, inv);
            ka->cen[3 * orig + 2] = centroid_of(sz0, R2, mz, inv);
            ka->flags[orig] = 0;
            ka->loc[self] = make_loc(0u, slot);
        }
        return true;
    }

    __device__ void write_empty(uint32_t orig) {
        if (ln == 0) {
            KArgs* ka = cold_args();
            ka->cnt_v[orig] = 0;
            ka->cnt_f[orig] = 0;
            ka->cnt_n[orig] = 0;
            ka->vol[orig] = 0.f;
            ka->cen[3 * orig] = px;
            ka->cen[3 * orig + 1] = py;
            ka->cen[3 * orig + 2] = pz;
            ka->flags[orig] = (uint8_t)kFlagEmpty;
            ka->loc[self] = make_loc(0u, 0u);
        }
    }
};

template <bool kW, bool kMixed>
__device__ void run_cells64(WaveMem64& M, const ClipArgs& A) {
    if (*cold_args()->err != 0u) return;  // rejected input
    Cell64<kW, kMixed> C(M, A);
    unsigned long long st_empty = 0;
    uint32_t missed = 0;  // cells in a row with a doubtful sign
    Work<kWaves64> work((uint32_t)A.n);
    for (;;) {
        const uint32_t k = work.next(uni((uint32_t)threadIdx.x >> 6));
        if (k == kNoCell) break;
        const uint32_t orig = cold_args()->order[k];
        int res = kEmptied;  // also a site that lost its position to a heavier one
        if (C.init(k)) {
            res = C.traverse();
            if (res == kNone && !C.finalize(k, orig)) res = kRestart;
        }
        if constexpr (kMixed) missed = res == kRestart ? missed : 0u;
        if (res == kEmptied) {
            C.write_empty(orig);
            ++st_empty;
        } else if (res == kRestart) {
            KArgs* kn = cold_args();
            if (C.ln == 0) {
                if constexpr (kMixed) kn->loc[k] = kLocRetry;  // listed by k_retries
                else kn->retry_list[atomicAdd(kn->retry_count, 1u)] = k | (C.deep ? 0u : kRetryChecked);
            }
            // Checked signs: after six such cells in a row the next 8 of the
            // wave's range go there untried, after one more the next 16, up to
            // 64 (a claim for each would cost 20 ns over the whole device).  A
            // set full of ties then costs the general pass and little else: a
            // lattice of 262k sites 5.3 ms with every cell tried, 4.8 so, 4.5
            // by the general pass alone; of 1M 20.3, 17.7 and 17.3.  Where one
            // cell in ten has a doubtful sign one in a million begins this.
            if constexpr (kMixed) {
                if (++missed >= 6u) {
                    uint32_t got = 0;
                    const uint32_t first = work.more(8u << min(missed - 6u, 3u), &got);
                    if (C.ln < got) kn->loc[first + C.ln] = kLocRetry;
                }
            }
        } else if (res == kOverflow) {
            KArgs* kn = cold_args();
            uint32_t pos = 0;
            if (C.ln == 0) {
                pos = atomicAdd(kn->next_count, 1u);
                kn->next_list[pos] = k;
                if constexpr (kMixed) kn->loc[k] = make_loc(1u, 0u);  // not kLocRetry, as it may stand there
            }
            pos = uni(pos);
            if (pos < kn->hand_out_cap) C.save(static_cast<HandoffT<64, kQueue0>*>(kn->hand_out)[pos]);
        }
    }
    if (C.ln == 0 && st_empty) atomicAdd(&cold_args()->stats[kStatEmpty], st_empty);
}

#pragma clang attribute pop

// 72 registers for 7 waves per SIMD: 21 values (22 with weights) go to scratch
// memory, none in a loop of a cell (60 bytes a lane and cell).  A build of
// clustered 1M sites, as first written: 20.7 ms at 4 waves, 18.8 at 5, 17.8 at
// 6, 17.2 at 7 and at 8 (64 registers, 44 spills).  With checked signs, two
// more values a lane, 6 waves (80 registers, 10 spills, 3 with weights).
template <bool kW, bool kMixed>
__global__ __launch_bounds__(64 * kWaves64, kMixed ? 6 : 7) void k_clip64(ClipArgs A) {
    __shared__ WaveMem64 mem[kWaves64];
    run_cells64<kW, kMixed>(mem[threadIdx.x >> 6], A);
}

// Cells marked kLocRetry, listed in (nearly) Morton order: a block lists those
// of kListCells cells in order.  The general pass gives each XCD a range of the
// list, and in the order in which waves finish its caches were of less use (1M
// sites of a lattice: 20.3 instead of 19.6 ms).
constexpr int kListItems = 16, kListCells = 256 * kListItems;
__global__ __launch_bounds__(256) void k_retries(const uint32_t* __restrict__ loc, int64_t n,
                                                 const uint32_t* __restrict__ err, uint32_t* __restrict__ list,
                                                 uint32_t* __restrict__ count) {
    if (*err != 0u) return;
    __shared__ uint32_t sums[4], base;
    const int ln = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t first = (int64_t)blockIdx.x * kListCells + (int64_t)threadIdx.x * kListItems;
    uint32_t m = 0;
    for (int i = 0; i < kListItems; ++i)
        if (first + i < n && loc[first + i] == kLocRetry) m |= 1u << i;
    const uint32_t own = (uint32_t)__popc(m), upto = wscan_u(own);
    if (ln == 63) sums[wv] = upto;
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t total = sums[0] + sums[1] + sums[2] + sums[3];
        base = total ? atomicAdd(count, total) : 0u;
    }
    __syncthreads();
    uint32_t at = base + upto - own;
    for (int k = 0; k < wv; ++k) at += sums[k];
    for (; m; m &= m - 1u) list[at++] = (uint32_t)(first + __builtin_ctz(m));
}

template <bool kW, bool kMixed>
hipError_t launch(const ClipArgs& a, int num_cu, hipStream_t s) {
    int per_cu = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_clip64<kW, kMixed>, 64 * kWaves64, 0);
    if (e != hipSuccess || per_cu < 1) per_cu = 4;
    int64_t blocks = (a.n + kWaves64 - 1) / kWaves64;
    if (blocks > (int64_t)per_cu * num_cu) blocks = (int64_t)per_cu * num_cu;
    hipLaunchKernelGGL((k_clip64<kW, kMixed>), dim3((unsigned)blocks), dim3(64 * kWaves64), 0, s, a);
    if (kMixed)
        hipLaunchKernelGGL(k_retries, dim3((unsigned)((a.n + kListCells - 1) / kListCells)), dim3(256), 0, s, a.loc, a.n,
                           a.err, a.retry_list, a.retry_count);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_clip64(const ClipArgs& a, int num_cu, hipStream_t s) {
    if (a.precision == 2) return a.weighted ? launch<true, true>(a, num_cu, s) : launch<false, true>(a, num_cu, s);
    return a.weighted ? launch<true, false>(a, num_cu, s) : launch<false, false>(a, num_cu, s);
}

}  // namespace vd
