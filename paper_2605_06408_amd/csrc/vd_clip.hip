// Per-site traversal and clipping: the hot loop of the method.
//
// What is computed (paper Sec. 4, Alg. 1, supplementary Sec. B): for every
// site p_i the cell starts as the clip box and is cut by the half-spaces
// a.y <= b (frame centred on p_i, a = p_j - p_i, b = (|a|^2 + w_i - w_j)/2)
// of candidate sites.  Candidates come from a best-first walk of the BVH:
// a node is skipped when the lower bound on the plane distance of any site
// in it (Sec. 4.2.2: d/2 + min(0, w_i - w_max)/(2d), d = distance from p_i
// to the node box) exceeds the directional radius of the cell toward the
// node (Sec. 4.2.1: distance from p_i to the far corner of the cell's AABB
// in each octant the node occupies); a site in a leaf is skipped when its
// plane distance b/|a| exceeds the directional radius of its own octant.
// Far children are queued with their bound as key, the minimum is popped and
// re-tested against the shrunken cell (Alg. 1).
//
// How it maps to CDNA4: one 64-wide wavefront owns one cell.  Vertex v lives
// in lane v % 64, slot v / 64: its position, the three planes meeting there,
// ordered so that their outward normals have a positive determinant, and the
// three vertices across its edges (edge k is the one that leaves plane k).
// Classifying all vertices against a plane is one ballot per slot; the hole
// left by removed vertices is closed by one new vertex per crossing edge
// (supplementary Sec. B): a kept vertex with a removed neighbour across edge
// k = (planes p_k+1, p_k+2) spawns the vertex (h, p_k+2, p_k+1), and new
// vertices find each other through two tables keyed by their old planes.  The
// node queue is spread one entry per lane (min-pop is a wave reduction), node
// children are tested by two lanes at once, and a leaf's sites by one lane
// each.
//
// Capacity tiers: 64 vertices (one slot; vertex state in registers, planes
// and tables in LDS), 128 (two slots, same layout), 1024 (16 slots; every
// per-cell array in LDS) and 16384 (256 slots; every per-cell array in an
// arena in global memory).  In the last two a workgroup of several waves
// builds one cell: the waves split every loop over vertex slots, combine
// their partial results through LDS (one barrier per exchange) and repeat
// the cell-wide control flow in step, so the few very large cells, which
// set the latency of the whole build, get many waves each; the node queue
// and the cell's final record belong to the first wave.  A cell that
// outgrows a tier is handed to the next.  The paper's own kernel keeps one cell per thread in
// global memory; that layout was made for its GPUs and is not used.
#include "vd_wave.h"

// The slot loops are written once for every tier and marked for unrolling,
// which the register tiers need (their vertex state is indexed by slot); in
// the memory tiers their bounds are run-time values and they stay loops.
#pragma clang diagnostic ignored "-Wpass-failed"

namespace vd {
namespace {

// Sizes and index packings of a tier.  Three vertex or plane indices are
// packed into one word: 10 bits each in 32-bit words up to 1024 vertices,
// 15 bits each in 64-bit words above.
template <int VPL>
struct Tier {
    static constexpr int CAP = 64 * VPL;
    static constexpr bool kReg = VPL <= 4;  // vertex state in registers, slot loops unrolled
    static constexpr bool kNarrow = CAP <= 1024;
    static constexpr int kB = kNarrow ? 10 : 15;
    using W = typename std::conditional<kNarrow, uint32_t, uint64_t>::type;
    static constexpr W kMask = (W(1) << kB) - 1;
    // new-vertex table entries: serial tag above the vertex index
    static constexpr int kTagShift = kNarrow ? 12 : 16;
    static constexpr uint32_t kTagMax = (1u << (32 - kTagShift)) - 2u;
    __device__ __forceinline__ static uint32_t fld(W w, int k) { return (uint32_t)((w >> (kB * k)) & kMask); }
    __device__ __forceinline__ static W setfld(W w, int k, uint32_t v) {
        return (w & ~(kMask << (kB * k))) | (W(v) << (kB * k));
    }
    __device__ __forceinline__ static W pack3(uint32_t a, uint32_t b, uint32_t c) {
        return W(a) | (W(b) << kB) | (W(c) << (2 * kB));
    }
};

// Per-slot values of one lane: a register array in the register tiers, a
// column of an arena array otherwise (element s at m[s * kStride]; stride 64
// for per-lane values, 1 for wave-uniform ones).
template <typename X, int N, bool kReg, int kStride>
struct Col {
    X r[kReg ? N : 1];
    X* m = nullptr;
    __device__ __forceinline__ X& operator[](int s) {
        if constexpr (kReg) return r[s];
        else return m[s * kStride];
    }
};

// Waves that build a cell together, and the slots of a cell of a memory tier
// whose positions and masks they hold in registers as well (kSlotsCached each).
constexpr int kGroupLds = 4;
constexpr int kGroupArena = 8;
constexpr int kSlotsCached = 4;
constexpr int kCachedSlots = kGroupLds * kSlotsCached;

// Per-cell state that the register tiers keep in registers and the larger
// tiers in LDS or the arena (index slot * 64 + lane for per-lane values, slot
// for wave-uniform masks).
template <int VPL, bool kArena = !Tier<VPL>::kReg>
struct ArenaState {};
template <int VPL>
struct ArenaState<VPL, true> {
    using W = typename Tier<VPL>::W;
    static constexpr int CAP = Tier<VPL>::CAP;
    float y0[CAP], y1[CAP], y2[CAP], ev[CAP];  // vertex positions and error scales
    W vt[CAP], va[CAP];                         // vertex planes and neighbours
    uint32_t qe[CAP];                           // node queue
    float qk[CAP];
    // clip: crossing edges of a vertex (low 3 bits) and their rank in its slot
    // (slots not kept in registers)
    uint32_t cross[VPL > kCachedSlots ? CAP : 1];
    uint32_t nb1[CAP], nb2[CAP];  // clip: links of the new vertices by rank (above 64 of them)
};

// What every clip of a memory tier exchanges between lanes and waves: per-slot
// masks and the tables of the new vertices.  In LDS in both memory tiers; the
// arena tier keeps only the first kHotRanks entries of the lists by rank here
// (a clip makes about six vertices), the rest in the arena.
constexpr int kHotRanks = 1024;
template <int VPL, bool kMem = !Tier<VPL>::kReg>
struct HotMem {};
template <int VPL>
struct HotMem<VPL, true> {
    using W = typename Tier<VPL>::W;
    static constexpr int CAP = Tier<VPL>::CAP;
    static constexpr int RANKS = CAP < kHotRanks ? CAP : kHotRanks;
    uint64_t alive[VPL], R[VPL], amb[VPL];
    uint32_t cnt[VPL];  // clip: crossing edges of each slot, free places (from bit 16), bounds lost (bit 31)
    uint32_t pre[VPL > 64 ? VPL : 1];  // the same, sums over the lower slots
    uint32_t ta[CAP];   // clip: new vertex by first old plane | finalize: plane rank
    uint32_t tb[CAP];   // clip: new vertex by second old plane | finalize: facet size
    uint32_t sor[RANKS];
    W edge[RANKS];
};
// The same tables of the register tiers, and what the memory tiers have
// beyond kHotRanks.
template <int VPL, bool kMem = !Tier<VPL>::kReg>
struct TableMem {
    using W = typename Tier<VPL>::W;
    static constexpr int CAP = Tier<VPL>::CAP;
    float4 psite[CAP];     // the plane's site (x, y, z, w) for exact re-evaluation
    uint32_t ta[CAP];      // clip: new vertex by first old plane | finalize: plane rank
    uint32_t tb[CAP];      // clip: new vertex by second old plane | finalize: facet size
    uint32_t sor[CAP];     // clip: free slot of rank | finalize: vertex renumbering
    W edge[CAP];           // clip: crossing edges by rank
    uint8_t outf[CAP];     // outside flags by vertex index (VPL > 1)
};
template <int VPL>
struct TableMem<VPL, true> {
    using W = typename Tier<VPL>::W;
    static constexpr int CAP = Tier<VPL>::CAP;
    uint32_t sor[CAP];
    W edge[CAP > kHotRanks ? CAP : 1];
};

// queue entries of the 64-vertex pass beyond the first 64
template <int VPL>
struct QueueExt {};
template <>
struct QueueExt<1> {
    uint32_t qxe[kQueue0 - 64];
    float qxk[kQueue0 - 64];
};
template <>
struct QueueExt<2> {
    uint32_t qxe[kQueue0 - 128];
    float qxk[kQueue0 - 128];
};

template <int VPL>
struct WaveMem : ArenaState<VPL>, QueueExt<VPL>, TableMem<VPL> {
    using W = typename Tier<VPL>::W;
    static constexpr int CAP = Tier<VPL>::CAP;
    float4 pl[CAP];        // planes: a.xyz, b (frame of the site)
    float psb[CAP];        // size of the terms b is formed from (error scale)
    int32_t pcode[CAP];    // Morton index of the plane's site, or box code -1..-6
    uint32_t anchor[CAP];  // finalize: lowest vertex of each facet
    W vtri[CAP];           // finalize: planes of each vertex
    W vadj[CAP];           // finalize: neighbours of each vertex
    double vpx[CAP], vpy[CAP], vpz[CAP];  // finalize: FP64 positions relative to vertex 0
    int32_t key[CAP];      // finalize and gc: output codes, used flags
};

// kLds: the per-cell arrays are in LDS (else in global memory).  kCount:
// count work units and cycles (a separate instantiation, so the timed
// kernels carry no counting code).  G: waves building the cell together
// (one in the register tiers).  kSoS: exact ties decided by the symbolic
// perturbation (its own instantiation: the checked exact evaluation would
// otherwise cost the default kernels registers).  kW: the sites carry
// weights; kOpt: the search options (culling, traversal order, warm start)
// are read at run time.  The passes of a build with the default options
// run instantiations with those options fixed, the register passes of an
// unweighted build also without the weight terms of the bounds and ball tests
// (every weight is zero there): the same results bit for bit, 4% less time
// for the fixed options (their checks and the scalar registers they held)
// and 2.5% for the weight terms.  Every wave of a group
// holds the same copy of the cell-wide scalars (site, bounds, plane and
// queue counts, flags) and changes it the same way, from values every wave
// has seen.
// Every member of Cell and the work loop are inlined into their kernel: as
// calls (the inliner's size limits give up on the larger instantiations)
// they cost a stack frame in scratch memory and spills around each call.
#pragma clang attribute push(__attribute__((always_inline)), apply_to = function)
template <int VPL, bool kLds, bool kCount, int G = 1, bool kSoS = false, bool kW = true, bool kOpt = true>
struct Cell {
    static_assert(G == 1 || !Tier<VPL>::kReg, "wave groups need the vertex state in memory");
    using T = Tier<VPL>;
    using W = typename T::W;
    static constexpr int CAP = T::CAP;
    static constexpr bool kReg = T::kReg;
    // hand-over: every pass but the last writes the state of the cells it
    // escalates; every pass but the first can take over such a state (from
    // the pass of capacity kPrevCap)
    static constexpr bool kSaves = CAP < kTierCap[kTiers - 1];
    static constexpr int kPrevCap = CAP == kTierCap[1] ? kTierCap[0]
                                    : (CAP == kTierCap[2] ? kTierCap[1] : (CAP == kTierCap[3] ? kTierCap[2] : 0));
    static constexpr bool kResumes = kPrevCap > 0;
    // queue capacity: one entry per vertex, but kQueue0 in the 64-vertex pass
    static constexpr bool kQExt = kReg && 64 * VPL < kQueue0;  // queue entries beyond the slots in LDS
    static constexpr int QCAP = queue_cap(CAP);
    static constexpr int kPrevQ = kPrevCap > 0 ? queue_cap(kPrevCap) : 64;
    using HIn = HandoffT<(kPrevCap > 0 ? kPrevCap : 64), (kPrevCap > 0 ? kPrevQ : 64)>;
    using HOut = HandoffT<(kSaves ? CAP : 64), (kSaves ? QCAP : 64)>;
    template <typename X>
    using Lane = Col<X, VPL, kReg, 64>;  // one value per slot of this lane
    template <typename X>
    using Wave = Col<X, VPL, kReg, 1>;   // one wave-uniform value per slot
    WaveMem<VPL>& M;
    HotMem<VPL>& H;
    const ClipArgs& A;
    const uint32_t ln;
    const uint32_t wid;  // wave of the group
    uint32_t* gx;        // group exchange tables in LDS: 2 x G x 8 words
    int gpar;            // table of the next exchange
    uint32_t serial;
    // site
    float px, py, pz, pw;
    // the site's weight where the arithmetic uses it (zero without weights)
    __device__ __forceinline__ float pwv() const { if constexpr (kW) return pw; else return 0.f; }
    // search options: the default instantiations fix them (directional plus
    // ball culling, best-first order, no warm start)
    __device__ __forceinline__ int culling() const { if constexpr (kOpt) return A.culling; else return 3; }
    __device__ __forceinline__ int traversal() const { if constexpr (kOpt) return A.traversal; else return 1; }
    __device__ __forceinline__ int warm_start() const { if constexpr (kOpt) return A.warm_start; else return 0; }
    uint32_t self;
    uint32_t flags;
    int robust;   // 0: FP32 signs; 1: doubtful signs in FP64; 2: every sign in FP64
    // vertices: slot s of this lane is vertex s*64 + lane
    Lane<float> y0, y1, y2, ev;
    Lane<W> vt, va;
    Wave<uint64_t> alive;
    float c0[kReg ? 1 : kSlotsCached], c1[kReg ? 1 : kSlotsCached], c2[kReg ? 1 : kSlotsCached];
    uint64_t cal[kReg ? 1 : kSlotsCached];
    bool bnd;  // the last effective clip may have moved the bounds
    int np;
    int vhi;  // one past the highest vertex index used since init
    // bounds of the current cell (uniform): AABB in the site's frame, the
    // squared far-corner coordinates, the directional and isotropic radii
    float blo0, blo1, blo2, bhi0, bhi1, bhi2;
    float hx2, hy2, hz2, lx2, ly2, lz2, rmax2, riso2;
    // 64-vertex pass: the vertex at each side of the AABB (min x, y, z, max
    // x, y, z) and the vertices the last effective clip removed; a clip that
    // removes none of the six leaves the AABB as it was (new vertices lie on
    // edges of the old cell)
    uint32_t ext[6];
    uint64_t cut_mask;
    // queue (entry q in lane q % 64, slot q / 64; in the 64-vertex pass entries
    // from 64 on are in LDS, M.qxe / M.qxk)
    Lane<uint32_t> qe;
    Lane<float> qk;
    int qn;
    // KNN warm start: the sites already clipped (Morton positions), lane t
    // holding the t-th; the leaves of the walk pass over them
    int nwarm;
    uint32_t wsite;
    // where the last capacity overflow struck: in leaf ov_leaf, with the
    // candidates ov_mask still to try (ov_ok), else somewhere not resumable
    bool ov_ok;
    uint32_t ov_leaf, ov_phase, ov_skip;
    uint64_t ov_mask;
    uint32_t leaf_phase = 1;  // 0 while clipping by the site's own leaf before any walk
    // work counters (uniform), accumulated over all cells of this wave
    uint64_t ctr[kCount ? kCtrCount : 1];
    static constexpr bool counting = kCount;

    // the first clip clears the new-vertex tables (the tag counter starts
    // at its wrap-around value)
    __device__ Cell(WaveMem<VPL>& m, HotMem<VPL>& hot, const ClipArgs& a, uint32_t* gxch)
        : M(m), H(hot), A(a), ln(lane_id()), wid(G > 1 ? uni((uint32_t)(threadIdx.x >> 6)) : 0u), gx(gxch), gpar(0),
          serial(T::kTagMax - 1) {
#pragma unroll
        for (int c = 0; c < (kCount ? kCtrCount : 1); ++c) ctr[c] = 0;
        if constexpr (!kReg) {
            y0.m = M.y0 + ln; y1.m = M.y1 + ln; y2.m = M.y2 + ln; ev.m = M.ev + ln;
            vt.m = M.vt + ln; va.m = M.va + ln;
            alive.m = H.alive;
            qe.m = M.qe + ln; qk.m = M.qk + ln;
        }
        vhi = CAP;
    }
    // tables of the new vertices and, when the cell is finished, of its facets
    __device__ __forceinline__ uint32_t& ta(uint32_t q) { if constexpr (kReg) return M.ta[q]; else return H.ta[q]; }
    __device__ __forceinline__ uint32_t& tb(uint32_t q) { if constexpr (kReg) return M.tb[q]; else return H.tb[q]; }
    // the plane's site (the memory tiers read it again where FP64 asks for it)
    __device__ __forceinline__ float4 site_of(uint32_t q) const {
        if constexpr (kReg) return M.psite[q];
        else return M.pcode[q] >= 0 ? A.pts[M.pcode[q]] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __device__ __forceinline__ void count(int c, uint64_t v) {
        if constexpr (kCount) ctr[c] += v;
    }
    // elapsed shader clock of this wave, accumulated per phase when counting
    __device__ __forceinline__ uint64_t tic() const {
        if constexpr (kCount) return (uint64_t)clock64();
        else return 0ull;
    }
    __device__ __forceinline__ void toc(int c, uint64_t t0) {
        if constexpr (kCount) ctr[c] += (uint64_t)clock64() - t0;
    }
    // wsync orders this wave's accesses; sync those of the whole group
    __device__ __forceinline__ void wsync() { wave_sync<kLds>(); }
    __device__ __forceinline__ void sync() {
        if constexpr (G > 1) __syncthreads();
        else wave_sync<kLds>();
    }
    // the first wave of the group (the only one without groups)
    __device__ __forceinline__ bool lead() const { return G == 1 || wid == 0; }
    // Group exchange: every wave posts N uniform words; returns the table
    // (word k of wave w at [w * 8 + k]) once all have posted.  The two tables
    // alternate, so one barrier per exchange is enough: a wave writes a table
    // again only after the barrier of the exchange in between, which every
    // wave reaches after reading it.
    template <int N>
    __device__ __forceinline__ const uint32_t* exch(const uint32_t (&v)[N]) {
        static_assert(N <= 8, "eight words per wave");
        uint32_t* t = gx + gpar * (G * 8);
        gpar ^= 1;
        if (ln == 0) {
#pragma unroll
            for (int k = 0; k < N; ++k) t[wid * 8 + k] = v[k];
        }
        __syncthreads();
        return t;
    }
    // Bitwise or over the group of kBits flags.
    template <int kBits>
    __device__ __forceinline__ uint32_t g_or(uint32_t f) {
        if constexpr (G == 1) {
            return f;
        } else {
            const uint32_t v[1] = {f};
            const uint32_t x = exch(v)[(ln % G) * 8];
            uint32_t r = 0;
#pragma unroll
            for (int k = 0; k < kBits; ++k) r |= ballot((x >> k) & 1u) != 0 ? 1u << k : 0u;
            return r;
        }
    }
    // the first wave's value, for every wave of the group
    __device__ __forceinline__ uint32_t bcast(uint32_t x) {
        if constexpr (G == 1) {
            return uni(x);
        } else {
            const uint32_t v[1] = {x};
            return uni(exch(v)[0]);
        }
    }
    // slots that may hold vertices (all of them in the register tiers)
    __device__ __forceinline__ int nsv() const { return kReg ? VPL : ((vhi + 63) >> 6); }
    // a wave-uniform value read from the memory of a memory tier
    __device__ __forceinline__ static uint64_t um(uint64_t v) {
        if constexpr (kReg) return v;
        else return uni(v);
    }
    // VD_EACH_SLOT runs its body for this wave's slots in use: s_ the slot, its
    // vertices' positions x_, y_, z_ and their mask al_.  In a group slot s
    // belongs to wave s % G, and its owner keeps the positions and the mask of
    // its first kC slots in registers: the tests of boxes, planes and
    // candidates then read no memory (they waited for LDS at every pair of
    // slots).  i_ is the place in the registers, kC for the slots beyond.
    // (A macro: with the body as a closure handed to a function the register
    // tiers kept their vertices in scratch memory and took four times as long.)
#define VD_EACH_SLOT(...)                                                                          \
    do {                                                                                           \
        if constexpr (kReg) {                                                                      \
            _Pragma("unroll") for (int s_ = 0; s_ < VPL; ++s_) {                                   \
                [[maybe_unused]] const int i_ = s_;                                                \
                [[maybe_unused]] const float x_ = y0[s_], y_ = y1[s_], z_ = y2[s_];                \
                [[maybe_unused]] const uint64_t al_ = alive[s_];                                   \
                __VA_ARGS__                                                                        \
            }                                                                                      \
        } else {                                                                                   \
            const int ns_ = nsv();                                                                 \
            _Pragma("unroll") for (int i_ = 0; i_ < kC; ++i_) {                                    \
                const int s_ = (int)wid + G * i_;                                                  \
                if (s_ < ns_) {                                                                    \
                    [[maybe_unused]] const float x_ = c0[i_], y_ = c1[i_], z_ = c2[i_];            \
                    [[maybe_unused]] const uint64_t al_ = cal[i_];                                 \
                    __VA_ARGS__                                                                    \
                }                                                                                  \
            }                                                                                      \
            if constexpr (VPL > G * kC) {                                                          \
                for (int s_ = (int)wid + G * kC; s_ < ns_; s_ += G) {                              \
                    [[maybe_unused]] constexpr int i_ = kC;                                        \
                    [[maybe_unused]] const float x_ = y0[s_], y_ = y1[s_], z_ = y2[s_];            \
                    [[maybe_unused]] const uint64_t al_ = uni(alive[s_]);                          \
                    __VA_ARGS__                                                                    \
                }                                                                                  \
            }                                                                                      \
        }                                                                                          \
    } while (0)
    static constexpr int kC = kReg ? VPL : kSlotsCached;
    __device__ __forceinline__ void load_slot(int i, int s) {
        c0[i] = y0[s];
        c1[i] = y1[s];
        c2[i] = y2[s];
    }
    // the registers of a cell just begun
    __device__ __forceinline__ void load_slots() {
        if constexpr (!kReg) {
            const int ns = nsv();
#pragma unroll
            for (int i = 0; i < kC; ++i) {
                const int s = (int)wid + G * i;
                cal[i] = 0;
                if (s < ns) {
                    load_slot(i, s);
                    cal[i] = uni(alive[s]);
                }
            }
        }
    }
    __device__ __forceinline__ uint64_t nalive() {
        uint64_t c = 0;
        const int ns = nsv();
#pragma unroll
        for (int s = 0; s < (kReg ? VPL : ns); ++s) c += (uint64_t)popc(um(alive[s]));
        return c;
    }

    __device__ __forceinline__ bool is_alive(uint32_t u) {
        const int sl = (int)(u >> 6);
        uint64_t al = 0;
        if constexpr (kReg) {
#pragma unroll
            for (int s = 0; s < VPL; ++s) al = s == sl ? alive[s] : al;
        } else {
            if (sl < nsv()) al = alive[sl];
        }
        return (al >> (u & 63)) & 1;
    }

    // ------------------------------------------------------------ setup
    __device__ bool init(uint32_t k) {
        if constexpr (G > 1) sync();  // every wave is done with the previous cell
        self = k;
        float4 s = A.pts[k];
        px = s.x; py = s.y; pz = s.z; pw = s.w;
        flags = 0;
        qn = 0;
        nwarm = 0;
        if (uni(pw) == -INFINITY) return false;  // coincident with a heavier site
        const float lo[3] = {A.bbox[0] - px, A.bbox[1] - py, A.bbox[2] - pz};
        const float hi[3] = {A.bbox[3] - px, A.bbox[4] - py, A.bbox[5] - pz};
        if (ln < 6 && lead()) {
            int ax = ln >> 1, side = ln & 1;
            float a[3] = {0.f, 0.f, 0.f};
            a[ax] = side ? 1.f : -1.f;
            float b = side ? hi[ax] : -lo[ax];
            M.pl[ln] = make_float4(a[0], a[1], a[2], b);
            M.psb[ln] = fabsf(b);
            M.pcode[ln] = -(int)(ln + 1);
            if constexpr (kReg) M.psite[ln] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        if constexpr (kReg) {
#pragma unroll
            for (int s2 = 0; s2 < VPL; ++s2) alive[s2] = 0;
        }
        // slots above the first are written by a clip before they are read
        if (lead()) alive[0] = 0xFFull;
        vhi = 8;
        if (lead()) {
            uint32_t c = ln & 7;
            uint32_t sx = c & 1, sy = (c >> 1) & 1, sz = (c >> 2) & 1;
            uint32_t X = sx, Y = 2 + sy, Z = 4 + sz;
            bool pos = ((sx ^ sy ^ sz) & 1) == 1;  // product of the three normal signs > 0
            uint32_t p1 = pos ? Y : Z, p2 = pos ? Z : Y;
            uint32_t ax1 = p1 >> 1, ax2 = p2 >> 1;
            vt[0] = T::pack3(X, p1, p2);
            va[0] = T::pack3(c ^ 1u, c ^ (1u << ax1), c ^ (1u << ax2));
            y0[0] = sx ? hi[0] : lo[0];
            y1[0] = sy ? hi[1] : lo[1];
            y2[0] = sz ? hi[2] : lo[2];
            ev[0] = fabsf(y0[0]) + fabsf(y1[0]) + fabsf(y2[0]);
        }
        np = 6;
        sync();
        load_slots();
        update_bounds();
        return true;
    }

    __device__ void update_bounds() {
        float mn0 = INFINITY, mn1 = INFINITY, mn2 = INFINITY, mx0 = -INFINITY, mx1 = -INFINITY, mx2 = -INFINITY,
              r2 = 0.f;
        VD_EACH_SLOT({
            if ((al_ >> ln) & 1) {
                mn0 = fminf(mn0, x_); mn1 = fminf(mn1, y_); mn2 = fminf(mn2, z_);
                mx0 = fmaxf(mx0, x_); mx1 = fmaxf(mx1, y_); mx2 = fmaxf(mx2, z_);
                if (culling() == 2) r2 = fmaxf(r2, fmaf(x_, x_, fmaf(y_, y_, z_ * z_)));
            }
        });
        float l0 = wmin(mn0), l1 = wmin(mn1), l2 = wmin(mn2);
        float h0 = wmax(mx0), h1 = wmax(mx1), h2 = wmax(mx2);
        riso2 = culling() == 2 ? wmax(r2) : 0.f;  // the isotropic radius only serves culling mode 2
        if constexpr (G > 1) {
            const uint32_t v[7] = {__float_as_uint(l0), __float_as_uint(l1), __float_as_uint(l2), __float_as_uint(h0),
                                   __float_as_uint(h1), __float_as_uint(h2), __float_as_uint(riso2)};
            const uint32_t* t = exch(v);
            l0 = l1 = l2 = INFINITY;
            h0 = h1 = h2 = -INFINITY;
            riso2 = 0.f;
#pragma unroll
            for (int w = 0; w < G; ++w) {
                const uint32_t* x = t + w * 8;
                l0 = fminf(l0, __uint_as_float(x[0])); l1 = fminf(l1, __uint_as_float(x[1]));
                l2 = fminf(l2, __uint_as_float(x[2]));
                h0 = fmaxf(h0, __uint_as_float(x[3])); h1 = fmaxf(h1, __uint_as_float(x[4]));
                h2 = fmaxf(h2, __uint_as_float(x[5]));
                riso2 = fmaxf(riso2, __uint_as_float(x[6]));
            }
            l0 = uni(l0); l1 = uni(l1); l2 = uni(l2);
            h0 = uni(h0); h1 = uni(h1); h2 = uni(h2);
            riso2 = uni(riso2);
        }
        blo0 = l0; blo1 = l1; blo2 = l2;
        bhi0 = h0; bhi1 = h1; bhi2 = h2;
        if constexpr (VPL == 1 && G == 1) {
            const bool al = (alive[0] >> ln) & 1;
            ext[0] = lowest(ballot(al && y0[0] == l0));
            ext[1] = lowest(ballot(al && y1[0] == l1));
            ext[2] = lowest(ballot(al && y2[0] == l2));
            ext[3] = lowest(ballot(al && y0[0] == h0));
            ext[4] = lowest(ballot(al && y1[0] == h1));
            ext[5] = lowest(ballot(al && y2[0] == h2));
        }
        derive_bounds();
    }
    __device__ __forceinline__ void derive_bounds() {
        hx2 = bhi0 * bhi0; hy2 = bhi1 * bhi1; hz2 = bhi2 * bhi2;
        lx2 = blo0 * blo0; ly2 = blo1 * blo1; lz2 = blo2 * blo2;
        rmax2 = fmaxf(hx2, lx2) + fmaxf(hy2, ly2) + fmaxf(hz2, lz2);
    }
    // After an effective clip: in the 64-vertex pass only the sides whose
    // vertex the clip removed are reduced again; in a group the bounds stay
    // unless the clip removed a vertex on one of them or put one outside.
    __device__ void bounds_after_clip() {
        if constexpr (G > 1) {
            if (culling() != 2 && !bnd) return;
        }
        if constexpr (VPL == 1 && G == 1) {
            if (culling() != 2) {
                uint32_t lost = 0;
#pragma unroll
                for (int k = 0; k < 6; ++k) lost |= (uint32_t)((cut_mask >> ext[k]) & 1ull) << k;
                if (lost == 0) return;
                const bool al = (alive[0] >> ln) & 1;
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    if ((lost >> k) & 1u) {
                        const float v = (k % 3 == 0) ? y0[0] : ((k % 3 == 1) ? y1[0] : y2[0]);
                        const float m = k < 3 ? wmin(al ? v : INFINITY) : wmax(al ? v : -INFINITY);
                        ext[k] = lowest(ballot(al && v == m));
                        if (k == 0) blo0 = m; else if (k == 1) blo1 = m; else if (k == 2) blo2 = m;
                        else if (k == 3) bhi0 = m; else if (k == 4) bhi1 = m; else bhi2 = m;
                    }
                }
                derive_bounds();
                return;
            }
        }
        update_bounds();
    }

    // Squared radius of the cell toward direction a (far AABB corner of the
    // octant of a; zero components count as positive).
    __device__ __forceinline__ float radius2_toward(float ax, float ay, float az) const {
        if (culling() == 2) return riso2;
        return (ax >= 0.f ? hx2 : lx2) + (ay >= 0.f ? hy2 : ly2) + (az >= 0.f ? hz2 : lz2);
    }

    // Power-ball test of a node box (frame of the site): a site p_j in the box
    // with w_j <= wmax cuts the cell only if some vertex v has
    // |v - p_j|^2 - w_j < |v|^2 - w_i, and |v - p_j|^2 >= dist(v, box)^2.
    // Returns true if some vertex might be cut (the box cannot be skipped).
    __device__ bool ball_hit(float lx, float ly, float lz, float hx, float hy, float hz, float wm) {
        if constexpr (kCount) count(kCtrBall, nalive());
        uint64_t hit = 0;
        VD_EACH_SLOT({
            float dx = fmaxf(fmaxf(lx - x_, x_ - hx), 0.f);
            float dy = fmaxf(fmaxf(ly - y_, y_ - hy), 0.f);
            float dz = fmaxf(fmaxf(lz - z_, z_ - hz), 0.f);
            float d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
            float r2 = fmaf(x_, x_, fmaf(y_, y_, z_ * z_));
            hit |= ballot(ball_test<kW>(d2, r2, wm, pwv())) & al_;
        });
        return g_or<1>(hit != 0 ? 1u : 0u) != 0;
    }

    // The ball test of both child records (lanes 0 and 1) in one pass over
    // the vertices (the vertex's own power is shared by the two boxes).
    __device__ void ball_hit_pair(const NodeChild& c, bool* hit0, bool* hit1) {
        if constexpr (kCount) count(kCtrBall, 2 * nalive());
        const float blx = c.lo[0] - px, bly = c.lo[1] - py, blz = c.lo[2] - pz;
        const float bhx = c.hi[0] - px, bhy = c.hi[1] - py, bhz = c.hi[2] - pz;
        const float l0x = rdl(blx, 0), l0y = rdl(bly, 0), l0z = rdl(blz, 0);
        const float h0x = rdl(bhx, 0), h0y = rdl(bhy, 0), h0z = rdl(bhz, 0), w0 = kW ? rdl(c.wmax, 0) : 0.f;
        const float l1x = rdl(blx, 1), l1y = rdl(bly, 1), l1z = rdl(blz, 1);
        const float h1x = rdl(bhx, 1), h1y = rdl(bhy, 1), h1z = rdl(bhz, 1), w1 = kW ? rdl(c.wmax, 1) : 0.f;
        uint64_t a0 = 0, a1 = 0;
        VD_EACH_SLOT({
            const float r2 = fmaf(x_, x_, fmaf(y_, y_, z_ * z_));
            float dx = fmaxf(fmaxf(l0x - x_, x_ - h0x), 0.f);
            float dy = fmaxf(fmaxf(l0y - y_, y_ - h0y), 0.f);
            float dz = fmaxf(fmaxf(l0z - z_, z_ - h0z), 0.f);
            float d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
            a0 |= ballot(ball_test<kW>(d2, r2, w0, pwv())) & al_;
            dx = fmaxf(fmaxf(l1x - x_, x_ - h1x), 0.f);
            dy = fmaxf(fmaxf(l1y - y_, y_ - h1y), 0.f);
            dz = fmaxf(fmaxf(l1z - z_, z_ - h1z), 0.f);
            d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
            a1 |= ballot(ball_test<kW>(d2, r2, w1, pwv())) & al_;
        });
        const uint32_t r = g_or<2>((a0 != 0 ? 1u : 0u) | (a1 != 0 ? 2u : 0u));
        *hit0 = (r & 1u) != 0;
        *hit1 = (r & 2u) != 0;
    }

    // Applies the ball test to the child record held by lane `l`.
    __device__ bool ball_hit_lane(const NodeChild& c, int l) {
        float lx = rdl(c.lo[0] - px, l), ly = rdl(c.lo[1] - py, l), lz = rdl(c.lo[2] - pz, l);
        float hx = rdl(c.hi[0] - px, l), hy = rdl(c.hi[1] - py, l), hz = rdl(c.hi[2] - pz, l);
        float wm = kW ? rdl(c.wmax, l) : 0.f;
        return ball_hit(lx, ly, lz, hx, hy, hz, wm);
    }

    // ------------------------------------------------------------ FP64 side test
    // Plane q in FP64, recomputed from the input coordinates: a = p_j - p_i
    // is exact in FP64, b = (|a|^2 + w_i - w_j) / 2 nearly so.
    __device__ P64 plane64(uint32_t q) const { return plane64(M.pcode[q], site_of(q)); }

    __device__ P64 plane64(int32_t code, float4 site) const {
        P64 r;
        const double qx = px, qy = py, qz = pz, qw = pw;
        if (code < 0) {
            int c = -code - 1, ax = c >> 1, side = c & 1;
            double p[3] = {qx, qy, qz};
            r.a0 = r.a1 = r.a2 = 0.0;
            double sgn = side ? 1.0 : -1.0;
            if (ax == 0) r.a0 = sgn; else if (ax == 1) r.a1 = sgn; else r.a2 = sgn;
            r.b = side ? ((double)A.bbox[3 + ax] - p[ax]) : (p[ax] - (double)A.bbox[ax]);
        } else {
            r.a0 = (double)site.x - qx; r.a1 = (double)site.y - qy; r.a2 = (double)site.z - qz;
            r.b = 0.5 * (r.a0 * r.a0 + r.a1 * r.a1 + r.a2 * r.a2 + (qw - (double)site.w));
        }
        return r;
    }

    // Side of the vertex with planes t w.r.t. plane h, recomputed in FP64 from
    // the input coordinates.  Returns +1 outside, -1 inside, 0 undecided.
    __device__ int side64(W t, const P64& h) const {
        const P64 P = plane64(T::fld(t, 0)), Q = plane64(T::fld(t, 1)), S = plane64(T::fld(t, 2));
        const Meet64 y(P, Q, S);
        const double det = y.det;
        double n[3];
        y.numerator(P, Q, S, n);
        // s * det = a_h . n - b_h det, evaluated without dividing
        double s = h.a0 * n[0] + h.a1 * n[1] + h.a2 * n[2] - h.b * det;
        if (det < 0) s = -s;
        double scale = (fabs(h.a0) + fabs(h.a1) + fabs(h.a2)) * (fabs(n[0]) + fabs(n[1]) + fabs(n[2])) +
                       fabs(h.b * det);
        if (fabs(s) <= 64.0 * kU64 * scale) return 0;
        return s > 0 ? 1 : -1;
    }

    // ------------------------------------------------------------ exact ties
    // Side of the vertex with planes t w.r.t. the plane of site hsite (code
    // hcode) when the FP64 filter cannot decide it: the test is evaluated
    // again in FP64 with every operation checked to be exact (the error of
    // each product by a fused multiply-add, of each sum by the two-sum
    // identity).  That holds for inputs with short dyadic coordinates, such
    // as lattices, which is where exact ties occur.  If the value is exact
    // and non-zero its sign decides (+-1).  If it is exactly zero the weights
    // are perturbed symbolically, w_k -> w_k + d^(k+1) for infinitesimal d
    // and original index k (Simulation of Simplicity): the test S is linear
    // in the plane offsets b = (|a|^2 + w_i - w_x) / 2, hence in the weights,
    // and its sign is that of the weight derivative of lowest original index
    // among the non-zero ones (+-2).  Returns 0 if some operation was not
    // exact (the sign stays undecided).
    //   S = det (a_h . y - b_h) = b_A a_h.(B x C) + b_B a_h.(C x A) + b_C a_h.(A x B) - b_h det
    //   dS/dw_x = -a_h.cross_X / 2 (X the plane of site x), dS/dw_m = det / 2
    //   (m the site of h), dS/dw_i = (sum of a_h.cross_X over site planes - det) / 2;
    // the vertex is outside iff S det > 0.
    struct PX {
        double a[3], b;
        uint32_t orig;  // original index of the plane's site (box faces: none)
        bool site;
    };
    __device__ static double xmul(double a, double b, bool& ok) {
        const double p = a * b;
        ok &= fma(a, b, -p) == 0.0;
        return p;
    }
    __device__ static double xadd(double a, double b, bool& ok) {
        const double s = a + b;
        const double bv = s - a;
        ok &= ((a - (s - bv)) + (b - bv)) == 0.0;
        return s;
    }
    __device__ PX plane_exact(int32_t code, float4 site, bool& ok) const {
        PX r;
        const double q[3] = {(double)px, (double)py, (double)pz};
        if (code < 0) {
            const int c = -code - 1, ax = c >> 1, side = c & 1;
            r.a[0] = r.a[1] = r.a[2] = 0.0;
            r.a[ax] = side ? 1.0 : -1.0;
            r.b = side ? xadd((double)A.bbox[3 + ax], -q[ax], ok) : xadd(q[ax], -(double)A.bbox[ax], ok);
            r.orig = 0u;
            r.site = false;
        } else {
            r.a[0] = xadd((double)site.x, -q[0], ok);
            r.a[1] = xadd((double)site.y, -q[1], ok);
            r.a[2] = xadd((double)site.z, -q[2], ok);
            double s2 = xadd(xadd(xmul(r.a[0], r.a[0], ok), xmul(r.a[1], r.a[1], ok), ok),
                             xmul(r.a[2], r.a[2], ok), ok);
            r.b = 0.5 * xadd(s2, xadd((double)pw, -(double)site.w, ok), ok);
            r.orig = cold_args()->order[code];
            r.site = true;
        }
        return r;
    }
    __device__ static void xcross(const double* u, const double* v, double* o, bool& ok) {
        o[0] = xadd(xmul(u[1], v[2], ok), -xmul(u[2], v[1], ok), ok);
        o[1] = xadd(xmul(u[2], v[0], ok), -xmul(u[0], v[2], ok), ok);
        o[2] = xadd(xmul(u[0], v[1], ok), -xmul(u[1], v[0], ok), ok);
    }
    __device__ static double xdot(const double* u, const double* v, bool& ok) {
        return xadd(xadd(xmul(u[0], v[0], ok), xmul(u[1], v[1], ok), ok), xmul(u[2], v[2], ok), ok);
    }
    __device__ int side_exact(W t, int32_t hcode) const {
        const float4 hsite = A.pts[hcode];
        bool ok = true;
        const PX P0 = plane_exact(M.pcode[T::fld(t, 0)], site_of(T::fld(t, 0)), ok);
        const PX P1 = plane_exact(M.pcode[T::fld(t, 1)], site_of(T::fld(t, 1)), ok);
        const PX P2 = plane_exact(M.pcode[T::fld(t, 2)], site_of(T::fld(t, 2)), ok);
        const PX H = plane_exact(hcode, hsite, ok);
        double cr[3][3];
        xcross(P1.a, P2.a, cr[0], ok);
        xcross(P2.a, P0.a, cr[1], ok);
        xcross(P0.a, P1.a, cr[2], ok);
        const double det = xdot(P0.a, cr[0], ok);
        const double hb[3] = {xdot(H.a, cr[0], ok), xdot(H.a, cr[1], ok), xdot(H.a, cr[2], ok)};
        double S = xadd(xadd(xmul(P0.b, hb[0], ok), xmul(P1.b, hb[1], ok), ok),
                        xadd(xmul(P2.b, hb[2], ok), -xmul(H.b, det, ok), ok), ok);
        if (!ok || det == 0.0) return 0;
        const int sd = det > 0.0 ? 1 : -1;
        if (S != 0.0) return (S > 0.0 ? 1 : -1) == sd ? 1 : -1;
        // exact tie: the lowest original index with a non-zero weight derivative
        uint32_t best = H.orig;
        int sgn = sd;  // dS/dw_m = det / 2
        double own = -det;
        const PX* X[3] = {&P0, &P1, &P2};
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            if (!X[r]->site) continue;
            own = xadd(own, hb[r], ok);
            if (hb[r] != 0.0 && X[r]->orig < best) {
                best = X[r]->orig;
                sgn = hb[r] > 0.0 ? -1 : 1;  // dS/dw_x = -a_h.cross_X / 2
            }
        }
        if (!ok) return 0;
        const uint32_t self_orig = cold_args()->order[self];
        if (own != 0.0 && self_orig < best) sgn = own > 0.0 ? 1 : -1;
        return sgn == sd ? 2 : -2;
    }

    // ------------------------------------------------------------ clip
    // mode 0: plain FP32 signs; 1: doubtful signs re-evaluated in FP64;
    // 2: doubtful signs taken as inside; 3: every sign evaluated in FP64.
    __device__ void classify(float ax, float ay, float az, float b, float sbh, int32_t hcode,
                             int mode, Wave<uint64_t>& R, bool* any_out, bool* all_out) {
        const float an1 = fabsf(ax) + fabsf(ay) + fabsf(az);
        if (kCount && mode != 2) count(kCtrClassify, nalive());
        bool anyo = false, allo = true, ambf = false;
        Wave<uint64_t> amb;
        if constexpr (!kReg) amb.m = H.amb;
        VD_EACH_SLOT({
            const float sv = fmaf(ax, x_, fmaf(ay, y_, fmaf(az, z_, -b)));
            uint64_t r = ballot(sv > 0.f) & al_, am = 0;
            if (mode != 0) {
                const float beta = doubt(an1, ev[s_], sbh);
                am = mode == 3 ? al_ : ballot(fabsf(sv) <= beta) & al_;
                if (mode == 2) r &= ~am;
            }
            amb[s_] = am;
            R[s_] = r;
            ambf |= am != 0;
            anyo |= r != 0;
            allo &= r == al_;
        });
        if constexpr (G > 1) {
            const uint32_t f = g_or<3>((anyo ? 1u : 0u) | (allo ? 0u : 2u) | (ambf ? 4u : 0u));
            anyo = (f & 1u) != 0;
            allo = (f & 2u) == 0;
            ambf = (f & 4u) != 0;
        }
        if ((mode == 1 || mode == 3) && ambf) {
            flags |= kFlagFP64;
            if constexpr (kCount) {
                uint64_t na = 0;
#pragma unroll
                for (int s = 0; s < nsv(); ++s) na += (uint64_t)popc(um(amb[s]));
                count(kCtrFP64, na);
            }
            P64 h = plane64(hcode, A.pts[hcode]);
            anyo = false;
            allo = true;
            bool uns = false, pert = false;
            const int ns = nsv();
#pragma unroll
            for (int s = kReg ? 0 : (int)wid; s < (kReg ? VPL : ns); s += G) {
                const uint64_t al = um(alive[s]);
                bool o = (um(R[s]) >> ln) & 1;
                bool unsure = false, tie = false;
                if ((um(amb[s]) >> ln) & 1) {
                    int sg = side64(vt[s], h);
                    if constexpr (kSoS) {
                        if (sg == 0) {
                            sg = side_exact(vt[s], hcode);
                            tie = sg == 2 || sg == -2;
                        }
                    }
                    o = sg > 0;
                    unsure = sg == 0;
                }
                const uint64_t r = ballot(o);
                R[s] = r;
                anyo |= r != 0;
                allo &= r == al;
                uns |= ballot(unsure) != 0;
                pert |= ballot(tie) != 0;
            }
            if constexpr (G > 1) {
                const uint32_t f = g_or<4>((anyo ? 1u : 0u) | (allo ? 0u : 2u) | (uns ? 4u : 0u) | (pert ? 8u : 0u));
                anyo = (f & 1u) != 0;
                allo = (f & 2u) == 0;
                uns = (f & 4u) != 0;
                pert = (f & 8u) != 0;
            }
            if (uns) flags |= kFlagUncertain;
            if (pert) flags |= kFlagPerturbed;
        }
        *any_out = anyo;
        *all_out = allo;
    }

    // Position and error scale of the vertex of planes (h, x, y), by Cramer's rule.
    __device__ void solve(uint32_t x, uint32_t y, float ax, float ay, float az, float b, float sbh, float* q0, float* q1,
                          float* q2, float* e) const {
        const Solve32 v(M.pl[x], M.pl[y], ax, ay, az, b);
        *q0 = v.y0;
        *q1 = v.y1;
        *q2 = v.y2;
        // error scale, for the doubtful-sign test (only read when signs are
        // checked: robust builds)
        if (robust != 0) *e = v.scale(sbh, M.psb[x], M.psb[y]);
    }

    // Tries the clip with the given outside masks; on an inconsistent
    // boundary sets *consistent = false and leaves the cell untouched.
    __device__ int apply(Wave<uint64_t>& R, bool any, bool all, float ax, float ay, float az, float b, float sbh,
                         int32_t hcode, bool* consistent) {
        *consistent = true;
        if (!any) return kNone;
        if (all) return kEmptied;
        if (np >= CAP) {
            gc();
            if (np >= CAP) return kOverflow;
        }
        if constexpr (VPL > 1) {
#pragma unroll
            for (int s = 0; s < VPL; ++s)
                M.outf[s * 64 + ln] = (uint8_t)((R[s] >> ln) & 1);
            sync();
        }
        auto is_out = [&](uint32_t v) -> bool {
            if constexpr (VPL == 1) return (R[0] >> v) & 1;
            else return M.outf[v] != 0;
        };
        Lane<uint32_t> cross, pre, frank, nb1, nb2;
        Lane<W> rec;
        Lane<uint8_t> isnew;
        Wave<uint64_t> fr;
        // crossing edges of kept vertices, ranked over the wave
        uint32_t m = 0;
#pragma unroll
        for (int s = 0; s < VPL; ++s) {
            bool kept = ((alive[s] & ~R[s]) >> ln) & 1;
            uint32_t c = 0, cnt = 0;
            if (kept) {
                const W nbr = va[s];
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if (is_out(T::fld(nbr, e))) {
                        c |= 1u << e;
                        ++cnt;
                    }
            }
            cross[s] = c;
            uint64_t b0 = ballot(cnt & 1), b1 = ballot(cnt & 2);
            pre[s] = m + mbcnt(b0) + 2 * mbcnt(b1);
            m += popc(b0) + 2 * popc(b1);
        }
        // free slots (dead or removed), ranked
        uint32_t nfree = 0;
#pragma unroll
        for (int s = 0; s < VPL; ++s) {
            const uint64_t f = ~alive[s] | R[s];
            fr[s] = f;
            frank[s] = nfree + mbcnt(f);
            nfree += popc(f);
        }
        if (m == 0) {  // some vertex is cut off but no edge crosses the plane
            *consistent = false;
            return kNone;
        }
        if (m > nfree) return kOverflow;
        const uint32_t h = (uint32_t)np;
        ++serial;
        if (serial >= T::kTagMax) {  // tag space exhausted: clear the tables
            for (int q = (int)ln; q < CAP; q += 64) { M.ta[q] = 0; M.tb[q] = 0; }
            serial = 1;
        }
        const uint32_t tag = serial << T::kTagShift;
        const uint32_t vmask = (1u << T::kTagShift) - 1u;
#pragma unroll
        for (int s = 0; s < VPL; ++s) {
            const uint32_t rk = frank[s];
            const bool nw = ((fr[s] >> ln) & 1) && rk < m;
            isnew[s] = nw;
            if (nw) M.sor[rk] = s * 64 + ln;
        }
#pragma unroll
        for (int s = 0; s < VPL; ++s) {
            const uint32_t c = cross[s];
            if (c) {
                uint32_t j = pre[s];
                const W t = vt[s];
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if ((c >> e) & 1) {
                        uint32_t x = T::fld(t, (e + 2) % 3), y = T::fld(t, (e + 1) % 3);
                        M.edge[j++] = T::pack3((uint32_t)(s * 64 + ln), x, y);
                    }
            }
        }
        sync();
#pragma unroll
        for (int s = 0; s < VPL; ++s) {
            W r = 0;
            if (isnew[s]) {
                r = M.edge[frank[s]];
                uint32_t me = tag | (uint32_t)(s * 64 + ln);
                M.ta[T::fld(r, 1)] = me;
                M.tb[T::fld(r, 2)] = me;
            }
            rec[s] = r;
        }
        sync();
        bool bad = false;
#pragma unroll
        for (int s = 0; s < VPL; ++s) {
            uint32_t n1 = 0, n2 = 0;
            if (isnew[s]) {
                const W r = rec[s];
                uint32_t me = tag | (uint32_t)(s * 64 + ln);
                uint32_t x = T::fld(r, 1), y = T::fld(r, 2);
                uint32_t a1 = M.ta[y], a2 = M.tb[x];
                bad |= M.ta[x] != me || M.tb[y] != me;
                bad |= (a1 & ~vmask) != tag || (a2 & ~vmask) != tag;
                n1 = a1 & vmask;
                n2 = a2 & vmask;
            }
            nb1[s] = n1;
            nb2[s] = n2;
        }
        bad = ballot(bad) != 0;
        if (!bad) {
            // the new vertices must form one cycle around the new facet:
            // following "next around h" from the first one returns after m steps
            const uint32_t start = uni(M.sor[0]);
            uint32_t v = start, steps = 0;
            do {
                const int sl = (int)(v >> 6), lv = (int)(v & 63);
                uint32_t nxt = 0xFFFFFFFFu;
#pragma unroll
                for (int s = 0; s < VPL; ++s) {
                    const uint32_t n1 = rdl(nb1[s], lv);
                    nxt = s == sl ? n1 : nxt;
                }
                v = nxt;
                ++steps;
            } while (v != start && steps <= m);
            bad = steps != m;
        }
        if (ballot(bad)) {
            *consistent = false;
            return kNone;
        }
        // commit: kept vertices point at their new neighbours
#pragma unroll
        for (int s = 0; s < VPL; ++s) {
            const uint32_t c = cross[s];
            if (c) {
                uint32_t j = pre[s];
                W a = va[s];
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if ((c >> e) & 1) a = T::setfld(a, e, M.sor[j++]);
                va[s] = a;
            }
        }
        // new vertices: planes (h, x, y), position by Cramer's rule
#pragma unroll
        for (int s = 0; s < VPL; ++s) {
            if (isnew[s]) {
                const W r = rec[s];
                uint32_t x = T::fld(r, 1), y = T::fld(r, 2);
                vt[s] = T::pack3(h, x, y);
                va[s] = T::pack3(T::fld(r, 0), nb1[s], nb2[s]);
                float q0, q1, q2, e = 0.f;
                solve(x, y, ax, ay, az, b, sbh, &q0, &q1, &q2, &e);
                y0[s] = q0;
                y1[s] = q1;
                y2[s] = q2;
                if (robust != 0) ev[s] = e;
            }
        }
#pragma unroll
        for (int s = 0; s < VPL; ++s) {
            const uint64_t keep = alive[s] & ~R[s];
            alive[s] = keep | ballot(isnew[s] != 0);
        }
        if (ln == 0) {
            M.pl[h] = make_float4(ax, ay, az, b);
            M.psb[h] = sbh;
            M.pcode[h] = hcode;
            M.psite[h] = A.pts[hcode];
        }
        np = (int)h + 1;
        sync();
        count(kCtrNewVertex, m);
        count(kCtrEffective, 1);
        return kChanged;
    }

    // apply() of the memory tiers.  A chain of LDS round trips, barriers and
    // short dependent sequences (one wave a SIMD), so what counts is their
    // number: every wave sums the counts of all slots by itself, finds the
    // crossing edges and free slots of its own slots and puts them into lists
    // by rank (two barriers); up to 64 new vertices every wave then works out
    // all of them, one a lane, with no exchange, and the first wave writes
    // them.  It had a barrier for each of outside flags, counts, lists, tables,
    // links and the result, followed the links one memory read at a time, kept
    // its tables in the arena in the 16384-vertex tier, and held every mask in
    // vector registers since nothing told the compiler that what waves
    // exchange is uniform.  Time of the passes, with the slots in registers
    // and the candidates tested two at a time: 1024 vertices 9.9 -> 7 ms (351
    // cells of 1M power cells), 16384 vertices 9.0 -> 4.6 ms (one cell of 1452
    // vertices).
    __device__ int apply_group(Wave<uint64_t>& R, bool any, bool all, float ax, float ay, float az, float b, float sbh,
                               int32_t hcode, bool* consistent) {
        *consistent = true;
        if (!any) return kNone;
        if (all) return kEmptied;
        if (np >= CAP) {
            gc();
            if (np >= CAP) return kOverflow;
        }
        const int ns = nsv();
        auto is_out = [&](uint32_t v) -> bool { return (H.R[v >> 6] >> (v & 63u)) & 1ull; };
        uint32_t cr[kC];  // crossing edges of the vertex (low 3 bits) and their rank in the slot
#pragma unroll
        for (int i = 0; i < kC; ++i) cr[i] = 0;
        VD_EACH_SLOT({
            const uint64_t r = uni(R[s_]);
            uint32_t c = 0, cnt = 0;
            if (((al_ & ~r) >> ln) & 1) {
                const W nbr = va[s_];
_Pragma("unroll")
                for (int e = 0; e < 3; ++e)
                    if (is_out(T::fld(nbr, e))) {
                        c |= 1u << e;
                        ++cnt;
                    }
            }
            const uint64_t b0 = ballot(cnt & 1), b1 = ballot(cnt & 2);
            c |= (mbcnt(b0) + 2 * mbcnt(b1)) << 3;
            if (i_ < kC) cr[i_ < kC ? i_ : 0] = c;
            else M.cross[s_ * 64 + ln] = c;
            const bool edge_of = x_ == blo0 || x_ == bhi0 || y_ == blo1 || y_ == bhi1 || z_ == blo2 || z_ == bhi2;
            H.cnt[s_] = (uint32_t)(popc(b0) + 2 * popc(b1)) | ((uint32_t)popc(~al_ | r) << 16) |
                       ((ballot(edge_of) & r) != 0 ? 1u << 31 : 0u);
        });
        sync();
        // sums over the slots, the same in every wave: crossing edges in the
        // low 16 bits (at most three a vertex), free places above
        uint32_t below64 = 0, total = 0;
        {
            uint32_t w = ln < (uint32_t)ns ? H.cnt[ln] : 0u;
            bnd = ballot(w >> 31) != 0;
            w &= ~(1u << 31);
            const uint32_t sum = wscan_u(w);
            below64 = sum - w;
            total = rdl(sum, 63);
            if constexpr (VPL > 64) {
                for (int s0 = 64; s0 < ns; s0 += 64) {
                    w = s0 + (int)ln < ns ? H.cnt[s0 + ln] : 0u;
                    bnd |= ballot(w >> 31) != 0;
                    w &= ~(1u << 31);
                    const uint32_t x = wscan_u(w) + total;
                    if (s0 + (int)ln < ns) H.pre[s0 + ln] = x - w;
                    total = rdl(x, 63);
                }
                if (ln < (uint32_t)ns) H.pre[ln] = below64;
                wave_sync<true>();
            }
        }
        auto below_slot = [&](int i, int s) -> uint32_t {
            if constexpr (VPL > 64) {
                if (i == kC) return uni(H.pre[s]);
            }
            return rdl(below64, s);
        };
        const uint32_t m = total & 0xFFFFu, used_free = total >> 16;  // used_free: free places in the slots in use
        if (m == 0) {  // some vertex is cut off but no edge crosses the plane
            *consistent = false;
            return kNone;
        }
        // slots above the used ones are free
        if (m > used_free + 64u * (uint32_t)(VPL - ns)) return kOverflow;
        const uint32_t h = (uint32_t)np;
        ++serial;
        if (serial >= T::kTagMax) {  // tag space exhausted: clear the tables
            for (int q = (int)(wid * 64 + ln); q < CAP; q += 64 * G) { H.ta[q] = 0; H.tb[q] = 0; }
            serial = 1;
        }
        const uint32_t tag = serial << T::kTagShift;
        const uint32_t vmask = (1u << T::kTagShift) - 1u;
        // lists by rank: the first in LDS
        auto sor = [&](uint32_t r) -> uint32_t& {
            if constexpr (CAP > kHotRanks) {
                if (r >= (uint32_t)kHotRanks) return M.sor[r];
            }
            return H.sor[r];
        };
        auto edge = [&](uint32_t r) -> W& {
            if constexpr (CAP > kHotRanks) {
                if (r >= (uint32_t)kHotRanks) return M.edge[r];
            }
            return H.edge[r];
        };
        auto place = [&](uint32_t r) -> uint32_t {  // the vertex of rank r
            return r < used_free ? sor(r) : (uint32_t)ns * 64u + (r - used_free);
        };
        VD_EACH_SLOT({
            const uint32_t below = below_slot(i_, s_), fb = below >> 16;
            const uint32_t c = i_ < kC ? cr[i_ < kC ? i_ : 0] : M.cross[s_ * 64 + ln];
            if (c & 7u) {
                uint32_t j = (below & 0xFFFFu) + (c >> 3);
                const W t = vt[s_];
_Pragma("unroll")
                for (int e = 0; e < 3; ++e)
                    if ((c >> e) & 1) {
                        const uint32_t x = T::fld(t, (e + 2) % 3), y = T::fld(t, (e + 1) % 3);
                        edge(j++) = T::pack3((uint32_t)(s_ * 64 + ln), x, y);
                    }
            }
            if (fb < m) {
                const uint64_t f = ~al_ | uni(R[s_]);
                const uint32_t rk = fb + mbcnt(f);
                if (((f >> ln) & 1) && rk < m) sor(rk) = (uint32_t)(s_ * 64 + ln);
            }
        });
        sync();
        // the vertex of rank r: links to the next and the previous around h
        auto links = [&](uint32_t r, W rec, uint32_t* n1, uint32_t* n2) -> bool {
            const uint32_t me = tag | r, x = T::fld(rec, 1), y = T::fld(rec, 2);
            const uint32_t a1 = H.ta[y], a2 = H.tb[x];
            *n1 = a1 & vmask;
            *n2 = a2 & vmask;
            return H.ta[x] == me && H.tb[y] == me && (a1 & ~vmask) == tag && (a2 & ~vmask) == tag;
        };
        auto put = [&](uint32_t r, W rec, uint32_t n1, uint32_t n2, float q0, float q1, float q2, float e) {
            const uint32_t v = place(r);
            M.vt[v] = T::pack3(h, T::fld(rec, 1), T::fld(rec, 2));
            M.va[v] = T::pack3(T::fld(rec, 0), place(n1), place(n2));
            M.y0[v] = q0;
            M.y1[v] = q1;
            M.y2[v] = q2;
            if (robust != 0) M.ev[v] = e;
        };
        if (m <= 64u) {
            // every wave writes the same words into the tables
            const bool nw = ln < m;
            W rec = 0;
            uint32_t n1 = 0, n2 = 0;
            bool bad = false;
            if (nw) {
                rec = edge(ln);
                H.ta[T::fld(rec, 1)] = tag | ln;
                H.tb[T::fld(rec, 2)] = tag | ln;
            }
            wave_sync<true>();
            if (nw) {
                bad = !links(ln, rec, &n1, &n2);
                // inverse permutations without fixed points: one cycle up to
                // five unless two point at each other (above two)
                bad |= m >= 4u && n1 == n2;
            }
            bad = ballot(bad) != 0;
            if (!bad && m >= 6u) {
                uint32_t v = 0, steps = 0;
                do {
                    v = rdl(n1, (int)v);
                    ++steps;
                } while (v != 0u && steps <= m);
                bad = steps != m;
            }
            if (bad) {
                *consistent = false;
                return kNone;
            }
            float q0 = 0.f, q1 = 0.f, q2 = 0.f, e = 0.f;
            bool beyond = false;
            if (nw) {
                solve(T::fld(rec, 1), T::fld(rec, 2), ax, ay, az, b, sbh, &q0, &q1, &q2, &e);
                beyond = q0 < blo0 || q0 > bhi0 || q1 < blo1 || q1 > bhi1 || q2 < blo2 || q2 > bhi2;
                if (lead()) put(ln, rec, n1, n2, q0, q1, q2, e);
            }
            bnd |= ballot(beyond) != 0;
        } else {
            bnd = true;
            const uint32_t step = 64u * G;
            for (uint32_t r = wid * 64u + ln; r < m; r += step) {
                const W rec = edge(r);
                H.ta[T::fld(rec, 1)] = tag | r;
                H.tb[T::fld(rec, 2)] = tag | r;
            }
            sync();
            bool bad = false;
            for (uint32_t r = wid * 64u + ln; r < m; r += step) {
                uint32_t n1, n2;
                bad |= !links(r, edge(r), &n1, &n2);
                M.nb1[r] = n1;
                M.nb2[r] = n2;
            }
            bad = g_or<1>(ballot(bad) != 0 ? 1u : 0u) != 0;
            if (!bad) {
                uint32_t v = 0, steps = 0;
                do {
                    v = uni(M.nb1[v]);
                    ++steps;
                } while (v != 0u && steps <= m);
                bad = steps != m;
            }
            if (bad) {
                *consistent = false;
                return kNone;
            }
            for (uint32_t r = wid * 64u + ln; r < m; r += step) {
                const W rec = edge(r);
                float q0, q1, q2, e = 0.f;
                solve(T::fld(rec, 1), T::fld(rec, 2), ax, ay, az, b, sbh, &q0, &q1, &q2, &e);
                put(r, rec, M.nb1[r], M.nb2[r], q0, q1, q2, e);
            }
        }
        // free places are taken in increasing order: the last rank's is the highest
        const int top = (int)uni(place(m - 1u)) + 1;
        if (top > vhi) vhi = top;
        // kept vertices point at their new neighbours; the masks; returns
        // the places of this slot that new vertices take
        auto commit = [&](int i, int s, uint64_t al, uint64_t* now) -> uint64_t {
            if (s >= ns) {  // a slot above those in use
                const uint32_t left = m - used_free - 64u * (uint32_t)(s - ns);
                *now = left >= 64u ? ~0ull : (1ull << left) - 1ull;
                alive[s] = *now;
                return *now;
            }
            const uint32_t below = below_slot(i, s), fb = below >> 16;
            const uint32_t c = i < kC ? cr[i < kC ? i : 0] : M.cross[s * 64 + ln];
            if (c & 7u) {
                uint32_t j = (below & 0xFFFFu) + (c >> 3);
                W nb = va[s];
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if ((c >> e) & 1) nb = T::setfld(nb, e, place(j++));
                va[s] = nb;
            }
            const uint64_t r = uni(R[s]), f = ~al | r;
            uint64_t fresh = 0;
            if (fb < m) fresh = ballot(fb + mbcnt(f) < m) & f;
            *now = (al & ~r) | fresh;
            alive[s] = *now;
            return fresh;
        };
        const int ns2 = nsv();
        uint64_t fresh[kC];
#pragma unroll
        for (int i = 0; i < kC; ++i) {
            const int s = (int)wid + G * i;
            fresh[i] = 0;
            if (s < ns2) fresh[i] = commit(i, s, cal[i], &cal[i]);
        }
        if constexpr (VPL > G * kC) {
            for (int s = (int)wid + G * kC; s < ns2; s += G) {
                uint64_t now;
                commit(kC, s, s < ns ? uni(alive[s]) : 0ull, &now);
            }
        }
        if (ln == 0 && lead()) {
            M.pl[h] = make_float4(ax, ay, az, b);
            M.psb[h] = sbh;
            M.pcode[h] = hcode;
        }
        np = (int)h + 1;
        sync();
#pragma unroll
        for (int i = 0; i < kC; ++i)
            if (fresh[i]) load_slot(i, (int)wid + G * i);
        count(kCtrNewVertex, m);
        count(kCtrEffective, 1);
        return kChanged;
    }

    __device__ int cut(Wave<uint64_t>& R, bool any, bool all, float ax, float ay, float az, float b, float sbh,
                       int32_t hcode, bool* consistent) {
        if constexpr (G > 1) return apply_group(R, any, all, ax, ay, az, b, sbh, hcode, consistent);
        else return apply(R, any, all, ax, ay, az, b, sbh, hcode, consistent);
    }

    // Plain FP32 signs unless the cell is being rebuilt robustly; an
    // inconsistent boundary in FP32 asks for that rebuild; in the robust modes
    // doubtful signs fall back to "inside" and, failing that, the plane is
    // skipped and the cell flagged.
    __device__ int clip(float ax, float ay, float az, float b, float sbh, int32_t hcode) {
        Wave<uint64_t> R;
        if constexpr (!kReg) R.m = H.R;
        count(kCtrClip, 1);
        bool any, all;
        classify(ax, ay, az, b, sbh, hcode, robust == 0 ? 0 : (robust == 1 ? 1 : 3), R, &any, &all);
        bool ok;
        int r = cut(R, any, all, ax, ay, az, b, sbh, hcode, &ok);
        if constexpr (VPL == 1 && G == 1) cut_mask = R[0];
        if (ok) return r;
        if (robust < 2) return kRestart;
        flags |= kFlagUncertain;
        classify(ax, ay, az, b, sbh, hcode, 2, R, &any, &all);
        r = cut(R, any, all, ax, ay, az, b, sbh, hcode, &ok);
        if constexpr (VPL == 1 && G == 1) cut_mask = R[0];
        return ok ? r : kNone;
    }

    // Drop planes no vertex uses (supplementary Sec. A, "Garbage collection").
    __device__ void gc() {
        const int ns = nsv();
        for (int q = (int)(wid * 64 + ln); q < np; q += 64 * G) M.key[q] = 0;
        sync();
#pragma unroll
        for (int s = kReg ? 0 : (int)wid; s < (kReg ? VPL : ns); s += G)
            if ((alive[s] >> ln) & 1) {
                const W t = vt[s];
                M.key[T::fld(t, 0)] = 1;
                M.key[T::fld(t, 1)] = 1;
                M.key[T::fld(t, 2)] = 1;
            }
        sync();
        uint32_t cnt = 0;
        if constexpr (kReg) {
            float4 pl[VPL], ps[VPL];
            float sb[VPL];
            int32_t pc[VPL];
            uint32_t dst[VPL];
            bool used[VPL];
#pragma unroll
            for (int s = 0; s < VPL; ++s) {
                int q = s * 64 + ln;
                used[s] = q < np && M.key[q] != 0;
                uint64_t u = ballot(used[s]);
                dst[s] = cnt + mbcnt(u);
                cnt += popc(u);
                if (used[s]) {
                    pl[s] = M.pl[q];
                    ps[s] = M.psite[q];
                    sb[s] = M.psb[q];
                    pc[s] = M.pcode[q];
                }
            }
            sync();
#pragma unroll
            for (int s = 0; s < VPL; ++s) {
                int q = s * 64 + ln;
                if (used[s]) {
                    M.pl[dst[s]] = pl[s];
                    M.psite[dst[s]] = ps[s];
                    M.psb[dst[s]] = sb[s];
                    M.pcode[dst[s]] = pc[s];
                    M.key[q] = (int32_t)dst[s];
                }
            }
        } else {
            // in place, 64 planes at a time, by the first wave of the group:
            // a destination never lies above its source, and every source of
            // a chunk is read before any of its destinations is written
            for (int q0 = 0; q0 < (lead() ? np : 0); q0 += 64) {
                const int q = q0 + (int)ln;
                const bool used = q < np && M.key[q] != 0;
                const uint64_t u = ballot(used);
                const uint32_t dst = cnt + mbcnt(u);
                cnt += popc(u);
                float4 pl = make_float4(0.f, 0.f, 0.f, 0.f);
                float sb = 0.f;
                int32_t pc = 0;
                if (used) {
                    pl = M.pl[q];
                    sb = M.psb[q];
                    pc = M.pcode[q];
                }
                wsync();
                if (used) {
                    M.pl[dst] = pl;
                    M.psb[dst] = sb;
                    M.pcode[dst] = pc;
                    M.key[q] = (int32_t)dst;
                }
                wsync();
            }
            if constexpr (G > 1) cnt = bcast(cnt);
        }
        sync();
#pragma unroll
        for (int s = kReg ? 0 : (int)wid; s < (kReg ? VPL : ns); s += G)
            if ((alive[s] >> ln) & 1) {
                const W t = vt[s];
                vt[s] = T::pack3((uint32_t)M.key[T::fld(t, 0)], (uint32_t)M.key[T::fld(t, 1)],
                                 (uint32_t)M.key[T::fld(t, 2)]);
            }
        np = (int)cnt;
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
        const float lbs = least_plane(d, dw, culling() == 3, [&] {
            const float fx = pmax(fabsf(blx), fabsf(bhx)), fy = pmax(fabsf(bly), fabsf(bhy)),
                        fz = pmax(fabsf(blz), fabsf(bhz));
            return __builtin_amdgcn_sqrtf(fmaf(fx, fx, fmaf(fy, fy, fz * fz)));
        });
        float rb2;
        if (culling() == 2) {
            rb2 = riso2;
        } else {
            // per axis: the far-corner square of each side the box reaches
            const float tx = pmax(bhx >= 0.f ? hx2 : 0.f, blx < 0.f ? lx2 : 0.f);
            const float ty = pmax(bhy >= 0.f ? hy2 : 0.f, bly < 0.f ? ly2 : 0.f);
            const float tz = pmax(bhz >= 0.f ? hz2 : 0.f, blz < 0.f ? lz2 : 0.f);
            rb2 = tx + ty + tz;
        }
        float rb = __builtin_amdgcn_sqrtf(rb2);
        *key = lbs;
        *cull = lbs > rb * (1.f + 16.f * kU);
        *delta = lbs - rb;
    }

    __device__ void push(uint32_t e, float k) {
        const int slot = qn >> 6, l = qn & 63;
        if constexpr (kQExt) {
            if (slot >= VPL) {
                if (ln == 0) {
                    M.qxe[(slot - VPL) * 64 + l] = e;
                    M.qxk[(slot - VPL) * 64 + l] = k;
                }
                wsync();  // read back by every lane
                ++qn;
                return;
            }
        }
        if constexpr (kReg) {
#pragma unroll
            for (int s = 0; s < VPL; ++s) {
                const bool here = s == slot && (int)ln == l;
                qe[s] = here ? e : qe[s];
                qk[s] = here ? k : qk[s];
            }
        } else {
            if ((int)ln == l && lead()) {
                qe[slot] = e;
                qk[slot] = k;
            }
        }
        ++qn;
    }

    // Removes and returns the entry with the smallest key (best-first), or
    // the last pushed one (depth-first).  The queue is kept by the first wave
    // of a group, which hands the entry to the others.
    __device__ void pop(uint32_t* e, float* k, bool least = false) {
        uint32_t ee = 0;
        float kk = 0.f;
        if (lead()) pop_lead(&ee, &kk, least || traversal() != 2);
        if constexpr (G > 1) {
            const uint32_t v[2] = {ee, __float_as_uint(kk)};
            const uint32_t* t = exch(v);
            ee = uni(t[0]);
            kk = __uint_as_float(uni(t[1]));
        }
        --qn;
        *e = ee;
        *k = kk;
    }
    __device__ void pop_lead(uint32_t* e, float* k, bool least) {
        const int nq = (qn + 63) >> 6;
        int S, L;
        if (!least) {
            S = (qn - 1) >> 6;
            L = (qn - 1) & 63;
        } else {
            float bk = INFINITY;
            int bs = 0;
            if constexpr (!kReg) {
                for (int s = 0; s < nq; s += 4) {  // four loads at a time (VPL is a multiple of four)
                    float kk[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) kk[k] = qk[s + k];
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if ((s + k) * 64 + (int)ln < qn && kk[k] < bk) {
                            bk = kk[k];
                            bs = s + k;
                        }
                }
            }
#pragma unroll
            for (int s = 0; s < (kReg ? VPL : 0); ++s) {
                int idx = s * 64 + (int)ln;
                if (idx < qn) {
                    const float kk = qk[s];
                    if (kk < bk) {
                        bk = kk;
                        bs = s;
                    }
                }
            }
            if constexpr (kQExt) {
                for (int s = VPL; s < (qn + 63) >> 6; ++s) {
                    const int idx = s * 64 + (int)ln;
                    if (idx < qn) {
                        const float kk = M.qxk[idx - 64 * VPL];
                        if (kk < bk) {
                            bk = kk;
                            bs = s;
                        }
                    }
                }
            }
            float m = wmin(bk);
            uint64_t msk = ballot(bk == m && (int)ln < qn);
            L = msk ? lowest(msk) : 0;
            S = rdl(bs, L);
        }
        uint32_t ee = 0, le = 0;
        float kk = 0.f, lk = 0.f;
        const int last = qn - 1, ls = last >> 6, ll = last & 63;
        if constexpr (kQExt) {
            if (ls >= VPL) {  // the last entry is beyond the register slots (LDS)
                if (S < VPL) {
#pragma unroll
                    for (int s = 0; s < VPL; ++s) {
                        const uint32_t e1 = rdl(qe[s], L);
                        const float k1 = rdl(qk[s], L);
                        ee = s == S ? e1 : ee;
                        kk = s == S ? k1 : kk;
                    }
                } else {
                    ee = uni(M.qxe[(S - VPL) * 64 + L]);
                    kk = uni(M.qxk[(S - VPL) * 64 + L]);
                }
                le = uni(M.qxe[last - 64 * VPL]);
                lk = uni(M.qxk[last - 64 * VPL]);
                if (S < VPL) {
#pragma unroll
                    for (int s = 0; s < VPL; ++s) {
                        const bool here = s == S && (int)ln == L;
                        qe[s] = here ? le : qe[s];
                        qk[s] = here ? lk : qk[s];
                    }
                } else {
                    if (ln == 0) {
                        M.qxe[(S - VPL) * 64 + L] = le;
                        M.qxk[(S - VPL) * 64 + L] = lk;
                    }
                    wsync();
                }
                *e = ee;
                *k = kk;
                return;
            }
        }
        if constexpr (kReg) {
#pragma unroll
            for (int s = 0; s < VPL; ++s) {
                const uint32_t e1 = rdl(qe[s], L), e2 = rdl(qe[s], ll);
                const float k1 = rdl(qk[s], L), k2 = rdl(qk[s], ll);
                ee = s == S ? e1 : ee;
                kk = s == S ? k1 : kk;
                le = s == ls ? e2 : le;
                lk = s == ls ? k2 : lk;
            }
#pragma unroll
            for (int s = 0; s < VPL; ++s) {
                const bool here = s == S && (int)ln == L;
                qe[s] = here ? le : qe[s];
                qk[s] = here ? lk : qk[s];
            }
        } else {
            ee = rdl(qe[S], L);
            kk = rdl(qk[S], L);
            le = rdl(qe[ls], ll);
            lk = rdl(qk[ls], ll);
            if ((int)ln == L) {
                qe[S] = le;
                qk[S] = lk;
            }
        }
        *e = ee;
        *k = kk;
    }

    // The candidates of `mask` (plane of lane L: a, b, size sb) that have
    // some vertex of the cell outside, or, when doubtful signs are
    // re-evaluated, within rounding of it.  The others are left out: one pass
    // over the vertices for the whole leaf (and for a wave group one exchange)
    // instead of a selection and a clip each.  The test is the FP32 side test
    // of classify.  Exactly, a plane that misses the cell misses every cell it
    // is later clipped to; in FP32 a vertex made by a later clip of this leaf
    // can come out beyond such a plane by its rounding, so this rule decides
    // some cells' signs at that level (those of the passes above 64 vertices:
    // the results of a build depend on it there, and it is the same in all).
    __device__ uint64_t cutting(uint64_t mask, float ax, float ay, float az, float b, float sb) {
        if constexpr (kCount) count(kCtrClassify, nalive() * (uint64_t)popc(mask));
        uint64_t cut = 0;  // candidates that put a vertex of this wave outside
        for (uint64_t m = mask; m;) {  // two candidates at a time
            const int L0 = lowest(m);
            m &= m - 1;
            const int L1 = m ? lowest(m) : L0;
            m &= m - 1;
            const float p0 = rdl(ax, L0), p1 = rdl(ay, L0), p2 = rdl(az, L0), pb = rdl(b, L0);
            const float q0 = rdl(ax, L1), q1 = rdl(ay, L1), q2 = rdl(az, L1), qb = rdl(b, L1);
            uint64_t o0 = 0, o1 = 0;
            if (robust == 0) {
                VD_EACH_SLOT({
                    o0 |= ballot(fmaf(p0, x_, fmaf(p1, y_, fmaf(p2, z_, -pb))) > 0.f) & al_;
                    o1 |= ballot(fmaf(q0, x_, fmaf(q1, y_, fmaf(q2, z_, -qb))) > 0.f) & al_;
                });
            } else {
                const float pn = fabsf(p0) + fabsf(p1) + fabsf(p2), ps = rdl(sb, L0);
                const float qn1 = fabsf(q0) + fabsf(q1) + fabsf(q2), qs = rdl(sb, L1);
                VD_EACH_SLOT({
                    const float e = ev[s_];
                    o0 |= ballot(fmaf(p0, x_, fmaf(p1, y_, fmaf(p2, z_, -pb))) >= -doubt(pn, e, ps)) & al_;
                    o1 |= ballot(fmaf(q0, x_, fmaf(q1, y_, fmaf(q2, z_, -qb))) >= -doubt(qn1, e, qs)) & al_;
                });
            }
            cut |= (o0 != 0 ? 1ull << L0 : 0ull) | (o1 != 0 ? 1ull << L1 : 0ull);
        }
        if constexpr (G > 1) {
            const uint32_t v2[2] = {(uint32_t)cut, (uint32_t)(cut >> 32)};
            const uint32_t* t = exch(v2);
            uint32_t lo = 0, hi = 0;
#pragma unroll
            for (int w = 0; w < G; ++w) {
                lo |= t[w * 8];
                hi |= t[w * 8 + 1];
            }
            cut = (uint64_t)uni(lo) | ((uint64_t)uni(hi) << 32);
        }
        return mask & cut;
    }

    // Clips by the candidate sites of one leaf (those of lanes in `allow`);
    // nearest plane first.
    __device__ int leaf(uint32_t ref, uint64_t allow) {
        const uint32_t first = leaf_first(ref), nsite = leaf_count(ref);
        count(kCtrLeaf, 1);
        count(kCtrSite, nsite);
        float ax = 0.f, ay = 0.f, az = 0.f, a2 = 0.f, b = 0.f, dw = 0.f, key = INFINITY;
        float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
        bool cand = false;
        {
            // every lane loads (lanes past the leaf repeat its last site) so
            // that the arithmetic runs without a divergent branch
            const uint32_t j = first + ((uint32_t)ln < nsite ? (uint32_t)ln : nsite - 1u);
            q = A.pts[j];
            ax = q.x - px; ay = q.y - py; az = q.z - pz;
            a2 = fmaf(ax, ax, fmaf(ay, ay, az * az));
            dw = kW ? pw - q.w : 0.f;
            b = 0.5f * (a2 + dw);
            cand = (uint32_t)ln < nsite && j != self && q.w != -INFINITY && a2 > 0.f;
            for (int t = 0; t < nwarm; ++t) cand = cand && j != rdl(wsite, t);
            key = cand ? b * __builtin_amdgcn_rsqf(a2) : INFINITY;  // orders candidates only
        }
        const float sbl = 0.5f * (a2 + fabsf(dw));  // size of the terms of b (error scale)
        auto keep = [&](bool c) -> bool {
            if (!c) return false;
            if (culling() == 3) {
                // the plane misses the cell's AABB: max over the box of a.y <= b
                float cx = ax >= 0.f ? bhi0 : blo0, cy = ay >= 0.f ? bhi1 : blo1, cz = az >= 0.f ? bhi2 : blo2;
                return reaches(ax, ay, az, b, cx, cy, cz, a2, dw);
            }
            float r2 = radius2_toward(ax, ay, az);
            float t = b - 4.f * kU * (2.f * a2 + fabsf(dw) + r2);
            return !(t > 0.f && t * t > a2 * r2);
        };
        uint64_t mask = ballot(keep(cand));
        if constexpr (kResumes) mask &= allow;
        // from 128 vertices up, the candidates that miss the cell are dropped
        // all at once (not when every sign is taken in FP64)
        if constexpr (G > 1 || VPL >= 2) {
            if (mask && robust < 2) mask = cutting(mask, ax, ay, az, b, sbl);
        }
        while (mask) {
            // nearest plane first (both traversal orders)
            int L;
            {
                float kk = ((mask >> ln) & 1) ? key : INFINITY;
                float m = wmin(kk);
                uint64_t mm = ballot(kk == m) & mask;
                L = lowest(mm ? mm : mask);
            }
            mask &= ~(1ull << L);
            float hx = rdl(ax, L), hy = rdl(ay, L), hz = rdl(az, L), hb = rdl(b, L);
            const float sb = rdl(sbl, L);
            const uint64_t t0 = tic();
            int r = clip(hx, hy, hz, hb, sb, (int32_t)(first + (uint32_t)L));
            toc(kCtrCycClip, t0);
            if constexpr (kSaves) {
                if (r == kOverflow) {  // the cell is as before this candidate
                    ov_ok = true;
                    ov_leaf = ref;
                    ov_mask = mask | (1ull << L);
                    ov_phase = leaf_phase;
                }
            }
            if (r == kEmptied || r == kOverflow || r == kRestart) return r;
            if (r == kChanged) {
                bounds_after_clip();
                mask &= ballot(keep(true));
                // (the candidates left are not tested again: a new vertex can
                // come out, by its rounding, on the far side of a plane that
                // passes close to the cell, or in doubt of it, where no vertex
                // was before, and what is decided of it then has to stay)
            }
        }
        return kNone;
    }

    __device__ void load_child(uint32_t node, int s, NodeChild* c) const {
        const float4* src = reinterpret_cast<const float4*>(&A.nodes[node].c[s]);
        float4 u = src[0], v = src[1];
        c->lo[0] = u.x; c->lo[1] = u.y; c->lo[2] = u.z; c->wmax = u.w;
        c->hi[0] = v.x; c->hi[1] = v.y; c->hi[2] = v.z; c->ref = __float_as_uint(v.w);
    }

    // KNN warm start (supplementary Sec. A): before the walk, the K sites
    // nearest to p_i are found by a best-first walk of the same BVH (queue
    // keyed by squared distance to the child boxes), and the cell is clipped
    // by their planes, nearest first.  Lanes 0..K-1 keep the K best squared
    // distances (best) and sites (bsite); `worst` is the K-th best (infinite
    // until K are found).  The walk that follows passes over these sites.
    // Returns kNone or what a clip returned (kEmptied, kOverflow, kRestart).
    __device__ int knn_warm(int K) {
        float best = INFINITY;
        uint32_t bsite = 0u;
        float worst = INFINITY;
        qn = 0;
        auto box_d2 = [&](const NodeChild& c) {
            const float dx = fmaxf(fmaxf(c.lo[0] - px, px - c.hi[0]), 0.f);
            const float dy = fmaxf(fmaxf(c.lo[1] - py, py - c.hi[1]), 0.f);
            const float dz = fmaxf(fmaxf(c.lo[2] - pz, pz - c.hi[2]), 0.f);
            return fmaf(dx, dx, fmaf(dy, dy, dz * dz));
        };
        auto take_leaf = [&](uint32_t ref) {
            const uint32_t first = leaf_first(ref), cnt = leaf_count(ref);
            const uint32_t j = first + ((uint32_t)ln < cnt ? (uint32_t)ln : cnt - 1u);
            const float4 q = A.pts[j];
            const float dx = q.x - px, dy = q.y - py, dz = q.z - pz;
            const float d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
            const bool ok = (uint32_t)ln < cnt && j != self && q.w != -INFINITY && d2 > 0.f;
            count(kCtrSite, cnt);
            uint64_t m = ballot(ok && d2 < worst);
            while (m) {
                const float c = wmin(((m >> ln) & 1) ? d2 : INFINITY);
                if (!(c < worst)) break;
                const uint64_t mm = ballot(((m >> ln) & 1) && d2 == c) & m;
                const int L = lowest(mm);
                m &= ~(1ull << L);
                const uint32_t js = rdl(j, L);
                // it replaces the worst of the K kept
                const float wv = wmax((int)ln < K ? best : -INFINITY);
                const int W = lowest(ballot((int)ln < K && best == wv));
                if ((int)ln == W) {
                    best = c;
                    bsite = js;
                }
                worst = wmax((int)ln < K ? best : -INFINITY);
            }
        };
        bool ok = true;
        {
            NodeChild c;
            load_child(A.root, (int)(ln & 1), &c);
            const float d = box_d2(c);
            count(kCtrNode, 2);
            push(A.root << 1, rdl(d, 0));
            push((A.root << 1) | 1u, rdl(d, 1));
        }
        int64_t budget = 4 * A.n + 1024;
        while (qn > 0 && ok) {
            if (--budget < 0) break;
            uint32_t e;
            float k;
            pop(&e, &k, true);
            if (!(k < worst)) break;
            NodeChild c;
            load_child(e >> 1, (int)(e & 1), &c);
            const uint32_t ref = uni(c.ref);
            if (ref_is_leaf(ref)) {
                take_leaf(ref);
                continue;
            }
            NodeChild cc;
            load_child(ref, (int)(ln & 1), &cc);
            const float d = box_d2(cc);
            count(kCtrNode, 2);
            for (int sd = 0; sd < 2; ++sd) {
                const float dd = rdl(d, sd);
                if (!(dd < worst)) continue;
                if (qn >= QCAP) {
                    ok = false;  // queue full: go on with the nearest found so far
                    break;
                }
                push((ref << 1) | (uint32_t)sd, dd);
            }
        }
        qn = 0;
        // clip by the found sites, nearest first
        float dd = (int)ln < K ? best : INFINITY;
        for (int t = 0; t < K; ++t) {
            const float c = wmin(dd);
            if (c == INFINITY) break;
            const int L = lowest(ballot(dd == c));
            if ((int)ln == L) dd = INFINITY;
            const uint32_t j = rdl(bsite, L);
            if ((int)ln == nwarm) wsite = j;
            ++nwarm;
            const float4 q = A.pts[j];
            const float ax = q.x - px, ay = q.y - py, az = q.z - pz;
            const float a2 = fmaf(ax, ax, fmaf(ay, ay, az * az));
            const float dw = kW ? pw - q.w : 0.f;
            const uint64_t t0 = tic();
            const int r = clip(ax, ay, az, 0.5f * (a2 + dw), 0.5f * (a2 + fabsf(dw)), (int32_t)j);
            toc(kCtrCycClip, t0);
            if (r == kEmptied || r == kOverflow || r == kRestart) return r;
            if (r == kChanged) update_bounds();
        }
        return kNone;
    }

    // The start of Alg. 1.  From the root, the walk first reaches the site's
    // own leaf (its bound is 0 there) and on the way down queues the sibling
    // of every node on that path, tested against the still uncut box.  Here
    // the own leaf (found through the site's leaf record) is clipped first;
    // then the siblings of its path are gathered by one scalar climb over the
    // parent links, one per lane, and tested together against the cut cell.
    // Only those that may still cut it are queued, with the keys Alg. 1 gives
    // them (a sibling culled here would be culled when popped: the cell only
    // shrinks), top of the path first so that the nearest is queued last.
    // Returns kNone, or what the leaf returned (kEmptied, kOverflow,
    // kRestart); *deep if the path has more than 64 siblings (nothing is
    // clipped then, and the walk starts at the root).
    __device__ int own_leaf_start(uint32_t* own, bool* deep) {
        KArgs* ka = cold_args();
        const uint32_t rec = uni(ka->leaf_of[self]);
        const uint32_t oref = uni(A.nodes[rec >> 1].c[rec & 1].ref);
        *own = oref;
        *deep = false;
        uint32_t e = rec ^ 1u;  // this lane's sibling record: (node << 1) | which child
        int ns = 1;
        for (uint32_t cur = rec;;) {
            const uint32_t u = uni(ka->up[cur >> 1]);
            if (u == kNoParent) break;
            if (ns == 64) {
                *deep = true;
                return kNone;
            }
            if ((int)ln == ns) e = u ^ 1u;
            ++ns;
            cur = u;
        }
        count(kCtrNode, (uint64_t)ns);
        // lanes past the path test the first sibling again (no divergent load)
        const uint32_t me = (int)ln < ns ? e : rdl(e, 0);
        NodeChild c;
        load_child(me >> 1, (int)(me & 1), &c);
        float key = 0.f, delta = 0.f;
        bool cull = true;
        const uint64_t t0 = tic();
        leaf_phase = 0;
        int r = leaf(oref, ~0ull);
        leaf_phase = 1;
        toc(kCtrCycLeaf, t0);
        if (r != kNone) return r;
        node_test(c, &key, &cull, &delta);
        uint64_t live = ballot(!cull && (int)ln < ns);
        while (live) {
            const int L = 63 - __builtin_clzll(live);
            live &= ~(1ull << L);
            if (culling() == 3 && !ball_hit_lane(c, L)) continue;
            if (qn >= QCAP) return kOverflow;
            push(rdl(me, L), rdl(key, L));
        }
        return kNone;
    }

    // Alg. 1.  Returns kNone when done, kEmptied, kOverflow or kRestart.
    // A cell taken over from the previous pass (resume) first finishes the
    // leaf it stopped in, then goes on with the queue it brought.
    __device__ int traverse(bool resume = false, uint32_t rleaf = 0, uint64_t rmask = 0, uint32_t rphase = 1,
                            uint32_t rskip = kNoParent) {
        uint32_t cur = A.root;
        bool have = true;
        uint64_t allow = ~0ull;  // candidates of the first leaf
        if constexpr (kSaves) ov_ok = false;
        uint32_t done_leaf = 0;
        bool skip_done = false;
        bool own_first = false;  // the first leaf is the site's own, then the walk starts at the root
        if constexpr (kResumes) {
            if (resume) {
                // the rest of the leaf it stopped in (one call site of leaf():
                // through the loop below)
                cur = rleaf;
                allow = rmask;
                own_first = rphase == 0;
                if (rphase != 0 && rskip != kNoParent) {  // the own leaf, clipped before this walk
                    done_leaf = rskip;
                    skip_done = true;
                }
            }
        }
        // own leaf first, then the siblings of its path (not for a cell taken
        // over), in the 64-vertex pass only: for the cells that outgrew it
        // the walk from the root is faster (starting them at their own leaf
        // made the larger passes 40-60% slower on the power and surface
        // workloads)
        if (!resume && A.leaf_of != nullptr) {
            if (warm_start() > 0) {
                const int rw = knn_warm(warm_start());
                if constexpr (kSaves) ov_ok = false;  // an overflow in the warm start starts over
                if (rw != kNone) return rw;
            }
            if constexpr (VPL == 1) {
                bool deep;
                const int r = own_leaf_start(&done_leaf, &deep);
                if (r != kNone) return r;
                have = deep;  // then from the root, the own leaf like any other
            }
        }
        // every node is visited at most once in a valid tree; the bound only
        // guarantees termination if the tree were ever malformed
        int64_t budget = 4 * A.n + 1024;
        for (;;) {
            while (have && !ref_is_leaf(cur)) {
                if (--budget < 0) return kOverflow;
                count(kCtrNode, 2);
                const uint32_t node = cur;
                float key = 0.f, delta = 0.f;
                bool cull = true;
                uint32_t ref = 0;
                NodeChild cc;
                load_child(node, (int)(ln & 1), &cc);
                node_test(cc, &key, &cull, &delta);
                ref = cc.ref;
                const uint64_t cm = ballot(cull);
                bool c0 = (cm & 1ull) != 0, c1 = (cm & 2ull) != 0;
                if (culling() == 3) {
                    if (!c0 && !c1) {
                        bool h0, h1;
                        ball_hit_pair(cc, &h0, &h1);
                        c0 = !h0;
                        c1 = !h1;
                    } else {
                        if (!c0 && !ball_hit_lane(cc, 0)) c0 = true;
                        if (!c1 && !ball_hit_lane(cc, 1)) c1 = true;
                    }
                }
                if (c0 && c1) {
                    have = false;
                    break;
                }
                // descend into the nearer child (smaller bound minus radius),
                // queue the other: the same in both traversal orders, which
                // differ only in what they pop next (Alg. 1: the least key;
                // depth-first: the last pushed)
                const float d0 = rdl(delta, 0), d1 = rdl(delta, 1);
                const int near = c1 ? 0 : (c0 ? 1 : (d0 <= d1 ? 0 : 1));
                const int far = 1 - near;
                if (!(far ? c1 : c0)) {
                    if (qn >= QCAP) return kOverflow;
                    push((node << 1) | (uint32_t)far, rdl(key, far));
                }
                cur = rdl(ref, near);
            }
            if (have && !(skip_done && cur == done_leaf)) {
                const uint64_t t0 = tic();
                if constexpr (kResumes) leaf_phase = own_first ? 0u : 1u;
                int r = leaf(cur, allow);
                if constexpr (kResumes) leaf_phase = 1;
                if constexpr (kSaves) ov_skip = skip_done ? done_leaf : kNoParent;
                if constexpr (kResumes) allow = ~0ull;
                toc(kCtrCycLeaf, t0);
                if (r != kNone) return r;
            }
            if constexpr (kResumes) {
                if (own_first) {  // the own leaf is done: from the root, passing over it
                    own_first = false;
                    done_leaf = cur;
                    skip_done = true;
                    cur = A.root;
                    continue;
                }
            }
            have = false;
            while (qn > 0) {
                if (--budget < 0) return kOverflow;
                uint32_t e;
                float k;
                pop(&e, &k);
                count(kCtrNode, 1);
                if (traversal() != 2 && k > __builtin_amdgcn_sqrtf(rmax2) * (1.f + 16.f * kU)) {
                    qn = 0;  // every key left is at least k: nothing can cut the cell
                    break;
                }
                float key = 0.f, delta = 0.f;
                bool cull = true;
                uint32_t ref = 0;
                NodeChild c;
                load_child(e >> 1, (int)(e & 1), &c);
                node_test(c, &key, &cull, &delta);
                ref = c.ref;
                bool culled = rdl((int)cull, 0) != 0;
                if (!culled && culling() == 3 && !ball_hit_lane(c, 0)) culled = true;
                if (!culled) {
                    cur = rdl(ref, 0);
                    have = true;
                    break;
                }
            }
            if (!have) return kNone;
        }
    }

    // ------------------------------------------------------------ hand-over
    // Writes the state of a cell that overflowed for the next pass; only the
    // header when the overflow is not resumable.
    __device__ void save(HOut& o) {
        if constexpr (kSaves) {
            sync();
            const int tid = (int)(wid * 64 + ln), step = 64 * G;
            if (ov_ok) {
                for (int q = tid; q < np; q += step) {
                    o.pl[q] = M.pl[q];
                    o.psite[q] = site_of((uint32_t)q);
                    o.psb[q] = M.psb[q];
                    o.pcode[q] = M.pcode[q];
                }
                if constexpr (kReg) {
#pragma unroll
                    for (int s = 0; s < VPL; ++s) {
                        const int q = s * 64 + (int)ln;
                        o.y0[q] = y0[s];
                        o.y1[q] = y1[s];
                        o.y2[q] = y2[s];
                        o.ev[q] = ev[s];
                        o.vt[q] = vt[s];
                        o.va[q] = va[s];
                        o.qe[q] = qe[s];
                        o.qk[q] = qk[s];
                        if (ln == 0) o.alive[s] = alive[s];
                    }
                    if constexpr (kQExt) {
                        for (int q = 64 * VPL + (int)ln; q < qn; q += 64) {
                            o.qe[q] = M.qxe[q - 64 * VPL];
                            o.qk[q] = M.qxk[q - 64 * VPL];
                        }
                    }
                } else {
                    for (int q = tid; q < vhi; q += step) {
                        o.y0[q] = M.y0[q];
                        o.y1[q] = M.y1[q];
                        o.y2[q] = M.y2[q];
                        o.ev[q] = M.ev[q];
                        o.vt[q] = M.vt[q];
                        o.va[q] = M.va[q];
                    }
                    for (int q = tid; q < qn; q += step) {
                        o.qe[q] = M.qe[q];
                        o.qk[q] = M.qk[q];
                    }
                    if (tid < nsv()) o.alive[tid] = H.alive[tid];
                }
            }
            if (tid < kMaxWarm) o.wsite[tid] = tid < nwarm ? wsite : 0u;  // lane t of wave 0 holds site t
            if (tid == 0) {
                o.nwarm = (uint32_t)nwarm;
                o.np = (uint32_t)np;
                o.vhi = (uint32_t)(kReg ? CAP : vhi);
                o.qn = (uint32_t)qn;
                o.flags = flags;
                o.robust = (uint32_t)robust;
                o.leaf = ov_leaf;
                o.mask = ov_mask;
                o.phase = ov_phase;
                o.skip = ov_phase == 0 ? kNoParent : ov_skip;
                o.valid = ov_ok ? 1u : 0u;
            }
        }
    }

    // Takes over a cell saved by the previous pass (instead of init): the
    // traversal then goes on with resume = true, H.leaf, H.mask, H.phase.
    // Vertex, plane and queue numbers are the same in every pass.
    __device__ void resume(uint32_t k, const HIn& in) {
        if constexpr (kResumes) {
            sync();  // every wave is done with the previous cell
            self = k;
            float4 s = A.pts[k];
            px = s.x; py = s.y; pz = s.z; pw = s.w;
            flags = uni(in.flags);
            robust = (int)uni(in.robust);
            nwarm = (int)uni(in.nwarm);
            wsite = (int)ln < kMaxWarm ? in.wsite[ln] : 0u;
            np = (int)uni(in.np);
            vhi = (int)uni(in.vhi);
            qn = (int)uni(in.qn);
            const int tid = (int)(wid * 64 + ln), step = 64 * G;
            for (int q = tid; q < np; q += step) {
                M.pl[q] = in.pl[q];
                if constexpr (kReg) M.psite[q] = in.psite[q];
                M.psb[q] = in.psb[q];
                M.pcode[q] = in.pcode[q];
            }
            if constexpr (kReg) {
#pragma unroll
                for (int s2 = 0; s2 < VPL; ++s2) {
                    const int q = s2 * 64 + (int)ln;
                    if (s2 < kPrevCap / 64) {
                        y0[s2] = in.y0[q];
                        y1[s2] = in.y1[q];
                        y2[s2] = in.y2[q];
                        ev[s2] = in.ev[q];
                        vt[s2] = in.vt[q];
                        va[s2] = in.va[q];
                        alive[s2] = in.alive[s2];
                    } else {
                        alive[s2] = 0ull;
                    }
                    if (s2 < kPrevQ / 64) {
                        qe[s2] = in.qe[q];
                        qk[s2] = in.qk[q];
                    }
                }
                if constexpr (kQExt) {
                    for (int q = 64 * VPL + (int)ln; q < qn; q += 64) {
                        M.qxe[q - 64 * VPL] = in.qe[q];
                        M.qxk[q - 64 * VPL] = in.qk[q];
                    }
                }
                vhi = CAP;
            } else {
                // vertex and plane indices: ten bits each there, wider here
                // above 1024 vertices
                auto wide = [](uint32_t x) -> W {
                    if constexpr (T::kNarrow) return (W)x;
                    else return T::pack3(x & 1023u, (x >> 10) & 1023u, (x >> 20) & 1023u);
                };
                for (int q = tid; q < vhi; q += step) {
                    M.y0[q] = in.y0[q];
                    M.y1[q] = in.y1[q];
                    M.y2[q] = in.y2[q];
                    M.ev[q] = in.ev[q];
                    M.vt[q] = wide(in.vt[q]);
                    M.va[q] = wide(in.va[q]);
                }
                for (int q = tid; q < qn; q += step) {
                    M.qe[q] = in.qe[q];
                    M.qk[q] = in.qk[q];
                }
                if (tid < nsv()) H.alive[tid] = in.alive[tid];
            }
            sync();
            load_slots();
            update_bounds();
        }
    }

    // ------------------------------------------------------------ output
    // FP64 position of a vertex (relative to the site) from its three planes.
    __device__ void pos64(W t, float fx, float fy, float fz, double* y) const {
        const P64 P = plane64(T::fld(t, 0)), Q = plane64(T::fld(t, 1)), S = plane64(T::fld(t, 2));
        const Meet64 m(P, Q, S);
        if (m.det != 0.0) {
            double n[3];
            m.numerator(P, Q, S, n);
            const double inv = 1.0 / m.det;
            y[0] = n[0] * inv; y[1] = n[1] * inv; y[2] = n[2] * inv;
        } else {
            y[0] = fx; y[1] = fy; y[2] = fz;
        }
    }

    // Writes the cell's record.  Returns false if the vertex/facet structure
    // is not a closed simple polytope (the caller then rebuilds the cell).
    // The planes are compacted by the group, the record written by its first
    // wave.
    __device__ bool finalize(uint32_t slot, uint32_t orig) {
        gc();
        bool ok = true;
        if (lead()) ok = finalize_lead(slot, orig);
        if constexpr (G > 1) ok = bcast(ok ? 1u : 0u) != 0;
        return ok;
    }
    __device__ bool finalize_lead(uint32_t slot, uint32_t orig) {
        const int F = np;
        const int ns = nsv();
        // facet order: ascending output code (box faces -6..-1, then original site ids)
        const uint32_t* order = cold_args()->order;
        for (int q = ln; q < F; q += 64) {
            int32_t c = M.pcode[q];
            M.key[q] = c >= 0 ? (int32_t)order[c] : c;
        }
        wsync();
        for (int q = ln; q < F; q += 64) {
            int32_t mine = M.key[q];
            uint32_t r = 0;
            for (int t = 0; t < F; ++t) r += M.key[t] < mine ? 1u : 0u;
            ta(q) = r;
            tb(q) = 0;
            M.anchor[q] = 0xFFFFFFFFu;
        }
        Stage st;
        {
            KArgs* ka = cold_args();
            st.cap = ka->stage.cap;
            st.vert = ka->stage.vert;
            st.tri64 = ka->stage.tri64;
            st.code = ka->stage.code;
            st.fsize = ka->stage.fsize;
            st.fv = ka->stage.fv;
        }
        int32_t* codes = st.code + (int64_t)slot * st.cap;
        for (int q = ln; q < F; q += 64) codes[ta(q)] = M.key[q];
        // vertex renumbering 0..nv-1 (slot-major)
        uint32_t nv = 0;
        int s0 = -1;
#pragma unroll
        for (int s = 0; s < (kReg ? VPL : ns); ++s) {
            const uint64_t al = alive[s];
            if (s0 < 0 && al) s0 = s;
            if ((al >> ln) & 1) M.sor[s * 64 + ln] = nv + mbcnt(al);
            nv += popc(al);
        }
        wsync();
        if (s0 < 0) return false;
        // reference point of the tetrahedral fan: vertex 0, in FP64
        double ref[3] = {0.0, 0.0, 0.0};
        {
            // (selects and no index: an array of the cell indexed at run time
            // would be kept in scratch memory, and the whole cell with it)
            uint64_t m0 = 0;
            if constexpr (kReg) {
#pragma unroll
                for (int s = 0; s < VPL; ++s) m0 = s == s0 ? alive[s] : m0;
            } else {
                m0 = uni(alive[s0]);
            }
            const int l0 = lowest(m0);
            double y[3] = {0.0, 0.0, 0.0};
            if constexpr (kReg) {
                W t = vt[0];
                float a = y0[0], b = y1[0], c = y2[0];
#pragma unroll
                for (int s = 1; s < VPL; ++s) {
                    t = s == s0 ? vt[s] : t;
                    a = s == s0 ? y0[s] : a;
                    b = s == s0 ? y1[s] : b;
                    c = s == s0 ? y2[s] : c;
                }
                if ((int)ln == l0) pos64(t, a, b, c, y);
            } else {
                if ((int)ln == l0) pos64(vt[s0], y0[s0], y1[s0], y2[s0], y);
            }
            for (int c = 0; c < 3; ++c) ref[c] = __shfl(y[c], l0);
        }
        // every neighbour must be a live vertex (its new number is then < nv;
        // numbers left from dead vertices are not trusted)
        bool bad = false;
#pragma unroll
        for (int s = 0; s < (kReg ? VPL : ns); ++s) {
            if ((alive[s] >> ln) & 1) {
                const W a = va[s];
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    const uint32_t u = T::fld(a, e);
                    bad |= !is_alive(u);
                }
            }
        }
        if (ballot(bad)) return false;
        float4* vout = st.vert + (int64_t)slot * st.cap;
        uint64_t* tri64 = st.tri64 ? st.tri64 + (int64_t)slot * st.cap : nullptr;
        const double p64[3] = {(double)px, (double)py, (double)pz};
#pragma unroll
        for (int s = 0; s < (kReg ? VPL : ns); ++s) {
            if ((alive[s] >> ln) & 1) {
                const W t = vt[s], a = va[s];
                uint32_t t0 = ta(T::fld(t, 0)), t1 = ta(T::fld(t, 1)), t2 = ta(T::fld(t, 2));
                uint32_t a0 = M.sor[T::fld(a, 0)], a1 = M.sor[T::fld(a, 1)], a2 = M.sor[T::fld(a, 2)];
                const uint32_t v = M.sor[s * 64 + ln];
                M.vtri[v] = T::pack3(t0, t1, t2);
                M.vadj[v] = T::pack3(a0, a1, a2);
                double y[3];
                pos64(t, y0[s], y1[s], y2[s], y);
                M.vpx[v] = y[0] - ref[0];
                M.vpy[v] = y[1] - ref[1];
                M.vpz[v] = y[2] - ref[2];
                uint32_t u0 = t0, u1 = t1, u2 = t2, tmp;
                if (u0 > u1) { tmp = u0; u0 = u1; u1 = tmp; }
                if (u1 > u2) { tmp = u1; u1 = u2; u2 = tmp; }
                if (u0 > u1) { tmp = u0; u0 = u1; u1 = tmp; }
                const uint32_t packed = tri64 ? 0u : (u0 | (u1 << 10) | (u2 << 20));
                vout[v] = make_float4((float)(p64[0] + y[0]), (float)(p64[1] + y[1]), (float)(p64[2] + y[2]),
                                      __uint_as_float(packed));
                if (tri64) tri64[v] = (uint64_t)u0 | ((uint64_t)u1 << 21) | ((uint64_t)u2 << 42);
                atomicAdd(&tb(t0), 1u);
                atomicAdd(&tb(t1), 1u);
                atomicAdd(&tb(t2), 1u);
                atomicMin(&M.anchor[t0], v);
                atomicMin(&M.anchor[t1], v);
                atomicMin(&M.anchor[t2], v);
            }
        }
        wsync();
        // facet rings in output (rank) order, counter-clockwise seen from outside;
        // sizes and anchors (lowest vertex) are indexed by facet rank
        uint16_t* fs = st.fsize + (int64_t)slot * st.cap;
        uint16_t* fvp = st.fv + (int64_t)slot * 3 * st.cap;
        uint32_t carry = 0;
        for (int r0 = 0; r0 < F; r0 += 64) {
            const uint32_t r = (uint32_t)(r0 + (int)ln);
            uint32_t sz = r < (uint32_t)F ? tb(r) : 0u;
            uint32_t x = sz;
            for (int o = 1; o < 64; o <<= 1) {
                uint32_t y = __shfl_up(x, o);
                if ((int)ln >= o) x += y;
            }
            if (r < (uint32_t)F) {
                fs[r] = (uint16_t)sz;
                const uint32_t base = carry + x - sz, start = M.anchor[r];
                if (sz < 3 || start >= nv) {
                    bad = true;
                } else {
                    uint32_t v = start, t = 0;
                    do {
                        fvp[base + t] = (uint16_t)v;
                        ++t;
                        W tri = M.vtri[v], adj = M.vadj[v];
                        uint32_t k = T::fld(tri, 0) == r ? 0u : (T::fld(tri, 1) == r ? 1u : 2u);
                        v = T::fld(adj, (k + 1) % 3);
                    } while (v != start && t < sz && v < nv);
                    bad |= (v != start) || (t != sz);
                }
            }
            carry += (uint32_t)__shfl(x, 63);
        }
        if (ballot(bad)) return false;
        // volume and centroid from the tetrahedra (ref, anchor_f, v, next_f(v)),
        // accumulated in FP64 (thin cells cancel badly in FP32)
        Fan64 sum;
        for (uint32_t v = ln; v < nv; v += 64) {
            const double Px = M.vpx[v], Py = M.vpy[v], Pz = M.vpz[v];
            W tri = M.vtri[v], adj = M.vadj[v];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                uint32_t an = M.anchor[T::fld(tri, k)];
                uint32_t nx = T::fld(adj, (k + 1) % 3);
                if (an == v || nx == an) continue;
                const double Qx = M.vpx[an], Qy = M.vpy[an], Qz = M.vpz[an];
                const double Nx = M.vpx[nx], Ny = M.vpy[nx], Nz = M.vpz[nx];
                sum.add(Qx, Qy, Qz, Px, Py, Pz, Nx, Ny, Nz);
            }
        }
        const double vol6 = wsum64(sum.vol6), mx = wsum64(sum.mx), my = wsum64(sum.my), mz = wsum64(sum.mz);
        uint32_t nbox = 0;
        for (int q = ln; q < F; q += 64) nbox += M.key[q] < 0 ? 1u : 0u;
        nbox = wsum_u(nbox);
        count(kCtrFinal, nv);
        if (ln == 0) {
            KArgs* ka = cold_args();
            ka->cnt_v[orig] = nv;
            ka->cnt_f[orig] = (uint32_t)F;
            ka->cnt_n[orig] = (uint32_t)F - nbox;
            ka->vol[orig] = (float)(vol6 / 6.0);
            double inv = vol6 != 0.0 ? 0.25 / vol6 : 0.0;
            ka->cen[3 * orig] = centroid_of(px, ref[0], mx, inv);
            ka->cen[3 * orig + 1] = centroid_of(py, ref[1], my, inv);
            ka->cen[3 * orig + 2] = centroid_of(pz, ref[2], mz, inv);
            ka->flags[orig] = (uint8_t)flags;
            ka->loc[self] = make_loc((uint32_t)A.tier, slot);
        }
        return true;
    }

    __device__ void write_empty(uint32_t orig, uint32_t extra) {
        if (ln == 0 && lead()) {
            KArgs* ka = cold_args();
            ka->cnt_v[orig] = 0;
            ka->cnt_f[orig] = 0;
            ka->cnt_n[orig] = 0;
            ka->vol[orig] = 0.f;
            ka->cen[3 * orig] = px;
            ka->cen[3 * orig + 1] = py;
            ka->cen[3 * orig + 2] = pz;
            ka->flags[orig] = (uint8_t)(flags | kFlagEmpty | extra);
            ka->loc[self] = make_loc((uint32_t)A.tier, 0);
        }
    }
};

constexpr int kWaves1 = 4, kWaves2 = 2;  // waves per block of the two register tiers

// The work loop shared by every tier (per wave, or per wave group with gx
// its exchange tables).
template <int VPL, bool kLds, bool kCount, int G = 1, bool kSoS = false, bool kW = true, bool kOpt = true>
__device__ void run_cells(WaveMem<VPL>& M, HotMem<VPL>& H, const ClipArgs& A, uint32_t* gx) {
    KArgs* ka = cold_args();
    // the input checks (non-finite values, a flat box) ran before this pass:
    // on such input no cell is built
    if (*ka->err != 0u) return;
    const uint32_t count = ka->list ? *ka->list_count : (uint32_t)A.n;
    if (count == 0) return;  // a larger pass with no cell
    Cell<VPL, kLds, kCount, G, kSoS, kW, kOpt> C(M, H, A, gx);
    unsigned long long st_empty = 0, st_large = 0, st_unc = 0, st_fail = 0, st_fp64 = 0, st_res = 0, st_pert = 0;
    constexpr uint32_t kWorkers = G > 1 ? 1u : (VPL == 1 ? kWaves1 : kWaves2);
    Work<kWorkers> work(count);
    for (;;) {
        uint32_t c = 0;
        if (C.lead()) c = work.next(G > 1 ? 0u : uni((uint32_t)threadIdx.x >> 6));
        c = C.bcast(c);
        if (c == kNoCell) break;
        KArgs* kc = cold_args();
        if (kc->list && c >= kc->slots) {
            // no staging slot: left undone and counted (the build runs the
            // passes again with more slots)
            if (C.ln == 0 && C.lead()) atomicAdd(kc->deferred, 1u);
            continue;
        }
        uint32_t k = kc->list ? kc->list[c] : c;
        bool checked = false;  // begin with checked signs
        if constexpr (VPL == 1) {
            checked = (k & kRetryChecked) != 0u;
            k &= ~kRetryChecked;
        }
        const uint32_t slot = kc->list && !(VPL == 1 && kc->retry) ? c : k;
        const uint32_t orig = kc->order[k];
        // a cell the previous pass handed over goes on from where it stopped
        using CellT = Cell<VPL, kLds, kCount, G, kSoS, kW, kOpt>;
        const typename CellT::HIn* hin = nullptr;
        if constexpr (CellT::kResumes) {
            if (kc->hand_in && c < kc->hand_in_cap) {
                const auto* h = static_cast<const typename CellT::HIn*>(kc->hand_in) + c;
                if (uni(h->valid)) hin = h;
            }
        }
        // a cell is built with plain FP32 signs first (mixed mode: with FP64
        // re-evaluation of doubtful ones); if that meets an inconsistent
        // configuration it is rebuilt with the FP64 re-evaluation, then with
        // every sign in FP64
        C.robust = A.precision == 2 || checked ? 1 : 0;
        bool done = false, escalated = false, loser = false;
        for (int attempt = checked ? 1 : 0; attempt < 3 && !done; ++attempt) {
            const bool res = attempt == 0 && hin != nullptr;
            if (res) {
                C.resume(k, *hin);
                ++st_res;
            } else if (!C.init(k)) {
                loser = true;
                break;
            }
            if (attempt > 0) C.flags |= kFlagFP64;
            if (A.tier > 0) C.flags |= kFlagLarge;
            const uint64_t t0 = C.tic();
            int r = C.traverse(res, res ? uni(hin->leaf) : 0u, res ? uni((uint64_t)hin->mask) : 0ull, res ? uni(hin->phase) : 1u,
                               res ? uni(hin->skip) : kNoParent);
            C.toc(kCtrCycTraverse, t0);
            if (r == kRestart) {
                C.robust = C.robust + 1;
                continue;
            }
            if (r == kOverflow) {
                KArgs* kn = cold_args();
                if (kn->next_list) {
                    uint32_t pos = 0;
                    if (C.ln == 0 && C.lead()) {
                        pos = atomicAdd(kn->next_count, 1u);
                        kn->next_list[pos] = k;
                    }
                    if constexpr (CellT::kSaves) {
                        pos = C.bcast(pos);
                        if (kn->hand_out && pos < kn->hand_out_cap)
                            C.save(static_cast<typename CellT::HOut*>(kn->hand_out)[pos]);
                    }
                    escalated = true;
                } else {
                    C.write_empty(orig, kFlagFailed);
                    ++st_fail;
                    ++st_empty;
                }
                done = true;
                break;
            }
            if (r == kEmptied) {
                C.write_empty(orig, 0);
                ++st_empty;
                done = true;
            } else if ([&] {
                           const uint64_t t1 = C.tic();
                           const bool ok = C.finalize(slot, orig);
                           C.toc(kCtrCycFinal, t1);
                           return ok;
                       }()) {
                done = true;
            } else if (C.robust < 2) {
                C.robust = C.robust + 1;
            } else {
                break;
            }
        }
        if (loser) {
            C.write_empty(orig, 0);
            ++st_empty;
            continue;
        }
        if (escalated) continue;
        if (!done) {
            // still inconsistent after the robust rebuilds: report an empty cell
            C.write_empty(orig, kFlagFailed | kFlagUncertain);
            ++st_fail;
            ++st_empty;
        }
        st_large += (C.flags & kFlagLarge) ? 1 : 0;
        st_unc += (C.flags & kFlagUncertain) ? 1 : 0;
        st_fp64 += (C.flags & kFlagFP64) ? 1 : 0;
        st_pert += (C.flags & kFlagPerturbed) ? 1 : 0;
    }
    if (C.ln == 0 && C.lead()) {
        ka = cold_args();
        if constexpr (kCount)
            for (int c = 0; c < kCtrCount; ++c)
                if (C.ctr[c]) atomicAdd(&ka->ctr[c], (unsigned long long)C.ctr[c]);
        if (st_empty) atomicAdd(&ka->stats[kStatEmpty], st_empty);
        if (st_large) atomicAdd(&ka->stats[kStatLarge], st_large);
        if (st_unc) atomicAdd(&ka->stats[kStatUncertain], st_unc);
        if (st_fail) atomicAdd(&ka->stats[kStatFailed], st_fail);
        if (st_fp64) atomicAdd(&ka->stats[kStatFP64], st_fp64);
        if (st_res) atomicAdd(&ka->stats[kStatResumed], st_res);
        if (st_pert) atomicAdd(&ka->stats[kStatPerturbed], st_pert);
    }
}

#pragma clang attribute pop

// Register tiers: per-cell arrays in LDS, WAVES independent waves per
// block.  Register budgets: the 64-vertex pass is held to 128 registers for
// 4 waves per SIMD (a few spills cost less than the lost occupancy: the pass
// issues VALU work back to back), the 128-vertex pass to 256 for 2.  (It was
// slower at 3 when it kept its cell in scratch memory; since it does not, 3
// waves in 168 registers have been measured faster where it has many cells, 390
// -> 383 ms on 20M surface sites, but are not in use: not tested enough.)
template <int VPL, int WAVES, bool kCount, bool kSoS = false, bool kW = true, bool kOpt = true>
__global__ __launch_bounds__(64 * WAVES, VPL == 1 ? 4 : 2) void k_clip(ClipArgs A) {
    __shared__ WaveMem<VPL> mem[WAVES];
    HotMem<VPL> none;
    run_cells<VPL, true, kCount, 1, kSoS, kW, kOpt>(mem[threadIdx.x >> 6], none, A, nullptr);
}

// 1024-vertex tier: the kGroupLds waves of a block build one cell, its
// arrays in LDS (one block per CU).
template <bool kCount, bool kSoS, bool kOpt>
__global__ __launch_bounds__(64 * kGroupLds, 1) void k_clip_lds(ClipArgs A) {
    __shared__ WaveMem<16> mem;
    __shared__ HotMem<16> hot;
    __shared__ uint32_t gx[2 * kGroupLds * 8];
    run_cells<16, true, kCount, kGroupLds, kSoS, true, kOpt>(mem, hot, A, gx);
}

// 16384-vertex tier: the kGroupArena waves of a block build one cell, its
// arrays in arena[blockIdx.x].
constexpr int kArenaVPL = kTierCap[3] / 64;
template <bool kCount, bool kSoS, bool kOpt>
__global__ __launch_bounds__(64 * kGroupArena) void k_clip_arena(ClipArgs A, WaveMem<kArenaVPL>* arena) {
    __shared__ HotMem<kArenaVPL> hot;
    __shared__ uint32_t gx[2 * kGroupArena * 8];
    run_cells<kArenaVPL, false, kCount, kGroupArena, kSoS, true, kOpt>(arena[blockIdx.x], hot, A, gx);
}

static_assert(kTierCap[0] == 64 && kTierCap[1] == 128 && kTierCap[2] == 1024,
              "the passes with a cell in registers or LDS are instantiated for 64, 128 and 1024 vertices");
static_assert(sizeof(WaveMem<16>) + sizeof(HotMem<16>) + 2 * kGroupLds * 8 * sizeof(uint32_t) <= 160 * 1024,
              "the 1024-vertex tier must fit the LDS of one CU");
static_assert(sizeof(HotMem<kArenaVPL>) + 2 * kGroupArena * 8 * sizeof(uint32_t) <= 160 * 1024,
              "the clip tables of the 16384-vertex tier must fit the LDS of one CU");
static_assert(Tier<kArenaVPL>::CAP <= (1 << Tier<kArenaVPL>::kB) && Tier<kArenaVPL>::CAP <= (1 << 16),
              "arena-tier indices must fit their packings and the 16-bit staged facet lists");

}  // namespace

size_t arena_bytes_per_worker() { return sizeof(WaveMem<kArenaVPL>); }

size_t handoff_bytes(int tier) {
    switch (tier) {
        case 0: return sizeof(HandoffT<kTierCap[0], kQueue0>);
        case 1: return sizeof(HandoffT<kTierCap[1], kQueue0>);
        case 2: return sizeof(HandoffT<kTierCap[2]>);
        default: return 0;
    }
}

int clip_grid_workers(int tier, int num_cu) {
    int per_cu = 0;
    hipError_t e = hipSuccess;
    if (tier == 0) {
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_clip<1, kWaves1, false>, 64 * kWaves1, 0);
        per_cu *= kWaves1;
    } else if (tier == 1) {
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_clip<2, kWaves2, false>, 64 * kWaves2, 0);
        per_cu *= kWaves2;
    } else if (tier == 2) {
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_clip_lds<false, false, true>, 64 * kGroupLds, 0);
        if (e == hipSuccess && per_cu > 0) return per_cu * num_cu;
        return num_cu;
    } else {
        return num_cu;  // arena groups: one per CU, bounded by arena memory
    }
    if (e != hipSuccess || per_cu < 1) per_cu = 4;
    return per_cu * num_cu;
}

template <bool kCount, bool kSoS>
void launch_tier(const ClipArgs& a, int workers, void* arena, hipStream_t s) {
    // Instantiations with the default search options fixed, in the register
    // passes also without weights (see Cell); in the large passes the code
    // falls from 94 to 61 KB and from 124 to 78 (1024 vertices 6.6 -> 6.3 ms on
    // 1M power sites).  Not in the register passes of perturbed builds: a
    // lattice of 27k took 1.56 ms instead of 1.52.
    const bool def = a.culling == 3 && a.traversal == 1 && a.warm_start == 0;
    auto* const ar = static_cast<WaveMem<kArenaVPL>*>(arena);
    switch (a.tier) {
        case 0: {
            const dim3 g((workers + kWaves1 - 1) / kWaves1), t(64 * kWaves1);
            if (kSoS || !def) hipLaunchKernelGGL((k_clip<1, kWaves1, kCount, kSoS>), g, t, 0, s, a);
            else if (a.weighted) hipLaunchKernelGGL((k_clip<1, kWaves1, kCount, false, true, false>), g, t, 0, s, a);
            else hipLaunchKernelGGL((k_clip<1, kWaves1, kCount, false, false, false>), g, t, 0, s, a);
            break;
        }
        case 1: {
            const dim3 g((workers + kWaves2 - 1) / kWaves2), t(64 * kWaves2);
            if (kSoS || !def) hipLaunchKernelGGL((k_clip<2, kWaves2, kCount, kSoS>), g, t, 0, s, a);
            else if (a.weighted) hipLaunchKernelGGL((k_clip<2, kWaves2, kCount, false, true, false>), g, t, 0, s, a);
            else hipLaunchKernelGGL((k_clip<2, kWaves2, kCount, false, false, false>), g, t, 0, s, a);
            break;
        }
        case 2: {
            const dim3 g(workers), t(64 * kGroupLds);
            if (!def) hipLaunchKernelGGL((k_clip_lds<kCount, kSoS, true>), g, t, 0, s, a);
            else hipLaunchKernelGGL((k_clip_lds<kCount, kSoS, false>), g, t, 0, s, a);
            break;
        }
        default: {
            const dim3 g(workers), t(64 * kGroupArena);
            if (!def) hipLaunchKernelGGL((k_clip_arena<kCount, kSoS, true>), g, t, 0, s, a, ar);
            else hipLaunchKernelGGL((k_clip_arena<kCount, kSoS, false>), g, t, 0, s, a, ar);
            break;
        }
    }
}

hipError_t launch_clip(const ClipArgs& a, int workers, void* arena, hipStream_t s) {
    if (a.tier >= 3 && !arena) return hipErrorInvalidValue;
    if (workers < 1) return hipErrorInvalidValue;
    // the perturbed build has no counting instantiation (counters stay zero)
    if (a.perturb) launch_tier<false, true>(a, workers, arena, s);
    else if (a.ctr) launch_tier<true, false>(a, workers, arena, s);
    else launch_tier<false, false>(a, workers, arena, s);
    return hipGetLastError();
}

}  // namespace vd
