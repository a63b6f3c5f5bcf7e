// Input packing and the power-augmented BVH (paper Sec. 4.3, supplementary
// Sec. A "Input packing" and "Power-augmented BVH").
//
// The paper packs each site as one 16-byte (x, y, z, w) record and builds a
// binary BVH whose nodes also store the largest weight below them.  Here the
// BVH is a linear BVH: 63-bit Morton codes (21 bits per axis inside the clip
// box), an LSD radix sort, the Karras (2012) binary radix tree over the sorted
// codes, subtrees of at most `leaf_size` sites collapsed into leaves, and every
// node's child boxes and max weights as reductions over its range of sites.
#include "vd_internal.h"

namespace vd {

// ------------------------------------------------------------------ packing

__device__ inline float4 pack_site(const float* __restrict__ xyz, const float* __restrict__ w, int64_t i, uint32_t* err) {
    const float x = xyz[3 * i], y = xyz[3 * i + 1], z = xyz[3 * i + 2];
    const float ww = w ? w[i] : 0.0f;
    if (!(isfinite(x) && isfinite(y) && isfinite(z) && isfinite(ww))) atomicOr(err, 1u);
    return make_float4(x, y, z, ww);
}

// The caller's box to device memory, and its check.
__device__ inline void put_box(const BoxArg& b, float* bbox, uint32_t* err) {
    for (int c = 0; c < 6; ++c) bbox[c] = b.v[c];
    for (int c = 0; c < 3; ++c)
        if (!(b.v[3 + c] > b.v[c]) || !isfinite(b.v[c]) || !isfinite(b.v[3 + c])) atomicOr(err, 2u);
}

// Bounding box of the sites: packing and per-block partial min/max, then one
// block folds them (a lane per partial, not one lane for all: at 1024 partials
// the serial fold took longer than the rest of the packing).
__device__ inline void fold_box(float* mn, float* mx, float (*red)[256], float* out) {
    for (int c = 0; c < 3; ++c) {
        red[c][threadIdx.x] = mn[c];
        red[3 + c][threadIdx.x] = mx[c];
    }
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            for (int c = 0; c < 3; ++c) {
                red[c][threadIdx.x] = fminf(red[c][threadIdx.x], red[c][threadIdx.x + o]);
                red[3 + c][threadIdx.x] = fmaxf(red[3 + c][threadIdx.x], red[3 + c][threadIdx.x + o]);
            }
        }
        __syncthreads();
    }
    if (threadIdx.x < 6) out[threadIdx.x] = red[threadIdx.x][0];
}

__global__ __launch_bounds__(256) void k_pack_box(const float* __restrict__ xyz, const float* __restrict__ w, int64_t n,
                                                  float4* __restrict__ pts, float* partial, uint32_t* err) {
    __shared__ float red[6][256];
    float mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float4 p = pack_site(xyz, w, i, err);
        pts[i] = p;
        mn[0] = fminf(mn[0], p.x); mn[1] = fminf(mn[1], p.y); mn[2] = fminf(mn[2], p.z);
        mx[0] = fmaxf(mx[0], p.x); mx[1] = fmaxf(mx[1], p.y); mx[2] = fmaxf(mx[2], p.z);
    }
    fold_box(mn, mx, red, partial + 6 * blockIdx.x);
}

__global__ __launch_bounds__(256) void k_box_final(const float* partial, int nblk, float* bbox, uint32_t* err) {
    __shared__ float red[6][256];
    float mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int k = threadIdx.x; k < nblk; k += 256)
        for (int c = 0; c < 3; ++c) {
            mn[c] = fminf(mn[c], partial[6 * k + c]);
            mx[c] = fmaxf(mx[c], partial[6 * k + 3 + c]);
        }
    fold_box(mn, mx, red, bbox);
    if (threadIdx.x < 3 && !(red[3 + threadIdx.x][0] > red[threadIdx.x][0])) atomicOr(err, 2u);  // flat point set
}

// ------------------------------------------------------------------ Morton

__device__ inline uint64_t spread21(uint32_t v) {
    uint64_t x = v & 0x1FFFFFu;
    x = (x | (x << 32)) & 0x001F00000000FFFFull;
    x = (x | (x << 16)) & 0x001F0000FF0000FFull;
    x = (x | (x << 8)) & 0x100F00F00F00F00Full;
    x = (x | (x << 4)) & 0x10C30C30C30C30C3ull;
    x = (x | (x << 2)) & 0x1249249249249249ull;
    return x;
}

__device__ inline uint32_t quantize21(float x, float lo, float inv_ext) {
    float f = (x - lo) * inv_ext;
    f = fminf(fmaxf(f, 0.0f), 2097151.0f);
    return (uint32_t)f;
}

__device__ inline uint64_t morton_code(float4 p, const float* bbox) {
    const float scale = 2097152.0f;
    uint32_t qx = quantize21(p.x, bbox[0], scale / (bbox[3] - bbox[0]));
    uint32_t qy = quantize21(p.y, bbox[1], scale / (bbox[4] - bbox[1]));
    uint32_t qz = quantize21(p.z, bbox[2], scale / (bbox[5] - bbox[2]));
    return (spread21(qx) << 2) | (spread21(qy) << 1) | spread21(qz);
}

__global__ void k_morton(const float4* __restrict__ pts, int64_t n, const float* __restrict__ bbox,
                         uint64_t* __restrict__ keys, uint32_t* __restrict__ vals) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    keys[i] = morton_code(pts[i], bbox);
    vals[i] = (uint32_t)i;
}

hipError_t launch_morton(const float4* pts, int64_t n, const float* bbox, uint64_t* keys, uint32_t* vals,
                         hipStream_t s) {
    hipLaunchKernelGGL(k_morton, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, pts, n, bbox, keys, vals);
    return hipGetLastError();
}

// ------------------------------------------------------------------ radix sort
// Stable LSD sort of the 63-bit codes, 8 bits a pass.  Three shapes, by size:
//
// Up to kSmallSort sites one block of 1024 threads does everything from the
// input arrays to the sorted codes in LDS: such a build is a chain of short
// kernels, and this one takes the place of 41.
//
// Above, one kernel makes the codes and the histograms of all eight digits at
// once (the keys are in registers), then each pass is one kernel in which a
// tile of keys finds its digits' places among the earlier tiles by looking
// back over what they have published (decoupled look-back, Merrill and Garland
// 2016): a word per tile
// and digit, 2 bits of state above the count.  A tile takes its number from a
// counter, so every earlier tile is running or done, and publishes its own
// counts before it waits: the wait ends.  Against a histogram, a three-kernel
// scan and a scatter for every pass (five launches and two reads of the keys
// instead of one): 10k sites 236 -> 75 us, 1M sites 336 -> 150 us for all passes.
//
// A wave ranks 64 keys at a time: the lanes that share a digit are found with
// 8 ballots, one for each of its bits.

constexpr int kSmallSort = 4096;
constexpr int kSortThreads = 256;
constexpr int kPasses = 8;
constexpr uint32_t kPartial = 1u << 30, kInclusive = 2u << 30, kCountMask = (1u << 30) - 1u;

// Keys per thread of a tile: few where there are few tiles, so that a small
// sort spreads over the compute units; 16 for large ones (less look-back).
static int sort_items(int64_t n) { return n <= 262144 ? 4 : (n <= 4194304 ? 8 : 16); }
static int64_t sort_tiles(int64_t n) {
    const int64_t tile = (int64_t)kSortThreads * sort_items(n);
    return (n + tile - 1) / tile;
}

// Words of scratch, all zero at the start: the digit counts of every pass,
// a tile counter a pass, and the published counts of every tile and pass.
constexpr size_t kSortHead = 256 * kPasses + 16;
size_t sort_scratch_words(int64_t n) {
    return n <= kSmallSort ? 16 : kSortHead + (size_t)sort_tiles(n) * 256 * kPasses;
}

// Lanes of this wave with the same digit (of those with ok set).
__device__ inline uint64_t same_digit(uint32_t d, bool ok) {
    uint64_t peers = __ballot(ok);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const bool bit = ((d >> b) & 1u) != 0u;
        const uint64_t bb = __ballot(bit);
        peers &= bit ? bb : ~bb;
    }
    return peers;
}
__device__ inline uint32_t lanes_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
__device__ inline void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// Exclusive sum over the 256 first threads of a block (all threads call it);
// part: 4 words of LDS.
__device__ inline uint32_t scan_256(uint32_t v, uint32_t* part) {
    const int ln = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t x = v;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o);
        if (ln >= o) x += y;
    }
    if (ln == 63 && wv < 4) part[wv] = x;
    __syncthreads();
    uint32_t base = 0;
    for (int k = 0; k < 3; ++k)
        if (k < wv) base += part[k];
    __syncthreads();
    return base + x - v;
}

// kBox: the box is given (packing, codes and sort from the input arrays);
// otherwise pts and bbox are there already.
template <bool kBox>
__global__ __launch_bounds__(1024) void k_sort_small(const float* __restrict__ xyz, const float* __restrict__ w, int n,
                                                     BoxArg box, float* bbox, float4* __restrict__ pts,
                                                     uint64_t* __restrict__ keys, uint32_t* __restrict__ vals,
                                                     uint32_t* err) {
    constexpr int kItems = kSmallSort / 1024;
    __shared__ uint64_t skey[kSmallSort];
    __shared__ uint32_t sval[kSmallSort];
    __shared__ uint32_t cnt[16][256];
    __shared__ uint32_t part[4];
    const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63;
    float b[6];
    for (int c = 0; c < 6; ++c) b[c] = kBox ? box.v[c] : bbox[c];
    if (kBox && threadIdx.x == 0) put_box(box, bbox, err);
    // a wave holds consecutive keys, 64 a round; it sorts only as many rounds as there are keys
    const int items = (n + 1023) >> 10;
    uint64_t key[kItems];
    uint32_t val[kItems];
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        const int i = wv * 64 * items + it * 64 + ln;
        key[it] = ~0ull;  // past the end: sorts last
        val[it] = 0u;
        if (it < items && i < n) {
            float4 p;
            if (kBox) {
                p = pack_site(xyz, w, i, err);
                pts[i] = p;
            } else {
                p = pts[i];
            }
            key[it] = morton_code(p, b);
            val[it] = (uint32_t)i;
        }
    }
    for (int pass = 0; pass < kPasses; ++pass) {
        for (int t = threadIdx.x; t < 16 * 256; t += 1024) (&cnt[0][0])[t] = 0u;
        __syncthreads();
        uint32_t rank[kItems];
#pragma unroll
        for (int it = 0; it < kItems; ++it) {
            if (it >= items) break;
            const uint32_t d = (uint32_t)(key[it] >> (8 * pass)) & 255u;
            const uint64_t peers = same_digit(d, true);
            const uint32_t below = lanes_below(peers), before = cnt[wv][d];
            rank[it] = before + below;
            wave_fence();
            if (below == 0) cnt[wv][d] = before + (uint32_t)__popcll(peers);
            wave_fence();
        }
        __syncthreads();
        uint32_t total = 0;
        if (threadIdx.x < 256) {
            for (int k = 0; k < 16; ++k) {
                const uint32_t c = cnt[k][threadIdx.x];
                cnt[k][threadIdx.x] = total;
                total += c;
            }
        }
        const uint32_t base = scan_256(threadIdx.x < 256 ? total : 0u, part);
        if (threadIdx.x < 256)
            for (int k = 0; k < 16; ++k) cnt[k][threadIdx.x] += base;
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kItems; ++it) {
            if (it >= items) break;
            const uint32_t pos = cnt[wv][(uint32_t)(key[it] >> (8 * pass)) & 255u] + rank[it];
            skey[pos] = key[it];
            sval[pos] = val[it];
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kItems; ++it) {
            if (it >= items) break;
            const int i = wv * 64 * items + it * 64 + ln;
            key[it] = skey[i];
            val[it] = sval[i];
        }
        __syncthreads();
    }
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        const int i = wv * 64 * items + it * 64 + ln;
        if (it < items && i < n) {
            keys[i] = key[it];
            vals[i] = val[it];
        }
    }
}

// Codes and the digit counts of all passes; blocks stride over the sites.
template <bool kBox>
__global__ __launch_bounds__(256) void k_codes(const float* __restrict__ xyz, const float* __restrict__ w, int64_t n,
                                               BoxArg box, float* bbox, float4* __restrict__ pts,
                                               uint64_t* __restrict__ keys, uint32_t* __restrict__ hist, uint32_t* err) {
    __shared__ uint32_t cnt[kPasses][256];
    for (int p = 0; p < kPasses; ++p) cnt[p][threadIdx.x] = 0u;
    float b[6];
    for (int c = 0; c < 6; ++c) b[c] = kBox ? box.v[c] : bbox[c];
    if (kBox && blockIdx.x == 0 && threadIdx.x == 0) put_box(box, bbox, err);
    __syncthreads();
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        float4 q;
        if (kBox) {
            q = pack_site(xyz, w, i, err);
            pts[i] = q;
        } else {
            q = pts[i];
        }
        const uint64_t key = morton_code(q, b);
        keys[i] = key;
#pragma unroll
        for (int p = 0; p < kPasses; ++p) atomicAdd(&cnt[p][(uint32_t)(key >> (8 * p)) & 255u], 1u);
    }
    __syncthreads();
    for (int p = 0; p < kPasses; ++p) {
        const uint32_t c = cnt[p][threadIdx.x];
        if (c) atomicAdd(&hist[256 * p + threadIdx.x], c);
    }
}

// One pass.  kFirst: the values are the site numbers themselves.
template <int kItems, bool kFirst>
__global__ __launch_bounds__(kSortThreads) void k_sort_pass(const uint64_t* __restrict__ kin,
                                                            const uint32_t* __restrict__ vin,
                                                            uint64_t* __restrict__ kout, uint32_t* __restrict__ vout,
                                                            int64_t n, int pass, uint32_t* __restrict__ scratch,
                                                            int ntiles) {
    __shared__ uint32_t cnt[4][256];
    __shared__ uint32_t part[4];
    __shared__ uint32_t ticket;
    const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63;
    if (threadIdx.x == 0) ticket = atomicAdd(&scratch[256 * kPasses + pass], 1u);
    for (int k = 0; k < 4; ++k) cnt[k][threadIdx.x] = 0u;
    // digit bases of this pass
    const uint32_t digit_base = scan_256(scratch[256 * pass + threadIdx.x], part);
    const uint32_t tile = ticket;  // the barriers above are passed
    uint32_t* const state = scratch + kSortHead + (size_t)pass * 256 * ntiles;
    const int64_t base = (int64_t)tile * (kSortThreads * kItems) + (int64_t)wv * 64 * kItems;
    uint64_t key[kItems];
    uint32_t val[kItems], rank[kItems];
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        const int64_t i = base + it * 64 + ln;
        const bool ok = i < n;
        key[it] = ok ? kin[i] : 0ull;
        val[it] = kFirst ? (uint32_t)i : (ok ? vin[i] : 0u);
    }
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        const bool ok = base + it * 64 + ln < n;
        const uint32_t d = (uint32_t)(key[it] >> (8 * pass)) & 255u;
        const uint64_t peers = same_digit(d, ok);
        const uint32_t below = lanes_below(peers), before = cnt[wv][d];
        rank[it] = before + below;
        wave_fence();
        if (ok && below == 0) cnt[wv][d] = before + (uint32_t)__popcll(peers);
        wave_fence();
    }
    __syncthreads();
    {
        const int d = threadIdx.x;
        uint32_t total = 0;
        for (int k = 0; k < 4; ++k) {
            const uint32_t c = cnt[k][d];
            cnt[k][d] = total;
            total += c;
        }
        uint32_t before = 0;  // keys of this digit in earlier tiles
        uint32_t* mine = state + (size_t)tile * 256 + d;
        if (tile == 0) {
            __hip_atomic_store(mine, kInclusive | total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            __hip_atomic_store(mine, kPartial | total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            for (uint32_t t = tile - 1;;) {
                const uint32_t v =
                    __hip_atomic_load(state + (size_t)t * 256 + d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (v < kPartial) {  // not published yet
                    __builtin_amdgcn_s_sleep(1);
                    continue;
                }
                before += v & kCountMask;
                if (v >= kInclusive) break;  // tile 0 always is
                --t;
            }
            __hip_atomic_store(mine, kInclusive | (before + total), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        for (int k = 0; k < 4; ++k) cnt[k][d] += digit_base + before;
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        if (base + it * 64 + ln >= n) continue;
        const uint32_t pos = cnt[wv][(uint32_t)(key[it] >> (8 * pass)) & 255u] + rank[it];
        kout[pos] = key[it];
        vout[pos] = val[it];
    }
}

template <int kItems>
static void sort_passes(uint64_t* keys, uint32_t* vals, uint64_t* keys_tmp, uint32_t* vals_tmp, int64_t n,
                        uint32_t* scratch, hipStream_t s) {
    const int64_t tiles = sort_tiles(n);
    uint64_t *ka = keys, *kb = keys_tmp;
    uint32_t *va = vals, *vb = vals_tmp;
    for (int p = 0; p < kPasses; ++p) {
        if (p == 0)
            hipLaunchKernelGGL((k_sort_pass<kItems, true>), dim3((unsigned)tiles), dim3(kSortThreads), 0, s, ka, va, kb,
                               vb, n, p, scratch, (int)tiles);
        else
            hipLaunchKernelGGL((k_sort_pass<kItems, false>), dim3((unsigned)tiles), dim3(kSortThreads), 0, s, ka, va,
                               kb, vb, n, p, scratch, (int)tiles);
        uint64_t* tk = ka; ka = kb; kb = tk;
        uint32_t* tv = va; va = vb; vb = tv;
    }
}

hipError_t launch_sort_sites(const float* xyz, const float* w, int64_t n, const BoxArg* box, float* bbox, float* bpart,
                             float4* pts, uint64_t* keys, uint32_t* vals, uint64_t* keys_tmp, uint32_t* vals_tmp,
                             uint32_t* scratch, uint32_t* err, hipStream_t s) {
    BoxArg b{};
    if (box) {
        b = *box;
    } else {
        const int64_t want = (n + 1023) / 1024;
        const int nblk = (int)(want < kBoxPartials ? want : kBoxPartials);
        hipLaunchKernelGGL(k_pack_box, dim3(nblk), dim3(256), 0, s, xyz, w, n, pts, bpart, err);
        hipLaunchKernelGGL(k_box_final, dim3(1), dim3(256), 0, s, bpart, nblk, bbox, err);
    }
    if (n <= kSmallSort) {
        if (box)
            hipLaunchKernelGGL(k_sort_small<true>, dim3(1), dim3(1024), 0, s, xyz, w, (int)n, b, bbox, pts, keys, vals,
                               err);
        else
            hipLaunchKernelGGL(k_sort_small<false>, dim3(1), dim3(1024), 0, s, xyz, w, (int)n, b, bbox, pts, keys,
                               vals, err);
        return hipGetLastError();
    }
    // (the counts of a block cost up to 2048 global additions, so the blocks are few)
    const int64_t want = (n + 1023) / 1024;
    const unsigned nblk = (unsigned)(want < 512 ? want : 512);
    if (box)
        hipLaunchKernelGGL(k_codes<true>, dim3(nblk), dim3(256), 0, s, xyz, w, n, b, bbox, pts, keys, scratch, err);
    else
        hipLaunchKernelGGL(k_codes<false>, dim3(nblk), dim3(256), 0, s, xyz, w, n, b, bbox, pts, keys, scratch, err);
    switch (sort_items(n)) {
        case 4: sort_passes<4>(keys, vals, keys_tmp, vals_tmp, n, scratch, s); break;
        case 8: sort_passes<8>(keys, vals, keys_tmp, vals_tmp, n, scratch, s); break;
        default: sort_passes<16>(keys, vals, keys_tmp, vals_tmp, n, scratch, s); break;
    }
    return hipGetLastError();  // an even number of passes: the result is in keys, vals
}

// ------------------------------------------------------------------ tree
// One kernel over the sorted positions: the sites in Morton order, coincident
// sites, the boxes of aligned blocks of 64 sites (a wave's own), and the
// binary radix tree (Karras 2012; equal codes are made distinct by their
// position).
//
// Coincident sites share a Morton code, so after the sort they sit in one run
// of equal codes.  Among sites with one position the heaviest keeps its cell
// (ties: lowest original index); the others get weight -inf: their cells are
// empty and their planes, implied by the winner's, are skipped.

__device__ inline int kdelta(const uint64_t* keys, int n, int i, int j) {
    if (j < 0 || j >= n) return -1;
    uint64_t a = keys[i], b = keys[j];
    return a != b ? __clzll((long long)(a ^ b)) : 64 + __clz(i ^ j);
}

__device__ inline float wave_min_f(float v) {
    for (int o = 32; o > 0; o >>= 1) v = fminf(v, __shfl_xor(v, o));
    return v;
}
__device__ inline float wave_max_f(float v) {
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}

// Box and largest weight of some sites, gathered over a wave.
struct BoxAcc {
    float lo[3], hi[3], w;
    __device__ void init() {
        lo[0] = lo[1] = lo[2] = INFINITY;
        hi[0] = hi[1] = hi[2] = -INFINITY;
        w = -INFINITY;
    }
    __device__ void add(float4 p) {
        lo[0] = fminf(lo[0], p.x); lo[1] = fminf(lo[1], p.y); lo[2] = fminf(lo[2], p.z);
        hi[0] = fmaxf(hi[0], p.x); hi[1] = fmaxf(hi[1], p.y); hi[2] = fmaxf(hi[2], p.z);
        w = fmaxf(w, p.w);
    }
    __device__ void add(const NodeChild& c) {
        for (int k = 0; k < 3; ++k) {
            lo[k] = fminf(lo[k], c.lo[k]);
            hi[k] = fmaxf(hi[k], c.hi[k]);
        }
        w = fmaxf(w, c.wmax);
    }
    __device__ NodeChild fold(uint32_t ref) const {
        NodeChild c;
        for (int k = 0; k < 3; ++k) {
            c.lo[k] = wave_min_f(lo[k]);
            c.hi[k] = wave_max_f(hi[k]);
        }
        c.wmax = wave_max_f(w);
        c.ref = ref;
        return c;
    }
};

// Lanes of this wave whose site (p, original index oi, code key, at position i)
// loses its position to another one; open: the lanes that share their code
// with a neighbour.  The runs are read 64 positions at a time, one candidate a
// lane, and the sites that have lost to nobody yet are held against all 64 in
// turn: nearly every site of a run of coincident ones is out after its own
// wave's 64.  One lane for each site, reading its whole run by itself, made the
// hierarchy of 50 places of 8000 sites take 32 ms (400k sites without
// coincident ones: 0.2); this makes it 0.36.
__device__ uint64_t losers(const float4* __restrict__ pts, const uint64_t* __restrict__ keys,
                           const uint32_t* __restrict__ order, int n, int i, float4 p, uint32_t oi, uint64_t key,
                           uint64_t open) {
    const int ln = threadIdx.x & 63, w0 = i - ln;
    uint64_t lost = 0;
    auto lane = [](float v, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); };
    auto against = [&](bool ok, float4 q, uint32_t oq, uint64_t who) {
        for (uint64_t m = who & ~lost; m; m &= m - 1ull) {
            const int L = __builtin_ctzll(m);
            const float w = lane(p.w, L);
            const bool same = ok && q.x == lane(p.x, L) && q.y == lane(p.y, L) && q.z == lane(p.z, L);
            const bool better = q.w > w || (q.w == w && oq < (uint32_t)__builtin_amdgcn_readlane((int)oi, L));
            if (__ballot(same && better)) lost |= 1ull << L;
        }
    };
    against(i < n, p, oi, open);
    // what is left of the runs that begin before this wave or end after it
    for (int dir = -1; dir <= 1; dir += 2) {
        const int edge = dir < 0 ? 0 : min(n - 1 - w0, 63);
        const uint64_t k = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)key, edge) |
                           ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(key >> 32), edge) << 32);
        const uint64_t who = open & __ballot(key == k);
        bool more = true;
        for (int j = w0 + 64 * dir + ln; more && (who & ~lost) != 0; j += 64 * dir) {
            const bool ok = j >= 0 && j < n && keys[j] == k;
            const uint32_t oq = ok ? order[j] : 0u;
            against(ok, ok ? pts[oq] : p, oq, who);
            more = __ballot(ok) == ~0ull;  // the run goes on
        }
    }
    return lost;
}

__global__ __launch_bounds__(256) void k_tree(const float4* __restrict__ pts, const uint64_t* __restrict__ keys,
                                              const uint32_t* __restrict__ order, int n, float4* __restrict__ spts,
                                              uint32_t* __restrict__ inv, NodeChild* __restrict__ blocks, int want_tree,
                                              int* __restrict__ split, uint32_t* __restrict__ up,
                                              int2* __restrict__ range) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    BoxAcc acc;
    acc.init();
    const bool in = i < n;
    const uint32_t oi = in ? order[i] : 0u;
    float4 p = in ? pts[oi] : make_float4(0.f, 0.f, 0.f, 0.f);
    const uint64_t key = in ? keys[i] : 0ull;
    const bool twin = in && ((i > 0 && keys[i - 1] == key) || (i + 1 < n && keys[i + 1] == key));
    const uint64_t twins = __ballot(twin);
    if (twins && ((losers(pts, keys, order, n, i, p, oi, key, twins) >> (threadIdx.x & 63)) & 1ull)) p.w = -INFINITY;
    if (in) {
        inv[oi] = (uint32_t)i;
        spts[i] = p;
        acc.add(p);
    }
    const NodeChild box = acc.fold(0u);
    if ((threadIdx.x & 63) == 0 && i < n) blocks[i >> 6] = box;
    if (!want_tree || i >= n - 1) return;
    const int d = (kdelta(keys, n, i, i + 1) - kdelta(keys, n, i, i - 1)) >= 0 ? 1 : -1;
    const int dmin = kdelta(keys, n, i, i - d);
    int lmax = 2;
    while (kdelta(keys, n, i, i + lmax * d) > dmin) lmax <<= 1;
    int l = 0;
    for (int t = lmax >> 1; t >= 1; t >>= 1)
        if (kdelta(keys, n, i, i + (l + t) * d) > dmin) l += t;
    const int j = i + l * d;
    const int dnode = kdelta(keys, n, i, j);
    int s = 0, t = l;
    do {
        t = (t + 1) >> 1;
        if (kdelta(keys, n, i, i + (s + t) * d) > dnode) s += t;
    } while (t > 1);
    const int gamma = i + s * d + (d < 0 ? -1 : 0);
    const int first = i < j ? i : j, last = i < j ? j : i;
    split[i] = gamma;  // children: positions [first, gamma] and [gamma + 1, last]
    range[i] = make_int2(first, last);
    // parent link of each internal child: parent index and which child it is
    if (first != gamma) up[gamma] = (uint32_t)i << 1;
    if (last != gamma + 1) up[gamma + 1] = ((uint32_t)i << 1) | 1u;
    if (i == 0) up[0] = kNoParent;
}

// ------------------------------------------------------------------ bounds
// Every node covers a contiguous range of sites in Morton order, so each
// child's box and max weight is a reduction over that range (min and max:
// any grouping gives the same bits).  Boxes of aligned blocks of 64, 64^2 and
// 64^3 sites are kept; a range is its partial head and tail at each level and
// the whole blocks between, and one wave reads 64 of them at a time.  One
// lane for each node, walking up to 128 sites by itself, and a table of every
// power of two of blocks (a launch for each) took 44 us for the nodes of a
// thousand sites and 210 us for those of a million; this takes 6 and 60.

// level k + 1 from level k: one wave per block of 64
__global__ __launch_bounds__(256) void k_box_level(const NodeChild* __restrict__ prev, int nprev,
                                                   NodeChild* __restrict__ cur, int ncur) {
    const int b = (int)((blockIdx.x * 256 + threadIdx.x) >> 6), ln = threadIdx.x & 63;
    if (b >= ncur) return;
    BoxAcc a;
    a.init();
    if (b * 64 + ln < nprev) a.add(prev[b * 64 + ln]);
    const NodeChild c = a.fold(0u);
    if (ln == 0) cur[b] = c;
}

constexpr int kBoxLevels = 3;
struct BoxTable {
    const NodeChild* lv[kBoxLevels];
};

// Wave-wide: the box of positions [f, l].
__device__ inline NodeChild range_box(const float4* __restrict__ spts, const BoxTable& t, int f, int l, uint32_t ref) {
    const int ln = threadIdx.x & 63;
    BoxAcc a;
    a.init();
    int lo = f, hi = l + 1;  // of the current level, [lo, hi)
    if (hi - lo <= 128) {
        for (int i = lo + ln; i < hi; i += 64) a.add(spts[i]);
        return a.fold(ref);
    }
    int b0 = (lo + 63) >> 6, b1 = hi >> 6;
    if (lo + ln < b0 * 64) a.add(spts[lo + ln]);
    if (b1 * 64 + ln < hi) a.add(spts[b1 * 64 + ln]);
#pragma unroll
    for (int k = 0; k < kBoxLevels; ++k) {
        lo = b0;
        hi = b1;
        if (k == kBoxLevels - 1 || hi - lo <= 128) {
            for (int i = lo + ln; i < hi; i += 64) a.add(t.lv[k][i]);
            break;
        }
        b0 = (lo + 63) >> 6;
        b1 = hi >> 6;
        if (lo + ln < b0 * 64) a.add(t.lv[k][lo + ln]);
        if (b1 * 64 + ln < hi) a.add(t.lv[k][b1 * 64 + ln]);
    }
    return a.fold(ref);
}

// Both child records of the nodes above the leaves, and the leaf record of
// every site below them: (node << 1) | which child.  A wave looks at 64 nodes
// and works on those of more than leaf_size sites (about four) in turn.
__global__ __launch_bounds__(256) void k_nodes(const float4* __restrict__ spts, int n, const int* __restrict__ split,
                                               const int2* __restrict__ range, BoxTable table,
                                               Node* __restrict__ nodes, uint32_t* __restrict__ leaf_of, int leaf_size) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    const int ln = threadIdx.x & 63;
    int2 r = make_int2(0, -1);
    int g = 0;
    if (i < n - 1) {
        r = range[i];
        g = split[i];
    }
    for (uint64_t m = __ballot(r.y - r.x + 1 > leaf_size); m; m &= m - 1ull) {
        const int L = __builtin_ctzll(m);
        const int node = i - ln + L;
        const int first = __builtin_amdgcn_readlane(r.x, L), last = __builtin_amdgcn_readlane(r.y, L);
        const int gamma = __builtin_amdgcn_readlane(g, L);
        for (int s = 0; s < 2; ++s) {
            const int f = s ? gamma + 1 : first, l = s ? last : gamma;
            const int cnt = l - f + 1;
            const bool leaf = cnt <= leaf_size;
            const NodeChild c =
                range_box(spts, table, f, l, leaf ? leaf_ref((uint32_t)f, (uint32_t)cnt) : (uint32_t)(gamma + s));
            if (ln == 0) nodes[node].c[s] = c;
            if (leaf && ln < cnt) leaf_of[f + ln] = ((uint32_t)node << 1) | (uint32_t)s;
        }
    }
}

size_t box_table_size(int64_t n) {
    size_t total = 0;
    for (int k = 0; k < kBoxLevels; ++k) {
        n = (n + 63) / 64;
        total += (size_t)n;
    }
    return total;
}

hipError_t launch_tree(const float4* pts, const uint64_t* keys, const uint32_t* order, int64_t n, float4* spts,
                       uint32_t* inv, NodeChild* table, int* split, uint32_t* up, int2* range, Node* nodes,
                       uint32_t* leaf_of, int leaf_size, hipStream_t s) {
    const bool tree = n > leaf_size;
    const unsigned blocks = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(k_tree, dim3(blocks), dim3(256), 0, s, pts, keys, order, (int)n, spts, inv, table, tree ? 1 : 0,
                       split, up, range);
    if (!tree) return hipGetLastError();
    BoxTable t;
    int64_t size[kBoxLevels];
    NodeChild* at = table;
    int64_t c = n;
    for (int k = 0; k < kBoxLevels; ++k) {
        c = (c + 63) / 64;
        size[k] = c;
        t.lv[k] = at;
        // a level is read only where the one below has more than 128 blocks
        if (k > 0 && size[k - 1] > 128)
            hipLaunchKernelGGL(k_box_level, dim3((unsigned)((c * 64 + 255) / 256)), dim3(256), 0, s, t.lv[k - 1],
                               (int)size[k - 1], at, (int)c);
        at += c;
    }
    hipLaunchKernelGGL(k_nodes, dim3(blocks), dim3(256), 0, s, spts, (int)n, split, range, t, nodes, leaf_of,
                       leaf_size);
    return hipGetLastError();
}

}  // namespace vd
