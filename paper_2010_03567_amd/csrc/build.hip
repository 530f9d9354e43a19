// build.hip -- integer mapping, curve keys, the octree's nodes from the sorted
// keys (all levels at once) and the upward multipole pass on gfx950.
//
// Paper: Sec. "Integer coordinates" (fixed-point positions, two's-complement
// nearest image), Sec. "Non-periodic potentials" (isolated root mapped into a
// sub-range of the integer space), Sec. "Geometry of the tree" (nested cubes
// along a space-filling curve, node split only above B particles),
// Sec. "One-sided multipole expansion" (moments about the centre of mass),
// Sec. "Fast multipole method" first phase (moments from daughter moments).
//
// Design: the build is enqueued without a host round trip; sizes that only the
// device knows are read there.  The nodes of all levels are found from the
// sorted keys at once (see "nodes"); each level occupies one contiguous index
// range, in curve order.  Multipoles go level by level from the deepest up.
#include <cstring>
#include <utility>

#include "g4_internal.h"

#define TWO32 4294967296.0
#define TWO31 2147483648.0
#define TWO30 1073741824.0

static const int kBlock = 256;

static inline int grid_for(int64_t work, int max_blocks = 4096)
{
    int64_t b = (work + kBlock - 1) / kBlock;
    if (b < 1) b = 1;
    if (b > max_blocks) b = max_blocks;
    return (int)b;
}

// ------------------------------------------------------------------ layout
int g4_layout(const g4_tree_params *tp, int64_t n, WsLayout *L)
{
    int B = tp->leaf_max < 1 ? 1 : tp->leaf_max;
    int maxd = tp->max_depth < 1 ? 1 : (tp->max_depth > G4_MAXLEV ? G4_MAXLEV : tp->max_depth);
    // every node is a leaf (disjoint, non-empty: <= n) or an internal node
    // (disjoint within a level, > B particles each: <= n/(B+1) per level)
    int64_t cap = n + (int64_t)maxd * (n / (B + 1)) + 2;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off += (bytes + 255) & ~(size_t)255;
        return o;
    };
    L->cap = cap;
    L->ctr = take(sizeof(DevCounters));
    L->keys0 = take((size_t)n * 8);
    L->keys1 = take((size_t)n * 8);
    L->perm0 = take((size_t)n * 4);
    L->perm1 = take((size_t)n * 4);
    L->parts = take((size_t)n * 16);
    L->bfirst = take((size_t)cap * 4);
    L->bcount = take((size_t)cap * 4);
    L->parent = take((size_t)cap * 4);
    L->wn = take((size_t)cap * sizeof(WNode));
    L->q3 = take((size_t)cap * 10 * 4);
    L->mom = take((size_t)cap * MOM_STRIDE * 8);
    L->aseed = take((size_t)n * 4);
    L->leafof = take((size_t)n * 4);
    // a walk grid never has more wavefronts than work items (<= n), rounded up to whole blocks of 4
    int64_t waves = ((n > 0 ? n : 1) + 3) / 4 * 4;
    if (waves > G4_WALK_MAX_WAVES) waves = G4_WALK_MAX_WAVES;
    L->spill_waves = waves;
    L->spill = take((size_t)waves * G4_WALK_SPILL * 16);
    L->srtab = take((size_t)G4_SRTAB_FUNCS * G4_SRTAB_MAX * 16);
    // digit tables of the key sort and of the forest's sort by box
    L->sort_bytes = g4_radix_sort_temp_bytes(n > 0 ? n : 1);
    L->sort_tmp = take(L->sort_bytes);
    L->total = off;
    return G4_OK;
}

// ------------------------------------------------------------ quantisation
__global__ void k_quantize(const double *__restrict__ pos, int64_t n, int periodic, double inv, double ox,
                           double oy, double oz, uint32_t *__restrict__ X, uint32_t *__restrict__ Y,
                           uint32_t *__restrict__ Z, int32_t *flag)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        double o[3] = {ox, oy, oz};
        uint32_t out[3];
        for (int k = 0; k < 3; k++) {
            double t = (pos[3 * i + k] - o[k]) * inv;
            double f = floor(t);
            if (periodic) {
                double w = f - TWO32 * floor(f * (1.0 / TWO32));
                out[k] = (uint32_t)(uint64_t)w;
            } else {
                if (f < 0.0 || f >= TWO31) {
                    atomicOr(flag, 1);
                    f = f < 0.0 ? 0.0 : TWO31 - 1.0;
                }
                out[k] = (uint32_t)(TWO30 + f);
            }
        }
        X[i] = out[0];
        Y[i] = out[1];
        Z[i] = out[2];
    }
}

int g4_launch_quantize(g4_ctx *ctx, const double *pos, int64_t n, const g4_tree_params *tp, uint32_t *x,
                       uint32_t *y, uint32_t *z, int32_t *flag)
{
    double inv = tp->periodic ? TWO32 / tp->box : TWO31 / tp->box;
    if (!tp->periodic)
        if (int st = g4_launch_zero(ctx, flag, 4)) return st;
    if (n > 0)
        k_quantize<<<grid_for(n), kBlock, 0, ctx->stream>>>(pos, n, tp->periodic, inv, tp->origin[0], tp->origin[1],
                                                           tp->origin[2], x, y, z, flag);
    G4_HIP(ctx, hipGetLastError());
    // the periodic map cannot fail: no read-back, so the host does not wait here
    if (tp->periodic) return G4_OK;
    int32_t h = 0;
    G4_HIP(ctx, hipMemcpyAsync(&h, flag, 4, hipMemcpyDeviceToHost, ctx->stream));
    G4_HIP(ctx, hipStreamSynchronize(ctx->stream));
    if (h) return g4_set_err(ctx, G4_EROOT, "particle outside the isolated root cube");
    return G4_OK;
}

// ------------------------------------------------------------------- keys
__device__ __forceinline__ uint64_t spread3(uint32_t v)
{
    uint64_t x = v & 0x1fffffu;
    x = (x | x << 32) & 0x1f00000000ffffull;
    x = (x | x << 16) & 0x1f0000ff0000ffull;
    x = (x | x << 8) & 0x100f00f00f00f00full;
    x = (x | x << 4) & 0x10c30c30c30c30c3ull;
    x = (x | x << 2) & 0x1249249249249249ull;
    return x;
}

// Peano-Hilbert index of a cell of the 2^21 grid, from its 21-bit
// coordinates, by Skilling's method ("Programming the Hilbert curve", AIP
// Conf. Proc. 707, 2004): from the top bit down, the coordinates are reflected
// and exchanged so that each level's sub-cube is entered in the curve's own
// orientation, then Gray-decoded; the result interleaved x, y, z from the top
// bit is the index.  Its level-l digit (bits 3 (21 - l) .. +2) labels one
// octant of the level-(l - 1) cube, as the Morton digit does, so both keys
// cut the same nested cubes.
__device__ __forceinline__ uint64_t ph_key21(uint32_t x, uint32_t y, uint32_t z)
{
    uint32_t c[3] = {x, y, z};
    for (uint32_t q = 1u << 20; q > 1u; q >>= 1) {
        const uint32_t p = q - 1u;
        for (int i = 0; i < 3; i++) {
            if (c[i] & q) {
                c[0] ^= p;  // reflect the low bits of the first coordinate
            } else {
                const uint32_t t = (c[0] ^ c[i]) & p;  // exchange the low bits with coordinate i
                c[0] ^= t;
                c[i] ^= t;
            }
        }
    }
    c[1] ^= c[0];
    c[2] ^= c[1];
    uint32_t t = 0;
    for (uint32_t q = 1u << 20; q > 1u; q >>= 1)
        if (c[2] & q) t ^= q - 1u;
    return (spread3(c[0] ^ t) << 2) | (spread3(c[1] ^ t) << 1) | spread3(c[2] ^ t);
}

// Curve key from the top 21 bits of each root-relative coordinate: Morton
// (bit interleaving; the level-l octant digit (x<<2 | y<<1 | z) sits at bit
// 3 (21 - l)) or Peano-Hilbert.
__device__ __forceinline__ uint64_t curve_key(uint32_t x, uint32_t y, uint32_t z, int drop, uint32_t corner, int kind)
{
    const uint32_t rx = (x - corner) >> drop, ry = (y - corner) >> drop, rz = (z - corner) >> drop;
    return kind == 1 ? ph_key21(rx, ry, rz) : (spread3(rx) << 2) | (spread3(ry) << 1) | spread3(rz);
}

// Curve keys, the identity permutation, and the particles packed as one
// 16-byte record each in caller order (pk), so that the gather into key
// order reads one record per particle instead of four separate words.
__global__ void k_keys(const uint32_t *__restrict__ X, const uint32_t *__restrict__ Y,
                       const uint32_t *__restrict__ Z, const float *__restrict__ m, int64_t n, int drop,
                       uint32_t corner, int kind, uint64_t *__restrict__ keys, uint32_t *__restrict__ perm,
                       uint4 *__restrict__ pk)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t x = X[i], y = Y[i], z = Z[i];
        keys[i] = curve_key(x, y, z, drop, corner, kind);
        perm[i] = (uint32_t)i;
        pk[i] = make_uint4(x, y, z, __float_as_uint(m[i]));
    }
}

__global__ void k_gather(const uint4 *__restrict__ pk, const uint32_t *__restrict__ perm, int64_t n,
                         uint4 *__restrict__ parts)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        parts[i] = pk[perm[i]];
}

// the packed caller-order records live in the moments buffer, which is
// free from the key pass until the upward pass (it holds >= 160 bytes per
// particle, the records 16)
static inline uint4 *packed_staging(g4_tree *t) { return reinterpret_cast<uint4 *>(t->mom); }

// sum over the eight lanes of a group; every lane ends with the same bits
template <typename T>
__device__ __forceinline__ T grp8_sum(T v)
{
    v += __shfl_xor(v, 1, 8);
    v += __shfl_xor(v, 2, 8);
    v += __shfl_xor(v, 4, 8);
    return v;
}

// ------------------------------------------------------------------ nodes
// All levels of the octree at once, from the sorted keys.  With
//   d(i) = common leading octants of the keys of particles i - 1 and i (-1 where
//          a box starts) and
//   D(i) = the largest number of common octants of any B + 1 consecutive
//          particles around i (-1 if there are none),
// the level-l cell of particle i starts at i iff d(i) < l, and holds more than B
// particles iff l <= D(i); so the leaf of i is at level L(i) = min(D(i) + 1, max
// depth), and the nodes that start at i are those of levels d(i) + 1 .. L(i).
// A node's number is its level's base plus the count of earlier starts of that
// level (nodes of a level are in curve order, the children of a node
// consecutive); the particle that ends a cell, d(j) < l <= L(j - 1), knows the
// end and the last child of the node before it.
//
// Four launches in place of one per level: k_levels (d, L, starts per block and
// level), k_level_scan, k_emit, k_records.  Bound by reading the keys; a level by
// level split cost a launch and a chain of dependent loads per level, 22 of them:
// 0.89 -> 0.41 ms at 2^24 particles (leaf 32), 0.09 -> 0.02 ms at 8192 (leaf 8).
#define LV_TILE 1024          // particles per block, one per thread
#define LV_WAVES (LV_TILE / 64)
#define LV_MAXB 1024          // leaf sizes whose windows fit the block's LDS
#define NLEV (G4_MAXLEV + 1)

// common leading octants of two 63-bit keys
__device__ __forceinline__ int common_octants(uint64_t a, uint64_t b)
{
    const uint64_t x = a ^ b;
    return x ? (__builtin_clzll(x) - 1) / 3 : G4_MAXLEV;
}

// 1 + common octants of particles s and s + B (0: not both in one box)
__device__ __forceinline__ uint32_t window_octants(const uint64_t *__restrict__ keys, const uint32_t *__restrict__ box,
                                                   int64_t s, int64_t n, int64_t B)
{
    if (s < 0 || s + B >= n || (box && box[s] != box[s + B])) return 0u;
    return 1u + (uint32_t)common_octants(keys[s], keys[s + B]);
}

// bits lo .. hi (none if lo > hi)
__device__ __forceinline__ uint32_t level_bits(int lo, int hi) { return lo > hi ? 0u : (2u << hi) - (1u << lo); }

// or of the 64 lanes' masks (uniform)
__device__ __forceinline__ uint32_t wave_or(uint32_t m)
{
    for (int off = 32; off > 0; off >>= 1) m |= (uint32_t)__shfl_xor((int)m, off);
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)m);
}

// Running maxima are taken on four bytes (in memory 16) at a time, at any alignment; bytes are below 128.
__device__ __forceinline__ uint32_t load4(const uint8_t *p)
{
    uint32_t v;
    __builtin_memcpy(&v, p, 4);
    return v;
}
__device__ __forceinline__ uint32_t max4(uint32_t a, uint32_t b)
{
    const uint32_t ge = ((a | 0x80808080u) - b) & 0x80808080u, mask = (ge >> 7) * 255u;
    return (a & mask) | (b & ~mask);
}

// For leaf sizes beyond LV_MAXB: windows in memory (LV_PAD zero bytes before and after),
// and their running maxima over `taps` values `step` apart, the last one at most `most` back.
// Eight values a pass: doubling, byte by byte, took 17 launches at B = 10^5.  Whole builds, ms,
// by a split per level / by doubling / now: 2 10^6 particles at leaf 10^5 0.37 / 0.42 / 0.37,
// 1.6 10^7 at leaf 4097 2.30 / 2.55 / 2.40.
#define LV_PAD 16
__global__ void k_window(const uint64_t *__restrict__ keys, const uint32_t *__restrict__ box, int64_t n, int64_t B,
                         uint8_t *__restrict__ out, uint8_t *__restrict__ other)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        out[i] = (uint8_t)window_octants(keys, box, i, n, B);
    if (blockIdx.x == 0 && threadIdx.x < LV_PAD) {
        out[(int)threadIdx.x - LV_PAD] = out[n + threadIdx.x] = 0;
        other[(int)threadIdx.x - LV_PAD] = 0;
    }
}
__global__ void k_window_max(const uint8_t *__restrict__ in, int64_t n, int64_t step, int taps, int64_t most,
                             uint8_t *__restrict__ out)
{
    const int64_t stride = 16 * (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = 16 * (blockIdx.x * (int64_t)blockDim.x + threadIdx.x); i < n; i += stride) {
        uint4 v, u;
        __builtin_memcpy(&v, in + i, 16);
        for (int t = 1; t < taps; t++) {
            const int64_t j = i - (t * step < most ? t * step : most);
            if (j > -16) {
                __builtin_memcpy(&u, in + j, 16);
                v = make_uint4(max4(v.x, u.x), max4(v.y, u.y), max4(v.z, u.z), max4(v.w, u.w));
            }
        }
        *reinterpret_cast<uint4 *>(out + i) = v;
    }
}

// lev[i] = (d(i) + 1) | L(i) << 8, and the starts of every level per block
// (cnt[level][block]).  wmax: 1 + D(i) already in memory, or null (then B <= LV_MAXB, or n <= B: no windows).
__global__ __launch_bounds__(LV_TILE) void k_levels(const uint64_t *__restrict__ keys, const uint32_t *__restrict__ box,
                                                    const uint8_t *__restrict__ wmax, int64_t n, int64_t B, int maxd,
                                                    uint16_t *__restrict__ lev, uint32_t *__restrict__ cnt, uint32_t nblk)
{
    __shared__ __attribute__((aligned(16))) uint8_t wbuf[2][LV_PAD + LV_TILE + LV_MAXB + 4];
    __shared__ uint32_t total[NLEV];
    const int64_t base = blockIdx.x * (int64_t)LV_TILE, i = base + threadIdx.x;
    if (threadIdx.x < NLEV) total[threadIdx.x] = 0;
    uint32_t top = 0;  // 1 + D(i)
    if (wmax || B >= n) {
        if (wmax && i < n) top = wmax[i];
        __syncthreads();
    } else {
        // window maxima over [i - B, i], from B particles before the tile on: four values a pass
        const int len = LV_TILE + (int)B, words = (len + 3) / 4;
        auto w = [&](int c, int k) { return &wbuf[c][LV_PAD + k]; };
        for (int k = threadIdx.x; k < 4 * words; k += LV_TILE)
            *w(0, k) = k < len ? (uint8_t)window_octants(keys, box, base - B + k, n, B) : (uint8_t)0;
        if (threadIdx.x < 2 * LV_PAD) wbuf[threadIdx.x / LV_PAD][threadIdx.x % LV_PAD] = 0;
        __syncthreads();
        int cur = 0, span = 1;
        for (; 4 * span <= (int)B + 1; span *= 4) {
            for (int q = threadIdx.x; q < words; q += LV_TILE) {
                uint32_t v = load4(w(cur, 4 * q));
#pragma unroll
                for (int t = 1; t < 4; t++) {
                    const int j = 4 * q - t * span;
                    if (j > -4) v = max4(v, load4(w(cur, j)));
                }
                *reinterpret_cast<uint32_t *>(w(cur ^ 1, 4 * q)) = v;
            }
            cur ^= 1;
            __syncthreads();
        }
        const int k = (int)B + threadIdx.x, most = (int)B + 1 - span;
        for (int o = 0; o < most; o += span) top = max(top, (uint32_t)*w(cur, k - o));
        top = max(top, (uint32_t)*w(cur, k - most));
    }
    int d1 = NLEV + 1, L = 0;  // d + 1 and L; past the end nothing starts
    if (i < n) {
        d1 = i == 0 || (box && box[i] != box[i - 1]) ? 0 : 1 + common_octants(keys[i - 1], keys[i]);
        L = min((int)top, maxd);
        lev[i] = (uint16_t)(d1 | L << 8);
    }
    for (uint32_t m = wave_or(level_bits(d1, L)); m; m &= m - 1) {  // the few levels that start among 64 neighbours
        const int l = __builtin_ctz(m);
        const uint32_t c = (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(d1 <= l && l <= L));
        if ((threadIdx.x & 63) == 0) atomicAdd(&total[l], c);
    }
    __syncthreads();
    if (threadIdx.x < NLEV) cnt[(size_t)threadIdx.x * nblk + blockIdx.x] = total[threadIdx.x];
}

// exclusive scan of one level's block counts (block = level), its size; block 0 resets the tree's counters
__global__ __launch_bounds__(1024) void k_level_scan(uint32_t *__restrict__ cnt, uint32_t nblk, DevCounters *__restrict__ C)
{
    __shared__ uint32_t wsum[16];
    uint32_t *row = cnt + (size_t)blockIdx.x * nblk;
    const uint32_t lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t carry = 0;
    for (uint32_t c0 = 0; c0 < nblk; c0 += 1024) {
        const uint32_t k = c0 + threadIdx.x, x = k < nblk ? row[k] : 0u;
        uint32_t incl = x;
#pragma unroll
        for (uint32_t off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(incl, off);
            if (lane >= off) incl += y;
        }
        if (lane == 63) wsum[wv] = incl;
        __syncthreads();
        uint32_t before = carry, all = carry;
        for (uint32_t v = 0; v < 16; v++) {
            before += v < wv ? wsum[v] : 0u;
            all += wsum[v];
        }
        if (k < nblk) row[k] = before + incl - x;
        carry = all;
        __syncthreads();
    }
    if (threadIdx.x == 0) C->lvl_count[blockIdx.x] = carry;
    if (blockIdx.x == 0 && threadIdx.x < 18) C->stat[threadIdx.x] = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) C->flags = 0;
    if (blockIdx.x == 0 && threadIdx.x >= NLEV && threadIdx.x < G4_MAXLEV + 4) C->lvl_count[threadIdx.x] = 0;
}

__global__ __launch_bounds__(LV_TILE) void k_emit(const uint16_t *__restrict__ lev, int64_t n, int maxd,
                                                  const uint32_t *__restrict__ cnt, uint32_t nblk,
                                                  DevCounters *__restrict__ C, uint32_t *__restrict__ bfirst,
                                                  uint32_t *__restrict__ bend, uint32_t *__restrict__ parent,
                                                  uint32_t *__restrict__ cfirst, uint32_t *__restrict__ cend, int64_t cap)
{
    __shared__ uint32_t off[NLEV][LV_WAVES];  // starts per wavefront, then the number of its first one
    const int64_t i = blockIdx.x * (int64_t)LV_TILE + threadIdx.x;
    const uint32_t lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int d1 = NLEV + 1, L = 0, Lp = 0;  // Lp: leaf level of particle i - 1
    if (i < n) {
        const uint16_t v = lev[i];
        d1 = v & 0xff;
        L = v >> 8;
        Lp = i > 0 ? lev[i - 1] >> 8 : -1;
    }
    if (lane < NLEV) off[lane][wv] = 0;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const bool last = i == n - 1;
    const uint32_t ms = wave_or(level_bits(d1, L));
    for (uint32_t m = ms; m; m &= m - 1) {
        const int l = __builtin_ctz(m);
        const uint32_t c = (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(d1 <= l && l <= L));
        if (lane == 0) off[l][wv] = c;
    }
    // levels to go through: those that start or end here, the ones above (parents) and below (last children)
    uint32_t mt = ms | wave_or(level_bits(d1, Lp) | (last ? level_bits(0, L) : 0u));
    mt = (mt | mt >> 1 | mt << 1) & level_bits(0, maxd);
    __syncthreads();
    uint32_t size = 0, run = 0;
    if (wv == 0) {
        // each level's base: the sizes of the levels above it, summed across the lanes
        size = lane <= (uint32_t)maxd ? C->lvl_count[lane] : 0u;
        run = size;
#pragma unroll
        for (uint32_t o = 1; o < 32; o <<= 1) {
            const uint32_t y = __shfl_up(run, o);
            if (lane >= o) run += y;
        }
        run -= size;
    }
    if (threadIdx.x <= (unsigned)maxd) {
        const uint32_t l = threadIdx.x;
        if (blockIdx.x == 0) {
            C->lvl_start[l] = run;
            if (l == (uint32_t)maxd) C->node_count = (uint32_t)min((int64_t)run + size, cap);
        }
        run += cnt[(size_t)l * nblk + blockIdx.x];
        for (uint32_t w = 0; w < LV_WAVES; w++) {
            const uint32_t c = off[l][w];
            off[l][w] = run;
            run += c;
        }
    }
    __syncthreads();
    uint32_t up = 0xffffffffu;  // node of the level above that holds particle i
    bool up_starts = false;
    uint32_t closed = 0xffffffffu;  // node of the level above that ends before particle i
    bool over = false;
    auto put = [&](uint32_t *a, uint32_t q, uint32_t v) {
        if ((int64_t)q < cap) a[q] = v;
        else over = true;
    };
    for (; mt; mt &= mt - 1) {
        const int l = __builtin_ctz(mt);
        const bool starts = d1 <= l && l <= L;
        const uint64_t m = __builtin_amdgcn_ballot_w64(starts);
        const uint32_t q = off[l][wv] + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        if (i >= n) continue;
        if (closed != 0xffffffffu) put(cend, closed, q);  // its children end where the next ones start
        closed = 0xffffffffu;
        if (d1 <= l && l <= Lp) {
            closed = q - 1;
            put(bend, closed, (uint32_t)i);
        }
        if (starts) {
            put(bfirst, q, (uint32_t)i);
            put(parent, q, up);
            if (up_starts) put(cfirst, up, q);
        }
        const uint32_t here = q + (starts ? 1u : 0u) - 1u;
        if (last && l <= L) put(bend, here, (uint32_t)n);
        if (last && l > 0 && l - 1 <= L) put(cend, up, here + 1u);
        up = here;
        up_starts = starts;
    }
    if (over) atomicOr(&C->flags, 2u);
}

__global__ void k_records(DevCounters *__restrict__ C, const uint16_t *__restrict__ lev, const uint4 *__restrict__ parts,
                          const uint32_t *__restrict__ bfirst, uint32_t *__restrict__ bcount,
                          const uint32_t *__restrict__ cfirst, const uint32_t *__restrict__ cend, WNode *__restrict__ wn,
                          int B, int maxd, int S, uint32_t corner)
{
    const uint32_t nn = C->node_count;
    uint32_t end[NLEV];  // end of every level but the last
#pragma unroll
    for (int l = 0; l < G4_MAXLEV; l++) end[l] = l < maxd ? C->lvl_start[l + 1] : 0xffffffffu;
    for (uint32_t q = blockIdx.x * blockDim.x + threadIdx.x; q < nn; q += gridDim.x * blockDim.x) {
        int level = 0;
#pragma unroll
        for (int l = 0; l < G4_MAXLEV; l++) level += q >= end[l] ? 1 : 0;
        const uint32_t first = bfirst[q], count = bcount[q] - first;  // k_emit left the end there
        bcount[q] = count;
        const bool split = (lev[first] >> 8) > level;
        // the geometric centre of the cube from any particle inside it
        const uint4 p0 = parts[first];
        const int sh = S - level;
        WNode w;
        uint32_t pc[3] = {p0.x, p0.y, p0.z}, g[3];
        for (int k = 0; k < 3; k++) {
            uint64_t rel = (uint64_t)(uint32_t)(pc[k] - corner);
            g[k] = (uint32_t)((uint64_t)corner + ((rel >> sh) << sh) + (1ull << (sh - 1)));
        }
        w.gx = g[0];
        w.gy = g[1];
        w.gz = g[2];
        w.cx = g[0];
        w.cy = g[1];
        w.cz = g[2];
        w.mass = 0.f;
        for (int k = 0; k < 6; k++) w.q[k] = 0.f;
        if (split) {
            w.next = cfirst[q];
            w.num = cend[q] - w.next;
            w.meta = (uint32_t)level;
        } else {
            w.next = first;
            w.num = count;
            w.meta = (uint32_t)level | WN_LEAF;
            if (count > (uint32_t)B) atomicOr(&C->flags, 1u);
        }
        wn[q] = w;
    }
}

// stable sort of the 63-bit curve keys (keys0, values perm0); the result is
// left in keys1 / perm1 (the views are swapped when the passes end in the
// first pair)
static int sort_keys(g4_ctx *ctx, g4_tree *t)
{
    int alt = 0;
    if (int st = g4_radix_sort_u64(ctx, t->keys0, t->keys1, t->perm0, t->perm1, t->n, 0, 3 * G4_MAXLEV, t->sort_tmp,
                                   t->sort_tmp_bytes, &alt))
        return st;
    if (!alt) {
        std::swap(t->keys0, t->keys1);
        std::swap(t->perm0, t->perm1);
    }
    return G4_OK;
}

// nodes from the sorted keys (keys1, parts); box: box of every sorted particle
// of a forest, or null.  Scratch: keys0 (levels, window maxima), the sort's
// tables (starts per block), the octupoles' place (children of each node).
static int launch_nodes(g4_ctx *ctx, g4_tree *t, const uint32_t *box)
{
    hipStream_t s = ctx->stream;
    const int64_t n = t->n, B = t->tp.leaf_max;
    const int maxd = t->tp.max_depth < 1 ? 1 : (t->tp.max_depth > G4_MAXLEV ? G4_MAXLEV : t->tp.max_depth);
    uint16_t *lev = reinterpret_cast<uint16_t *>(t->keys0);
    uint32_t *cnt = static_cast<uint32_t *>(t->sort_tmp);
    uint32_t *cfirst = reinterpret_cast<uint32_t *>(t->q3), *cend = cfirst + t->cap;
    const uint32_t nblk = (uint32_t)((n + LV_TILE - 1) / LV_TILE);
    if ((size_t)NLEV * nblk * sizeof(uint32_t) > t->sort_tmp_bytes)
        return g4_set_err(ctx, G4_ENOMEM, "level tables exceed the sort scratch");
    const uint8_t *wmax = nullptr;
    if (B > LV_MAXB && n > B) {  // a set of at most B particles has no window
        // levels, then two byte arrays between their pads: 4 n bytes and 100 of the 8 n
        auto at = [&](int64_t bytes) { return reinterpret_cast<uint8_t *>(t->keys0) + (bytes + 15) / 16 * 16; };
        uint8_t *w[2] = {at(2 * n + LV_PAD), at(2 * n + LV_PAD) + (n + 15) / 16 * 16 + 2 * LV_PAD};
        const unsigned grid = grid_for((n + 15) / 16);
        int cur = 0;
        int64_t span = 1;
        k_window<<<grid_for(n), kBlock, 0, s>>>(t->keys1, box, n, B, w[0], w[1]);
        for (; 8 * span <= B + 1; span *= 8, cur ^= 1)
            k_window_max<<<grid, kBlock, 0, s>>>(w[cur], n, span, 8, 7 * span, w[cur ^ 1]);
        const int64_t most = B + 1 - span;
        k_window_max<<<grid, kBlock, 0, s>>>(w[cur], n, span, 1 + (int)((most + span - 1) / span), most, w[cur ^ 1]);
        wmax = w[cur ^ 1];
    }
    k_levels<<<nblk, LV_TILE, 0, s>>>(t->keys1, box, wmax, n, B, maxd, lev, cnt, nblk);
    k_level_scan<<<NLEV, 1024, 0, s>>>(cnt, nblk, t->ctr);
    k_emit<<<nblk, LV_TILE, 0, s>>>(lev, n, maxd, cnt, nblk, t->ctr, t->bfirst, t->bcount, t->parent, cfirst, cend, t->cap);
    // the node count is known on the device only; about n / 3 at small leaves, n / 8 at 32
    k_records<<<grid_for(n, 2048), kBlock, 0, s>>>(t->ctr, lev, t->parts, t->bfirst, t->bcount, cfirst, cend, t->wn, (int)B,
                                                  maxd, t->S, t->corner);
    G4_HIP(ctx, hipGetLastError());
    return G4_OK;
}

int g4_launch_build(g4_ctx *ctx, g4_tree *t, const g4_particles *p)
{
    hipStream_t s = ctx->stream;
    const int64_t n = t->n;
    k_keys<<<grid_for(n), kBlock, 0, s>>>(p->x, p->y, p->z, p->mass, n, t->S - G4_MAXLEV, t->corner,
                                          t->tp.key_kind, t->keys0, t->perm0, packed_staging(t));
    G4_HIP(ctx, hipGetLastError());
    if (int st = sort_keys(ctx, t)) return st;
    // sorted keys now live in keys1, the permutation in perm1
    k_gather<<<grid_for(n), kBlock, 0, s>>>(packed_staging(t), t->perm1, n, t->parts);
    G4_HIP(ctx, hipGetLastError());
    return launch_nodes(ctx, t, nullptr);
}

// ---------------------------------------------------------------- moments
// packed symmetric index tables
__constant__ int c_i3[10][3] = {{0, 0, 0}, {0, 0, 1}, {0, 0, 2}, {0, 1, 1}, {0, 1, 2},
                                {0, 2, 2}, {1, 1, 1}, {1, 1, 2}, {1, 2, 2}, {2, 2, 2}};

__device__ __forceinline__ int p2i(int i, int j)
{
    // packed index of (i, j) in xx xy xz yy yz zz
    if (i > j) { int t = i; i = j; j = t; }
    return i == 0 ? j : (i == 1 ? 2 + j : 5);
}

// Upward pass for one level: leaves from their particles (P2M), internal
// nodes from their children (M2M by the parallel-axis shift):
//   Q2 = sum_c [Q2_c + M_c d d],
//   Q3 = sum_c [Q3_c + d(x)Q2_c (three placements) + M_c d d d],  d = s_c - s.
// Eight lanes take one node: a leaf's particles go to the lanes in turn, an
// internal node's children one per lane; the sums close with a fixed
// butterfly over the group, so the result does not depend on timing.
template <typename T>
__device__ __forceinline__ void moments_level(const DevCounters *__restrict__ C, const uint4 *__restrict__ parts,
                                              WNode *wn, double *mom, float *__restrict__ q3out,
                                              uint32_t *__restrict__ leafof, int level, double unit_d, uint32_t gid,
                                              uint32_t ngroups)
{
    const uint32_t beg = C->lvl_start[level], end = beg + C->lvl_count[level];
    const T unit = (T)unit_d;
    const uint32_t d8 = threadIdx.x & 7;
    for (uint32_t q = beg + gid; q < end; q += ngroups) {
        WNode w = wn[q];
        const uint32_t g[3] = {w.gx, w.gy, w.gz};
        T M = 0, c1[3] = {0, 0, 0}, s[3];
        T Q2[6] = {0, 0, 0, 0, 0, 0}, Q3[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
        if (sizeof(T) == 4 && (w.meta & WN_LEAF) && w.num <= 32) {
            // up to four particles per lane, loaded together (clamped
            // indices) and kept in registers for both passes (measured
            // faster for the single-precision levels only)
            const uint32_t stop = w.next + w.num;
            uint4 pv[4];
#pragma unroll
            for (uint32_t u = 0; u < 4; u++) {
                const uint32_t j = w.next + d8 + 8 * u;
                pv[u] = parts[j < stop ? j : stop - 1];
                if (j < stop) leafof[j] = q;
            }
#pragma unroll
            for (uint32_t u = 0; u < 4; u++) {
                const T m = w.next + d8 + 8 * u < stop ? (T)__uint_as_float(pv[u].w) : (T)0;
                const T d[3] = {(T)(int32_t)(pv[u].x - g[0]) * unit, (T)(int32_t)(pv[u].y - g[1]) * unit,
                                (T)(int32_t)(pv[u].z - g[2]) * unit};
                M += m;
                for (int k = 0; k < 3; k++) c1[k] += m * d[k];
            }
            M = grp8_sum(M);
            for (int k = 0; k < 3; k++) s[k] = M > 0 ? grp8_sum(c1[k]) / M : (T)0;
#pragma unroll
            for (uint32_t u = 0; u < 4; u++) {
                const T m = w.next + d8 + 8 * u < stop ? (T)__uint_as_float(pv[u].w) : (T)0;
                const T d[3] = {(T)(int32_t)(pv[u].x - g[0]) * unit - s[0], (T)(int32_t)(pv[u].y - g[1]) * unit - s[1],
                                (T)(int32_t)(pv[u].z - g[2]) * unit - s[2]};
                Q2[0] += m * d[0] * d[0]; Q2[1] += m * d[0] * d[1]; Q2[2] += m * d[0] * d[2];
                Q2[3] += m * d[1] * d[1]; Q2[4] += m * d[1] * d[2]; Q2[5] += m * d[2] * d[2];
                for (int a = 0; a < 10; a++) Q3[a] += m * d[c_i3[a][0]] * d[c_i3[a][1]] * d[c_i3[a][2]];
            }
        } else if (w.meta & WN_LEAF) {
            const uint32_t stop = w.next + w.num;
            for (uint32_t j = w.next + d8; j < stop; j += 8) {
                leafof[j] = q;
                uint4 p = parts[j];
                T m = (T)__uint_as_float(p.w);
                T d[3] = {(T)(int32_t)(p.x - g[0]) * unit, (T)(int32_t)(p.y - g[1]) * unit,
                          (T)(int32_t)(p.z - g[2]) * unit};
                M += m;
                for (int k = 0; k < 3; k++) c1[k] += m * d[k];
            }
            M = grp8_sum(M);
            for (int k = 0; k < 3; k++) s[k] = M > 0 ? grp8_sum(c1[k]) / M : (T)0;
            for (uint32_t j = w.next + d8; j < stop; j += 8) {
                uint4 p = parts[j];
                T m = (T)__uint_as_float(p.w);
                T d[3] = {(T)(int32_t)(p.x - g[0]) * unit - s[0], (T)(int32_t)(p.y - g[1]) * unit - s[1],
                          (T)(int32_t)(p.z - g[2]) * unit - s[2]};
                Q2[0] += m * d[0] * d[0]; Q2[1] += m * d[0] * d[1]; Q2[2] += m * d[0] * d[2];
                Q2[3] += m * d[1] * d[1]; Q2[4] += m * d[1] * d[2]; Q2[5] += m * d[2] * d[2];
                for (int a = 0; a < 10; a++) Q3[a] += m * d[c_i3[a][0]] * d[c_i3[a][1]] * d[c_i3[a][2]];
            }
        } else {
            const bool has = d8 < w.num;
            T Mc = 0, dl[3] = {0, 0, 0}, q2c[6] = {0, 0, 0, 0, 0, 0};
            const double *mc = mom + (size_t)(w.next + (has ? d8 : 0)) * MOM_STRIDE;
            if (has) {
                const WNode &wc = wn[w.next + d8];
                Mc = (T)mc[0];
                dl[0] = (T)(int32_t)(wc.gx - g[0]) * unit + (T)mc[1];
                dl[1] = (T)(int32_t)(wc.gy - g[1]) * unit + (T)mc[2];
                dl[2] = (T)(int32_t)(wc.gz - g[2]) * unit + (T)mc[3];
                for (int a = 0; a < 6; a++) q2c[a] = (T)mc[4 + a];
            }
            M = grp8_sum(Mc);
            for (int k = 0; k < 3; k++) s[k] = M > 0 ? grp8_sum(Mc * dl[k]) / M : (T)0;
            if (has) {
                const T d[3] = {dl[0] - s[0], dl[1] - s[1], dl[2] - s[2]};
                Q2[0] = q2c[0] + Mc * d[0] * d[0]; Q2[1] = q2c[1] + Mc * d[0] * d[1];
                Q2[2] = q2c[2] + Mc * d[0] * d[2]; Q2[3] = q2c[3] + Mc * d[1] * d[1];
                Q2[4] = q2c[4] + Mc * d[1] * d[2]; Q2[5] = q2c[5] + Mc * d[2] * d[2];
                for (int a = 0; a < 10; a++) {
                    const int i = c_i3[a][0], j = c_i3[a][1], k = c_i3[a][2];
                    Q3[a] = (T)mc[10 + a] + d[i] * q2c[p2i(j, k)] + d[j] * q2c[p2i(i, k)] + d[k] * q2c[p2i(i, j)] +
                            Mc * d[i] * d[j] * d[k];
                }
            }
        }
        for (int a = 0; a < 6; a++) Q2[a] = grp8_sum(Q2[a]);
        for (int a = 0; a < 10; a++) Q3[a] = grp8_sum(Q3[a]);
        if (d8 == 0) {
            double *mo = mom + (size_t)q * MOM_STRIDE;
            mo[0] = (double)M;
            for (int k = 0; k < 3; k++) mo[1 + k] = (double)s[k];
            for (int a = 0; a < 6; a++) mo[4 + a] = (double)Q2[a];
            for (int a = 0; a < 10; a++) mo[10 + a] = (double)Q3[a];
            // walk record: COM on the integer grid, single-precision moments
            uint32_t cg[3];
            for (int k = 0; k < 3; k++) cg[k] = g[k] + (uint32_t)(int64_t)rint((double)s[k] / unit_d);
            w.cx = cg[0];
            w.cy = cg[1];
            w.cz = cg[2];
            w.mass = (float)M;
            for (int a = 0; a < 6; a++) w.q[a] = (float)Q2[a];
            wn[q] = w;
            for (int a = 0; a < 10; a++) q3out[(size_t)q * 10 + a] = (float)Q3[a];
        }
    }
}

#define G4_FP64_LEVELS 8

template <typename T>
__global__ void k_moments(const DevCounters *__restrict__ C, const uint4 *__restrict__ parts, WNode *wn, double *mom,
                          float *__restrict__ q3out, uint32_t *__restrict__ leafof, int level, double unit)
{
    moments_level<T>(C, parts, wn, mom, q3out, leafof, level, unit, (blockIdx.x * blockDim.x + threadIdx.x) >> 3,
                     (gridDim.x * blockDim.x) >> 3);
}

// levels hi .. lo in one block, for levels of few nodes
template <typename T>
__global__ __launch_bounds__(512) void k_moments_block(const DevCounters *__restrict__ C,
                                                       const uint4 *__restrict__ parts, WNode *wn, double *mom,
                                                       float *__restrict__ q3out, uint32_t *__restrict__ leafof, int hi,
                                                       int lo, double unit)
{
    for (int l = hi; l >= lo; l--) {
        moments_level<T>(C, parts, wn, mom, q3out, leafof, l, unit, threadIdx.x >> 3, 64);
        __syncthreads();
    }
}

// Levels 0 to MOM_TOP hold at most 73 nodes (per box): one block takes them, a launch
// instead of one per level, unless they may hold large leaves, which one compute unit reads
// more slowly (2 10^6 particles, leaf 10^5 or two levels: 11.8 ms by level, 13.2 by the block;
// leaf 1000 0.88 and 0.89).  So do the levels from MOM_DEEP on of a set of at most
// MOM_DEEP_N particles.  A larger set may have thousands of nodes that deep, where it is
// the dense core of a larger one, and 64 groups of lanes are too few for them: 16384
// particles in 10^-4 of the box side, leaf 4, 155 us with a launch per level and 707 with
// the block (leaf 16: 144, 353); 1024 in 10^-4, leaf 1, 181, 200; 500 184, 168; ordinary
// sets of 1000 87, 78, of 8192 (leaf 16) 97, 91.
#define MOM_TOP 2
#define MOM_TOP_LEAF 1024
#define MOM_DEEP 17
#define MOM_DEEP_N 512

int g4_launch_moments(g4_ctx *ctx, g4_tree *t)
{
    hipStream_t s = ctx->stream;
    int l = t->tp.max_depth < 1 ? 1 : (t->tp.max_depth > G4_MAXLEV ? G4_MAXLEV : t->tp.max_depth);
    if (t->n <= MOM_DEEP_N && l >= MOM_DEEP) {
        k_moments_block<float><<<1, 512, 0, s>>>(t->ctr, t->parts, t->wn, t->mom, t->q3, t->leafof, l, MOM_DEEP, t->unit);
        l = MOM_DEEP - 1;
    }
    const int top = t->nbox <= 8 && l > MOM_TOP && t->tp.leaf_max <= MOM_TOP_LEAF ? MOM_TOP : -1;
    for (; l > top; l--) {
        if (l <= G4_FP64_LEVELS)
            k_moments<double><<<grid_for(t->n, 1024), kBlock, 0, s>>>(t->ctr, t->parts, t->wn, t->mom, t->q3, t->leafof, l,
                                                                     t->unit);
        else
            k_moments<float><<<grid_for(t->n, 1024), kBlock, 0, s>>>(t->ctr, t->parts, t->wn, t->mom, t->q3, t->leafof, l,
                                                                    t->unit);
    }
    if (l >= 0)
        k_moments_block<double><<<1, 512, 0, s>>>(t->ctr, t->parts, t->wn, t->mom, t->q3, t->leafof, l, 0, t->unit);
    G4_HIP(ctx, hipGetLastError());
    return G4_OK;
}

// Fourth moments Q4 (15 packed components, multi-index order xxxx xxxy ...
// zzzz) about every node's centre of mass, for the walk at p = 4, 5; FP64, one
// thread per node, levels from the deepest up.  A leaf sums m d^(a,b,c) over its
// particles; an internal node shifts its children's moments to its own centre
// of mass: for d = s_child - s,
//   Q4_alpha = sum_{beta <= alpha} C(alpha, beta) Qc_beta d^(alpha - beta),
// C the product of binomial coefficients per axis, Qc_beta the child's moment
// of order |beta| (its mass for 0, zero for 1 about its centre of mass).
__device__ __forceinline__ int m4_idx(int a, int b, int c)
{
    // position of a multi-index within its order: (b + c)(b + c + 1)/2 + c
    return (b + c) * (b + c + 1) / 2 + c;
}

__global__ __launch_bounds__(128) void k_moments4(const DevCounters *__restrict__ C, const uint4 *__restrict__ parts,
                                                  const WNode *__restrict__ wn, const double *__restrict__ mom,
                                                  double *__restrict__ q4, int level, double unit)
{
    const uint32_t beg = C->lvl_start[level], end = beg + C->lvl_count[level];
    constexpr double binom[5][5] = {{1, 0, 0, 0, 0}, {1, 1, 0, 0, 0}, {1, 2, 1, 0, 0}, {1, 3, 3, 1, 0}, {1, 4, 6, 4, 1}};
    for (uint32_t q = beg + blockIdx.x * blockDim.x + threadIdx.x; q < end; q += gridDim.x * blockDim.x) {
        const WNode w = wn[q];
        const double *mo = mom + (size_t)q * MOM_STRIDE;
        double Q[15];
#pragma unroll
        for (int k = 0; k < 15; k++) Q[k] = 0.0;
        if (w.meta & WN_LEAF) {
            for (uint32_t j = w.next; j < w.next + w.num; j++) {
                const uint4 p = parts[j];
                const double m = (double)__uint_as_float(p.w);
                const double d[3] = {(double)(int32_t)(p.x - w.gx) * unit - mo[1],
                                     (double)(int32_t)(p.y - w.gy) * unit - mo[2],
                                     (double)(int32_t)(p.z - w.gz) * unit - mo[3]};
                double pw[3][5];
#pragma unroll
                for (int k = 0; k < 3; k++) {
                    pw[k][0] = 1.0;
#pragma unroll
                    for (int e = 1; e < 5; e++) pw[k][e] = pw[k][e - 1] * d[k];
                }
#pragma unroll
                for (int a = 4; a >= 0; a--)
#pragma unroll
                    for (int b = 4 - a; b >= 0; b--) Q[m4_idx(a, b, 4 - a - b)] += m * pw[0][a] * pw[1][b] * pw[2][4 - a - b];
            }
        } else {
            for (uint32_t ch = w.next; ch < w.next + w.num; ch++) {
                const WNode wc = wn[ch];
                const double *mc = mom + (size_t)ch * MOM_STRIDE;
                const double *qc4 = q4 + (size_t)ch * 15;
                const double d[3] = {(double)(int32_t)(wc.gx - w.gx) * unit + mc[1] - mo[1],
                                     (double)(int32_t)(wc.gy - w.gy) * unit + mc[2] - mo[2],
                                     (double)(int32_t)(wc.gz - w.gz) * unit + mc[3] - mo[3]};
                double pw[3][5], qc[5][15];
#pragma unroll
                for (int k = 0; k < 3; k++) {
                    pw[k][0] = 1.0;
#pragma unroll
                    for (int e = 1; e < 5; e++) pw[k][e] = pw[k][e - 1] * d[k];
                }
                // the child's moments by order: mass, (no dipole), Q2, Q3, Q4 (packed)
                qc[0][0] = mc[0];
#pragma unroll
                for (int k = 0; k < 6; k++) qc[2][k] = mc[4 + k];
#pragma unroll
                for (int k = 0; k < 10; k++) qc[3][k] = mc[10 + k];
#pragma unroll
                for (int k = 0; k < 15; k++) qc[4][k] = qc4[k];
#pragma unroll
                for (int a = 4; a >= 0; a--)
#pragma unroll
                    for (int b = 4 - a; b >= 0; b--) {
                        const int c = 4 - a - b;
                        double sum = 0.0;
#pragma unroll
                        for (int ba = 0; ba <= 4; ba++)
#pragma unroll
                            for (int bb = 0; bb <= 4; bb++)
#pragma unroll
                                for (int bc = 0; bc <= 4; bc++) {
                                    const int n = ba + bb + bc;
                                    if (ba > a || bb > b || bc > c || n == 1) continue;
                                    sum += binom[a][ba] * binom[b][bb] * binom[c][bc] * qc[n][m4_idx(ba, bb, bc)] *
                                           pw[0][a - ba] * pw[1][b - bb] * pw[2][c - bc];
                                }
                        Q[m4_idx(a, b, c)] += sum;
                    }
            }
        }
#pragma unroll
        for (int k = 0; k < 15; k++) q4[(size_t)q * 15 + k] = Q[k];
    }
}

int g4_launch_moments4(g4_ctx *ctx, g4_tree *t, double *q4)
{
    const int maxd = t->tp.max_depth < 1 ? 1 : (t->tp.max_depth > G4_MAXLEV ? G4_MAXLEV : t->tp.max_depth);
    for (int l = maxd; l >= 0; l--)
        k_moments4<<<2048, 128, 0, ctx->stream>>>(t->ctr, t->parts, t->wn, t->mom, q4, l, t->unit);
    G4_HIP(ctx, hipGetLastError());
    return G4_OK;
}

// ------------------------------------------------------------------ export
__global__ void k_export(const DevCounters *__restrict__ C, const WNode *__restrict__ wn,
                         const uint32_t *__restrict__ bfirst, const uint32_t *__restrict__ bcount,
                         const double *__restrict__ mom, int S, uint32_t corner, double unit, int32_t *level,
                         uint32_t *cell, int64_t *count, int64_t *first, int32_t *leaf, double *mass, double *com,
                         double *q2, double *q3)
{
    const uint32_t nn = C->node_count;
    for (uint32_t q = blockIdx.x * blockDim.x + threadIdx.x; q < nn; q += gridDim.x * blockDim.x) {
        const WNode w = wn[q];
        const int l = (int)(w.meta & 0xff);
        const uint32_t g[3] = {w.gx, w.gy, w.gz};
        if (level) level[q] = l;
        if (leaf) leaf[q] = (w.meta & WN_LEAF) ? 1 : 0;
        if (count) count[q] = bcount[q];
        if (first) first[q] = bfirst[q];
        for (int k = 0; k < 3; k++) {
            uint64_t rel = (uint64_t)(uint32_t)(g[k] - corner) - (1ull << (S - l - 1));
            if (cell) cell[3 * (size_t)q + k] = (uint32_t)(rel >> (S - l));
            if (com) com[3 * (size_t)q + k] = (double)(uint32_t)(g[k] - corner) * unit + mom[(size_t)q * MOM_STRIDE + 1 + k];
        }
        if (mass) mass[q] = mom[(size_t)q * MOM_STRIDE];
        if (q2)
            for (int a = 0; a < 6; a++) q2[6 * (size_t)q + a] = mom[(size_t)q * MOM_STRIDE + 4 + a];
        if (q3)
            for (int a = 0; a < 10; a++) q3[10 * (size_t)q + a] = mom[(size_t)q * MOM_STRIDE + 10 + a];
    }
}

int g4_launch_export(g4_ctx *ctx, const g4_tree *t, int32_t *level, uint32_t *cell, int64_t *count,
                     int64_t *first, int32_t *leaf, double *mass, double *com, double *q2, double *q3)
{
    k_export<<<grid_for(t->cap), kBlock, 0, ctx->stream>>>(t->ctr, t->wn, t->bfirst, t->bcount, t->mom, t->S,
                                                           t->corner, t->unit, level, cell, count, first, leaf, mass,
                                                           com, q2, q3);
    G4_HIP(ctx, hipGetLastError());
    return G4_OK;
}

// ------------------------------------------------------------------ zeroing
__global__ void k_zero_words(uint32_t *__restrict__ p, size_t nwords)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < nwords; i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

int g4_launch_zero(g4_ctx *ctx, void *p, size_t bytes)
{
    const size_t nw = bytes / 4;
    if (nw == 0) return G4_OK;
    k_zero_words<<<grid_for((int64_t)nw), kBlock, 0, ctx->stream>>>(static_cast<uint32_t *>(p), nw);
    G4_HIP(ctx, hipGetLastError());
    return G4_OK;
}

// ------------------------------------------------------------- seed gather
__global__ void k_gather_seed(const float *__restrict__ a_caller, const uint32_t *__restrict__ perm, int64_t n,
                              float *__restrict__ a_sorted)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        a_sorted[i] = a_caller[perm[i]];
}

int g4_launch_gather_seed(g4_ctx *ctx, g4_tree *t, const float *a_seed_caller)
{
    k_gather_seed<<<grid_for(t->n), kBlock, 0, ctx->stream>>>(a_seed_caller, t->perm1, t->n, t->aseed);
    G4_HIP(ctx, hipGetLastError());
    return G4_OK;
}

// ------------------------------------------------------------------ forest
// Many independent boxes in one node array: particles sorted by (box, curve
// key), one root per box at level 0 (nodes 0..nbox-1); nodes and moments as for
// a single tree, with a new root wherever the box changes.

// box of each Morton-sorted particle (caller index -> box by binary search)
__global__ void k_boxkey(const uint32_t *__restrict__ perm, int64_t n, const int64_t *__restrict__ off, int nbox,
                         uint32_t *__restrict__ bkey)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t c = perm[i];
        int lo = 0, hi = nbox - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (off[mid] <= c) lo = mid;
            else hi = mid - 1;
        }
        bkey[i] = (uint32_t)lo;
    }
}

// the particles and their curve keys in the final (box, key) order
__global__ void k_gather_keys(const uint4 *__restrict__ pk, const uint32_t *__restrict__ perm, int64_t n, int drop,
                              uint32_t corner, int kind, uint4 *__restrict__ parts, uint64_t *__restrict__ keys)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const uint4 q = pk[perm[i]];
        parts[i] = q;
        keys[i] = curve_key(q.x, q.y, q.z, drop, corner, kind);
    }
}

int g4_launch_build_forest(g4_ctx *ctx, g4_tree *t, const g4_particles *p, const int64_t *off_dev, uint32_t *bkey0,
                           uint32_t *bkey1)
{
    hipStream_t s = ctx->stream;
    const int64_t n = t->n;
    k_keys<<<grid_for(n), kBlock, 0, s>>>(p->x, p->y, p->z, p->mass, n, t->S - G4_MAXLEV, t->corner,
                                          t->tp.key_kind, t->keys0, t->perm0, packed_staging(t));
    G4_HIP(ctx, hipGetLastError());
    if (int st = sort_keys(ctx, t)) return st;
    k_boxkey<<<grid_for(n), kBlock, 0, s>>>(t->perm1, n, off_dev, t->nbox, bkey0);
    int bits = 1;
    while ((1 << bits) < t->nbox) bits++;
    // stable: particles of a box keep their curve order
    int alt = 0;
    if (int st = g4_radix_sort_u32(ctx, bkey0, bkey1, t->perm1, t->perm0, n, 0, bits, t->sort_tmp, t->sort_tmp_bytes,
                                   &alt))
        return st;
    if (alt) std::swap(t->perm0, t->perm1);
    k_gather_keys<<<grid_for(n), kBlock, 0, s>>>(packed_staging(t), t->perm1, n, t->S - G4_MAXLEV, t->corner,
                                                  t->tp.key_kind, t->parts, t->keys1);
    G4_HIP(ctx, hipGetLastError());
    return launch_nodes(ctx, t, alt ? bkey1 : bkey0);
}
