// sort.hip -- stable least-significant-digit radix sort of (key, value)
// pairs on gfx950: the ordering of the particles along the space-filling
// curve (Sec. "Geometry of the tree": particles sorted by their curve key) and
// the regrouping of a forest's particles by box.
//
// One pass per 8-bit digit, three steps each:
//   1. k_rs_hist:    every block counts the digits of its tile of RS_TILE keys
//                    (LDS atomics) into hist[digit][block];
//   2. k_rs_scan_*:  the table is scanned digit-major (one block per digit row,
//                    then the 256 row totals), so hist[d][b] becomes the first
//                    output slot of block b's keys with digit d;
//   3. k_rs_scatter: every block ranks its tile stably -- each wavefront
//                    takes its quarter in chunks of 64 keys in order; lanes
//                    with equal digits find each other with 8 ballots, rank by
//                    the lanes below them and by a per-wavefront running count
//                    -- then places the tile in LDS in digit order and writes
//                    it out so that consecutive threads write consecutive
//                    slots of each digit's run.
// Small sets (up to RS_SMALL_BLOCKS tiles) take one launch per digit: every
// block of the scatter sums the histogram's rows itself, and adds the keys it
// places to the next digit's histogram at the tile of their new position.  Their
// sort is bound by launches and latency, so a block has 16 wavefronts, a tile as
// few keys as that leaves, and a quarter of its threads take every fourth row.
// 63-bit keys, kernel time: four launches a digit 0.15 ms (8192) and 0.17 (50 k), one
// launch on tiles of 512 keys by four wavefronts 0.06 and 0.09; whole tree builds then
// 89 us (8192), 111 (32768), 133 (50 k), now 85, 91, 106.
// Equal keys keep their input order (every rank follows chunk, wavefront and
// block order), which the tree build relies on for ties.
#include <algorithm>

#include "g4_internal.h"

#define RS_BITS 8
#define RS_BINS 256
#define RS_THREADS 256
#define RS_ITEMS 8                         // keys per lane and wavefront chunk count
#define RS_TILE (RS_THREADS * RS_ITEMS)    // 2048 keys per block
#define RS_SMALL_THREADS 1024              // a block of a small set
#define RS_SMALL_BLOCKS 128                // tiles of a small set: a block reads every tile's histogram
// Keys per lane of a small set: 1 up to 2^17 keys, 2 up to 2^18, and the general form
// beyond, where the additions to the next histogram cost more than launches.  Tree builds,
// us, at 1 / 2 / general: 80 k 116 / 121 / 178, 131 k 132 / 138 / 182, 160 k 155 / 149 / 184
// (192 tiles), 262 k - / 181 / 189, 320 k - / 207 / 198 (192 tiles), 500 k at 8 315 / 210.
#define RS_SMALL_N ((int64_t)RS_SMALL_BLOCKS * RS_SMALL_THREADS)

__device__ __forceinline__ uint64_t rs_ballot(bool c) { return __builtin_amdgcn_ballot_w64(c); }
__device__ __forceinline__ uint32_t rs_below(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
__device__ __forceinline__ void rs_wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <typename K>
__device__ __forceinline__ uint32_t rs_digit(K k, int shift)
{
    return (uint32_t)(k >> shift) & (RS_BINS - 1);
}

template <typename K>
__global__ __launch_bounds__(RS_THREADS) void k_rs_hist(const K *__restrict__ keys, int64_t n, int shift,
                                                        uint32_t *__restrict__ hist, uint32_t nb)
{
    __shared__ uint32_t h[RS_BINS];
    h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * RS_TILE;
#pragma unroll
    for (int c = 0; c < RS_ITEMS; c++) {
        const int64_t i = base + c * RS_THREADS + threadIdx.x;
        if (i < n) atomicAdd(&h[rs_digit(keys[i], shift)], 1u);
    }
    __syncthreads();
    hist[(size_t)threadIdx.x * nb + blockIdx.x] = h[threadIdx.x];
}

// exclusive scan of one digit row hist[d][0..nb) in place; the row total to tot[d]
__global__ __launch_bounds__(RS_THREADS) void k_rs_scan_rows(uint32_t *__restrict__ hist, uint32_t nb,
                                                             uint32_t *__restrict__ tot)
{
    __shared__ uint32_t part[RS_THREADS];
    uint32_t *row = hist + (size_t)blockIdx.x * nb;
    const uint32_t per = (nb + RS_THREADS - 1) / RS_THREADS;
    const uint32_t lo = threadIdx.x * per, hi = min(nb, lo + per);
    uint32_t s = 0;
    for (uint32_t k = lo; k < hi; k++) s += row[k];
    part[threadIdx.x] = s;
    __syncthreads();
    // Hillis-Steele inclusive scan of the 256 partial sums
    for (int off = 1; off < RS_THREADS; off <<= 1) {
        const uint32_t v = threadIdx.x >= (unsigned)off ? part[threadIdx.x - off] : 0u;
        __syncthreads();
        part[threadIdx.x] += v;
        __syncthreads();
    }
    uint32_t run = part[threadIdx.x] - s;
    for (uint32_t k = lo; k < hi; k++) {
        const uint32_t v = row[k];
        row[k] = run;
        run += v;
    }
    if (threadIdx.x == RS_THREADS - 1) tot[blockIdx.x] = part[RS_THREADS - 1];
}

// exclusive scan of the 256 digit totals: the first output slot of each digit
__global__ __launch_bounds__(RS_BINS) void k_rs_scan_digits(const uint32_t *__restrict__ tot,
                                                            uint32_t *__restrict__ dbase)
{
    __shared__ uint32_t v[RS_BINS];
    const uint32_t own = tot[threadIdx.x];
    v[threadIdx.x] = own;
    __syncthreads();
    for (int off = 1; off < RS_BINS; off <<= 1) {
        const uint32_t a = threadIdx.x >= (unsigned)off ? v[threadIdx.x - off] : 0u;
        __syncthreads();
        v[threadIdx.x] += a;
        __syncthreads();
    }
    dbase[threadIdx.x] = v[threadIdx.x] - own;
}

// the first digit's histogram of a small set, and the next table cleared
template <typename K, int ITEMS>
__global__ __launch_bounds__(RS_SMALL_THREADS) void k_rs_hist_small(const K *__restrict__ keys, int64_t n, int shift,
                                                                    uint32_t *__restrict__ hist,
                                                                    uint32_t *__restrict__ next)
{
    __shared__ uint32_t h[RS_BINS];
    if (threadIdx.x < RS_BINS) h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * (RS_SMALL_THREADS * ITEMS);
#pragma unroll
    for (int c = 0; c < ITEMS; c++) {
        const int64_t i = base + c * RS_SMALL_THREADS + threadIdx.x;
        if (i < n) atomicAdd(&h[rs_digit(keys[i], shift)], 1u);
    }
    __syncthreads();
    if (threadIdx.x < RS_BINS) {
        hist[(size_t)blockIdx.x * RS_BINS + threadIdx.x] = h[threadIdx.x];
        next[(size_t)blockIdx.x * RS_BINS + threadIdx.x] = 0u;
    }
}

// SMALL: hist is the raw histogram [tile][digit]; the keys placed are added to
// `next`, the next digit's one (digit 8 bits up; null on the last pass), and
// `clear` is zeroed for the pass after that.
template <typename K, int THREADS, int ITEMS, bool SMALL>
__global__ __launch_bounds__(THREADS) void k_rs_scatter(const K *__restrict__ kin, const uint32_t *__restrict__ vin,
                                                        K *__restrict__ kout, uint32_t *__restrict__ vout, int64_t n,
                                                        int shift, const uint32_t *__restrict__ hist, uint32_t nb,
                                                        const uint32_t *__restrict__ dbase, uint32_t *__restrict__ next,
                                                        uint32_t *__restrict__ clear)
{
    constexpr int TILE = THREADS * ITEMS, WAVES = THREADS / 64, WTILE = TILE / WAVES, GROUPS = THREADS / RS_BINS;
    __shared__ uint32_t cnt[WAVES][RS_BINS];  // per wavefront: running count, then the wavefront's base
    __shared__ uint32_t wtot[2][4];
    __shared__ uint32_t bpre[RS_BINS];    // block-local first slot of each digit
    __shared__ uint32_t gpos[RS_BINS];    // global first slot of this block's run of each digit
    __shared__ uint2 psum[SMALL ? GROUPS : 1][SMALL ? RS_BINS : 1];  // sums over a part of the tiles
    __shared__ K skey[TILE];
    __shared__ uint32_t sval[TILE];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int k = threadIdx.x; k < WAVES * RS_BINS; k += THREADS) (&cnt[0][0])[k] = 0u;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * TILE + (int64_t)w * WTILE;
    K key[ITEMS];
    uint32_t val[ITEMS], rank[ITEMS];
#pragma unroll
    for (int c = 0; c < ITEMS; c++) {
        const int64_t i = base + c * 64 + lane;
        const bool valid = i < n;
        key[c] = valid ? kin[i] : (K)0;
        val[c] = valid ? vin[i] : 0u;
        const uint32_t d = rs_digit(key[c], shift);
        // lanes of this chunk with the same digit
        uint64_t m = rs_ballot(valid);
#pragma unroll
        for (int b = 0; b < RS_BITS; b++) {
            const uint64_t bal = rs_ballot((d >> b) & 1u);
            m &= ((d >> b) & 1u) ? bal : ~bal;
        }
        const uint32_t before = cnt[w][d];
        rank[c] = before + rs_below(m);
        rs_wave_fence();
        if (valid && (uint32_t)lane == (uint32_t)__builtin_ctzll(m)) cnt[w][d] = before + (uint32_t)__builtin_popcountll(m);
        rs_wave_fence();
    }
    if constexpr (SMALL) {
        // this block's first slot of each digit within the digit's run, and the digit's total:
        // the threads of a digit take the tiles in turn
        const uint32_t d = threadIdx.x % RS_BINS, g = threadIdx.x / RS_BINS;
        uint32_t mine = 0, all = 0;
        if (g == 0) clear[(size_t)blockIdx.x * RS_BINS + d] = 0u;
#pragma unroll 8
        for (uint32_t b = g; b < nb; b += GROUPS) {
            const uint32_t v = hist[(size_t)b * RS_BINS + d];
            mine += b < blockIdx.x ? v : 0u;
            all += v;
        }
        psum[g][d] = make_uint2(mine, all);
    }
    __syncthreads();
    // one thread per digit: wavefront bases, the block's digit prefix, the global start
    const int d = threadIdx.x;
    uint32_t total = 0, mine = 0, all = 0, x = 0, y = 0;
    if (threadIdx.x < RS_BINS) {
#pragma unroll
        for (int k = 0; k < WAVES; k++) {
            const uint32_t v = cnt[k][d];
            cnt[k][d] = total;
            total += v;
        }
        if constexpr (SMALL)
            for (int g = 0; g < GROUPS; g++) {
                mine += psum[g][d].x;
                all += psum[g][d].y;
            }
        // exclusive scans over the digits: of the block's totals and, SMALL, of all totals
        x = total;
        y = all;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t a = __shfl_up(x, off), b = SMALL ? __shfl_up(y, off) : 0u;
            if (lane >= off) {
                x += a;
                y += b;
            }
        }
        if (lane == 63) {
            wtot[0][w] = x;
            wtot[1][w] = y;
        }
    }
    __syncthreads();
    if (threadIdx.x < RS_BINS) {
        for (int k = 0; k < w; k++) {
            x += wtot[0][k];
            y += wtot[1][k];
        }
        bpre[d] = x - total;
        gpos[d] = SMALL ? mine + y - all : hist[(size_t)d * nb + blockIdx.x] + dbase[d];
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < ITEMS; c++) {
        const int64_t i = base + c * 64 + lane;
        if (i < n) {
            const uint32_t d = rs_digit(key[c], shift);
            const uint32_t lp = bpre[d] + cnt[w][d] + rank[c];
            skey[lp] = key[c];
            sval[lp] = val[c];
        }
    }
    __syncthreads();
    const int64_t b0 = (int64_t)blockIdx.x * TILE;
    const uint32_t valid_n = (uint32_t)std::min<int64_t>(TILE, n - b0);
    for (uint32_t j0 = 0; j0 < valid_n; j0 += THREADS) {
        const uint32_t j = j0 + threadIdx.x;
        K k = 0;
        uint32_t o = 0;
        if (j < valid_n) {
            k = skey[j];
            const uint32_t d = rs_digit(k, shift);
            o = gpos[d] + (j - bpre[d]);
            kout[o] = k;
            vout[o] = sval[j];
        }
        if constexpr (SMALL)
            if (next) {
                // slot of the next digit's table; there is one, so shift + RS_BITS is below the key's width
                const uint32_t slot = j < valid_n ? o / TILE * RS_BINS + rs_digit(k, shift + RS_BITS) : 0xffffffffu;
                // one addition per run of equal slots in the wavefront: keys that share a digit
                // would otherwise queue on one address
                const uint32_t up = (uint32_t)__shfl_up((int)slot, 1);
                const uint64_t heads = rs_ballot(lane == 0 || up != slot);
                const uint64_t above = lane < 63 ? heads >> (lane + 1) : 0ull;
                const uint32_t run = above ? (uint32_t)__builtin_ctzll(above) + 1u : 64u - (uint32_t)lane;
                if (((heads >> lane) & 1ull) && slot != 0xffffffffu) atomicAdd(&next[slot], run);
            }
    }
}

size_t g4_radix_sort_temp_bytes(int64_t n)
{
    auto tiles = [](int64_t m, int64_t tile) { return (size_t)std::max<int64_t>((m + tile - 1) / tile, 1); };
    const size_t large = (size_t)RS_BINS * tiles(n, RS_TILE) * 4 + 2 * RS_BINS * 4;
    // grow with n throughout, so that a scratch sized for more keys serves fewer
    const size_t one = 3 * (size_t)RS_BINS * tiles(std::min(n, RS_SMALL_N), RS_SMALL_THREADS) * 4;
    const size_t two = 3 * (size_t)RS_BINS * tiles(std::min(n, 2 * RS_SMALL_N), 2 * RS_SMALL_THREADS) * 4;
    return (std::max(std::max(large, one), two) + 255) & ~(size_t)255;
}

template <typename K, int ITEMS>
static int radix_sort_small(g4_ctx *ctx, K *ki, K *ko, uint32_t *vi, uint32_t *vo, int64_t n, int bit_lo, int bit_hi,
                            uint32_t *hist, int *in_alt)
{
    const uint32_t ns = (uint32_t)((n + RS_SMALL_THREADS * ITEMS - 1) / (RS_SMALL_THREADS * ITEMS));
    uint32_t *t[3];  // this digit's histogram, the next one's, the one being cleared
    for (int k = 0; k < 3; k++) t[k] = hist + (size_t)k * RS_BINS * ns;
    hipStream_t s = ctx->stream;
    k_rs_hist_small<K, ITEMS><<<ns, RS_SMALL_THREADS, 0, s>>>(ki, n, bit_lo, t[0], t[1]);
    for (int shift = bit_lo; shift < bit_hi; shift += RS_BITS) {
        const bool more = shift + RS_BITS < bit_hi;
        k_rs_scatter<K, RS_SMALL_THREADS, ITEMS, true><<<ns, RS_SMALL_THREADS, 0, s>>>(
            ki, vi, ko, vo, n, shift, t[0], ns, nullptr, more ? t[1] : nullptr, t[2]);
        std::swap(ki, ko);
        std::swap(vi, vo);
        *in_alt ^= 1;
        std::rotate(t, t + 1, t + 3);
    }
    G4_HIP(ctx, hipGetLastError());
    return G4_OK;
}

template <typename K>
static int radix_sort(g4_ctx *ctx, K *k0, K *k1, uint32_t *v0, uint32_t *v1, int64_t n, int bit_lo, int bit_hi,
                      void *temp, size_t temp_bytes, int *in_alt)
{
    *in_alt = 0;
    if (n <= 1 || bit_hi <= bit_lo) return G4_OK;
    if (n > 0xFFFFFFFFll) return g4_set_err(ctx, G4_EINVAL, "radix sort: more than 2^32 - 1 keys");
    if (temp_bytes < g4_radix_sort_temp_bytes(n)) return g4_set_err(ctx, G4_ENOMEM, "radix sort: temp too small");
    uint32_t *hist = (uint32_t *)temp;
    if (n <= RS_SMALL_N) return radix_sort_small<K, 1>(ctx, k0, k1, v0, v1, n, bit_lo, bit_hi, hist, in_alt);
    if (n <= 2 * RS_SMALL_N) return radix_sort_small<K, 2>(ctx, k0, k1, v0, v1, n, bit_lo, bit_hi, hist, in_alt);
    const uint32_t nb = (uint32_t)((n + RS_TILE - 1) / RS_TILE);
    uint32_t *tot = hist + (size_t)RS_BINS * nb;
    uint32_t *dbase = tot + RS_BINS;
    hipStream_t s = ctx->stream;
    K *ki = k0, *ko = k1;
    uint32_t *vi = v0, *vo = v1;
    for (int shift = bit_lo; shift < bit_hi; shift += RS_BITS) {
        k_rs_hist<K><<<nb, RS_THREADS, 0, s>>>(ki, n, shift, hist, nb);
        k_rs_scan_rows<<<RS_BINS, RS_THREADS, 0, s>>>(hist, nb, tot);
        k_rs_scan_digits<<<1, RS_BINS, 0, s>>>(tot, dbase);
        k_rs_scatter<K, RS_THREADS, RS_ITEMS, false><<<nb, RS_THREADS, 0, s>>>(ki, vi, ko, vo, n, shift, hist, nb, dbase, nullptr,
                                                                   nullptr);
        std::swap(ki, ko);
        std::swap(vi, vo);
        *in_alt ^= 1;
    }
    G4_HIP(ctx, hipGetLastError());
    return G4_OK;
}

int g4_radix_sort_u64(g4_ctx *ctx, uint64_t *k0, uint64_t *k1, uint32_t *v0, uint32_t *v1, int64_t n, int bit_lo,
                      int bit_hi, void *temp, size_t temp_bytes, int *in_alt)
{
    return radix_sort<uint64_t>(ctx, k0, k1, v0, v1, n, bit_lo, bit_hi, temp, temp_bytes, in_alt);
}

int g4_radix_sort_u32(g4_ctx *ctx, uint32_t *k0, uint32_t *k1, uint32_t *v0, uint32_t *v1, int64_t n, int bit_lo,
                      int bit_hi, void *temp, size_t temp_bytes, int *in_alt)
{
    return radix_sort<uint32_t>(ctx, k0, k1, v0, v1, n, bit_lo, bit_hi, temp, temp_bytes, in_alt);
}
