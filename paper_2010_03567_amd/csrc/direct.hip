// direct.hip -- direct summation on the device, FP64 throughout: the exact
// reference against which the paper measures every force algorithm (Sec.
// "Softened potential in periodic systems").  Kernel 0: spline-softened
// Newtonian; kernel 1: the short-range force of eq. (eqnpo4) over the nearest
// image only, optionally truncated at r_cut; kernel 2: periodic gravity, the
// softened nearest image plus the correction psi of the other images summed
// exactly by Ewald's method for every pair (Sec. "Periodic boundary
// conditions", eqs. eqnpo1, eqnewal) -- about a thousand terms per pair, for
// sampled targets.  Kernels 0 and 1: a block takes a few targets and its lanes
// split the sources (see k_direct).
#include <algorithm>

#include "g4_internal.h"

#define DT 256

struct DirectArgs {
    const uint32_t *x, *y, *z;
    const float *m;
    int64_t n;
    const int64_t *targets;
    int64_t nt;
    int64_t t0;  // first target of this launch
    double unit, h, hinv, asplit, rskip2, rcut2, G, L;
    float near2;  // squared reach of a pair in grid steps, rounded up (kernel 1, or truncated sums)
    uint32_t reach16;  // the reach in steps of 2^16 grid units, rounded up, plus one for the dropped bits (FAR)
    int truncate;
    double *ax, *ay, *az, *pot;
};

__device__ __forceinline__ void soft_kw(double u, double hinv, double &K, double &W)
{
    double h3 = hinv * hinv * hinv, u2 = u * u;
    if (u < 0.5) {
        K = h3 * (32.0 / 3.0 + u2 * (-192.0 / 5.0 + 32.0 * u));
        W = hinv * (14.0 / 5.0 + u2 * (-16.0 / 3.0 + u2 * (48.0 / 5.0 - 32.0 / 5.0 * u)));
    } else {
        K = h3 * (64.0 / 3.0 - 48.0 * u + 192.0 / 5.0 * u2 - 32.0 / 3.0 * u2 * u - 1.0 / (15.0 * u2 * u));
        W = hinv * (16.0 / 5.0 - 1.0 / (15.0 * u) + u2 * (-32.0 / 3.0 + u * (16.0 + u * (-48.0 / 5.0 + 32.0 / 15.0 * u))));
    }
}

// (erf x - 2x e^{-x^2}/sqrt(pi)) / x^3 and erf(x)/x, series below x = 0.5
__device__ __forceinline__ double lrf(double x)
{
    if (x < 0.5) {
        double s = 0, t = 1, x2 = x * x;
        for (int k = 0; k < 14; k++) { s += t / (2 * k + 3); t *= -x2 / (k + 1); }
        return 4.0 / 1.7724538509055160273 * s;
    }
    return (erf(x) - 2.0 * x / 1.7724538509055160273 * exp(-x * x)) / (x * x * x);
}
__device__ __forceinline__ double erfx(double x)
{
    if (x < 0.5) {
        double s = 0, t = 1, x2 = x * x;
        for (int k = 0; k < 14; k++) { s += t / (2 * k + 1); t *= -x2 / (k + 1); }
        return 2.0 / 1.7724538509055160273 * s;
    }
    return erf(x) / x;
}

// psi(d) and grad psi(d) of a cube of side L by the Ewald sums with alpha = 2/L:
// the n = 0 image combined with 1/|d| as erf(alpha r)/r, 342 further real
// images (|n_i| <= 3) and 728 wave vectors (|n_i| <= 4).
__device__ void ewald_exact(double dx, double dy, double dz, double L, double &psi, double &gx, double &gy,
                            double &gz)
{
    const double alpha = 2.0 / L, V = L * L * L, c2 = 2.0 * alpha / 1.7724538509055160273;
    const double r2 = dx * dx + dy * dy + dz * dz, r = sqrt(r2);
    // erf(alpha r)/r and its r^-1 d/dr = -(erf(ar) - 2ar e^{-a^2 r^2}/sqrt(pi))/r^3
    psi = alpha * erfx(alpha * r) + M_PI / (alpha * alpha * V);
    double g1 = -alpha * alpha * alpha * lrf(alpha * r);
    gx = g1 * dx;
    gy = g1 * dy;
    gz = g1 * dz;
    for (int nx = -3; nx <= 3; nx++)
        for (int ny = -3; ny <= 3; ny++)
            for (int nz = -3; nz <= 3; nz++) {
                if (!nx && !ny && !nz) continue;
                const double px = dx + nx * L, py = dy + ny * L, pz = dz + nz * L;
                const double q2 = px * px + py * py + pz * pz, q = sqrt(q2), x = alpha * q;
                const double ec = erfc(x);
                psi -= ec / q;
                // d/dx_i [erfc(alpha q)/q] = -(erfc + 2 x e^{-x^2}/sqrt(pi)) x_i / q^3
                const double f = (ec + c2 * q * exp(-x * x)) / (q2 * q);
                gx += f * px;
                gy += f * py;
                gz += f * pz;
            }
    const double tp = 2.0 * M_PI / L;
    for (int nx = -4; nx <= 4; nx++)
        for (int ny = -4; ny <= 4; ny++)
            for (int nz = -4; nz <= 4; nz++) {
                if (!nx && !ny && !nz) continue;
                const double kx = tp * nx, ky = tp * ny, kz = tp * nz, k2 = kx * kx + ky * ky + kz * kz;
                const double w = 4.0 * M_PI / V * exp(-k2 / (4.0 * alpha * alpha)) / k2;
                double sn, cs;
                sincos(kx * dx + ky * dy + kz * dz, &sn, &cs);
                psi -= w * cs;
                gx += w * sn * kx;
                gy += w * sn * ky;
                gz += w * sn * kz;
            }
}

// Force factor K (a += m K d) and potential factor W (phi -= m W) of one pair.
template <int KER>
__device__ __forceinline__ void direct_pair(const DirectArgs &A, double r2, double &K, double &W)
{
    const double r = sqrt(r2);
    if (r >= A.h) {
        if (KER == 0) {
            K = 1.0 / (r2 * r);
            W = 1.0 / r;
        } else {
            const double x = A.asplit * r, ec = erfc(x);
            K = (ec + 2.0 * x / 1.7724538509055160273 * exp(-x * x)) / (r2 * r);
            W = ec / r;
        }
    } else {
        soft_kw(r * A.hinv, A.hinv, K, W);
        if (KER == 1) {
            const double x = A.asplit * r;
            K -= A.asplit * A.asplit * A.asplit * lrf(x);
            W -= A.asplit * erfx(x);
        }
    }
}

// FP64 pair sums.  A block takes TB targets and all sources: every lane holds
// the TB targets and strides over the sources, so a sampled sum of few targets
// still fills the chip (one thread per target left 96 of 10^4 targets' 256
// compute units idle), and the partial sums of the lanes close in a fixed order.
//
// FAR (a reach below half the box side): a pair beyond the reach adds nothing,
// and 99 of 100 are, but each heavy FP64 evaluation stalled all 64 lanes of its
// wavefront.  Three stages, each on full wavefronts, joined by lists in LDS:
// * a source against all targets of the block at once, on the upper 16 bits of
//   the coordinates, two targets per packed 16-bit instruction: with c = X - r
//   the offset is within [-r, r] exactly if px - c <= 2r modulo 2^16, so the
//   largest of the three axes decides, and the least of them over the targets
//   (28 instructions for 8 targets; the FP32 test of every pair took 15 each);
// * the sources near some target against every target, in FP32 on the grid
//   against a reach rounded up;
// * the near pairs with the exact FP64 test, so the terms of every sum are the
//   same.  Near pairs of one target come together: their atomics go to SL sums
//   per target (at one sum they took as long as the kernel functions).
// 10^4 targets of 10^6 sources at a reach of 0.075 box sides: 288 ms with one
// thread per target, 10.7 with the FP32 test of every pair and one sum, 4.3
// with the packed test, 3.7 with both; all 50 k on themselves (reach 0.2) 24.8,
// 3.85, 2.9, 2.3; 8192 Newtonian (no reach) 2.35 -> 0.18.  Bound by the packed test
// where near pairs are few (2.9 ms at a reach of 0.02), then by erfc and exp in FP64.
#define DIRECT_TB 8                       // most targets of a block
#define DIRECT_STEP 4                     // sources of a lane per step, all loaded before the first is tested
                                          // (10^4 of 10^6: 5.35 ms at 2, 4.93 at 4, 4.79 at 8; 50 k: 3.04, 2.96, 3.02)
#define DIRECT_WINDOW ((int64_t)1 << 28)  // sources of one pass: a list entry holds the source and target in 32 bits

typedef uint16_t us2 __attribute__((ext_vector_type(2)));

// FAR needs 4 wavefronts per SIMD (128 VGPRs; 10^4 of 10^6: 3.7 ms, 5.0 at 3, 4.9 at 5, where the FP64 part spills)
template <int KER, int TB, int NW, bool FAR>
__global__ __launch_bounds__(64 * NW, FAR ? 4 : 1) void k_direct(const DirectArgs A)
{
    constexpr uint32_t QCAP = 64 * TB + 64;  // pending pairs of a wavefront: < 64 left, 64 TB appended per step
    constexpr int SL = FAR ? (NW < 16 ? 8 : 4) : 1;  // partial sums per wavefront and target
    __shared__ double acc[NW][TB][4][SL];
    __shared__ uint32_t list[FAR ? NW : 1][FAR ? QCAP : 1];
    __shared__ uint32_t seen[FAR ? NW : 1][FAR ? 64 + 64 * DIRECT_STEP : 1];  // pending sources
    __shared__ uint32_t tx[TB], ty[TB], tz[TB];
    __shared__ int64_t ti[TB];
    const int64_t q0 = A.t0 + blockIdx.x * (int64_t)TB;
    const int nt = (int)min((int64_t)TB, A.nt - q0);
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (threadIdx.x < TB) {
        const int64_t q = q0 + min((int)threadIdx.x, nt - 1);  // the last block repeats its last target
        const int64_t i = A.targets ? A.targets[q] : q;
        ti[threadIdx.x] = i;
        tx[threadIdx.x] = A.x[i];
        ty[threadIdx.x] = A.y[i];
        tz[threadIdx.x] = A.z[i];
    }
    for (int k = threadIdx.x; k < NW * TB * 4 * SL; k += 64 * NW) (&acc[0][0][0][0])[k] = 0.0;
    __syncthreads();
    uint32_t X[TB], Y[TB], Z[TB];
#pragma unroll
    for (int t = 0; t < TB; t++) {
        // the same for every lane: scalar registers
        X[t] = (uint32_t)__builtin_amdgcn_readfirstlane((int)tx[t]);
        Y[t] = (uint32_t)__builtin_amdgcn_readfirstlane((int)ty[t]);
        Z[t] = (uint32_t)__builtin_amdgcn_readfirstlane((int)tz[t]);
    }
    if constexpr (FAR) {
        uint32_t *L = list[wv], *S = seen[wv];
        // two targets per word: the upper 16 bits of their coordinates less the reach
        constexpr int TP = (TB + 1) / 2;
        us2 cx[TP], cy[TP], cz[TP];
#pragma unroll
        for (int t = 0; t < TP; t++) {
            const int u = 2 * t, v = min(2 * t + 1, TB - 1);
            const uint16_t r = (uint16_t)A.reach16;
            cx[t] = us2{(uint16_t)((X[u] >> 16) - r), (uint16_t)((X[v] >> 16) - r)};
            cy[t] = us2{(uint16_t)((Y[u] >> 16) - r), (uint16_t)((Y[v] >> 16) - r)};
            cz[t] = us2{(uint16_t)((Z[u] >> 16) - r), (uint16_t)((Z[v] >> 16) - r)};
        }
        for (int64_t w0 = 0; w0 < A.n; w0 += DIRECT_WINDOW) {
            const uint32_t wn = (uint32_t)min(DIRECT_WINDOW, A.n - w0);
            const uint32_t *sx = A.x + w0, *sy = A.y + w0, *sz = A.z + w0;
            uint32_t cnt = 0, ns = 0;  // pending pairs and sources (uniform)
            // the last `k` pending pairs, one per lane
            auto eval = [&](uint32_t k) {
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
                if ((uint32_t)lane < k) {
                    const uint32_t e = L[cnt - k + lane], j = e / DIRECT_TB, t = e % DIRECT_TB;
                    if (w0 + j != ti[t]) {
                        const double dx = (double)(int32_t)(sx[j] - tx[t]) * A.unit;
                        const double dy = (double)(int32_t)(sy[j] - ty[t]) * A.unit;
                        const double dz = (double)(int32_t)(sz[j] - tz[t]) * A.unit;
                        const double r2 = dx * dx + dy * dy + dz * dz;
                        if (!(r2 > A.rskip2 || (A.truncate && r2 > A.rcut2))) {
                            const double m = (double)A.m[w0 + j];
                            double K, W;
                            direct_pair<KER>(A, r2, K, W);
                            __hip_atomic_fetch_add(&acc[wv][t][0][lane % SL], m * K * dx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                            __hip_atomic_fetch_add(&acc[wv][t][1][lane % SL], m * K * dy, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                            __hip_atomic_fetch_add(&acc[wv][t][2][lane % SL], m * K * dz, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                            __hip_atomic_fetch_add(&acc[wv][t][3][lane % SL], -m * W, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                        }
                    }
                }
                cnt -= k;
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
            };
            // the last `k` pending sources, one per lane, against every target
            auto pairs = [&](uint32_t k) {
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
                const bool have = (uint32_t)lane < k;
                const uint32_t j = S[ns - k + (have ? lane : 0)];
                const uint32_t px = sx[j], py = sy[j], pz = sz[j];
#pragma unroll
                for (int t = 0; t < TB; t++) {
                    const float dx = (float)(int32_t)(px - tx[t]), dy = (float)(int32_t)(py - ty[t]),
                                dz = (float)(int32_t)(pz - tz[t]);
                    const bool near = have && fmaf(dx, dx, fmaf(dy, dy, dz * dz)) <= A.near2;
                    const uint64_t m = __builtin_amdgcn_ballot_w64(near);
                    if (near)
                        L[cnt + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
                            j * DIRECT_TB + t;
                    cnt += (uint32_t)__builtin_popcountll(m);
                }
                ns -= k;
            };
            for (uint32_t b = wv * (64 * DIRECT_STEP);; b += 64 * DIRECT_STEP * NW) {
                const bool last = b >= wn;
                if (!last) {
                    uint32_t px[DIRECT_STEP], py[DIRECT_STEP], pz[DIRECT_STEP];
#pragma unroll
                    for (int u = 0; u < DIRECT_STEP; u++) {
                        const uint32_t j = min(b + 64 * u + lane, wn - 1);
                        px[u] = sx[j];
                        py[u] = sy[j];
                        pz[u] = sz[j];
                    }
#pragma unroll
                    for (int u = 0; u < DIRECT_STEP; u++) {
                        const uint32_t j = b + 64 * u + lane;
                        const us2 hx = us2((uint16_t)(px[u] >> 16)), hy = us2((uint16_t)(py[u] >> 16)),
                                  hz = us2((uint16_t)(pz[u] >> 16));
                        us2 least = us2((uint16_t)0xffff);
#pragma unroll
                        for (int t = 0; t < TP; t++)
                            least = __builtin_elementwise_min(
                                least, __builtin_elementwise_max(hx - cx[t], __builtin_elementwise_max(hy - cy[t], hz - cz[t])));
                        const bool near = j < wn && min((uint32_t)least.x, (uint32_t)least.y) <= 2u * A.reach16;
                        const uint64_t m = __builtin_amdgcn_ballot_w64(near);
                        if (near)
                            S[ns + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] = j;
                        ns += (uint32_t)__builtin_popcountll(m);
                    }
                }
                // 64 pending sources at a time (in the end the rest): their pairs, and the pairs' terms
                while (ns >= 64 || (last && ns + cnt)) {
                    if (ns) pairs(min(ns, 64u));
                    while (cnt >= 64 || (last && cnt)) eval(min(cnt, 64u));
                }
                if (last) break;
            }
        }
    } else {
        double s[TB][4];
#pragma unroll
        for (int t = 0; t < TB; t++) s[t][0] = s[t][1] = s[t][2] = s[t][3] = 0.0;
        for (int64_t j = threadIdx.x; j < A.n; j += 64 * NW) {
            const uint32_t px = A.x[j], py = A.y[j], pz = A.z[j];
            const double m = (double)A.m[j];
#pragma unroll
            for (int t = 0; t < TB; t++) {
                if (j == ti[t]) continue;
                const double dx = (double)(int32_t)(px - X[t]) * A.unit;
                const double dy = (double)(int32_t)(py - Y[t]) * A.unit;
                const double dz = (double)(int32_t)(pz - Z[t]) * A.unit;
                const double r2 = dx * dx + dy * dy + dz * dz;
                if (r2 > A.rskip2 || (A.truncate && r2 > A.rcut2)) continue;
                double K, W;
                direct_pair<KER>(A, r2, K, W);
                s[t][0] += m * K * dx;
                s[t][1] += m * K * dy;
                s[t][2] += m * K * dz;
                s[t][3] -= m * W;
            }
        }
#pragma unroll
        for (int t = 0; t < TB; t++)
#pragma unroll
            for (int c = 0; c < 4; c++) {
                double v = s[t][c];
                for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
                if (lane == 0) acc[wv][t][c][0] = v;
            }
    }
    __syncthreads();
    if (threadIdx.x < (unsigned)(4 * nt)) {
        const int t = threadIdx.x >> 2, c = threadIdx.x & 3;
        double v = 0.0;
        for (int w = 0; w < NW; w++)
            for (int k = 0; k < SL; k++) v += acc[w][t][c][k];
        double *out = c == 0 ? A.ax : c == 1 ? A.ay : c == 2 ? A.az : A.pot;
        if (out) out[q0 + t] = A.G * v;
    }
}

// Kernel 2 costs about a thousand terms per pair, so a target gets a whole
// block: its threads split the sources and their FP64 sums are reduced in LDS.
__global__ __launch_bounds__(DT) void k_direct_ewald(const DirectArgs A)
{
    __shared__ double red[4][DT];
    const int64_t q = blockIdx.x;
    const int64_t i = A.targets ? A.targets[q] : q;
    const uint32_t xi = A.x[i], yi = A.y[i], zi = A.z[i];
    double ax = 0, ay = 0, az = 0, ph = 0;
    for (int64_t j = threadIdx.x; j < A.n; j += DT) {
        if (j == i) continue;
        const double dx = (double)(int32_t)(A.x[j] - xi) * A.unit;
        const double dy = (double)(int32_t)(A.y[j] - yi) * A.unit;
        const double dz = (double)(int32_t)(A.z[j] - zi) * A.unit;
        const double r2 = dx * dx + dy * dy + dz * dz, r = sqrt(r2);
        const double m = (double)A.m[j];
        double K, W;
        if (r >= A.h) {
            K = 1.0 / (r2 * r);
            W = 1.0 / r;
        } else {
            soft_kw(r * A.hinv, A.hinv, K, W);
        }
        double ps, gx, gy, gz;
        ewald_exact(dx, dy, dz, A.L, ps, gx, gy, gz);
        ax += m * (K * dx + gx);
        ay += m * (K * dy + gy);
        az += m * (K * dz + gz);
        ph += m * (ps - W);
    }
    red[0][threadIdx.x] = ax;
    red[1][threadIdx.x] = ay;
    red[2][threadIdx.x] = az;
    red[3][threadIdx.x] = ph;
    __syncthreads();
    for (int s = DT / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s)
            for (int c = 0; c < 4; c++) red[c][threadIdx.x] += red[c][threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        A.ax[q] = A.G * red[0][0];
        A.ay[q] = A.G * red[1][0];
        A.az[q] = A.G * red[2][0];
        if (A.pot) A.pot[q] = A.G * red[3][0];
    }
}

// Blocks of one launch: a grid holds fewer than 2^32 threads, which 2^26 targets reach
// at 8 targets to a block of 512.  More targets take more launches, one after the other.
#define DIRECT_BLOCKS ((int64_t)1 << 22)

template <int KER, int TB, bool FAR>
static void launch_direct_tb(DirectArgs A, hipStream_t s)
{
    // few targets: larger blocks, so that a block's lanes are more of the chip and its near
    // pairs, which differ much from block to block, more evenly spread (reach 0.075: 300
    // targets of 10^6 0.66 ms at 16 wavefronts, 0.68 at 8, 0.97 at 4; 10^4 targets 4.92, 4.28, 4.91)
    const int64_t blocks = (A.nt + TB - 1) / TB;
    if constexpr (TB < 8) {  // 8 targets a block only from 8192 on
        if (blocks < 1024) {
            k_direct<KER, TB, 16, FAR><<<(unsigned)blocks, 1024, 0, s>>>(A);
            return;
        }
    }
    for (int64_t b = 0; b < blocks; b += DIRECT_BLOCKS) {
        A.t0 = b * TB;
        k_direct<KER, TB, FAR ? 8 : 4, FAR><<<(unsigned)std::min(DIRECT_BLOCKS, blocks - b), FAR ? 512 : 256, 0, s>>>(A);
    }
}

// Targets per block: 8 (4 without lists, where the sums stay in registers)
// spare most source tests; fewer where that would leave less than four blocks
// per compute unit (5000 targets of 200 k, reach 0.2: 1.49 ms at 8, 1.30 at 4).
// The lists pay at every reach that the packed test can hold, below half the
// box side: 10^4 targets of 10^6 take 3.0 ms with and 24.6 without at a reach
// of 0.02, 18.5 and 58.9 at 0.33, 39.9 and 59.4 at 0.49 (300 targets of 50 k
// to 10^6 at 0.49: 12 % less with lists); beyond that a box has nothing to skip.
template <int KER>
static void launch_direct(const DirectArgs &A, double reach2, double box, hipStream_t s)
{
    if (reach2 * 4.1 <= box * box) {
        if (A.nt >= 8192) launch_direct_tb<KER, 8, true>(A, s);
        else if (A.nt >= 2048) launch_direct_tb<KER, 4, true>(A, s);
        else if (A.nt >= 1024) launch_direct_tb<KER, 2, true>(A, s);
        else launch_direct_tb<KER, 1, true>(A, s);
    } else {
        if (A.nt >= 2048) launch_direct_tb<KER, 4, false>(A, s);
        else if (A.nt >= 1024) launch_direct_tb<KER, 2, false>(A, s);
        else launch_direct_tb<KER, 1, false>(A, s);
    }
}

int g4_launch_direct(g4_ctx *ctx, const g4_particles *p, const g4_tree_params *tp, const g4_walk_params *wp,
                     int truncate, const int64_t *targets, int64_t ntargets, double *ax, double *ay, double *az,
                     double *pot)
{
    DirectArgs A;
    A.x = p->x; A.y = p->y; A.z = p->z; A.m = p->mass; A.n = p->n;
    A.targets = targets;
    A.nt = targets ? ntargets : p->n;
    A.t0 = 0;
    A.unit = tp->box / (tp->periodic ? 4294967296.0 : 2147483648.0);
    A.L = tp->box;
    A.h = 2.8 * wp->eps0;
    A.hinv = A.h > 0 ? 1.0 / A.h : 0.0;
    A.asplit = wp->kernel == 1 ? 0.5 / wp->r_s : 0.0;
    // beyond alpha r = 6, erfc < 3e-17: such sources add nothing in FP64
    A.rskip2 = wp->kernel == 1 ? (6.0 / A.asplit) * (6.0 / A.asplit) : 1e300;
    A.truncate = truncate;
    A.rcut2 = wp->r_cut * wp->r_cut;
    A.G = wp->G;
    A.ax = ax; A.ay = ay; A.az = az; A.pot = pot;
    const double reach2 = std::min(A.rskip2, truncate ? A.rcut2 : 1e300);
    A.near2 = (float)(reach2 / (A.unit * A.unit)) * 1.00001f;
    // at most 0.494 2^16 + 2 where the lists are used
    A.reach16 = (uint32_t)std::min(sqrt((double)A.near2) / 65536.0 + 2.0, 32767.0);
    if (A.nt > 0 && wp->kernel == 2) k_direct_ewald<<<(unsigned)A.nt, DT, 0, ctx->stream>>>(A);
    else if (A.nt > 0 && wp->kernel == 1) launch_direct<1>(A, reach2, tp->box, ctx->stream);
    else if (A.nt > 0) launch_direct<0>(A, reach2, tp->box, ctx->stream);
    G4_HIP(ctx, hipGetLastError());
    return G4_OK;
}
