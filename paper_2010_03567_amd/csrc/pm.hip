// pm.hip -- long-range force of the TreePM split on a periodic mesh (gfx950).
//
// Paper: Sec. "TreePM approach": the long-range potential is the k-space
// sum of the Ewald decomposition with the Green's function
// exp(-k^2 r_s^2) / k^2, evaluated with a particle-mesh method -- clouds-in-
// cell assignment, FFT, multiplication with the Green's function, inverse
// FFT, a 4th-order finite-difference gradient on the mesh and CIC
// interpolation to the particles, the smoothing of assignment and
// interpolation deconvolved by dividing by the CIC window (a squared sinc per
// axis) once for each.  The potential carries the sign of the Newtonian one
// (attractive): phi_lr = -G (4 pi / V) sum_{k != 0} exp(-k^2 r_s^2)/k^2 ...
//
// Layout: an ng^3 real FP32 mesh (z fastest), mesh point c at c h, h = L / ng,
// and its transform along z as ng/2 + 1 complex values per row (the rest is
// their conjugate).  The particles come from a built tree in curve order (so
// that neighbouring threads touch neighbouring cells) with 32-bit integer
// coordinates: for ng = 2^g the cell is the top g bits and the CIC weight
// the remaining bits, both exact.
//
// Steps: k_pm_deposit (8 atomics per particle; on small meshes FP64 sums that k_pm_round
// rounds; dense boxes by tiles in LDS, k_pm_deposit_tile, k_pm_interp_tile) -> k_pm_z_forward (two
// real lines as one complex transform) -> k_pm_lines along y -> k_pm_lines
// along x: forward, Green's function and inverse in one pass -> inverse along
// y -> k_pm_z_inverse, which leaves the real potential -> k_pm_interp
// (gradient and interpolation fused: each particle reads the potential around
// its 8 CIC points).
#include <algorithm>
#include <cmath>

#include "g4_internal.h"

// Complex values per row of the half spectrum: ng/2 + 1, padded so that rows
// of the larger meshes start on 64-byte boundaries.
__host__ __device__ constexpr int pm_pitch(int ng) { return ng / 2 + (ng >= 64 ? 8 : 1); }

// Tables, in FP64 rounded once: tw[m] = exp(-2 pi i m / ng), m < ng, and per
// axis gt[i] = exp(-k^2 r_s^2) / sinc^4(pi n / ng), k = 2 pi n / L, n the signed
// wave number of index i (the Gaussian and the twice deconvolved CIC window of
// the Green's function factorise over the axes).
__global__ void k_pm_tables(float2 *__restrict__ tw, float *__restrict__ gt, int ng, double box, double r_s)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ng) return;
    double s, c;
    sincospi(-2.0 * (double)i / (double)ng, &s, &c);
    tw[i] = make_float2((float)c, (float)s);
    const int n = i < ng / 2 ? i : i - ng;
    const double k = 2.0 * M_PI * n / box, u = M_PI * n / ng, w = n ? sin(u) / u : 1.0;
    // an infinite split scale leaves the mean alone, which the force drops: zero, not NaN
    gt[i] = n ? (float)(exp(-k * k * r_s * r_s) / (w * w * w * w)) : 1.f;
}

__global__ void k_pm_clear(float4 *__restrict__ m, size_t nvec)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < nvec; i += (size_t)gridDim.x * blockDim.x)
        m[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

// CIC cell and upper weight of one coordinate: top g bits, remaining bits / 2^(32-g)
__device__ __forceinline__ void pm_cell(uint32_t X, int shift, float wscale, int &i, float &f)
{
    i = (int)(X >> shift);
    f = (float)(X & ((1u << shift) - 1u)) * wscale;
}

// Particles arrive in curve order, so particles that share a mesh cell sit
// in consecutive lanes (the cell index is a prefix of the curve key; each CIC
// corner is the same shift of it).  Every corner's contributions are summed
// over such runs by a segmented scan across the wavefront and the last lane
// of a run issues the one atomic: in haloes most atomics disappear.  A wavefront
// takes RUN times 64 consecutive particles and carries the run at the end of each 64
// over to the next.
//
// The atomics come in any order.  Where the mesh is small they add in FP64, rounded
// once after (k_pm_round): two calls then differ in no bit but for a rare flip of that
// rounding.  With FP32 sums the particle that differs most between two calls of
// 30000 particles at 32^3 was off by 6e-5 of its force in the median, and by
// more than 1e-4 in 16 of 100 pairs of calls.  On larger meshes the wider sums would
// cost memory traffic (8 bytes more cleared and read a point), so there the longer runs
// leave fewer sums to the order instead.
#define PM_WIDE 64  // largest mesh side with FP64 sums
#define PM_RUN 4
template <typename T, int RUN>
__global__ void k_pm_deposit(const uint4 *__restrict__ parts, int64_t n, int ng, int shift, float wscale,
                             T *__restrict__ mesh)
{
    const int lane = threadIdx.x & 63;
    const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6, nwaves = (gridDim.x * (int64_t)blockDim.x) >> 6;
    for (int64_t base = wave * (64 * RUN); base < n; base += nwaves * (64 * RUN)) {
        uint32_t ckey[8];  // the run carried over, per corner (uniform; ~0: none)
        float cval[8];
#pragma unroll
        for (int c = 0; c < 8; c++) {
            ckey[c] = 0xffffffffu;
            cval[c] = 0.f;
        }
        for (int r = 0; r < RUN; r++) {
            const int64_t p = base + 64 * r + lane;
            const bool act = p < n;
            const uint4 q = act ? parts[p] : make_uint4(0u, 0u, 0u, 0u);
            const float m = act ? __uint_as_float(q.w) : 0.f;
            int ix, iy, iz;
            float fx, fy, fz;
            pm_cell(q.x, shift, wscale, ix, fx);
            pm_cell(q.y, shift, wscale, iy, fy);
            pm_cell(q.z, shift, wscale, iz, fz);
            const int mask = ng - 1;
#pragma unroll
            for (int c = 0; c < 8; c++) {
                const int dx = c >> 2, dy = (c >> 1) & 1, dz = c & 1;
                float v = m * (dx ? fx : 1.f - fx) * (dy ? fy : 1.f - fy) * (dz ? fz : 1.f - fz);
                const uint32_t key =
                    act ? (uint32_t)((((ix + dx) & mask) * ng + ((iy + dy) & mask)) * ng + ((iz + dz) & mask)) : 0xffffffffu;
                if (lane == 0 && ckey[c] != 0xffffffffu) {
                    if (ckey[c] == key) v += cval[c];
                    else atomicAdd(&mesh[ckey[c]], (T)cval[c]);
                }
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const uint32_t ku = (uint32_t)__shfl_up((int)key, off);
                    const float vu = __shfl_up(v, off);
                    if (lane >= off && ku == key) v += vu;
                }
                const uint32_t kd = (uint32_t)__shfl_down((int)key, 1);
                if (act && lane != 63 && kd != key) atomicAdd(&mesh[key], (T)v);
                ckey[c] = (uint32_t)__shfl((int)key, 63);
                cval[c] = __shfl(v, 63);
            }
        }
#pragma unroll
        for (int c = 0; c < 8; c++)
            if (lane == 0 && ckey[c] != 0xffffffffu) atomicAdd(&mesh[ckey[c]], (T)cval[c]);
    }
}

__global__ void k_pm_round(const double2 *__restrict__ wide, size_t npair, float2 *__restrict__ mesh)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < npair; i += (size_t)gridDim.x * blockDim.x) {
        const double2 v = wide[i];
        mesh[i] = make_float2((float)v.x, (float)v.y);
    }
}

// ---------------------------------------------------------------- transforms
// An N-point line (N = 8 .. 1024) is held by N / 8 threads, 8 points each in
// registers: thread j holds points j + q N / 8.  Radix-8 steps (self-sorting
// order, the last one of radix 2 or 4 where log2 N is no multiple of 3) exchange
// through LDS in between, so 512 points cross it twice (an in-place transform
// in LDS with fused radix-2 pairs crossed it ten times).  Global loads and stores
// go straight between registers and memory.  Every pass is bound by HBM: 8 or
// 6 bytes per mesh point and pass, 44 for a call where the complex mesh moved
// 120.  Mesh 512^3, 2^24 particles: transforms and Green's function 6.3 -> 1.24 ms, 5.1 TB/s.
__device__ __forceinline__ float2 c_add(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 c_sub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 c_mul(float2 a, float2 w) { return make_float2(a.x * w.x - a.y * w.y, a.x * w.y + a.y * w.x); }
// times exp(SIGN i pi / 2)
template <int SIGN>
__device__ __forceinline__ float2 c_quarter(float2 a)
{
    return SIGN < 0 ? make_float2(a.y, -a.x) : make_float2(-a.y, a.x);
}

template <int SIGN>
__device__ __forceinline__ void dft2(float2 &a, float2 &b)
{
    const float2 t = c_sub(a, b);
    a = c_add(a, b);
    b = t;
}
template <int SIGN>
__device__ __forceinline__ void dft4(float2 &a, float2 &b, float2 &c, float2 &d)
{
    const float2 s0 = c_add(a, c), s1 = c_sub(a, c), s2 = c_add(b, d), s3 = c_quarter<SIGN>(c_sub(b, d));
    a = c_add(s0, s2);
    b = c_add(s1, s3);
    c = c_sub(s0, s2);
    d = c_sub(s1, s3);
}
template <int SIGN>
__device__ __forceinline__ void dft8(float2 v[8])
{
    constexpr float r = 0.70710678118654752f;
    dft4<SIGN>(v[0], v[2], v[4], v[6]);
    dft4<SIGN>(v[1], v[3], v[5], v[7]);
    // odd half times exp(SIGN 2 pi i k / 8)
    const float2 o1 = make_float2(r * (v[3].x - SIGN * v[3].y), r * (SIGN * v[3].x + v[3].y));
    const float2 o2 = c_quarter<SIGN>(v[5]);
    const float2 o3 = make_float2(r * (-v[7].x - SIGN * v[7].y), r * (SIGN * v[7].x - v[7].y));
    const float2 e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6], o0 = v[1];
    v[0] = c_add(e0, o0);
    v[4] = c_sub(e0, o0);
    v[1] = c_add(e1, o1);
    v[5] = c_sub(e1, o1);
    v[2] = c_add(e2, o2);
    v[6] = c_sub(e2, o2);
    v[3] = c_add(e3, o3);
    v[7] = c_sub(e3, o3);
}

constexpr int ilog2c(int v) { return v <= 1 ? 0 : 1 + ilog2c(v / 2); }

// The transform of one line: v[q] is point j + q N/8 before and after.  sm: LDS
// of the block, at(p) the place of point p of this line in it; tw: exp(-2 pi i m / N)
// in LDS.  Every thread of the block calls this (barriers).  Unnormalised.
template <int N, int SIGN, typename At>
__device__ __forceinline__ void fft_line(float2 v[8], int j, float2 *sm, const At &at, const float2 *tw)
{
    constexpr int T = N / 8, LG = ilog2c(N), S8 = LG / 3, R = 1 << (LG % 3);
    auto twid = [&](int m) {
        const float2 w = tw[m];
        return SIGN < 0 ? w : make_float2(w.x, -w.y);
    };
    int ns = 1;
#pragma unroll
    for (int s = 0; s < S8; s++) {
        if (s > 0) {
            const int e = (j & (ns - 1)) * (N / (8 * ns));
#pragma unroll
            for (int k = 1; k < 8; k++) v[k] = c_mul(v[k], twid(e * k));
        }
        dft8<SIGN>(v);
        if (s + 1 < S8 || R > 1) {
            const int base = (j / ns) * ns * 8 + (j & (ns - 1));
#pragma unroll
            for (int k = 0; k < 8; k++) sm[at(base + k * ns)] = v[k];
            __syncthreads();
#pragma unroll
            for (int k = 0; k < 8; k++) v[k] = sm[at(j + k * T)];
            __syncthreads();
        }
        ns *= 8;
    }
    if constexpr (R == 2) {
#pragma unroll
        for (int m = 0; m < 4; m++) {
            v[m + 4] = c_mul(v[m + 4], twid(j + m * T));
            dft2<SIGN>(v[m], v[m + 4]);
        }
    } else if constexpr (R == 4) {
#pragma unroll
        for (int m = 0; m < 2; m++) {
            const int b = j + m * T;
#pragma unroll
            for (int k = 1; k < 4; k++) v[m + 2 * k] = c_mul(v[m + 2 * k], twid(b * k));
            dft4<SIGN>(v[m], v[m + 2], v[m + 4], v[m + 6]);
        }
    }
}

// threads of a z pass: 256 / (N / 8) pairs of lines per block
#define PM_Z_THREADS 256

// Forward along z: rows 2 p and 2 p + 1 of the real mesh as the real and
// imaginary part of one transform Z; A_k = (Z_k + Z*_{N-k})/2, B_k = (Z_k - Z*_{N-k})/2i.
template <int N>
__global__ __launch_bounds__(PM_Z_THREADS) void k_pm_z_forward(const float *__restrict__ real, float2 *__restrict__ half,
                                                               const float2 *__restrict__ tw)
{
    constexpr int T = N / 8, LP = PM_Z_THREADS / T, LINE = N + N / 8 + 1, PZ = pm_pitch(N);
    __shared__ float2 tws[N], sm[LP * LINE];
    for (int k = threadIdx.x; k < N; k += PM_Z_THREADS) tws[k] = tw[k];
    const int t = threadIdx.x / T, j = threadIdx.x % T;
    const size_t pr = (size_t)blockIdx.x * LP + t;
    const bool have = pr < (size_t)N * N / 2;
    const auto at = [&](int p) { return t * LINE + p + (p >> 3); };
    float2 v[8];
    const float *r0 = real + (have ? 2 * pr : 0) * N;
#pragma unroll
    for (int q = 0; q < 8; q++) v[q] = make_float2(r0[j + q * T], r0[N + j + q * T]);
    __syncthreads();
    fft_line<N, -1>(v, j, sm, at, tws);
#pragma unroll
    for (int q = 0; q < 8; q++) sm[at(j + q * T)] = v[q];
    __syncthreads();
    if (!have) return;
    float2 *a = half + 2 * pr * PZ, *b = a + PZ;
#pragma unroll
    for (int m = 0; m < 5; m++) {
        const int k = j + m * T;
        if (m == 4 && j > 0) break;  // k = N / 2 by the first thread
        const float2 z = sm[at(k)], y = sm[at((N - k) & (N - 1))];
        a[k] = make_float2(0.5f * (z.x + y.x), 0.5f * (z.y - y.y));
        b[k] = make_float2(0.5f * (z.y + y.y), 0.5f * (y.x - z.x));
    }
}

// Inverse along z: Z = A + i B over the full line from the two half rows (the
// values at 0 and N / 2 are real), whose transform has line A in its real and line
// B in its imaginary part.
template <int N>
__global__ __launch_bounds__(PM_Z_THREADS) void k_pm_z_inverse(const float2 *__restrict__ half, float *__restrict__ real,
                                                               const float2 *__restrict__ tw)
{
    constexpr int T = N / 8, LP = PM_Z_THREADS / T, LINE = N + N / 8 + 1, PZ = pm_pitch(N);
    __shared__ float2 tws[N], sm[LP * LINE];
    for (int k = threadIdx.x; k < N; k += PM_Z_THREADS) tws[k] = tw[k];
    const int t = threadIdx.x / T, j = threadIdx.x % T;
    const size_t pr = (size_t)blockIdx.x * LP + t;
    const bool have = pr < (size_t)N * N / 2;
    const auto at = [&](int p) { return t * LINE + p + (p >> 3); };
    const float2 *a = half + (have ? 2 * pr : 0) * PZ, *b = a + PZ;
    float2 v[8];
#pragma unroll
    for (int q = 0; q < 8; q++) {
        const int k = j + q * T;
        const bool low = k <= N / 2;
        const float2 x = a[low ? k : N - k], y = b[low ? k : N - k];
        if (k == 0 || k == N / 2) v[q] = make_float2(x.x, y.x);
        else v[q] = low ? make_float2(x.x - y.y, x.y + y.x) : make_float2(x.x + y.y, y.x - x.y);
    }
    __syncthreads();
    fft_line<N, 1>(v, j, sm, at, tws);
    if (!have) return;
    float *r0 = real + 2 * pr * N;
#pragma unroll
    for (int q = 0; q < 8; q++) {
        r0[j + q * T] = v[q].x;
        r0[N + j + q * T] = v[q].y;
    }
}

// Lines along y or x of the half spectrum, in place: a block takes PM_COLS lines
// neighbouring in z, so that every row of the tile is a run of 64 to 128 bytes.
// MODE 0: forward along y, 1: inverse along y, 2: along x forward, times the
// Green's function with the CIC window deconvolved twice,
// F(k) = -G (4 pi / V) exp(-k^2 r_s^2) / k^2 / W(k)^2, W = prod_d sinc^2(pi n_d / N),
// F(0) = 0, and inverse: the points of a line stay in registers between the two.
constexpr int pm_cols(int n) { return n >= 1024 ? 8 : 16; }

template <int N, int MODE>
__global__ __launch_bounds__(pm_cols(N) *N / 8) void k_pm_lines(float2 *__restrict__ half, const float2 *__restrict__ tw,
                                                               const float *__restrict__ gt, float pref)
{
    constexpr int T = N / 8, TL = pm_cols(N), NZ = N / 2 + 1, PZ = pm_pitch(N), TILES = (NZ + TL - 1) / TL;
    __shared__ float2 tws[N], sm[(N + N / 8) * TL];
    for (int k = threadIdx.x; k < N; k += TL * T) tws[k] = tw[k];
    const int t = threadIdx.x % TL, j = threadIdx.x / TL;
    const int outer = blockIdx.x / TILES, z = (blockIdx.x % TILES) * TL + t;
    const bool have = z < NZ;
    const auto at = [&](int p) { return (p + (p >> 3)) * TL + t; };
    // y: rows outer N + p; x: rows p N + outer
    const size_t stride = MODE == 2 ? (size_t)N * PZ : (size_t)PZ;
    float2 *line = half + (MODE == 2 ? (size_t)outer * PZ : (size_t)outer * N * PZ) + (have ? z : 0);
    float2 v[8];
#pragma unroll
    for (int q = 0; q < 8; q++) v[q] = line[(size_t)(j + q * T) * stride];
    __syncthreads();
    if constexpr (MODE == 0) fft_line<N, -1>(v, j, sm, at, tws);
    if constexpr (MODE == 1) fft_line<N, 1>(v, j, sm, at, tws);
    if constexpr (MODE == 2) {
        fft_line<N, -1>(v, j, sm, at, tws);
        const int ny = outer < N / 2 ? outer : outer - N;
        const float gyz = gt[outer] * gt[have ? z : 0] * pref;
        const int n2 = ny * ny + z * z;
#pragma unroll
        for (int q = 0; q < 8; q++) {
            const int ix = j + q * T, nx = ix < N / 2 ? ix : ix - N;
            const int k2 = nx * nx + n2;
            const float f = k2 ? gyz * gt[ix] / (float)k2 : 0.f;
            v[q].x *= f;
            v[q].y *= f;
        }
        fft_line<N, 1>(v, j, sm, at, tws);
    }
    if (!have) return;
#pragma unroll
    for (int q = 0; q < 8; q++) line[(size_t)(j + q * T) * stride] = v[q];
}

// real mesh -> real potential, through the half spectrum
template <int N>
static void pm_potential(float *real, float2 *half, const float2 *tw, const float *gt, float pref, hipStream_t s)
{
    constexpr int T = N / 8, LP = PM_Z_THREADS / T, TL = pm_cols(N), TILES = (N / 2 + 1 + TL - 1) / TL;
    const unsigned zb = (unsigned)(((size_t)N * N / 2 + LP - 1) / LP), lb = (unsigned)N * TILES;
    k_pm_z_forward<N><<<zb, PM_Z_THREADS, 0, s>>>(real, half, tw);
    k_pm_lines<N, 0><<<lb, TL * T, 0, s>>>(half, tw, gt, pref);
    k_pm_lines<N, 2><<<lb, TL * T, 0, s>>>(half, tw, gt, pref);
    k_pm_lines<N, 1><<<lb, TL * T, 0, s>>>(half, tw, gt, pref);
    k_pm_z_inverse<N><<<zb, PM_Z_THREADS, 0, s>>>(half, real, tw);
}

// gradient (4th-order differences) and CIC interpolation at one particle;
// at(x, y, z): the potential at a mesh point
template <typename At>
__device__ __forceinline__ void pm_gradient(const At &at, int ix, int iy, int iz, float fx, float fy, float fz, bool pot,
                                            float &gx, float &gy, float &gz, float &ph)
{
    gx = gy = gz = ph = 0.f;
#pragma unroll
    for (int c = 0; c < 8; c++) {
        const int dx = c >> 2, dy = (c >> 1) & 1, dz = c & 1;
        const float w = (dx ? fx : 1.f - fx) * (dy ? fy : 1.f - fy) * (dz ? fz : 1.f - fz);
        const int x = ix + dx, y = iy + dy, z = iz + dz;
        const float d1x = at(x + 1, y, z) - at(x - 1, y, z), d2x = at(x + 2, y, z) - at(x - 2, y, z);
        const float d1y = at(x, y + 1, z) - at(x, y - 1, z), d2y = at(x, y + 2, z) - at(x, y - 2, z);
        const float d1z = at(x, y, z + 1) - at(x, y, z - 1), d2z = at(x, y, z + 2) - at(x, y, z - 2);
        gx = fmaf(w, (2.f / 3.f) * d1x - (1.f / 12.f) * d2x, gx);
        gy = fmaf(w, (2.f / 3.f) * d1y - (1.f / 12.f) * d2y, gy);
        gz = fmaf(w, (2.f / 3.f) * d1z - (1.f / 12.f) * d2z, gz);
        if (pot) ph = fmaf(w, at(x, y, z), ph);
    }
}

struct PmOut {
    float inv_h;
    int accumulate;
    double *ax, *ay, *az, *pot;
};
__device__ __forceinline__ void pm_write(const PmOut &O, uint32_t o, float gx, float gy, float gz, float ph)
{
    const double a0 = -(double)gx * O.inv_h, a1 = -(double)gy * O.inv_h, a2 = -(double)gz * O.inv_h;
    if (O.accumulate) {
        O.ax[o] += a0;
        O.ay[o] += a1;
        O.az[o] += a2;
        if (O.pot) O.pot[o] += (double)ph;
    } else {
        O.ax[o] = a0;
        O.ay[o] = a1;
        O.az[o] = a2;
        if (O.pot) O.pot[o] = (double)ph;
    }
}

// staged results (g_x, g_y, g_z, phi; caller order) into the output arrays
__global__ void k_pm_finish(const float4 *__restrict__ staged, int64_t n, const PmOut O)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float4 v = staged[i];
        pm_write(O, (uint32_t)i, v.x, v.y, v.z, v.w);
    }
}

// one particle per thread, the potential read from memory
__global__ void k_pm_interp(const uint4 *__restrict__ parts, const uint32_t *__restrict__ perm, int64_t n,
                            const float *__restrict__ phi, int ng, int lg, int shift, float wscale, const PmOut O)
{
    const int mask = ng - 1;
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x) {
        const uint4 q = parts[p];
        int ix, iy, iz;
        float fx, fy, fz, gx, gy, gz, ph;
        pm_cell(q.x, shift, wscale, ix, fx);
        pm_cell(q.y, shift, wscale, iy, fy);
        pm_cell(q.z, shift, wscale, iz, fz);
        const auto at = [&](int x, int y, int z) {
            return phi[((size_t)(x & mask) << (2 * lg)) + ((size_t)(y & mask) << lg) + (size_t)(z & mask)];
        };
        pm_gradient(at, ix, iy, iz, fx, fy, fz, O.pot != nullptr, gx, gy, gz, ph);
        pm_write(O, perm[p], gx, gy, gz, ph);
    }
}

// ------------------------------------------------------------------- tiles
// A cube of PM_CUBE^3 mesh cells is a node of the curve, so its particles are one
// run of the sorted ones.  With enough particles per cube the mesh around a cube
// is staged in LDS: the deposit adds there and then once per cell to memory, where
// the 8 float atomics per particle were the bound; the interpolation
// reads its 56 potentials per particle from LDS instead of through L1.
//
// The rule: at least PM_TILE_MIN particles per cube on average, which pay for
// staging its 4913 and 9261 mesh points, and PM_TILE_N in all (a third of it from 128^3
// on, where the mesh fills the chip's blocks with cubes), which pay for the work
// list.  Whole call by memory / by tiles, ms: 2e5 particles at 128^3 (391 a cube)
// 0.125 / 0.103, at 64^3 (3125) 0.066 / 0.071, at 256^3 (49) 0.262 / 0.257; 10^6 at
// 64^3 0.139 / 0.122, at 256^3 (244) 0.433 / 0.305; 4e6 at 512^3 (122) 2.84 / 2.18; 2^24
// at 512^3 (512) 6.03 / 2.95.
#define PM_TILE_MIN 100
#define PM_TILE_N 500000
#define PM_CUBE_BITS 4
#define PM_CUBE (1 << PM_CUBE_BITS)
#define PM_DT (PM_CUBE + 1)      // deposit tile side: the cube and its upper neighbours
#define PM_IT (PM_CUBE + 5)      // interpolation tile side: two points more on either side
#define PM_ITEM 4096             // particles of one work item at most (denser cubes are shared by several)
#define PM_DEP_THREADS 256
#define PM_INT_THREADS 512

// first particle of every cube (in key order), from the steps of the sorted keys' prefixes
__global__ void k_pm_starts(const uint64_t *__restrict__ keys, int64_t n, int kshift, uint32_t ncube,
                            uint32_t *__restrict__ start, uint32_t *__restrict__ nitems)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i == 0) *nitems = 0;
    if (i > n) return;
    const uint32_t lo = i == 0 ? 0u : (uint32_t)(keys[i - 1] >> kshift) + 1u;
    const uint32_t hi = i == n ? ncube : (uint32_t)(keys[i] >> kshift);
    for (uint32_t c = lo; c <= hi; c++) start[c] = (uint32_t)i;
}

// work items (first particle, count)
__global__ __launch_bounds__(256) void k_pm_items(const uint32_t *__restrict__ start, uint32_t ncube,
                                                  uint4 *__restrict__ items, uint32_t *__restrict__ nitems)
{
    const uint32_t c = blockIdx.x * 256 + threadIdx.x;
    const int lane = threadIdx.x & 63;
    const uint32_t first = c < ncube ? start[c] : 0u, count = c < ncube ? start[c + 1] - first : 0u;
    const uint32_t parts = (count + PM_ITEM - 1) / PM_ITEM;
    uint32_t incl = parts;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t v = (uint32_t)__shfl_up((int)incl, off);
        if (lane >= off) incl += v;
    }
    uint32_t base = 0;
    if (lane == 63 && incl) base = atomicAdd(nitems, incl);
    base = (uint32_t)__shfl((int)base, 63) + incl - parts;
    for (uint32_t k = 0; k < parts; k++)
        items[base + k] = make_uint4(first + k * PM_ITEM, min(count - k * PM_ITEM, (uint32_t)PM_ITEM), 0u, 0u);
}

// A thread takes a run of consecutive particles: particles of one cell follow
// each other, so it adds them up in registers and goes to LDS only when the cell
// changes, and the threads of a wavefront work in different cells.
__global__ __launch_bounds__(PM_DEP_THREADS) void k_pm_deposit_tile(const uint4 *__restrict__ parts,
                                                                    const uint4 *__restrict__ items,
                                                                    const uint32_t *__restrict__ nitems, int ng, int lg,
                                                                    int shift, float wscale, float *__restrict__ mesh)
{
    __shared__ float tile[PM_DT * PM_DT * PM_DT];
    if (blockIdx.x >= *nitems) return;
    const uint4 it = items[blockIdx.x];
    for (int e = threadIdx.x; e < PM_DT * PM_DT * PM_DT; e += PM_DEP_THREADS) tile[e] = 0.f;
    const uint4 q0 = parts[it.x];
    const int bx = (int)(q0.x >> shift) & ~(PM_CUBE - 1),
              by = (int)(q0.y >> shift) & ~(PM_CUBE - 1),
              bz = (int)(q0.z >> shift) & ~(PM_CUBE - 1);
    __syncthreads();
    const uint32_t per = (it.y + PM_DEP_THREADS - 1) / PM_DEP_THREADS;
    const uint32_t p0 = it.x + min(it.y, threadIdx.x * per), p1 = it.x + min(it.y, (threadIdx.x + 1) * per);
    int cell = -1;
    float s[8];
#pragma unroll
    for (int c = 0; c < 8; c++) s[c] = 0.f;
    auto flush = [&]() {
#pragma unroll
        for (int c = 0; c < 8; c++) {
            atomicAdd(&tile[cell + (c >> 2) * PM_DT * PM_DT + ((c >> 1) & 1) * PM_DT + (c & 1)], s[c]);
            s[c] = 0.f;
        }
    };
    for (uint32_t p = p0; p < p1; p++) {
        const uint4 q = parts[p];
        int ix, iy, iz;
        float fx, fy, fz;
        pm_cell(q.x, shift, wscale, ix, fx);
        pm_cell(q.y, shift, wscale, iy, fy);
        pm_cell(q.z, shift, wscale, iz, fz);
        const int here = ((ix - bx) * PM_DT + (iy - by)) * PM_DT + (iz - bz);
        if (here != cell) {
            if (cell >= 0) flush();
            cell = here;
        }
        const float m = __uint_as_float(q.w);
#pragma unroll
        for (int c = 0; c < 8; c++) {
            const int dx = c >> 2, dy = (c >> 1) & 1, dz = c & 1;
            s[c] += m * (dx ? fx : 1.f - fx) * (dy ? fy : 1.f - fy) * (dz ? fz : 1.f - fz);
        }
    }
    if (cell >= 0) flush();
    __syncthreads();
    const int mask = ng - 1;
    // 16 lanes add a row of the cube, one line of memory, then the points above the rows
    // follow.  (Points that no other cube reaches need no atomic, but storing those and adding
    // only the cube's shell broke every row into three requests: mesh 512^3, 2^24 particles
    // 1.02 ms with the stores, 0.62 all atomic, 0.58 row by row.)
    auto add = [&](int row, int z) {
        const float v = tile[row * PM_DT + z];
        const int x = row / PM_DT, y = row - x * PM_DT;
        if (v != 0.f)
            atomicAdd(&mesh[((size_t)((bx + x) & mask) << (2 * lg)) + ((size_t)((by + y) & mask) << lg) +
                            (size_t)((bz + z) & mask)], v);
    };
    for (int row = threadIdx.x / PM_CUBE; row < PM_DT * PM_DT; row += PM_DEP_THREADS / PM_CUBE)
        add(row, threadIdx.x % PM_CUBE);
    for (int row = threadIdx.x; row < PM_DT * PM_DT; row += PM_DEP_THREADS) add(row, PM_CUBE);
}

__global__ __launch_bounds__(PM_INT_THREADS) void k_pm_interp_tile(const uint4 *__restrict__ parts,
                                                                   const uint32_t *__restrict__ perm,
                                                                   const uint4 *__restrict__ items,
                                                                   const uint32_t *__restrict__ nitems,
                                                                   const float *__restrict__ phi, int ng, int lg,
                                                                   int shift, float wscale, const PmOut O,
                                                                   float4 *__restrict__ staged)
{
    __shared__ float tile[PM_IT * PM_IT * PM_IT];
    if (blockIdx.x >= *nitems) return;
    const uint4 it = items[blockIdx.x];
    const uint4 q0 = parts[it.x];
    const int bx = ((int)(q0.x >> shift) & ~(PM_CUBE - 1)) - 2,
              by = ((int)(q0.y >> shift) & ~(PM_CUBE - 1)) - 2,
              bz = ((int)(q0.z >> shift) & ~(PM_CUBE - 1)) - 2;
    const int mask = ng - 1;
    // several loads in flight (512^3, 2^24 particles: 1.01 ms one by one, 0.85 by 2, 0.83 by 6, 0.90 by 10)
#pragma unroll 6
    for (int e = threadIdx.x; e < PM_IT * PM_IT * PM_IT; e += PM_INT_THREADS) {
        const int x = e / (PM_IT * PM_IT), y = e / PM_IT % PM_IT, z = e % PM_IT;
        tile[e] = phi[((size_t)((bx + x) & mask) << (2 * lg)) + ((size_t)((by + y) & mask) << lg) +
                      (size_t)((bz + z) & mask)];
    }
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < it.y; k += PM_INT_THREADS) {
        const uint4 q = parts[it.x + k];
        int ix, iy, iz;
        float fx, fy, fz, gx, gy, gz, ph;
        pm_cell(q.x, shift, wscale, ix, fx);
        pm_cell(q.y, shift, wscale, iy, fy);
        pm_cell(q.z, shift, wscale, iz, fz);
        const auto at = [&](int x, int y, int z) { return tile[(x * PM_IT + y) * PM_IT + z]; };
        pm_gradient(at, ix - bx, iy - by, iz - bz, fx, fy, fz, O.pot != nullptr, gx, gy, gz, ph);
        if (staged) staged[perm[it.x + k]] = make_float4(gx, gy, gz, ph);
        else pm_write(O, perm[it.x + k], gx, gy, gz, ph);
    }
}

static int ilog2(int v)
{
    int g = 0;
    while ((1 << g) < v) g++;
    return g;
}

// real mesh (density, then potential), half spectrum, tables
struct PmLayout {
    size_t real, half, tw, gt, spare, total;
};
static int pm_layout(int ng, PmLayout *L)
{
    if (ng < 8 || ng > 1024 || (ng & (ng - 1))) return G4_EINVAL;
    auto al = [](size_t b) { return (b + 255) / 256 * 256; };
    const size_t ncell = (size_t)ng * ng * ng;
    L->real = 0;
    L->half = al(ncell * 4);
    L->tw = L->half + al((size_t)ng * ng * pm_pitch(ng) * 8);
    L->gt = L->tw + al((size_t)ng * 8);
    L->spare = L->gt + al((size_t)ng * 4);
    L->total = std::max(L->spare, al((size_t)ng / 2 * 8) + al(ncell * 8) + al(ncell * 4));
    return G4_OK;
}

int g4_pm_layout_bytes(int ng, size_t *bytes)
{
    PmLayout L;
    if (pm_layout(ng, &L)) return G4_EINVAL;
    *bytes = L.total;
    return G4_OK;
}

int g4_launch_pm(g4_ctx *ctx, const g4_tree *t, const g4_pm_params *pp, void *ws, size_t ws_bytes, int accumulate,
                 double *ax, double *ay, double *az, double *pot)
{
    const int ng = pp->ng, lg = ilog2(ng);
    PmLayout L;
    if (pm_layout(ng, &L)) return g4_set_err(ctx, G4_EINVAL, "ng must be a power of two in [8, 1024]");
    if (ws_bytes < L.total) return g4_set_err(ctx, G4_ENOMEM, "pm workspace too small");
    char *b = (char *)ws;
    const size_t ncell = (size_t)ng * ng * ng;
    float *phi = (float *)(b + L.real), *gt = (float *)(b + L.gt);
    float2 *half = (float2 *)(b + L.half), *tw = (float2 *)(b + L.tw);
    hipStream_t s = ctx->stream;
    const int shift = 32 - lg;
    const float wscale = ldexpf(1.f, -shift);
    auto clear = [&](void *p, size_t bytes) {
        k_pm_clear<<<(unsigned)std::min<size_t>(4096, (bytes / 16 + 255) / 256), 256, 0, s>>>((float4 *)p, bytes / 16);
    };
    const int64_t n = t->n;
    const unsigned pblocks = (unsigned)std::min<int64_t>(8192, (n + 255) / 256);
    // work items of the tiles, if the particles are dense enough for them and the lists fit
    const uint32_t ncube = lg >= PM_CUBE_BITS ? 1u << (3 * (lg - PM_CUBE_BITS)) : 0u;
    const size_t max_items = ncube + (size_t)(n / PM_ITEM);
    uint32_t *nitems = (uint32_t *)(b + L.spare), *start = nitems + 64;
    uint4 *items = (uint4 *)(b + L.spare + 256 + ((size_t)ncube + 1 + 63) / 64 * 256);
    const bool tiles = ncube && n >= (int64_t)PM_TILE_MIN * ncube && n >= (ng >= 128 ? PM_TILE_N / 3 : PM_TILE_N) &&
                       (char *)(items + max_items) <= b + L.total;
    // the FP64 mesh lies behind the real one, where the spectrum and the tables come later
    const bool wide = !tiles && ng <= PM_WIDE && L.half + ncell * sizeof(double) <= L.total;
    if (tiles) {
        clear(phi, ncell * 4);
        k_pm_starts<<<(unsigned)((n + 1 + 255) / 256), 256, 0, s>>>(t->keys1, n, 3 * (G4_MAXLEV - lg + PM_CUBE_BITS), ncube,
                                                                  start, nitems);
        k_pm_items<<<(ncube + 255) / 256, 256, 0, s>>>(start, ncube, items, nitems);
        k_pm_deposit_tile<<<(unsigned)max_items, PM_DEP_THREADS, 0, s>>>(t->parts, items, nitems, ng, lg, shift, wscale,
                                                                         phi);
    } else if (wide) {
        double *mesh = (double *)(b + L.half);
        clear(mesh, ncell * 8);
        k_pm_deposit<double, 1><<<pblocks, 256, 0, s>>>(t->parts, n, ng, shift, wscale, mesh);
        k_pm_round<<<(unsigned)std::min<size_t>(1024, (ncell / 2 + 255) / 256), 256, 0, s>>>((const double2 *)mesh, ncell / 2,
                                                                                          (float2 *)phi);
    } else {
        clear(phi, ncell * 4);
        k_pm_deposit<float, PM_RUN><<<pblocks, 256, 0, s>>>(t->parts, n, ng, shift, wscale, phi);
    }
    k_pm_tables<<<(ng + 255) / 256, 256, 0, s>>>(tw, gt, ng, t->tp.box, pp->r_s);
    // -G 4 pi / V / (2 pi / L)^2: the sum over wave numbers in units of 2 pi / L
    const float pref = (float)(-pp->G / (M_PI * t->tp.box));
    switch (lg) {
    case 3: pm_potential<8>(phi, half, tw, gt, pref, s); break;
    case 4: pm_potential<16>(phi, half, tw, gt, pref, s); break;
    case 5: pm_potential<32>(phi, half, tw, gt, pref, s); break;
    case 6: pm_potential<64>(phi, half, tw, gt, pref, s); break;
    case 7: pm_potential<128>(phi, half, tw, gt, pref, s); break;
    case 8: pm_potential<256>(phi, half, tw, gt, pref, s); break;
    case 9: pm_potential<512>(phi, half, tw, gt, pref, s); break;
    default: pm_potential<1024>(phi, half, tw, gt, pref, s); break;
    }
    const PmOut O{(float)(ng / t->tp.box), accumulate, ax, ay, az, pot};
    if (tiles) {
        // Every output array written in the caller's order costs a particle one line of
        // memory each; staged as one 16-byte record in the spectrum's place (free by now,
        // if it is large enough) it costs one, and the arrays are then streamed.
        // Whole call by scattered arrays / staged, ms: 5e5 particles at 256^3 0.307 / 0.296,
        // 4e6 0.660 / 0.510, 2^24 at 512^3 4.17 / 3.55 (added to the outputs: 4.86 / 3.63).
        float4 *staged = (size_t)n * sizeof(float4) <= L.tw - L.half ? (float4 *)half : nullptr;
        k_pm_interp_tile<<<(unsigned)max_items, PM_INT_THREADS, 0, s>>>(t->parts, t->perm1, items, nitems, phi, ng, lg, shift,
                                                                        wscale, O, staged);
        if (staged) k_pm_finish<<<4096, 256, 0, s>>>(staged, n, O);
    } else
        k_pm_interp<<<pblocks, 256, 0, s>>>(t->parts, t->perm1, n, phi, ng, lg, shift, wscale, O);
    G4_HIP(ctx, hipGetLastError());
    return G4_OK;
}
