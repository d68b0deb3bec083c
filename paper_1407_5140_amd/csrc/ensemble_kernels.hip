// Kernels of the n-run error analysis and of the canonical averages:
//   k_boot_mean  the bin-wise mean of n runs' pieces per window, for the
//                ensemble itself and for bootstrap resamples (Sec. II.B)
//   k_thermo     u, c and f per spin from a density of states over a grid of
//                temperatures (the specific-heat analysis of Sec. IV.A)
// The joining of the mean pieces is k_concat, one block per resample.
#pragma once
#include "rewl_device.hpp"

namespace rewl {

enum : uint32_t { kTagBoot = 4 };

// Grid (h, R + 1), 256 threads, n pointers of dynamic LDS.  runs[i] points at
// run i's window tables [h][WB]; mean receives [R + 1][h][WB].  Resample 0
// takes run j for draw j; resample r >= 1 takes run floor(x0 n / 2^32) for
// draw j of window a, x0 the first Philox word at counter (r, j, a, kTagBoot).
// The sum runs in draw order and is then divided by n.
__global__ void __launch_bounds__(256) k_boot_mean(const double* const* __restrict__ runs, int n,
                                                   int h, int WB, uint32_t k0, uint32_t k1,
                                                   double* __restrict__ mean)
{
    extern __shared__ const double* piece[];   // draw j -> the picked run's table of window a
    const int a = blockIdx.x, r = blockIdx.y;
    const size_t off = (size_t)a * WB;
    for (int j = threadIdx.x; j < n; j += blockDim.x) {
        int p = j;
        if (r > 0) {
            const u32x4 x = philox10((uint32_t)r, (uint32_t)j, (uint32_t)a, kTagBoot, k0, k1);
            p = (int)(((uint64_t)x.x * (uint64_t)n) >> 32);
        }
        piece[j] = runs[p] + off;
    }
    __syncthreads();
    double* o = mean + ((size_t)r * h + a) * WB;
    for (int b = threadIdx.x; b < WB; b += blockDim.x) {
        double acc = 0.0;
        for (int j = 0; j < n; ++j) acc += piece[j][b];
        o[b] = acc / (double)n;
    }
}

// ------------------------------------------------------------------ thermo
// u, c and f of rows of ln g on a grid of temperatures.  The sums over the levels
// are a contraction: in a block of 64 bins about the energy Ek,
//   e^{ln g(E) - E/T} = e^{ln g(Ek') - Ek/T} G(row, E) K(E, T),
// G = e^{ln g - ln g(Ek') - b (E - Ek)} scaled to at most 1, K = e^{-(1/T - b)(E - Ek)}
// with b in the middle of the tile's 1/T: so one exponential per row and level and a
// table of 64 per temperature (the same for every block) take the place of one per
// row, level and temperature, and sums of w, w (E - Er) and w (E - Er)^2 for 16 rows
// x 16 temperatures are FP64 matrix instructions, Er the row's level of most weight in
// the block at b.  A block's sums join the running ones under their scale, kept to twice
// the double precision, about the Er of the largest block so far (so the variance loses
// little; about Ek instead, a tile with nearly all its weight in one level lost digits
// and was done again: a call of 16 rows of 20 001 levels at 1000 temperatures of 0.05 to
// 0.5 took 887 us, level by level alone 761, now 636).  One block per tile, its 8
// waves taking every 8th block of bins.  201 rows of 20 001 levels at 601
// temperatures: 2.47 ms level by level, now 0.72.
// Tiles whose 1/T spread so far that K would leave e^+-kSpread are marked, and taken by a
// second launch level by level (k_thermo_direct): one block per row and 8 temperatures,
// pass 1 for the largest exponent and its bin, pass 2 for the sums about that energy.
// Terms below e^-745.2 of the largest are zero in double precision.  Redone by the waves
// of the contraction's own block instead, the marked tiles of 16 rows of 20 001 levels at
// 300 temperatures of 0.3 to 5 made a call of 1.61 ms out of 0.62.
constexpr double kSpread = 64.0;
constexpr int kThermoT = 8;

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Grid (ceil(nT / 8), S).  redo: null for every tile, or k_thermo's mark per tile of 8.
// A block's waves take every 64 waves-th bin; up to 8 of them while that leaves a wave 4
// steps of 64 bins and the grid has at most 2048 waves, 2 to a SIMD: each wave pays about
// 300 cross-lane steps for its sums (4 x 552 temperatures, 513 levels: 91 us a call with one
// wave, 106 with 8; 20 001 levels: 432 and 207.  With up to 8192 waves, 2 x 10 000
// temperatures and 513 levels took 1.14 times as long as with one wave to a block).
constexpr int kDirectWaves = 8;
inline int direct_threads(int S, int nT, int W)
{
    int w = 1;
    while (w < kDirectWaves && W >= 512 * w && (int64_t)S * ((nT + kThermoT - 1) / kThermoT) * w * 2 <= 2048) w *= 2;
    return 64 * w;
}
__global__ void __launch_bounds__(64 * kDirectWaves) k_thermo_direct(const double* __restrict__ lng, int W, int model, int N,
                                                                  const double* __restrict__ temp, int nT,
                                                                  const uint8_t* __restrict__ redo,
                                                                  double* __restrict__ u, double* __restrict__ c,
                                                                  double* __restrict__ f)
{
    constexpr int n = kThermoT;
    const int waves = blockDim.x >> 6;
    const int t0 = blockIdx.x * n, s = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (redo && !redo[(size_t)s * gridDim.x + blockIdx.x]) return;
    const double* T = temp + t0;
    const double* row = lng + (size_t)s * W;
    const int nt = nT - t0 < n ? nT - t0 : n;
    const double twoN = 2.0 * N;
    __shared__ double part[kDirectWaves][3][n];
    __shared__ int at[kDirectWaves][n];
    double beta[n], mx[n];
    int arg[n];
#pragma unroll
    for (int i = 0; i < n; ++i) {
        beta[i] = 1.0 / T[i < nt ? i : nt - 1];
        mx[i] = -__builtin_inf();
        arg[i] = W;
    }
    for (int b = threadIdx.x; b < W; b += blockDim.x) {
        const double v = row[b];
        if (!(v > -__builtin_inf())) continue;
        const double E = model == 0 ? 4.0 * b - twoN : (double)b - twoN;
#pragma unroll
        for (int i = 0; i < n; ++i) {
            const double x = v - beta[i] * E;
            if (x > mx[i]) {
                mx[i] = x;
                arg[i] = b;
            }
        }
    }
    // the maximum with the lowest bin on ties: over the wave, then over the waves
#pragma unroll
    for (int i = 0; i < n; ++i) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const double m2 = __shfl_xor(mx[i], o, 64);
            const int a2 = __shfl_xor(arg[i], o, 64);
            if (m2 > mx[i] || (m2 == mx[i] && a2 < arg[i])) {
                mx[i] = m2;
                arg[i] = a2;
            }
        }
        if (waves > 1 && lane == 0) {
            part[wave][0][i] = mx[i];
            at[wave][i] = arg[i];
        }
    }
    if (waves > 1) __syncthreads();
    double Em[n], Z[n], S1[n], S2[n];
#pragma unroll
    for (int i = 0; i < n; ++i) {
        for (int w = 0; w < waves && waves > 1; ++w) {
            const double m2 = part[w][0][i];
            const int a2 = at[w][i];
            if (m2 > mx[i] || (m2 == mx[i] && a2 < arg[i])) {
                mx[i] = m2;
                arg[i] = a2;
            }
        }
        Em[i] = model == 0 ? 4.0 * arg[i] - twoN : (double)arg[i] - twoN;
        Z[i] = S1[i] = S2[i] = 0.0;
    }
    if (waves > 1) __syncthreads();
    for (int b = threadIdx.x; b < W; b += blockDim.x) {
        const double v = row[b];
        if (!(v > -__builtin_inf())) continue;
        const double E = model == 0 ? 4.0 * b - twoN : (double)b - twoN;
#pragma unroll
        for (int i = 0; i < n; ++i) {
            const double d = (v - beta[i] * E) - mx[i];
            if (d >= -745.2) {
                const double w = exp(d), e = E - Em[i], we = w * e;
                Z[i] += w;
                S1[i] += we;
                S2[i] += we * e;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < n; ++i) {
        Z[i] = wave_sum(Z[i]);
        S1[i] = wave_sum(S1[i]);
        S2[i] = wave_sum(S2[i]);
        if (waves > 1 && lane == 0) {
            part[wave][0][i] = Z[i];
            part[wave][1][i] = S1[i];
            part[wave][2][i] = S2[i];
        }
    }
    if (waves > 1) __syncthreads();
    if (threadIdx.x < nt) {
        double zz = 0, s1 = 0, s2 = 0, em = 0, m = 0;
#pragma unroll
        for (int i = 0; i < n; ++i)
            if (i == lane) {
                zz = Z[i]; s1 = S1[i]; s2 = S2[i]; em = Em[i]; m = mx[i];
            }
        if (waves > 1) {
            zz = s1 = s2 = 0;
            for (int w = 0; w < waves; ++w) {
                zz += part[w][0][lane];
                s1 += part[w][1][lane];
                s2 += part[w][2][lane];
            }
        }
        const double t = T[lane], mean = s1 / zz;
        const size_t o = (size_t)s * nT + t0 + lane;
        if (u) u[o] = (em + mean) / N;
        if (c) c[o] = (s2 / zz - mean * mean) / ((double)N * t * t);
        if (f) f[o] = -t * (m + log(zz)) / N;
    }
}

// Sums of one (row, temperature) about the energy E0: weights w = Z e^{-(hi + lo)}.
struct Moments {
    double hi, lo, E0, Z, S1, S2;
};
__device__ __forceinline__ void merge(Moments& a, const Moments& b)
{
    if (b.hi == -__builtin_inf()) return;
    double d = (b.hi - a.hi) + (b.lo - a.lo);             // +inf for the first block
    if (a.hi == -__builtin_inf()) d = __builtin_inf();
    const bool up = d > 0.0;
    const double w = exp(-fabs(d)), wa = up ? w : 1.0, wb = up ? 1.0 : w;
    const double E0 = up ? b.E0 : a.E0, da = a.E0 - E0, db = b.E0 - E0;
    a.S2 = wa * (a.S2 + da * (2.0 * a.S1 + da * a.Z)) + wb * (b.S2 + db * (2.0 * b.S1 + db * b.Z));
    a.S1 = wa * (a.S1 + da * a.Z) + wb * (b.S1 + db * b.Z);
    a.Z = wa * a.Z + wb * b.Z;
    a.hi = up ? b.hi : a.hi;
    a.lo = up ? b.lo : a.lo;
    a.E0 = E0;
}

// Grid (ceil(nT / 16), ceil(S / 16)).  Rows without a finite level or with NaN or +inf do no
// harm; what comes out for them is nowhere used (the host looks at the rows meanwhile).
typedef double f64x4 __attribute__((ext_vector_type(4)));
__global__ void __launch_bounds__(512) k_thermo(const double* __restrict__ lng, int S, int W, int model, int N,
                                                const double* __restrict__ T, int nT, uint8_t* __restrict__ redo, double* __restrict__ u,
                                                double* __restrict__ c, double* __restrict__ f)
{
    __shared__ double K[64][16];
    __shared__ Moments part[4][256];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
    const int s0 = blockIdx.y * 16, t0 = blockIdx.x * 16, nt = nT - t0 < 16 ? nT - t0 : 16;
    const double step = model == 0 ? 4.0 : 1.0, twoN = 2.0 * N;
    const double beta = 1.0 / T[t0 + (li < nt ? li : nt - 1)];
    double lo = beta, hi = beta;
    for (int o = 1; o < 16; o <<= 1) {
        const double l2 = __shfl_xor(lo, o), h2 = __shfl_xor(hi, o);
        lo = l2 < lo ? l2 : lo;
        hi = h2 > hi ? h2 : hi;
    }
    const int nt8 = (nT + kThermoT - 1) / kThermoT, mark = 2 * blockIdx.x + (tid & 1);
    const size_t mine = (size_t)(s0 + (tid >> 1)) * nt8 + mark;
    const bool marks = tid < 32 && s0 + (tid >> 1) < S && mark < nt8;
    if (!((hi - lo) * (16.0 * step) <= kSpread)) {           // block-uniform
        if (marks) redo[mine] = 1;
        return;
    }
    const double mid = 0.5 * (lo + hi);
    for (int e = tid; e < 64 * 16; e += 512)                  // column e % 16 is this lane's
        K[e >> 4][li] = exp(-(beta - mid) * (step * (double)((e >> 4) - 32)));
    __syncthreads();

    const int srow = s0 + li < S ? s0 + li : S - 1;
    const double* row = lng + (size_t)srow * W;
    Moments m[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) m[r] = {-__builtin_inf(), 0.0, 0.0, 0.0, 0.0, 0.0};
    for (int k = wave; k * 64 < W; k += 8) {
        // rows li, bins 4 q + lk of the block
        double a[16], top = -__builtin_inf();
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int b = k * 64 + 4 * q + lk;
            a[q] = b < W ? row[b] : -__builtin_inf();
            top = a[q] > top ? a[q] : top;
        }
        for (int o = 16; o < 64; o <<= 1) {
            const double t2 = __shfl_xor(top, o);
            top = t2 > top ? t2 : top;
        }
        const bool some = top > -__builtin_inf();
        double mx = -__builtin_inf();
        int at = 32;                                          // the level of most weight at mid
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            a[q] = some ? (a[q] - top) - mid * (step * (double)(4 * q + lk - 32)) : -__builtin_inf();
            if (a[q] > mx) {
                mx = a[q];
                at = 4 * q + lk;
            }
        }
        for (int o = 16; o < 64; o <<= 1) {
            const double m2 = __shfl_xor(mx, o);
            const int a2 = __shfl_xor(at, o);
            if (m2 > mx || (m2 == mx && a2 < at)) {
                mx = m2;
                at = a2;
            }
        }
        const double e0 = step * (double)(lk - at);
        f64x4 Z = {}, S1 = {}, S2 = {};
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const double g = some ? exp(a[q] - mx) : 0.0, kk = K[4 * q + lk][li];
            const double e = e0 + step * (double)(4 * q), g1 = g * e;
            Z = __builtin_amdgcn_mfma_f64_16x16x4f64(g, kk, Z, 0, 0, 0);
            S1 = __builtin_amdgcn_mfma_f64_16x16x4f64(g1, kk, S1, 0, 0, 0);
            S2 = __builtin_amdgcn_mfma_f64_16x16x4f64(g1 * e, kk, S2, 0, 0, 0);
        }
        // entry r: row 4 r + lk, temperature li; scale top + mx - beta Ek
        const double Ek = step * (double)(k * 64 + 32) - twoN, p = beta * Ek, pe = __builtin_fma(beta, Ek, -p);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const double tp = __shfl(top, 4 * r + lk), mr = __shfl(mx, 4 * r + lk);
            const double Er = Ek + step * (double)(__shfl(at, 4 * r + lk) - 32);
            Moments b = {-__builtin_inf(), 0.0, Er, Z[r], S1[r], S2[r]};
            if (tp > -__builtin_inf()) {
                const dd sum = two_sum(tp, -p);
                b.hi = sum.hi;
                b.lo = (sum.lo - pe) + mr;
            }
            merge(m[r], b);
        }
    }
    // the 8 waves' sums, pairwise
    for (int w = 4; w > 0; w >>= 1) {
        if (wave >= w && wave < 2 * w)
#pragma unroll
            for (int r = 0; r < 4; ++r) part[wave - w][r * 64 + lane] = m[r];
        __syncthreads();
        if (wave < w)
#pragma unroll
            for (int r = 0; r < 4; ++r) merge(m[r], part[wave][r * 64 + lane]);
        __syncthreads();
    }
    __shared__ int weak[16][2];
    if (tid < 32) weak[tid >> 1][tid & 1] = 0;
    __syncthreads();
    if (wave == 0 && li < nt) {
        const double t = T[t0 + li];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int s = s0 + 4 * r + lk;
            if (s >= S) continue;
            const double mean = m[r].S1 / m[r].Z, sq = m[r].S2 / m[r].Z, var = sq - mean * mean;
            const size_t o = (size_t)s * nT + t0 + li;
            if (u) u[o] = (m[r].E0 + mean) / N;
            if (c) c[o] = var / ((double)N * t * t);
            if (f) f[o] = -t * (m[r].hi + (m[r].lo + log(m[r].Z))) / N;
            if (!(var >= 0x1p-8 * sq)) weak[4 * r + lk][li >= kThermoT] = 1;
        }
    }
    __syncthreads();
    // a variance far below the mean square about Er has lost digits (the level of most weight
    // at this temperature is far from the one at b): those again about the level itself
    if (marks) redo[mine] = (uint8_t)weak[tid >> 1][tid & 1];
}

}  // namespace rewl
