// rewl_kernels.hip -- the REWL hot path on gfx950.
//
// One interval of replica-exchange Wang-Landau (arXiv:1407.5140 Sec. II.A):
//   k_sweep    X single-site attempts per walker, one walker per lane, the
//              walker's lattice and histogram and its window's ln g base in LDS,
//              drawn by a second wave (k_sweep_persist: the same from a queue of tiles;
//              k_sweep_far: with the draws in device memory; k_sweep_wave: one walker
//              per wave); flatness test in the epilogue
//   k_merge    per window: when all m walkers are flat, average ln g, reset H,
//              halve ln f, detect convergence
//   k_exchange Eq. (1) between neighbouring windows, alternating pairings
//   k_advance  interval counter, termination bookkeeping, order of the sweep's blocks
// All interval state lives in device memory, so an interval is a fixed
// sequence of launches that can be captured once and replayed.
#include "host_copy.hpp"
#include "rewl_device.hpp"

namespace rewl {

// ------------------------------------------------------------------- sweep
// LDS of one tile of nw walkers of window a:
//   base [kPad + WB + kPad]         window ln g base, +inf in the pads
//   H    [(kPad + WB + kPad) << lnw] per-walker counts, bin-major (lane minor)
//   lat  Ising [L*wpr << lnw] u64 words / Potts [N << lnw] bytes
//   draws [2][8 (Ising) or 4 (Potts) << lnw]: the next attempts of every walker, twice (in
//                                    device memory where one walker's tables leave no room)
// A block is two waves: wave 0 walks, wave 1 draws the next attempts of its walkers
// meanwhile, down to the sites whose spins an attempt reads.  (Drawn by the whole GPU in
// a launch of its own, through a buffer of 12 bytes per attempt in memory, the
// 65 280-walker batch took 3.9 + 13.1 ms per interval, now 10.9.)
// A move changes the bin by at most 2 (Ising) or 4 (Potts), so a proposal
// outside the window lands in a pad, sees ln g = +inf and is rejected.
constexpr int kPad = 4;
constexpr int kDrawBytes = 64;      // of one walker: 8 draws of 8 bytes or 4 of 16

__host__ __device__ inline size_t sweep_lds_bytes(int model, int L, int wpr, int WB, int nw, bool far_draws = false)
{
    const size_t nb = (size_t)WB + 2 * kPad, al = far_draws ? 7 : 15;
    const size_t s = (nb * 8 + nb * nw * 4 + al) & ~al, lat = (model == 0 ? (size_t)L * wpr * 8 : (size_t)L * L) * nw;
    return far_draws ? s + lat : s + ((lat + al) & ~al) + (size_t)2 * kDrawBytes * nw;
}

// How many bytes of the word x differ from the byte v.
__device__ __forceinline__ int bytes_unlike(uint32_t x, uint32_t v)
{
    const uint32_t y = x ^ __builtin_amdgcn_perm(v, v, 0u);
    return __builtin_popcount((((y & 0x7f7f7f7fu) + 0x7f7f7f7fu) | y) & 0x80808080u);
}

// The decision of decide_fast and accept_slow on the attempt's own draw: bit 0
// accepted, bit 1 taken by the slow path.  For the attempts that the bounds of
// bounds_of leave open.
__device__ __noinline__ int decide_draw(const Inst& I, uint64_t T, uint32_t slot, double delta)
{
    const uint64_t u53 = u53_of(draw(I.k0, I.k1, T, slot, kTagFlip));
    const int f = decide_fast(delta, threshold_of(u53, I.band), I.band);
    return f == 2 ? 2 | (accept_slow(delta, u53) ? 1 : 0) : f;
}

// Lane l's value of a wave-uniform lane index l (v_readlane).
__device__ __forceinline__ uint32_t rl(uint32_t v, int l)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}
__device__ __forceinline__ uint64_t rl64(uint64_t v, int l)
{
    return ((uint64_t)rl((uint32_t)(v >> 32), l) << 32) | rl((uint32_t)v, l);
}
__device__ __forceinline__ float rlf(float v, int l)
{
    return __builtin_bit_cast(float, rl(__builtin_bit_cast(uint32_t, v), l));
}
__device__ __forceinline__ double rld(double v, int l)
{
    return __builtin_bit_cast(double, rl64(__builtin_bit_cast(uint64_t, v), l));
}

template <int MODEL, int WPR, bool FAR>
__device__ void sweep_tile(const Inst& I, const Tile& tile, char* smem, char* draws)
{
    const int a = tile.window, nw = tile.nw, tid = threadIdx.x, lane = tid & 63;
    const bool walks = tid < 64;                                 // wave 0; wave 1 draws
    const int WB = I.WB, L = I.L, N = I.N;
    const int slot0 = a * I.m + tile.r0;
    const int lo = I.lo[a];
    const int nbins = WB + 2 * kPad;
    double* lbase = (double*)smem;                               // index kPad + bin
    uint32_t* lH = (uint32_t*)(lbase + nbins);                   // index (kPad + bin) << lnw | lane
    constexpr size_t kAlign = FAR ? 7 : 15;
    char* latp = smem + ((nbins * 8 + (size_t)nbins * nw * 4 + kAlign) & ~kAlign);
    // Ising: .x row | col<<8 | row_up<<16 | row_down<<24 (periodic rows);
    // Potts: .x site | off<<16, off = floor(x1 (q-1) / 2^32), .y and .z the neighbours' sites;
    // last word: the bound of the threshold (upper_of)
    typedef uint32_t Draw __attribute__((ext_vector_type(MODEL ? 4 : 2)));
    constexpr int kDraws = kDrawBytes / (int)sizeof(Draw);
    Draw* ring;
    if constexpr (FAR) ring = (Draw*)draws;
    else ring = (Draw*)(latp + (((MODEL == 0 ? (size_t)L * WPR * 8 : (size_t)N) * nw + 15) & ~size_t(15)));
    const int nthr = blockDim.x;
    const int lnw = __builtin_ctz(nw);                           // nw is a power of two

    // ---- stage the window table, the tile's histograms and lattices in LDS.
    //      A walker's counts enter LDS relative to an offset cw of its own (kept by
    //      lane l for walker l): every decision of the sweep compares two ln g
    //      values of one walker, so a per-walker constant cancels, and the 32-bit
    //      LDS entries only need to hold the counts' spread around the offset.
    //      cw = H(current bin) - 2^31 when that count is past 2^31, else 0 (so
    //      counts below 2^31 enter as they are).  Levels that never occur carry
    //      the sentinel 0xffffffff (never visited, excluded from the flatness
    //      minimum, written back as 0).
    // bins b >= width (a window narrower than WB) are outside the window: +inf
    // table (moves there are rejected) and the never-visited sentinel
    const int width = I.hi[a] - lo + 1;
    for (int i = tid; i < nbins; i += nthr) {
        const int b = i - kPad;
        lbase[i] = (b >= 0 && b < width) ? I.base[(size_t)a * WB + b] : __builtin_inf();
    }
    uint64_t cw = 0;
    if (lane < nw) {
        const uint64_t hc0 = I.H[(size_t)(slot0 + lane) * WB + (I.bin[slot0 + lane] - lo)];
        cw = hc0 > (1ull << 31) ? hc0 - (1ull << 31) : 0ull;
    }
    // counts must lie in [cw, cw + 2^32 - 1 - X) so that this interval's X
    // updates stay below the sentinel; otherwise the run reports an overflow
    const uint64_t span = 0xffffffffull - (uint64_t)I.X;
    // global H is walker-major: H[slot][bin]; consecutive threads take consecutive bins
    bool bad = false;
    for (int l = 0; l < nw; ++l) {
        const uint64_t cl = rl64(cw, l);
        for (int i = tid; i < nbins; i += nthr) {
            const int b = i - kPad;
            uint32_t hv = 0;
            if (b >= 0 && b < WB) {
                hv = 0xffffffffu;
                if (b < width && I.mask[lo + b]) {
                    const uint64_t v = I.H[(size_t)(slot0 + l) * WB + b] - cl;   // wraps if below cl
                    bad |= v >= span;
                    hv = (uint32_t)v;
                }
            }
            lH[(i << lnw) + l] = hv;
        }
    }
    if (bad) atomicOr(&I.ctr->err, kErrOverflow);
    // lattices are walker-major too: lat[slot][word] / plat[slot][site]
    if (MODEL == 0) {
        uint64_t* lat = (uint64_t*)latp;
        const int nwords = L * WPR;
        for (int l = 0; l < nw; ++l)
            for (int w = tid; w < nwords; w += nthr) lat[(w << lnw) + l] = I.lat[(size_t)(slot0 + l) * nwords + w];
    } else {
        uint8_t* lat = (uint8_t*)latp;
        for (int l = 0; l < nw; ++l)
            for (int w = tid; w < N; w += nthr) lat[(w << lnw) + l] = I.plat[(size_t)(slot0 + l) * N + w];
    }
    const int k = I.k[a];
    const uint32_t inc = I.done[a] == 0 ? 1u : 0u;               // converged: frozen
    const double scale = __builtin_ldexp(1.0, -k);
    const uint32_t X = (uint32_t)I.X, nchunk = (X + kDraws - 1) / kDraws;
    const uint64_t T0 = (uint64_t)I.ctr->t * (uint64_t)X;
    const float e32 = kErrLane + (float)I.band;

    if (!walks) {
        // entry i << lnw | l of a chunk: attempt i of the chunk, walker l, at the site
        // floor(x0 N / 2^32)
        const uint32_t qm1 = I.q - 1;
        const float rL = 1.0f / (float)L;
        for (uint32_t c = 0; c <= nchunk; ++c) {
            if (c < nchunk) {
                Draw* r = ring + (size_t)(c & 1) * kDraws * nw;
                for (int e = lane; e < kDraws << lnw; e += 64) {
                    const u32x4 x = draw(I.k0, I.k1, T0 + (uint64_t)(c * kDraws + (e >> lnw)),
                                         (uint32_t)(slot0 + (e & (nw - 1))), kTagFlip);
                    const uint32_t site = (uint32_t)(((uint64_t)x.x * (uint32_t)N) >> 32);
                    // row = site / L: site < 2^24 is exact in FP32, the product's rounding
                    // puts the estimate at most one off, corrected below
                    int row = (int)((float)site * rL);
                    int col = (int)site - (int)__umul24((uint32_t)row, (uint32_t)L);
                    if (col < 0) { --row; col += L; }
                    else if (col >= L) { ++row; col -= L; }
                    const uint32_t hi = __builtin_bit_cast(uint32_t, upper_of(x.z, x.w, e32));
                    if constexpr (MODEL) {
                        const uint32_t off = (uint32_t)(((uint64_t)x.y * qm1) >> 32);
                        const uint32_t up = row == 0 ? site + (N - L) : site - L;
                        const uint32_t dn = row == L - 1 ? site - (N - L) : site + L;
                        const uint32_t lf = col == 0 ? site + (L - 1) : site - 1;
                        const uint32_t rt = col == L - 1 ? site - (L - 1) : site + 1;
                        r[e] = Draw{site | (off << 16), up | (dn << 16), lf | (rt << 16), hi};
                    } else {
                        const int ru = row == 0 ? L - 1 : row - 1, rd = row == L - 1 ? 0 : row + 1;
                        r[e] = Draw{(uint32_t)(row | (col << 8) | (ru << 16) | (rd << 24)), hi};
                    }
                }
            }
            __syncthreads();                  // chunk c is there, chunk c - 1 has been walked
        }
    } else {
        __syncthreads();                      // everything is staged, and chunk 0 is there
        const int slot = slot0 + lane;
        const bool active = lane < nw;
        int b = active ? I.bin[slot] - lo + kPad : kPad;         // padded bin index
        const int wl = active ? lane : 0;
        uint32_t hc = lH[(b << lnw) + wl];
        double lngc = __builtin_fma((double)hc, scale, lbase[b]);
        const double incv = inc ? scale : 0.0;

        const int q = I.q;
        // one flip attempt with draw D, attempt j;
        // lH always holds the walker's current counts, including bin b
        auto attempt = [&](const Draw& D, uint32_t j) {
            const uint32_t pk = D.x, hw = D[MODEL ? 3 : 1];
            const float hi = __builtin_bit_cast(float, hw);
            int nb;
            int waddr;                                           // LDS index of the flipped word/byte
            uint64_t wold = 0, wnew = 0;
            uint8_t pold = 0, pnew = 0;
            if constexpr (MODEL == 0) {
                const uint64_t* lat = (const uint64_t*)latp;
                const int r = pk & 0xff, c = (pk >> 8) & 0xff;
                const int ru = (pk >> 16) & 0xff, rd = pk >> 24;
                if (WPR == 1) {
                    const int cl = c == 0 ? L - 1 : c - 1, cr = c == L - 1 ? 0 : c + 1;
                    waddr = (r << lnw) + lane;
                    const uint64_t w = lat[waddr];
                    const uint64_t wu = lat[(ru << lnw) + lane];
                    const uint64_t wd = lat[(rd << lnw) + lane];
                    const uint32_t sp = (uint32_t)(w >> c) & 1u;
                    const uint32_t ones = ((uint32_t)(wu >> c) & 1u) + ((uint32_t)(wd >> c) & 1u) +
                                          ((uint32_t)(w >> cl) & 1u) + ((uint32_t)(w >> cr) & 1u);
                    // aligned neighbours al: dE = 4 al - 8, bin change al - 2
                    nb = b + (sp ? (int)ones : 4 - (int)ones) - 2;
                    wold = w;
                    wnew = w ^ (1ull << c);
                } else {
                    const int cl = c == 0 ? L - 1 : c - 1, cr = c == L - 1 ? 0 : c + 1;
                    auto spin = [&](int rr, int cc) -> uint32_t {
                        return (uint32_t)(lat[((rr * WPR + (cc >> 6)) << lnw) + lane] >> (cc & 63)) & 1u;
                    };
                    waddr = ((r * WPR + (c >> 6)) << lnw) + lane;
                    const uint64_t w = lat[waddr];
                    const uint32_t sp = (uint32_t)(w >> (c & 63)) & 1u;
                    const uint32_t ones = spin(ru, c) + spin(rd, c) + spin(r, cl) + spin(r, cr);
                    nb = b + (sp ? (int)ones : 4 - (int)ones) - 2;
                    wold = w;
                    wnew = w ^ (1ull << (c & 63));
                }
            } else {
                const uint8_t* lat = (const uint8_t*)latp + lane;
                waddr = ((int)(pk & 0xffff) << lnw) + lane;
                const uint32_t s0 = ((const uint8_t*)latp)[waddr];
                const uint32_t n0 = lat[(D.y & 0xffff) << lnw], n1 = lat[(D.y >> 16) << lnw];
                const uint32_t n2 = lat[(D.z & 0xffff) << lnw], n3 = lat[(D.z >> 16) << lnw];
                int nv = (int)s0 + 1 + (int)(pk >> 16);
                nv = nv >= q ? nv - q : nv;
                pold = (uint8_t)s0;
                pnew = (uint8_t)nv;
                const uint32_t n = n0 | (n1 << 8) | (n2 << 16) | (n3 << 24);
                nb = b + bytes_unlike(n, (uint32_t)nv) - bytes_unlike(n, s0);   // dE = n(old) - n(new)
            }
            const double bn = lbase[nb];
            const uint32_t hn = lH[(nb << lnw) + lane];
            const double lngn = __builtin_fma((double)hn, scale, bn);   // +inf in a pad
            const double delta = lngc - lngn;                    // exact (or -inf)
            // above hi accepts for certain, below its lower bound rejects for certain
            const float df = (float)delta;
            bool f = df > hi;
            const bool open = !f && df >= lower_of(hi, e32);
            if (__builtin_expect(__any(open), 0)) {
                if (open) {
                    const int r = decide_draw(I, T0 + (uint64_t)j, (uint32_t)slot, delta);
                    f = r & 1;
                    if (r & 2) atomicAdd((unsigned long long*)&I.ctr->slow, 1ull);
                }
            }
            // written either way: a store under a mask of its own costs a branch
            if (MODEL == 0) ((uint64_t*)latp)[waddr] = f ? wnew : wold;
            else ((uint8_t*)latp)[waddr] = f ? pnew : pold;
            b = f ? nb : b;
            hc = (f ? hn : hc) + inc;
            lH[(b << lnw) + lane] = hc;
            lngc = (f ? lngn : lngc) + incv;                     // exact: base + 2^-k H
        };

        for (uint32_t c = 0; c < nchunk; ++c) {
            if (active) {
                const Draw* r = ring + (size_t)(c & 1) * kDraws * nw + lane;
                Draw D[kDraws];
#pragma unroll
                for (int i = 0; i < kDraws; ++i) D[i] = r[i << lnw];
                const uint32_t j0 = c * kDraws;
                if (j0 + kDraws <= X) {
#pragma unroll
                    for (int i = 0; i < kDraws; ++i) attempt(D[i], j0 + i);
                } else {
#pragma unroll
                    for (int i = 0; i < kDraws; ++i)
                        if (j0 + i < X) attempt(D[i], j0 + i);
                }
            }
            __syncthreads();
        }
        if (active) {
            I.bin[slot] = b - kPad + lo;
            I.swaps[slot] = -1;
        }
    }

    // ---- write back (absolute counts: the walker's offset added back)
    for (int l = 0; l < nw; ++l) {
        const uint64_t cl = rl64(cw, l);
        for (int bb = tid; bb < WB; bb += nthr) {
            const uint32_t hv = lH[((bb + kPad) << lnw) + l];
            I.H[(size_t)(slot0 + l) * WB + bb] = hv == 0xffffffffu ? 0ull : (uint64_t)hv + cl;
        }
    }
    if (MODEL == 0) {
        const uint64_t* lat = (const uint64_t*)latp;
        const int nwords = L * WPR;
        for (int l = 0; l < nw; ++l)
            for (int w = tid; w < nwords; w += nthr) I.lat[(size_t)(slot0 + l) * nwords + w] = lat[(w << lnw) + l];
    } else {
        const uint8_t* lat = (const uint8_t*)latp;
        for (int l = 0; l < nw; ++l)
            for (int w = tid; w < N; w += nthr) I.plat[(size_t)(slot0 + l) * N + w] = lat[(w << lnw) + l];
    }

    // ---- flatness of each walker (Sec. II.A, or Eq. (8)) over the levels of the
    //      window that occur; latched until the window merges
    if (inc && walks && lane < nw) {
        uint32_t mn = 0xffffffffu;
        uint64_t sum = 0;
        for (int bb = kPad; bb < WB + kPad; ++bb) {
            const uint32_t v = lH[(bb << lnw) + lane];
            mn = v < mn ? v : mn;                                // the sentinel never wins the min
            sum += v == 0xffffffffu ? 0u : v;
        }
        const int slot = slot0 + lane;
        const int64_t n = I.nreach[a];
        if (walker_flat(I, (uint64_t)mn + cw, sum + (uint64_t)n * cw, n, k)) I.flat[slot] = 1;
    }
}

template <bool FAR>
__device__ __forceinline__ void sweep_one_tile(const Inst* __restrict__ insts, const Tile& tile, char* smem, char* draws)
{
    const Inst& I = insts[tile.inst];
    if (I.ctr->all_done) return;
    if (I.model == 0) {
        // (Ising rows of one word have at most 4097 levels, 48 KB of tables)
        if (!FAR && I.wpr == 1) sweep_tile<0, 1, false>(I, tile, smem, draws);
        else sweep_tile<0, 2, FAR>(I, tile, smem, draws);
    } else {
        sweep_tile<1, 1, FAR>(I, tile, smem, draws);
    }
}

__global__ void __launch_bounds__(128) k_sweep(const Inst* __restrict__ insts,
                                              const Tile* __restrict__ tiles, int ntiles)
{
    extern __shared__ __align__(16) char smem[];
    sweep_one_tile<false>(insts, tiles[blockIdx.x], smem, nullptr);
}

// Tiles of one walker whose draws lie in device memory, 2 kDrawBytes a tile.
__global__ void __launch_bounds__(128) k_sweep_far(const Inst* __restrict__ insts, const Tile* __restrict__ tiles,
                                                  char* __restrict__ draws)
{
    extern __shared__ __align__(16) char smem[];
    sweep_one_tile<true>(insts, tiles[blockIdx.x], smem, draws + (size_t)blockIdx.x * 2 * kDrawBytes);
}

// Persistent form: a grid sized to the blocks the GPU holds at once; each block
// takes the next tile from a queue counter until the tiles run out (the tiles
// are ordered longest-first by the host).  The counter is reset by k_advance at
// the end of the interval, so the launch sequence needs no memset.
__global__ void __launch_bounds__(128) k_sweep_persist(const Inst* __restrict__ insts,
                                                      const Tile* __restrict__ tiles, int ntiles,
                                                      int32_t* __restrict__ queue)
{
    extern __shared__ __align__(16) char smem[];
    __shared__ int next;
    for (;;) {
        if (threadIdx.x == 0) next = atomicAdd(queue, 1);
        __syncthreads();
        const int t = next;
        __syncthreads();
        if (t >= ntiles) break;             // block-uniform: every wave of the grid ends here
        sweep_one_tile<false>(insts, tiles[t], smem, nullptr);
        __syncthreads();                    // the tile's LDS is free before the next one is staged
    }
}

// -------------------------------------------------------------- wave sweep
// One wave per walker, for workloads with few walkers: the walker's Markov
// chain runs on wave-uniform (scalar) values, and the 64 lanes draw the Philox
// numbers of the next 64 attempts in parallel (no draw buffer).
// LDS: the window's base table (shared by the block's walkers, all of one
// window), then per wave its counts (LDS placement only), then per wave its site
// map, then per wave its lattice (Potts one byte per site, Ising wpr 64-bit words
// per row).  The site map holds one 64-bit attempt mask per entry: one entry per
// site, or M = 2^j < N entries shared by the sites equal modulo M, which only
// adds attempts to the out-of-date sets, never removes one (so a smaller map
// trades extra re-evaluations for LDS).
// site-map entries per walker for a lattice of N sites and a cap of 2^map_log2
// entries (0: 2^12)
__host__ __device__ inline int wave_map_entries(int N, int map_log2 = 0)
{
    const int cap = 1 << (map_log2 > 0 ? map_log2 : 12);
    return N <= cap ? N : cap;
}
__host__ __device__ inline size_t wave_lds_bytes(int model, int L, int WB, int G, bool hglobal, int mapn)
{
    const size_t nb = (size_t)WB + 2 * kPad, N = (size_t)L * L;
    size_t s = nb * 8 + (hglobal ? 0 : (size_t)G * nb * 4);
    s = (s + 7) & ~size_t(7);
    s += (size_t)G * mapn * 8;
    s += model == 1 ? (size_t)G * N : (size_t)G * L * ((L + 63) / 64) * 8;
    return s;
}

// Lane (byte offset / 4)'s value of v.
__device__ __forceinline__ float bperm_f(float v, int byte)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(byte, __builtin_bit_cast(int, v)));
}

// Index of the lowest set bit of a wave-uniform mask, 2^32 - 1 if there is none.
__device__ __forceinline__ uint32_t first_bit(uint64_t m)
{
    uint32_t r;
    asm("s_ff1_i32_b64 %0, %1" : "=s"(r) : "s"(m));
    return r;
}

// c if bit i (modulo 64) of the wave-uniform mask m is set, else 0.
__device__ __forceinline__ uint32_t bit_then(uint64_t m, uint32_t i, uint32_t c)
{
    uint32_t r;
    asm("s_bitcmp1_b64 %1, %2\n\ts_cselect_b32 %0, %3, 0" : "=s"(r) : "s"(m), "s"(i), "s"(c) : "scc");
    return r;
}

// a if bit i (modulo 64) of the wave-uniform mask m is set, else b.
__device__ __forceinline__ uint32_t bit_pick(uint64_t m, uint32_t i, uint32_t a, uint32_t b)
{
    uint32_t r;
    asm("s_bitcmp1_b64 %1, %2\n\ts_cselect_b32 %0, %3, %4" : "=s"(r) : "s"(m), "s"(i), "s"(a), "s"(b) : "scc");
    return r;
}

// Bit i of a wave-uniform mask set.
__device__ __forceinline__ void set_bit(uint64_t& m, uint32_t i) { asm("s_bitset1_b64 %0, %1" : "+s"(m) : "s"(i)); }

// Exact decision of one walker's attempt, taken by the whole wave alike.
__device__ __forceinline__ bool wave_decide(const Inst& I, uint64_t T, uint32_t slot, double delta, int lane)
{
    const int f = __builtin_amdgcn_readfirstlane(decide_draw(I, T, slot, delta));
    if ((f & 2) && lane == 0) atomicAdd((unsigned long long*)&I.ctr->slow, 1ull);
    return f & 1;
}

// Bin change of flipping Ising spin (r, c): rows w (row r), wu (r-1), wd (r+1).
__device__ __forceinline__ int ising_d(uint64_t w, uint64_t wu, uint64_t wd, int c, int L)
{
    const int cl = c == 0 ? L - 1 : c - 1, cr = c == L - 1 ? 0 : c + 1;
    const uint32_t sp = (uint32_t)(w >> c) & 1u;
    const uint32_t ones = ((uint32_t)(wu >> c) & 1u) + ((uint32_t)(wd >> c) & 1u) +
                          ((uint32_t)(w >> cl) & 1u) + ((uint32_t)(w >> cr) & 1u);
    return (sp ? (int)ones : 4 - (int)ones) - 2;
}

// Bin change of flipping Ising spin (r, c) on rows of wpr 64-bit words.
__device__ __forceinline__ int ising_d_words(const uint64_t* rows, int wpr, int r, int ru, int rd, int c,
                                             int L)
{
    if (wpr == 1) return ising_d(rows[r], rows[ru], rows[rd], c, L);
    auto spin = [&](int rr, int cc) -> uint32_t {
        return (uint32_t)(rows[rr * wpr + (cc >> 6)] >> (cc & 63)) & 1u;
    };
    const int cl = c == 0 ? L - 1 : c - 1, cr = c == L - 1 ? 0 : c + 1;
    const uint32_t sp = spin(r, c);
    const uint32_t ones = spin(ru, c) + spin(rd, c) + spin(r, cl) + spin(r, cr);
    return (sp ? (int)ones : 4 - (int)ones) - 2;
}

// Wave variant: one walker per wave.
// * The walker's ln g over 64 consecutive bins lives in registers, one bin per
//   lane, so that no table memory is on the dependent chain; the window moves
//   when the walker comes within four bins of its edge.
// * Per chunk of 64 attempts the lanes draw the numbers and evaluate every
//   attempt's bin change d on the lattice.  A per-site bit map in LDS gives each
//   attempt the earlier attempts of the chunk whose site lies in its
//   neighbourhood (P); an attempt is out of date once one of those has flipped.
// * The chain advances a run at a time.  From attempt i on, every lane j >= i
//   evaluates its attempt as if the walker were still in its bin, with ln g
//   raised by the (j - i) updates of the attempts in between: that holds while
//   those attempts were rejected or were accepted with d = 0 (a move within the
//   bin, always accepted).  The run ends at the first accepted move with d != 0,
//   or before the first attempt that a flip of the run made out of date.
// WIDE: Ising rows of several 64-bit words (L > 64); the narrow form keeps one
// word per row.
// HG: the walker's counts stay in device memory (the 64-bit H array) instead of
// an LDS copy: they are touched only when the register window is loaded or
// stored and by the flatness test, so LDS then holds only the window's base table,
// the site maps and the lattices, and more walkers fit a block.  Both placements
// compute identical results.
// A walker alone on its SIMD is bound by the issue of its own instructions and the
// hand-overs between the lanes and the scalar side, not by memory or arithmetic: a step is
// 28 instructions and about 195 cycles, a round's start and end 600, a chunk's draws and
// sets 600 (Ising L=64, middle windows: 26 steps and 2.2 rounds per chunk).  A step in
// FP64 on exact values took 390 cycles, one of 34 instructions 270.  Interval of 10^4
// attempts, us, with FP64 steps / 34 instructions / now: Ising L=32, 128 walkers 1090 / 695
// / 554; L=64, 1024: 1100 / 656 / 517; L=128, 2048: 1249 / 811 / 608; Potts q=10 L=32, 4096
// (4 to a SIMD): 1699 / 970 / 633; L=64, 4096: 1725 / 1180 / 821 (the last three by the
// order of the blocks too, order_tiles).  All with the walkers spread over their windows; a
// run's first 40 intervals are shorter (Potts L=32 547, L=64 637).
template <int MODEL, bool WIDE, bool HG>
__device__ void sweep_wave(const Inst& I, const Tile& tile, char* smem, uint32_t* __restrict__ cost)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int G = tile.nw;
    const int a = tile.window, WB = I.WB, L = I.L, N = I.N;
    const int nbins = WB + 2 * kPad;
    const int lo = I.lo[a];
    double* lbase = (double*)smem;
    // bins b >= width (a window narrower than WB) lie outside the window
    const int width = I.hi[a] - lo + 1;
    for (int i = threadIdx.x; i < nbins; i += blockDim.x) {
        const int b = i - kPad;
        lbase[i] = (b >= 0 && b < width) ? I.base[(size_t)a * WB + b] : __builtin_inf();
    }
    const bool active = wave < G;
    const int r = tile.r0 + wave, slot = a * I.m + r;
    uint32_t* lH = (uint32_t*)(lbase + nbins) + (size_t)wave * nbins;           // LDS placement only
    uint64_t* gH = I.H + (size_t)slot * WB;                                      // the walker's counts
    const int M = I.mapn;                                     // site-map entries
    // site -> map entry: the site itself when every site has one, else site mod M
    const uint32_t mmask = M >= N ? 0xffffffffu : (uint32_t)(M - 1);
    const int wpr = WIDE ? I.wpr : 1;                         // Ising words per row
    const size_t off_map = ((size_t)nbins * 8 + (HG ? 0 : (size_t)G * nbins * 4) + 7) & ~size_t(7);
    uint64_t* lmap = (uint64_t*)(smem + off_map) + (size_t)wave * M;
    uint8_t* llat = (uint8_t*)(smem + off_map + (size_t)G * M * 8) + (size_t)wave * N;
    uint64_t* lrow = (uint64_t*)(smem + off_map + (size_t)G * M * 8) + (size_t)wave * L * wpr;
    auto ent = [&](int site) { return (int)((uint32_t)site & mmask); };
    // the walker's counts relative to an offset of its own (a per-walker constant
    // cancels from every decision), chosen and checked as in sweep_tile
    uint64_t cw = 0;
    if (active && !HG) {
        const uint64_t hc0 = I.H[(size_t)slot * WB + (I.bin[slot] - lo)];
        cw = hc0 > (1ull << 31) ? hc0 - (1ull << 31) : 0ull;
        const uint64_t span = 0xffffffffull - (uint64_t)I.X;
        bool bad = false;
        for (int i = lane; i < nbins; i += 64) {
            const int b = i - kPad;
            uint32_t hv = 0;
            if (b >= 0 && b < WB) {
                hv = 0xffffffffu;
                if (b < width && I.mask[lo + b]) {
                    const uint64_t v = I.H[(size_t)slot * WB + b] - cw;
                    bad |= v >= span;
                    hv = (uint32_t)v;
                }
            }
            lH[i] = hv;
        }
        if (bad) atomicOr(&I.ctr->err, kErrOverflow);
    }
    if (active) {
        for (int i = lane; i < M; i += 64) lmap[i] = 0;
        if (MODEL == 0) {
            for (int i = lane; i < L * wpr; i += 64) lrow[i] = I.lat[(size_t)slot * L * wpr + i];
        } else {
            for (int i = lane; i < N; i += 64) llat[i] = I.plat[(size_t)slot * N + i];
        }
    }
    __syncthreads();
    if (!active) return;

    const int k = I.k[a];
    const uint32_t inc = I.done[a] == 0 ? 1u : 0u;
    const double scale = __builtin_ldexp(1.0, -k);
    const double incv = inc ? scale : 0.0;
    const int64_t X = I.X;
    const uint64_t T0 = (uint64_t)I.ctr->t * (uint64_t)X;
    const uint32_t q = (uint32_t)I.q, qm1 = q - 1;
    const double band = I.band;
    const int b = __builtin_amdgcn_readfirstlane(I.bin[slot] - lo + kPad);

    // register window of the walker's table: lane l holds ln g of bin b0 + l
    // (+inf beyond the table).  Every value is a multiple of 2^-(k + log2 m)
    // below 2^21, so every step here is exact; the counts are recovered as
    // H = (ln g - base) 2^k when the window moves.
    const int b0max = nbins > 64 ? nbins - 64 : 0;
    int b0 = b - 32 < 0 ? 0 : (b - 32 > b0max ? b0max : b - 32);
    int idx = b - b0;                     // the walker's bin, as a lane of the window
    const double unscale = __builtin_ldexp(1.0, k);
    double gl;
    // with HG the table entries are absolute counts (below 2^53: exact in FP64)
    auto occurs = [&](int i) { return i >= kPad && i < kPad + width && I.mask[lo + i - kPad]; };
    auto load_window = [&]() {
        const int i = b0 + lane;
        if (HG) {
            // the window's entries may have been stored by other lanes of this wave
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
            gl = i < nbins ? (occurs(i) ? __builtin_fma((double)gH[i - kPad], scale, lbase[i]) : lbase[i])
                           : __builtin_inf();
        } else {
            gl = i < nbins ? __builtin_fma((double)lH[i], scale, lbase[i]) : __builtin_inf();
        }
    };
    auto store_window = [&]() {
        const int i = b0 + lane;
        // pads and levels that do not occur are never visited: leave them
        if (HG) {
            if (occurs(i)) gH[i - kPad] = (uint64_t)((gl - lbase[i]) * unscale);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        } else if (i >= kPad && i < kPad + WB && lH[i] != 0xffffffffu) {
            lH[i] = (uint32_t)((gl - lbase[i]) * unscale);
        }
    };
    load_window();
    // The steps compare in FP32: g0 = ln g of each bin of the window less that of
    // the bin the walker was in when it was taken, gl holding the exact values of
    // that moment; cnt = visits since then of the bins that the walker has left,
    // cur = g0 + cnt 2^-k.  The walker's own bin (hot = 1) has in cnt less the attempt
    // of the chunk at which the walker came, and lb + j 2^-k is its ln g before
    // attempt j.  The walker may step to the bins of `safe`, whose g0 is below 64, away
    // from the window's edge; when it leaves them, and at the end of a chunk, the visits
    // go into gl (exact) and g0 is taken afresh.  Every quantity that a decision can
    // depend on then stays below 512, the seven roundings on its way (six of at most
    // 2^-16) below kErr32, and an attempt closer to its threshold than that is decided
    // on the exact values.
    constexpr float kErr32 = 0x1p-13f;
    const float inc32 = (float)incv, laneinc = (float)lane * inc32;       // exact
    float g0, cur, cnt = 0.0f, hot = lane == idx ? 1.0f : 0.0f, lb;
    uint64_t safe;
    auto settle = [&](int j) {            // attempts below j of the chunk are decided
        cnt = __builtin_fmaf((float)j, hot, cnt);
        gl = __builtin_fma((double)cnt, incv, gl);            // exact
        if (__builtin_expect((unsigned)(idx - 4) > 55u, 0)) { // idx < 4 or idx > 59
            store_window();                                   // move the window around the walker
            const int bb = b0 + idx;
            b0 = bb - 32 < 0 ? 0 : (bb - 32 > b0max ? b0max : bb - 32);
            idx = bb - b0;
            load_window();
            hot = lane == idx ? 1.0f : 0.0f;
        }
        cur = g0 = (float)(gl - rld(gl, idx));
        safe = __builtin_amdgcn_ballot_w64(__builtin_fabsf(g0) < 64.0f) & 0x0ffffffffffffff0ull;
        cnt = -(float)j * hot;
        lb = -(float)j * inc32;
    };
    settle(0);
    uint32_t work = 0;                    // of the interval, in steps
    const float rL = 1.0f / (float)L;
    const float band32 = (float)band + kErr32;
    const uint64_t lanebit = 1ull << lane;

    for (int64_t j0 = 0; j0 < X; j0 += 64) {
        const int n = (int)((X - j0) < 64 ? (X - j0) : 64);
        const uint64_t live = n == 64 ? ~0ull : ((1ull << n) - 1);
        // ---- lanes: draws and sites of the chunk's attempts
        const u32x4 x = draw(I.k0, I.k1, T0 + (uint64_t)(j0 + lane), (uint32_t)slot, kTagFlip);
        const int site = (int)(((uint64_t)x.x * (uint32_t)N) >> 32);
        int rr = (int)((float)site * rL);          // site / L, at most one off, corrected below
        int cc = site - (int)__umul24((uint32_t)rr, (uint32_t)L);
        const int fix = cc < 0 ? -1 : (cc >= L ? 1 : 0);
        rr += fix;
        cc -= fix * L;
        const bool top = rr == 0, bottom = rr == L - 1;
        const int ru = top ? L - 1 : rr - 1, rd = bottom ? 0 : rr + 1;
        const int s_up = top ? site + (N - L) : site - L, s_dn = bottom ? site - (N - L) : site + L;
        const int s_lf = cc == 0 ? site + (L - 1) : site - 1, s_rt = cc == L - 1 ? site - (L - 1) : site + 1;
        // attempts of the chunk at this attempt's site or one of its neighbours.
        // Neighbourhoods are symmetric, so the later ones among them (qm) are
        // exactly the attempts whose evaluation a flip of this one makes out of
        // date, and the earlier ones (pm) those whose flip makes this one out of
        // date.  (Sites sharing a map entry only add attempts to either set.)
        uint64_t* const home = lmap + ent(site);
        atomicOr((unsigned long long*)home, lane < n ? lanebit : 0ull);
        const uint64_t e0 = *home, e1 = lmap[ent(s_up)], e2 = lmap[ent(s_dn)], e3 = lmap[ent(s_lf)], e4 = lmap[ent(s_rt)];
        *home = 0;
        const uint32_t off = MODEL == 0 ? 0u : (uint32_t)(((uint64_t)x.y * qm1) >> 32);
        // bounds of the acceptance threshold less the lane's updates: with y = lb minus
        // cur of the candidate bin, y > whi accepts and y < wlo rejects for certain
        const Bound32 tb = bounds_of(x.z, x.w, band32);
        const float whi = tb.hi - laneinc, wlo = tb.lo - laneinc;
        const uint64_t nbh = e0 | e1 | e2 | e3 | e4;
        const uint64_t pm = nbh & (lanebit - 1);
        const uint64_t qm = nbh & ~(lanebit | (lanebit - 1));
        uint64_t* const fword = lrow + (WIDE ? rr * wpr + (cc >> 6) : rr);   // Ising: the flip's word
        const uint64_t fbit = 1ull << (cc & 63);

        // the first attempt that this one's flip makes out of date (64: there is none), in
        // the upper half of the word that a step reads of its move
        const uint32_t cut = (uint32_t)__builtin_popcountll((qm - 1) & ~qm) << 16;

        // the chain: rounds from one evaluation of the lattice to the next
        uint32_t i = 0;                   // first attempt of the round
        for (;;) {
            int d;                        // bin change of this lane's attempt
            uint32_t nv = 0;              // Potts: proposed state
            if (MODEL == 0) {
                d = ising_d_words(lrow, wpr, rr, ru, rd, cc, L);
            } else {
                const uint32_t s0 = llat[site];
                const uint32_t n0 = llat[s_up], n1 = llat[s_dn], n2 = llat[s_lf], n3 = llat[s_rt];
                nv = s0 + 1u + off;
                nv = nv >= q ? nv - q : nv;
                const int nold = (n0 == s0) + (n1 == s0) + (n2 == s0) + (n3 == s0);
                const int nnew = (n0 == nv) + (n1 == nv) + (n2 == nv) + (n3 == nv);
                d = nold - nnew;
            }
            const uint32_t word = cut + ((uint32_t)d & 63u);
            int addr = (idx + d) << 2;
            float gp = bperm_f(cur, addr);
            __builtin_amdgcn_sched_barrier(0);
            // zall: moves within the bin (d = 0, always accepted); stale: attempts with
            // one of them in the neighbourhood; lim: the first attempt that is out of date,
            // as far as the moves made go; after: the attempts behind the last move.  An
            // attempt of no concern to the round has no threshold it could pass.
            const uint64_t run = live & (~0ull << i);
            const uint64_t zall = __builtin_amdgcn_ballot_w64(d == 0) & run;
            const uint64_t stale = __builtin_amdgcn_ballot_w64((pm & zall) != 0) & run;
            const uint64_t nz = run & ~zall;
            const bool mine = __builtin_amdgcn_inverse_ballot_w64(nz);
            const float wh = mine ? whi : __builtin_inff(), wl = mine ? wlo : __builtin_inff();
            uint64_t after = ~0ull;
            uint32_t lim = min(first_bit(stale), 64u);
            uint64_t moved = 0;           // accepted moves with d != 0 of the round
            for (;;) {
                // Steps from one accepted move with d != 0 to the next.  A step is one
                // dependent chain (look up, compare, first not certainly rejected, its bin
                // change) whose instructions a wave alone on its SIMD issues one by one (4.5
                // cycles for most, 11 for v_readlane, 24 for a branch): so there is one
                // branch, the next step's lookup is issued before this one is known to be a
                // move, and the bookkeeping runs while it is under way.  at: the
                // walker's bin, modulo 64, under the words' upper halves; addr: 4 (at + d).
                uint64_t gt, ge;
                uint32_t ja, at = (uint32_t)idx, w, lim1 = bit_then(safe, at, lim);
                float jf, gn;
                auto step = [&]() {
                    const float y = lb - gp;
                    ge = __builtin_amdgcn_ballot_w64(y >= wl);        // holds gt
                    gt = __builtin_amdgcn_ballot_w64(y > wh);
                    ja = first_bit(ge & after);
                    jf = (float)(int)ja;
                    w = (uint32_t)__builtin_amdgcn_readlane((int)word, (int)ja);
                    cnt = __builtin_fmaf(jf, hot, cnt);               // the old bin's visits
                    gn = rlf(gp, (int)ja);                            // the new bin's entry
                    addr += (int)(w << 2);
                    cur = __builtin_fmaf(cnt, inc32, g0);
                    gp = bperm_f(cur, addr);                          // lane: bits 2 to 7
                    __builtin_amdgcn_sched_barrier(0);
                    // none, or one between the bounds, or in a bin outside `safe`: left to
                    // the code below
                    return ja < bit_then(gt, ja, lim1);
                };
                auto move = [&]() {
                    at += w;
                    lim = min(lim, w >> 16);
                    after = ~1ull << (ja & 63);
                    hot = __builtin_amdgcn_inverse_ballot_w64(1ull << (at & 63)) ? 1.0f : 0.0f;
                    cnt = __builtin_fmaf(-jf, hot, cnt);
                    lb = __builtin_fmaf(-jf, inc32, gn);
                    set_bit(moved, ja);
                };
                bool go = step();
                while (go) {
                    move();
                    lim1 = bit_then(safe, at, lim);
                    __builtin_amdgcn_sched_barrier(0);
                    go = step();
                }
                // the step not taken (cur of the walker's own bin is of no use to any attempt)
                cnt = __builtin_fmaf(-jf, hot, cnt);
                idx = (int)(at & 63);
                const uint32_t end = bit_pick(safe, at, lim, 65);
                if (__builtin_expect(min(ja, 64u) >= end, 1)) break;  // the usual end of a round
                if (end == 65) {
                    settle(64 - (int)__builtin_clzll(moved));         // up to the last move
                    addr = (idx + d) << 2;
                    gp = bperm_f(cur, addr);
                    continue;
                }
                // attempts between the bounds are decided exactly, in order, up to the
                // first accepted one
                const uint64_t open = nz & after & (~0ull >> (64 - lim));
                uint64_t acc = gt & open, amb = ge & ~gt & open & (acc - 1) & ~acc;
                while (amb) {
                    const uint32_t kk = first_bit(amb);
                    const int cand = idx + __builtin_amdgcn_readlane(d, (int)kk);
                    const double here = __builtin_fma((double)(rlf(cnt, idx) + (float)kk), incv, rld(gl, idx));
                    const double there = __builtin_fma((double)rlf(cnt, cand), incv, rld(gl, cand));
                    if (wave_decide(I, T0 + (uint64_t)j0 + (uint64_t)kk, (uint32_t)slot, here - there, lane)) {
                        acc = 1ull << kk;
                        break;
                    }
                    amb &= amb - 1;
                }
                if (!acc) break;
                ja = first_bit(acc);
                jf = (float)(int)ja;
                cnt = __builtin_fmaf(jf, hot, cnt);
                cur = __builtin_fmaf(cnt, inc32, g0);
                w = (uint32_t)__builtin_amdgcn_readlane((int)word, (int)ja);
                gn = rlf(cur, (int)((at + w) & 63));
                move();
                idx = (int)(at & 63);
                addr = (idx + d) << 2;
                gp = bperm_f(cur, addr);
            }
            // the round's flips: its accepted moves, and its d = 0 moves before the first
            // out-of-date attempt
            const uint64_t flips = (zall & (~0ull >> (64 - lim))) | moved;
            if (__builtin_amdgcn_inverse_ballot_w64(flips)) {
                if (MODEL == 0) atomicXor((unsigned long long*)fword, fbit);
                else llat[site] = (uint8_t)nv;
            }
            work += (uint32_t)__builtin_popcountll(moved) + 4;           // a round costs about 4
            i = lim;
            if (i >= (uint32_t)n) break;  // else evaluated again on the lattice as it stands now
        }
        settle(n);
        cnt = lb = 0.0f;
    }
    store_window();
    if (lane == 0 && cost) atomicMax(cost, work);

    // ---- write back (HG: the window's store above is the write back)
    if (!HG)
        for (int i = lane; i < WB; i += 64) {
            const uint32_t hv = lH[i + kPad];
            gH[i] = hv == 0xffffffffu ? 0ull : (uint64_t)hv + cw;
        }
    else
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    if (MODEL == 0) {
        for (int i = lane; i < L * wpr; i += 64) I.lat[(size_t)slot * L * wpr + i] = lrow[i];
    } else {
        for (int i = lane; i < N; i += 64) I.plat[(size_t)slot * N + i] = llat[i];
    }
    if (lane == 0) {
        I.bin[slot] = b0 + idx - kPad + lo;
        I.swaps[slot] = -1;
    }
    // ---- flatness (Sec. II.A): wave-wide min and sum of the walker's counts
    if (inc) {
        // minimum and sum of the counts over the levels that occur (relative to cw
        // with LDS placement, absolute with HG)
        uint64_t mn = ~0ull, sum = 0;
        for (int i = lane + kPad; i < WB + kPad; i += 64) {
            if (HG) {
                if (!occurs(i)) continue;
                const uint64_t v = gH[i - kPad];
                mn = v < mn ? v : mn;
                sum += v;
            } else {
                const uint32_t v = lH[i];
                if (v == 0xffffffffu) continue;
                mn = v < mn ? v : mn;
                sum += v;
            }
        }
        for (int off = 32; off > 0; off >>= 1) {
            const uint64_t m2 = shfl_xor_u64(mn, off), s2 = shfl_xor_u64(sum, off);
            mn = m2 < mn ? m2 : mn;
            sum += s2;
        }
        if (lane == 0) {
            const int64_t n = I.nreach[a];
            if (walker_flat(I, mn + cw, sum + (uint64_t)n * cw, n, k)) I.flat[slot] = 1;
        }
    }
}

__global__ void __launch_bounds__(512) k_sweep_wave(const Inst* __restrict__ insts,
                                                    const Tile* __restrict__ tiles, uint32_t* __restrict__ cost)
{
    extern __shared__ __align__(16) char smem[];
    const Tile tile = tiles[blockIdx.x];
    const Inst& I = insts[tile.inst];
    if (I.ctr->all_done) return;
    if (cost) cost += blockIdx.x;
    const bool wide = I.wpr > 1;
    if (I.hglobal) {
        if (I.model == 0) {
            if (wide) sweep_wave<0, true, true>(I, tile, smem, cost);
            else sweep_wave<0, false, true>(I, tile, smem, cost);
        } else {
            sweep_wave<1, false, true>(I, tile, smem, cost);
        }
    } else {
        if (I.model == 0) {
            if (wide) sweep_wave<0, true, false>(I, tile, smem, cost);
            else sweep_wave<0, false, false>(I, tile, smem, cost);
        } else {
            sweep_wave<1, false, false>(I, tile, smem, cost);
        }
    }
}

// ------------------------------------------------------------------- merge
// One block per (instance, window).  When all m walkers are flat:
// ln g := mean_w ln g_w = base + 2^-(k + log2 m) sum_w H_w (exact), then the
// table is shifted by the integer part of its minimum over occurring levels.
__global__ void __launch_bounds__(256) k_merge(const Inst* __restrict__ insts,
                                               const int2* __restrict__ items)
{
    __shared__ double red[256];
    __shared__ int okflag, skip;
    const int2 it = items[blockIdx.x];
    const Inst& I = insts[it.x];
    const int a = it.y, tid = threadIdx.x;
    if (tid == 0) skip = I.ctr->all_done || I.done[a];   // one read, block-uniform
    __syncthreads();
    if (skip) return;
    int ok = 1;
    for (int r = tid; r < I.m; r += blockDim.x) ok &= I.flat[a * I.m + r];
    ok = __syncthreads_and(ok);
    if (!ok) return;
    const int WB = I.WB, m = I.m, k = I.k[a], lo = I.lo[a];
    const int sh = k + I.log2m;
    double* base = I.base + (size_t)a * WB;
    uint64_t* H = I.H + (size_t)a * m * WB;                    // the window's walkers, H[r][bin]
    double mn = __builtin_inf(), mx = 0.0;
    bool big = false;
    for (int b = tid; b < WB; b += blockDim.x) {
        uint64_t s = 0;
        for (int r = 0; r < m; ++r) s += H[(size_t)r * WB + b];
        big |= s >= (1ull << 53);                             // (double)s would round
        const double nb = base[b] + __builtin_ldexp((double)s, -sh);
        base[b] = nb;
        if (b <= I.hi[a] - lo && I.mask[lo + b]) mn = nb < mn ? nb : mn;
        mx = fabs(nb) > mx ? fabs(nb) : mx;
    }
    red[tid] = mn;
    __syncthreads();
    for (int st = blockDim.x / 2; st > 0; st >>= 1) {
        if (tid < st) red[tid] = red[tid + st] < red[tid] ? red[tid + st] : red[tid];
        __syncthreads();
    }
    const double shift = floor(red[0]);
    __syncthreads();
    red[tid] = mx;
    __syncthreads();
    for (int st = blockDim.x / 2; st > 0; st >>= 1) {
        if (tid < st) red[tid] = red[tid + st] > red[tid] ? red[tid + st] : red[tid];
        __syncthreads();
    }
    // values are multiples of 2^-sh, or of 2^-20 after a warm start: exact below 2^(52 - that)
    if (tid == 0) okflag = red[0] < __builtin_ldexp(1.0, 52 - (sh > 20 ? sh : 20));
    __syncthreads();
    if (__syncthreads_or(big) && tid == 0) okflag = 0;
    for (int b = tid; b < WB; b += blockDim.x) base[b] = base[b] - shift;
    for (size_t i = tid; i < (size_t)WB * m; i += blockDim.x) H[i] = 0ull;
    for (int r = tid; r < m; r += blockDim.x) I.flat[a * m + r] = 0;
    if (tid == 0) {
        if (!okflag) atomicOr(&I.ctr->err, kErrExactness);
        I.k[a] = k + 1;
        I.merges[a] = (int32_t)I.ctr->t;
        if (k + 1 >= I.kfinal) {
            I.done[a] = 1;
            const int nd = atomicAdd(&I.ctr->n_done, 1) + 1;
            if (nd == I.h) I.ctr->all_done = 1;
        }
    }
}

// ---------------------------------------------------------------- exchange
// Thread per (instance, window a < h-1, walker r); pairs with a = t (mod 2)
// are active.  Walker r of window a meets walker (r + c) mod m of window a+1,
// c drawn once per (t, a).  Eq. (1) in log form, decided exactly; on accept the
// two configurations (lattice and energy) change places, ln g and H stay.
__global__ void __launch_bounds__(256) k_exchange(const Inst* __restrict__ insts,
                                                  const int32_t* __restrict__ pair_start,
                                                  int n_inst)
{
    // one wave per proposing walker: every lane takes the same decision from the
    // same values, then the lanes swap the two configurations together
    const int lane = threadIdx.x & 63;
    const int gw = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
    if (gw >= pair_start[n_inst]) return;
    int lo_i = 0, hi_i = n_inst - 1;
    while (lo_i < hi_i) {
        int mid = (lo_i + hi_i + 1) >> 1;
        if (pair_start[mid] <= gw) lo_i = mid;
        else hi_i = mid - 1;
    }
    const Inst& I = insts[lo_i];
    if (!I.exch || I.ctr->all_done) return;
    const int local = gw - pair_start[lo_i];
    const int m = I.m, a = local / m, r = local - a * m;
    const int64_t t = I.ctr->t;
    if ((a & 1) != (int)(t & 1)) return;
    const u32x4 xc = draw(I.k0, I.k1, (uint64_t)t, (uint32_t)a, kTagPartner);
    const int c = (int)(((uint64_t)xc.x * (uint64_t)m) >> 32);
    const int rj = (r + c) & (m - 1);
    const int i = a * m + r, j = (a + 1) * m + rj;
    const int bi = I.bin[i], bj = I.bin[j];
    const int loa = I.lo[a], hia = I.hi[a], lob = I.lo[a + 1], hib = I.hi[a + 1];
    bool acc = false;
    if (bj >= loa && bj <= hia && bi >= lob && bi <= hib) {
        const int WB = I.WB;
        const double sa = __builtin_ldexp(1.0, -I.k[a]);
        const double sb = __builtin_ldexp(1.0, -I.k[a + 1]);
        const double* ba = I.base + (size_t)a * WB;
        const double* bb = I.base + (size_t)(a + 1) * WB;
        const uint64_t* Hi = I.H + (size_t)i * WB;
        const uint64_t* Hj = I.H + (size_t)j * WB;
        auto gi = [&](int bin) { return __builtin_fma((double)Hi[bin - loa], sa, ba[bin - loa]); };
        auto gj = [&](int bin) { return __builtin_fma((double)Hj[bin - lob], sb, bb[bin - lob]); };
        const double delta = (gi(bi) - gi(bj)) + (gj(bj) - gj(bi));
        const uint64_t u53 = u53_of(draw(I.k0, I.k1, (uint64_t)t, (uint32_t)i, kTagExchange));
        const int f = decide_fast(delta, threshold_of(u53, I.band), I.band);
        if (f == 2) {
            acc = accept_slow(delta, u53);
            if (lane == 0) atomicAdd((unsigned long long*)&I.ctr->slow, 1ull);
        } else {
            acc = f == 1;
        }
    }
    if (acc) {
        if (I.model == 0) {
            const int nwords = I.L * I.wpr;
            uint64_t* pi = I.lat + (size_t)i * nwords;
            uint64_t* pj = I.lat + (size_t)j * nwords;
            for (int w = lane; w < nwords; w += 64) {
                const uint64_t x = pi[w];
                pi[w] = pj[w];
                pj[w] = x;
            }
        } else {
            uint8_t* pi = I.plat + (size_t)i * I.N;
            uint8_t* pj = I.plat + (size_t)j * I.N;
            if ((I.N & 15) == 0) {                  // rows of 16-byte words (slots are N apart)
                uint4* qi = (uint4*)pi;
                uint4* qj = (uint4*)pj;
                for (int w = lane; w < (I.N >> 4); w += 64) {
                    const uint4 x = qi[w];
                    qi[w] = qj[w];
                    qj[w] = x;
                }
            } else {
                for (int w = lane; w < I.N; w += 64) {
                    const uint8_t x = pi[w];
                    pi[w] = pj[w];
                    pj[w] = x;
                }
            }
        }
    }
    if (lane == 0) {
        if (acc) {
            I.bin[i] = bj;
            I.bin[j] = bi;
            // replicas follow their configurations; a round trip is window 0,
            // then window h-1, then window 0 again (each replica takes part in
            // one proposal per interval, so these updates do not race)
            const int up = I.rid[i], down = I.rid[j];      // up: window a -> a+1
            I.rid[i] = down;
            I.rid[j] = up;
            if (a + 1 == I.h - 1 && I.rt_state[up] == 1) I.rt_state[up] = 2;
            if (a == 0) {
                if (I.rt_state[down] == 2) I.rt_count[down] += 1;
                I.rt_state[down] = 1;
            }
            atomicAdd((unsigned long long*)&I.ex_acc[a], 1ull);
        }
        atomicAdd((unsigned long long*)&I.ex_prop[a], 1ull);
        I.swaps[i] = acc ? 1 : 0;
        I.swaps[j] = acc ? 1 : 0;
    }
}

// ----------------------------------------------------------------- advance
// The wave sweep's blocks, those with most work first.  Windows differ by an order of
// magnitude in the work of an interval (moves and rounds per attempt); blocks start in
// their order, a SIMD serves its oldest wave first, and the launch ends with its slowest
// wave.  By one block, in 64 classes of the most work that a wave of the block had since
// the last time; which of a class comes first is left open.  us per interval of 10^4
// attempts, in the windows' order and so: Potts q=10 L=32, 4096 walkers 842 and 633; L=64
// 984 and 821; Ising L=128, 2048 walkers 690 and 608.  (Priorities instead, s_setprio by
// window: 650, 984 and 655; order and priorities: no better.)
constexpr int kOrderClasses = 64, kOrderEvery = 8;
__device__ void order_tiles(Tile* tiles, Tile* tmp, uint32_t* cost, int ntiles)
{
    __shared__ uint32_t top, start[kOrderClasses];
    const int tid = threadIdx.x;
    if (tid == 0) top = 0;
    if (tid < kOrderClasses) start[tid] = 0;
    __syncthreads();
    uint32_t mx = 0;
    for (int i = tid; i < ntiles; i += blockDim.x) mx = cost[i] > mx ? cost[i] : mx;
    atomicMax(&top, mx);
    __syncthreads();
    const uint64_t all = (uint64_t)top + 1;
    auto class_of = [&](int i) { return kOrderClasses - 1 - (int)((uint64_t)cost[i] * kOrderClasses / all); };
    for (int i = tid; i < ntiles; i += blockDim.x) atomicAdd(&start[class_of(i)], 1u);
    __syncthreads();
    if (tid == 0)
        for (uint32_t c = 0, sum = 0; c < kOrderClasses; ++c) {
            const uint32_t v = start[c];
            start[c] = sum;
            sum += v;
        }
    __syncthreads();
    for (int i = tid; i < ntiles; i += blockDim.x) tmp[atomicAdd(&start[class_of(i)], 1u)] = tiles[i];
    __syncthreads();
    for (int i = tid; i < ntiles; i += blockDim.x) {
        tiles[i] = tmp[i];
        cost[i] = 0;
    }
}

// queue[0]: the persistent sweep's tile queue; queue[1]: intervals so far.  ntiles: the wave
// sweep's blocks if their order matters, else 0.
__global__ void k_advance(const Inst* __restrict__ insts, int n_inst, int32_t* __restrict__ queue, Tile* tiles, Tile* tmp,
                          uint32_t* cost, int ntiles)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (blockIdx.x == 0 && ntiles > 0) {
        const int t = queue[1];
        __syncthreads();
        if (threadIdx.x == 0) queue[1] = (t + 1) & 0xffff;
        // the time it takes grows with the blocks: so does the time between (every 8th interval
        // of 10^2 attempts, 65 536 blocks 1545 us per interval, so 1506, never 1494; of 10^3,
        // 16 384 blocks 973, 964 and 1004)
        if (t % (kOrderEvery + (ntiles >> 7)) == 0) order_tiles(tiles, tmp, cost, ntiles);
    }
    if (i == 0) *queue = 0;
    if (i >= n_inst) return;
    InstCtr* c = insts[i].ctr;
    if (!c->stopped) {
        c->t += 1;
        if (c->all_done) c->stopped = 1;
    }
}

// -------------------------------------------------------------------- init
// Thread per slot.  Start from a ground state (Ising: all up, or the
// checkerboard for a window in the upper half; Potts: all 0) and take every
// proposal that does not increase the distance of the energy bin to the window.
__device__ int lattice_bin(const Inst& I, int slot)
{
    const int L = I.L;
    int broken = 0;
    for (int y = 0; y < L; ++y)
        for (int x = 0; x < L; ++x) {
            const int xr = x + 1 == L ? 0 : x + 1, yd = y + 1 == L ? 0 : y + 1;
            if (I.model == 0) {
                auto sp = [&](int yy, int xx) {
                    return (int)(I.lat[(size_t)slot * L * I.wpr + yy * I.wpr + (xx >> 6)] >> (xx & 63)) & 1;
                };
                broken += (sp(y, x) != sp(y, xr)) + (sp(y, x) != sp(yd, x));
            } else {
                auto sp = [&](int yy, int xx) { return (int)I.plat[(size_t)slot * I.N + yy * L + xx]; };
                broken += (sp(y, x) != sp(y, xr)) + (sp(y, x) != sp(yd, x));
            }
        }
    return I.model == 0 ? broken / 2 : broken;
}

__global__ void k_init(const Inst* __restrict__ insts, const int32_t* __restrict__ thread_start,
                       int n_inst)
{
    const int gid = blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= thread_start[n_inst]) return;
    int lo_i = 0, hi_i = n_inst - 1;
    while (lo_i < hi_i) {
        int mid = (lo_i + hi_i + 1) >> 1;
        if (thread_start[mid] <= gid) lo_i = mid;
        else hi_i = mid - 1;
    }
    const Inst& I = insts[lo_i];
    const int slot = gid - thread_start[lo_i];
    const int a = slot / I.m, L = I.L, N = I.N;
    const int wlo = I.lo[a], whi = I.hi[a];
    const bool upper = wlo + whi > I.W - 1;
    if (I.model == 0) {
        for (int y = 0; y < L; ++y)
            for (int wi = 0; wi < I.wpr; ++wi) {
                uint64_t word = 0;
                for (int xb = 0; xb < 64; ++xb) {
                    const int x = wi * 64 + xb;
                    if (x >= L) break;
                    const bool up = upper ? ((x + y) & 1) == 0 : true;
                    word |= (uint64_t)up << xb;
                }
                I.lat[(size_t)slot * L * I.wpr + y * I.wpr + wi] = word;
            }
    } else {
        for (int s = 0; s < N; ++s) I.plat[(size_t)slot * N + s] = 0;
    }
    int b = lattice_bin(I, slot);
    auto dist = [&](int bb) { return bb < wlo ? wlo - bb : (bb > whi ? bb - whi : 0); };
    const int64_t cap = 1000 * (int64_t)N;
    for (int64_t j = 0; b < wlo || b > whi; ++j) {
        if (j >= cap) {
            atomicOr(&I.ctr->err, kErrInitStuck);
            return;
        }
        const u32x4 x = draw(I.k0, I.k1, (uint64_t)j, (uint32_t)slot, kTagInit);
        const int site = (int)(((uint64_t)x.x * (uint64_t)N) >> 32);
        const int r = site / L, c = site - r * L;
        const int ru = r == 0 ? L - 1 : r - 1, rd = r == L - 1 ? 0 : r + 1;
        const int cl = c == 0 ? L - 1 : c - 1, cr = c == L - 1 ? 0 : c + 1;
        int nb;
        int nv = 0;
        if (I.model == 0) {
            auto sp = [&](int yy, int xx) {
                return (int)(I.lat[(size_t)slot * L * I.wpr + yy * I.wpr + (xx >> 6)] >> (xx & 63)) & 1;
            };
            const int s = sp(r, c);
            const int ones = sp(ru, c) + sp(rd, c) + sp(r, cl) + sp(r, cr);
            const int al = s ? ones : 4 - ones;
            nb = b + al - 2;
        } else {
            auto sp = [&](int yy, int xx) { return (int)I.plat[(size_t)slot * N + yy * L + xx]; };
            const int s = sp(r, c);
            nv = s + 1 + (int)(((uint64_t)x.y * (uint64_t)(I.q - 1)) >> 32);
            nv = nv >= I.q ? nv - I.q : nv;
            const int n[4] = {sp(ru, c), sp(rd, c), sp(r, cl), sp(r, cr)};
            int nold = 0, nnew = 0;
            for (int d = 0; d < 4; ++d) {
                nold += n[d] == s;
                nnew += n[d] == nv;
            }
            nb = b + nold - nnew;
        }
        if (dist(nb) <= dist(b)) {
            if (I.model == 0) {
                uint64_t* p = I.lat + (size_t)slot * L * I.wpr + r * I.wpr + (c >> 6);
                *p ^= 1ull << (c & 63);
            } else {
                I.plat[(size_t)slot * N + site] = (uint8_t)nv;
            }
            b = nb;
        }
    }
    I.bin[slot] = b;
}

// ------------------------------------------------------------ concatenate
// Sec. II.B: per overlap, 5-point derivative of both pieces with step d,
// join where they agree best (ties to the lower bin, joins ascending), shift
// the pieces, cut the tails, normalise to sum g = q^N.  One block per set of
// pieces: block r joins pieces[r][h][WB] into out[r][W] (join[r][max(h-1,1)],
// shift[r][h], status[r]); all sets share the windows of instance `inst`.
// The search of a window depends on the one before only through its lower end (joins
// ascend), so every wave first searches windows of its own in full, and wave 0 then
// goes through them in order, searching again only where the join found lies below
// that end.  (76 overlaps of 751 bins one after the other took 770 us for 201 sets, now 310.)
template <int U>
__device__ int join_of(const Inst& I, const double* __restrict__ fa, const double* __restrict__ fb, int loa, int lob,
                       int hia, int d, int first)
{
    const int lane = threadIdx.x & 63;
    const uint8_t* mk = I.mask;
    double best = __builtin_inf();
    int bestb = -1;
    const int last = hia - 2 * d;              // every load below stays inside both pieces
    for (int b0 = first; b0 <= last; b0 += U * 64) {
        bool ok[U];
        double diff[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {          // U at a time: one wait for all their loads
            const int b = b0 + 64 * u + lane, bc = b < last ? b : last, ia = bc - loa, ib = bc - lob;
            ok[u] = b <= last && (mk[bc] & mk[bc - d] & mk[bc + d] & mk[bc - 2 * d] & mk[bc + 2 * d]);
            const double na = ((fa[ia - 2 * d] - 8.0 * fa[ia - d]) + 8.0 * fa[ia + d]) - fa[ia + 2 * d];
            const double nbv = ((fb[ib - 2 * d] - 8.0 * fb[ib - d]) + 8.0 * fb[ib + d]) - fb[ib + 2 * d];
            diff[u] = fabs(na / (12.0 * d) - nbv / (12.0 * d));
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (ok[u] && (bestb < 0 || diff[u] < best)) {
                best = diff[u];
                bestb = b0 + 64 * u + lane;
            }
    }
    for (int o = 32; o > 0; o >>= 1) {
        const double d2 = __shfl_xor(best, o);
        const int b2 = __shfl_xor(bestb, o);
        if (b2 >= 0 && (bestb < 0 || d2 < best || (d2 == best && b2 < bestb))) {
            best = d2;
            bestb = b2;
        }
    }
    return bestb;
}

// Threads of a block for so many rows on n_cu CUs, U windows' loads at a time.  Alone on its
// CU a block is fastest with 16 waves and four loads under way (94 registers); of more rows
// as many blocks share a CU as its 32 waves allow with one load under way (54 registers).
// Kernel, us, with 1024 threads and U = 4 / so: 1001 rows of Ising L=16, 8 windows 64 / 20,
// L=64, 16 windows 259 / 158, Potts L=100, 77 windows 1494 / 1040; 4001 rows 234 / 42 and
// 1061 / 545; 201 rows of Potts L=100 353 / 451 (512 threads).
constexpr int kConcatThreads = 1024;
inline int concat_threads(int64_t rows, int n_cu)
{
    return rows <= n_cu ? kConcatThreads : rows <= 4 * (int64_t)n_cu ? 512 : rows <= 8 * (int64_t)n_cu ? 256 : 128;
}
template <int U>
__global__ void __launch_bounds__(kConcatThreads) k_concat(const Inst* __restrict__ insts, int inst,
                                                           const double* __restrict__ pieces,
                                                           double* __restrict__ out,
                                                           int32_t* __restrict__ join, double* __restrict__ shift,
                                                           int32_t* __restrict__ status)
{
    __shared__ double rd[kConcatThreads];
    const Inst& I = insts[inst];
    const int h = I.h, WB = I.WB, W = I.W, tid = threadIdx.x;
    const size_t set = blockIdx.x;
    pieces += set * h * WB;
    out += set * W;
    join += set * (h > 1 ? h - 1 : 1);
    shift += set * h;
    status += set;
    auto stencil = [&](int a) {                // step of the derivative in overlap a
        const int d = (I.hi[a] - I.lo[a + 1] + 1) / 8;
        return d < 1 ? 1 : (d > 10 ? 10 : d);
    };
    for (int a = tid >> 6; a + 1 < h; a += (int)(blockDim.x >> 6)) {
        const double* fa = pieces + (size_t)a * WB;
        const double* fb = pieces + (size_t)(a + 1) * WB;
        const int d = stencil(a), loa = I.lo[a], lob = I.lo[a + 1];
        const int bs = join_of<U>(I, fa, fb, loa, lob, I.hi[a], d, lob + 2 * d);
        if ((tid & 63) == 0) {
            join[a] = bs;
            shift[a + 1] = bs < 0 ? 0.0 : fa[bs - loa] - fb[bs - lob];
        }
    }
    __syncthreads();
    if (tid < 64) {
        double sh = 0.0;
        int before = -1, st = 0;               // the join of the window before
        if (tid == 0) shift[0] = 0.0;
        for (int a0 = 0; a0 + 1 < h; a0 += 64) {
            // lane l: window a0 + l
            const int n = h - 1 - a0 < 64 ? h - 1 - a0 : 64, al = a0 + (tid < n ? tid : 0);
            int jl = join[al];
            double sl = shift[al + 1];
            const int fl = I.lo[al + 1] + 2 * stencil(al);
            for (int i = 0; i < n; ++i) {
                const int a = a0 + i;
                int first = __builtin_amdgcn_readlane(fl, i), bs = __builtin_amdgcn_readlane(jl, i);
                double step = rld(sl, i);
                if (a > 0 && before + 1 > first) first = before + 1;
                if (bs >= 0 && bs < first) {
                    const double* fa = pieces + (size_t)a * WB;
                    const double* fb = pieces + (size_t)(a + 1) * WB;
                    const int loa = I.lo[a], lob = I.lo[a + 1];
                    bs = __builtin_amdgcn_readfirstlane(join_of<U>(I, fa, fb, loa, lob, I.hi[a], stencil(a), first));
                    step = bs < 0 ? 0.0 : fa[bs - loa] - fb[bs - lob];
                }
                if (bs < 0) {                  // no valid join: report, keep indices inside
                    st = -2;
                    const int lob = I.lo[a + 1], hia = I.hi[a];
                    bs = first < lob ? lob : (first > hia ? hia : first);
                }
                sh = sh + step;
                before = bs;
                if (tid == i) {
                    jl = bs;
                    sl = sh;
                }
            }
            if (tid < n) {
                join[al] = jl;
                shift[al + 1] = sl;
            }
        }
        if (tid == 0) *status = st;
    }
    __syncthreads();
    // assemble
    double mx = -__builtin_inf();
    for (int b = tid, a = 0; b < W; b += blockDim.x) {
        while (a + 1 < h && b > join[a]) ++a;  // ascending bins: the piece before is still the start
        const double v = pieces[(size_t)a * WB + (b - I.lo[a])] + shift[a];
        out[b] = v;
        if (I.mask[b] && v > mx) mx = v;
    }
    rd[tid] = mx;
    __syncthreads();
    for (int st = blockDim.x / 2; st > 0; st >>= 1) {
        if (tid < st) rd[tid] = rd[tid + st] > rd[tid] ? rd[tid + st] : rd[tid];
        __syncthreads();
    }
    const double gmax = rd[0];
    __syncthreads();
    double acc = 0.0;
    for (int b = tid; b < W; b += blockDim.x)
        if (I.mask[b]) acc += exp(out[b] - gmax);
    rd[tid] = acc;
    __syncthreads();
    for (int st = blockDim.x / 2; st > 0; st >>= 1) {
        if (tid < st) rd[tid] += rd[tid + st];
        __syncthreads();
    }
    const double lse = gmax + log(rd[0]);
    const double target = (double)I.N * log(I.model == 0 ? 2.0 : (double)I.q);
    __syncthreads();
    for (int b = tid; b < W; b += blockDim.x)
        out[b] = I.mask[b] ? out[b] + (target - lse) : -__builtin_inf();
}

// ---------------------------------------------------------------- collect
// Up to kCollect pieces of device memory into one buffer, a block each (host_copy.hpp).
__global__ void __launch_bounds__(256) k_collect(const Collect c, char* __restrict__ out)
{
    const int p = blockIdx.x;
    const uint32_t n16 = c.bytes[p] >> 4;
    const uint4* s = (const uint4*)c.src[p];
    uint4* o = (uint4*)(out + c.off[p]);
    for (uint32_t i = threadIdx.x; i < n16; i += blockDim.x) o[i] = s[i];
    for (uint32_t i = (n16 << 4) + threadIdx.x; i < c.bytes[p]; i += blockDim.x) out[c.off[p] + i] = c.src[p][i];
}

// ------------------------------------------------------ predicate probe
// Evaluates the full acceptance predicate (fast test against log(u53 2^-53)
// with the guard band, exact slow path inside it) on caller-given inputs.
__global__ void k_accept_probe(const double* __restrict__ delta, const uint64_t* __restrict__ u53,
                               int n, int32_t* __restrict__ out)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        const int f = decide_fast(delta[i], threshold_of(u53[i], kBand), kBand);
        out[i] = f == 2 ? (accept_slow(delta[i], u53[i]) ? 3 : 2) : f;
    }
}

__global__ void k_bounds_probe(const uint32_t* __restrict__ zw, int n, double band, float* __restrict__ out)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t z = zw[2 * i], w = zw[2 * i + 1];
    const Bound32 b = bounds_of(z, w, (float)band);
    const float e = kErrLane + (float)band, hi = upper_of(z, w, e);
    out[4 * i + 0] = b.lo;
    out[4 * i + 1] = b.hi;
    out[4 * i + 2] = hi;
    out[4 * i + 3] = lower_of(hi, e);
}

// worst: the bits of a non-negative double, whose order is that of the doubles.
__global__ void k_log2_probe(uint32_t first, int64_t n, unsigned long long* __restrict__ worst)
{
    double mx = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float u = __builtin_bit_cast(float, (uint32_t)(first + (uint32_t)i));
        const double l = log2((double)u), e = fabs((double)__builtin_amdgcn_logf(u) - l) / (0x1p-23 * (1.0 + fabs(l)));
        mx = e > mx ? e : mx;
    }
    atomicMax(worst, __builtin_bit_cast(unsigned long long, mx));
}

__global__ void k_philox_probe(const uint32_t* __restrict__ in, int n, uint32_t* __restrict__ out)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        const uint32_t* c = in + 6 * i;
        const u32x4 x = philox10(c[0], c[1], c[2], c[3], c[4], c[5]);
        out[4 * i + 0] = x.x;
        out[4 * i + 1] = x.y;
        out[4 * i + 2] = x.z;
        out[4 * i + 3] = x.w;
    }
}

}  // namespace rewl
