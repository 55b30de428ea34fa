// gfx950 kernels of the phase-space hot path and their host launchers.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>

#include "chain.h"
#include "device_util.h"
#include "launch.h"

namespace msx {

namespace {

// ---------------------------------------------------------------------------
// Kernels
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(kBlock) void k_uniform(uint64_t seed, uint64_t sid, uint64_t e0, int64_t n, int d,
                                                    double* __restrict__ y) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint64_t e = e0 + (uint64_t)i;
    for (int g = 0; g < (d + 3) / 4; ++g) {
        uint64_t c0 = e, c1 = (uint64_t)g, c2 = 0, c3 = 0;
        philox4x64_10(c0, c1, c2, c3, seed, sid);
        const uint64_t wv[4] = {c0, c1, c2, c3};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int k = 4 * g + j;
            if (k < d) y[(int64_t)k * n + i] = to_unit(wv[j]);
        }
    }
}

template <bool MIX>
__global__ __launch_bounds__(kBlock) void k_weight(const ChannelTab* __restrict__ ct, const ProcessTab* __restrict__ pt,
                                                   int np, int64_t n, const double* __restrict__ p,
                                                   const double* __restrict__ x1x2, const double* __restrict__ jac,
                                                   double* __restrict__ w, double* __restrict__ alpha) {
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    double j = jac[e];
    double wv = 0.0, av = 0.0;
    if (j != 0.0) {
        double x1 = 1.0, x2 = 1.0, L = 0.0;
        if (ct->hadronic) {
            x1 = x1x2[e];
            x2 = x1x2[n + e];
            L = t_log<MIX>(x1 * x2);
        }
        auto get = [&](int k, int c) -> double { return p[((int64_t)c * np + k + 2) * n + e]; };
        double pae = p[((int64_t)0 * np) * n + e], pax = p[((int64_t)1 * np) * n + e];
        double pay = p[((int64_t)2 * np) * n + e], paz = p[((int64_t)3 * np) * n + e];
        RegQ q;
        double af = integrand_alpha<MIX, kMaxFinal>(pt, ct->alpha_index, x1, x2, L, pae, pax, pay, paz, get, q, av);
        wv = af * j;
    }
    w[e] = wv;
    if (alpha) alpha[e] = av;
}

// Sum of the statistics of tiles [t0, t1) over the first kBlock threads of a
// workgroup, in a fixed order; the result is valid in thread 0.  Every thread
// of the workgroup calls it.
struct TileSum {
    double s1, s2, zeros, wmax;
};
__device__ __forceinline__ TileSum sum_tiles(const double* tile_stats, int64_t t0, int64_t t1,
                                             double (&red)[4][kWaves]) {
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t t = threadIdx.x < kBlock ? t0 + threadIdx.x : t1; t < t1; t += kBlock) {
        a[0] += tile_stats[t * 4 + 0];
        a[1] += tile_stats[t * 4 + 1];
        a[2] += tile_stats[t * 4 + 2];
        a[3] = fmax(a[3], tile_stats[t * 4 + 3]);
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double r0 = wave_sum(a[0]), r1 = wave_sum(a[1]), r2 = wave_sum(a[2]), r3 = wave_max(a[3]);
    if (lane == 0 && wave < kWaves) {
        red[0][wave] = r0;
        red[1][wave] = r1;
        red[2][wave] = r2;
        red[3][wave] = r3;
    }
    __syncthreads();
    TileSum r{red[0][0], red[1][0], red[2][0], red[3][0]};
    for (int v = 1; v < kWaves; ++v) {
        r.s1 += red[0][v];
        r.s2 += red[1][v];
        r.zeros += red[2][v];
        r.wmax = fmax(r.wmax, red[3][v]);
    }
    return r;
}

// A channel with more than kStatTiles tiles is reduced in two steps: first
// kStatSlices workgroups sum a contiguous run of its tiles each, in place
// (into the run's first entry), then the last of them to finish adds the runs.
// One workgroup per channel walking all its tiles is bound by the latency of its
// loads: 147 us for the 78125 tiles of 2e7 t tbar events, 11 us in two steps;
// up to 2048 tiles (eight loads a thread) the slices would cost more than they
// save.  A launch of its own for the slices, made whenever the buffers of a
// device-count call hold that many tiles, took 2.2 us of the 16 of a thousand
// two-dimensional events.
constexpr int kStatTiles = 2048, kStatSlices = 64;

// Reduce the tiles of channel c and add to its accumulators
// stats[c] = (sum w, sum w^2, n, n(w == 0), max w); every thread of a workgroup
// of at least kBlock calls it, for every slice: kStatSlices of them where a channel
// may have more than kStatTiles tiles (SLICED), else one, without the code of the
// others (0.4 us of a launch).
template <bool SLICED>
__device__ __forceinline__ void channel_stats(int c, int slice, const SampleCall* __restrict__ call,
                                              uint32_t* __restrict__ done, double* tile_stats,
                                              double* __restrict__ stats, double (&red)[4][kWaves]) {
    if (c >= call->n_chan || ((call->skip_mask >> c) & 1)) return;
    const int64_t t0 = call->tile_start[c], t1 = call->tile_start[c + 1];
    TileSum r;
    if (!SLICED || t1 - t0 <= kStatTiles) {
        if (slice) return;
        r = sum_tiles(tile_stats, t0, t1, red);
    } else {
        const int64_t per = (t1 - t0 + kStatSlices - 1) / kStatSlices;
        const int64_t b = t0 + slice * per, e = min(t1, b + per);
        if (b >= e) return;
        const int slices = (int)((t1 - t0 + per - 1) / per);  // that have tiles
        __shared__ int last;
        const TileSum own = sum_tiles(tile_stats, b, e, red);
        if (threadIdx.x == 0) {
            tile_stats[b * 4 + 0] = own.s1;
            tile_stats[b * 4 + 1] = own.s2;
            tile_stats[b * 4 + 2] = own.zeros;
            tile_stats[b * 4 + 3] = own.wmax;
            __threadfence();
            last = atomicAdd(&done[c], 1u) == (unsigned)slices - 1;
        }
        __syncthreads();
        if (!last) return;
        __threadfence();
        // the runs' sums sit in the first entry of each run
        const int64_t t = t0 + threadIdx.x * per;
        if (threadIdx.x < 64) {
            static_assert(kStatSlices == 64, "one lane per run");
            const bool has = t < t1;
            r.s1 = wave_sum(has ? tile_stats[t * 4 + 0] : 0.0);
            r.s2 = wave_sum(has ? tile_stats[t * 4 + 1] : 0.0);
            r.zeros = wave_sum(has ? tile_stats[t * 4 + 2] : 0.0);
            r.wmax = wave_max(has ? tile_stats[t * 4 + 3] : 0.0);
        }
    }
    if (threadIdx.x == 0) {
        double* st = stats + 5 * c;
        st[0] += r.s1;
        st[1] += r.s2;
        st[2] += (double)(call->ev_start[c + 1] - call->ev_start[c]);
        st[3] += r.zeros;
        st[4] = fmax(st[4], r.wmax);
    }
}

// The statistics of a call, a row of workgroups per channel.  After the sample
// has read it the caller's event counter may move on (null: it stays).
template <bool SLICED>
__global__ __launch_bounds__(kBlock) void k_stats_final(const SampleCall* __restrict__ call,
                                                        uint32_t* __restrict__ done, double* tile_stats,
                                                        double* __restrict__ stats, uint64_t* __restrict__ advance) {
    __shared__ double red[4][kWaves];
    if (advance && threadIdx.x == 0 && blockIdx.x == 0 && blockIdx.y == 0)
        *advance += (uint64_t)call->ev_start[call->n_chan];
    channel_stats<SLICED>(blockIdx.y, blockIdx.x, call, done, tile_stats, stats, red);
}

// Hit-or-miss unweighting (the paper's channel-wise unweighting against an
// estimated maximum weight): event i is kept when u_i w_max < w_i, u_i the
// Philox uniform of event id e0 + i (dimension 0, as msx_uniform), and
// carries the unit weight max(1, w_i / w_max) (overweight events above 1).
// Pass 1 decides: every wave writes its decisions as one 64-bit mask per 64
// events, and the kept events of every block of kUnwPer are counted; a one-
// workgroup scan turns the counts into offsets; pass 2 writes the kept
// indices in increasing order from the masks (ranks are bit counts).  The
// generator is most of the work, so it runs once: deciding again in pass 2
// made that pass as long as the first (59 us each for 1e7 weights; now 55
// and 8, and the scan 23 -> 13 with its 1024 run totals added by waves).
constexpr int kUnwPer = kBlock * 4;          // events per block
constexpr int kUnwMasks = kUnwPer / 64;      // masks per block

__global__ __launch_bounds__(kBlock) void k_unw_count(const double* __restrict__ w, int64_t n, double w_max,
                                                      uint64_t seed, uint64_t sid, uint64_t e0,
                                                      int64_t* __restrict__ blk, uint64_t* __restrict__ masks) {
    __shared__ int red[kWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t base = (int64_t)blockIdx.x * kUnwPer;
    double wv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int64_t i = base + q * kBlock + threadIdx.x;
        wv[q] = i < n ? w[i] : 0.0;
    }
    int c = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int64_t i = base + q * kBlock + threadIdx.x;
        uint64_t c0 = e0 + (uint64_t)i, c1 = 0, c2 = 0, c3 = 0;
        philox4x64_10(c0, c1, c2, c3, seed, sid);
        const uint64_t bal = __ballot(i < n && to_unit(c0) * w_max < wv[q]);
        if (lane == 0) masks[(int64_t)blockIdx.x * kUnwMasks + q * kWaves + wave] = bal;
        c += __popcll(bal);
    }
    if (lane == 0) red[wave] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t t = 0;
        for (int v = 0; v < kWaves; ++v) t += red[v];
        blk[blockIdx.x] = t;
    }
}

// Exclusive scan of nb block counts in place (one workgroup: every thread
// sums a contiguous run, the run totals are scanned by waves); total to
// *count.
__global__ __launch_bounds__(1024) void k_unw_scan(int64_t* __restrict__ blk, int64_t nb, int64_t* __restrict__ count) {
    __shared__ int64_t tot[16];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int64_t per = (nb + 1023) / 1024;
    const int64_t b0 = t * per, b1 = min(nb, b0 + per);
    int64_t s = 0;
    for (int64_t b = b0; b < b1; ++b) s += blk[b];
    int64_t run = s;  // inclusive over the wave
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t x = __shfl_up(run, o, 64);
        if (lane >= o) run += x;
    }
    if (lane == 63) tot[wave] = run;
    __syncthreads();
    int64_t acc = run - s;
    for (int v = 0; v < wave; ++v) acc += tot[v];
    if (t == 1023) *count = acc + s;
    for (int64_t b = b0; b < b1; ++b) {
        const int64_t x = blk[b];
        blk[b] = acc;
        acc += x;
    }
}

__global__ __launch_bounds__(kBlock) void k_unw_write(const double* __restrict__ w, double w_max,
                                                      const int64_t* __restrict__ blk,
                                                      const uint64_t* __restrict__ masks, int64_t* __restrict__ keep,
                                                      double* __restrict__ uw) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t* m = masks + (int64_t)blockIdx.x * kUnwMasks;
    int64_t base = blk[blockIdx.x];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        int off = 0, all = 0;
        uint64_t mine = 0;
#pragma unroll
        for (int v = 0; v < kWaves; ++v) {
            const uint64_t x = m[q * kWaves + v];
            const int c = __popcll(x);
            off += v < wave ? c : 0;
            all += c;
            mine = v == wave ? x : mine;
        }
        if ((mine >> lane) & 1) {
            const int64_t i = (int64_t)blockIdx.x * kUnwPer + q * kBlock + threadIdx.x;
            const int64_t pos = base + off + __popcll(mine & ((1ull << lane) - 1));
            keep[pos] = i;
            if (uw) uw[pos] = fmax(1.0, w[i] / w_max);
        }
        base += all;
    }
}

// ---------------------------------------------------------------------------
// Observables, cuts and weighted histograms of lab-frame events
// ---------------------------------------------------------------------------
struct ObsK {
    int32_t kind;   // MSX_OBS_* of msx.h
    uint32_t set;   // final-state particle labels
    int32_t rank;   // MSX_OBS_PT_RANK: 0 = hardest
    int32_t pad;
};
constexpr int kObsE = 0, kObsPt = 1, kObsEta = 2, kObsPhi = 3, kObsM = 4, kObsPtRank = 5, kObsDrHardest = 6;

__device__ __forceinline__ double pt_of(double px, double py) { return sqrt(px * px + py * py); }
__device__ __forceinline__ double eta_of(double px, double py, double pz) { return asinh(pz / pt_of(px, py)); }

// The kinds of a summed momentum.
__device__ __forceinline__ double of_sum(int kind, double E, double X, double Y, double Z) {
    switch (kind) {
        case kObsE: return E;
        case kObsPt: return pt_of(X, Y);
        case kObsEta: return eta_of(X, Y, Z);
        case kObsPhi: return atan2(Y, X);
        default: return sqrt(fmax(E * E - X * X - Y * Y - Z * Z, 0.0));
    }
}

struct ObsList {
    ObsK o[8];
    uint32_t need_e, need_xy, need_z;  // final-state particles whose components any observable reads
    uint32_t need_pt;                  // particles of the sets ordered by p_T
};

// One thread per event: the final-state components that the list needs go
// once into statically indexed registers (NF particles), their transverse
// momenta are formed once, and every observable is evaluated from there; the
// list and the sets are uniform, so a particle outside a set costs a scalar
// branch.  Read per observable (and per pair of particles for the ranks) from
// memory, three observables of 1e7 four-jet events took 1063 us; this way
// 383 us for 1.52 GB, 4.0 TB/s.
template <int NF>
__global__ __launch_bounds__(kBlock) void k_observables(const double* __restrict__ p, int64_t n, ObsList ol, int k,
                                                        double* __restrict__ out) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    constexpr int np = NF + 2;
    double FE[NF], FX[NF], FY[NF], FZ[NF], PT[NF];
#pragma unroll
    for (int i = 0; i < NF; ++i) {
        FE[i] = (ol.need_e >> i) & 1 ? p[((int64_t)0 * np + i + 2) * n + e] : 0.0;
        FX[i] = (ol.need_xy >> i) & 1 ? p[((int64_t)1 * np + i + 2) * n + e] : 0.0;
        FY[i] = (ol.need_xy >> i) & 1 ? p[((int64_t)2 * np + i + 2) * n + e] : 0.0;
        FZ[i] = (ol.need_z >> i) & 1 ? p[((int64_t)3 * np + i + 2) * n + e] : 0.0;
    }
#pragma unroll
    for (int i = 0; i < NF; ++i) PT[i] = (ol.need_pt >> i) & 1 ? pt_of(FX[i], FY[i]) : 0.0;
    for (int j = 0; j < k; ++j) {
        const uint32_t set = ol.o[j].set;
        const int kind = ol.o[j].kind;
        double v;
        if (kind == kObsPtRank) {
            // the rank-th largest by counting: p_T,i is the rank-th hardest when
            // exactly rank particles are harder (or as hard with a lower label)
            const int rank = ol.o[j].rank;
            v = 0.0;
#pragma unroll
            for (int i = 0; i < NF; ++i) {
                if (!((set >> i) & 1)) continue;
                int harder = 0;
#pragma unroll
                for (int q = 0; q < NF; ++q)
                    if (q != i && ((set >> q) & 1)) harder += (PT[q] > PT[i] || (PT[q] == PT[i] && q < i)) ? 1 : 0;
                v = harder == rank ? PT[i] : v;
            }
        } else if (kind == kObsDrHardest) {
            // the two hardest (p_T descending, lower label first on ties)
            double pa = -1.0, ax = 0.0, ay = 0.0, az = 0.0, pb = -1.0, bx = 0.0, by = 0.0, bz = 0.0;
#pragma unroll
            for (int i = 0; i < NF; ++i) {
                if (!((set >> i) & 1)) continue;
                if (PT[i] > pa) {
                    pb = pa;
                    bx = ax;
                    by = ay;
                    bz = az;
                    pa = PT[i];
                    ax = FX[i];
                    ay = FY[i];
                    az = FZ[i];
                } else if (PT[i] > pb) {
                    pb = PT[i];
                    bx = FX[i];
                    by = FY[i];
                    bz = FZ[i];
                }
            }
            v = 0.0;
            if (pa >= 0.0 && pb >= 0.0) {
                const double deta = asinh(az / pa) - asinh(bz / pb);
                double dphi = fabs(atan2(ay, ax) - atan2(by, bx));
                if (dphi > kPiD) dphi = 2.0 * kPiD - dphi;
                v = sqrt(deta * deta + dphi * dphi);
            }
        } else {
            double E = 0.0, X = 0.0, Y = 0.0, Z = 0.0;
#pragma unroll
            for (int i = 0; i < NF; ++i) {
                if (!((set >> i) & 1)) continue;
                E += FE[i];
                X += FX[i];
                Y += FY[i];
                Z += FZ[i];
            }
            v = of_sum(kind, E, X, Y, Z);
        }
        out[(int64_t)j * n + e] = v;
    }
}

// The same for a list without ordered kinds, every observable straight from
// memory, where the list reads no more particles than there are: the registers of
// all particles (131 to 193) then only cost waves.  5e6 events of eight particles,
// one p_T: 65 us through registers, 26 so (42 before); the mass of all 233 both
// ways; energy and mass of all, 16 reads, 247 and 391.
__global__ __launch_bounds__(kBlock) void k_observables_direct(const double* __restrict__ p, int np, int64_t n, ObsList ol,
                                                               int k, double* __restrict__ out) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    for (int j = 0; j < k; ++j) {
        const int kind = ol.o[j].kind;
        double E = 0.0, X = 0.0, Y = 0.0, Z = 0.0;
        // a loop per kind: the components of a particle are then in flight together
        auto each = [&](auto&& add) {
            for (uint32_t m = ol.o[j].set; m; m &= m - 1) {
                const double* at = p + (int64_t)(__builtin_ctz(m) + 2) * n + e;
                add([&](int c) { return at[(int64_t)c * np * n]; });
            }
        };
        switch (kind) {
            case kObsE: each([&](auto&& q) { E += q(0); }); break;
            case kObsPt:
            case kObsPhi:
                each([&](auto&& q) {
                    const double x = q(1), y = q(2);
                    X += x;
                    Y += y;
                });
                break;
            case kObsEta:
                each([&](auto&& q) {
                    const double x = q(1), y = q(2), z = q(3);
                    X += x;
                    Y += y;
                    Z += z;
                });
                break;
            default:
                each([&](auto&& q) {
                    const double t = q(0), x = q(1), y = q(2), z = q(3);
                    E += t;
                    X += x;
                    Y += y;
                    Z += z;
                });
        }
        out[(int64_t)j * n + e] = of_sum(kind, E, X, Y, Z);
    }
}

struct CutList {
    double lo[8], hi[8];
};

// w[e] = 0 unless lo_j <= x[j][e] < hi_j for every observable j.
__global__ __launch_bounds__(kBlock) void k_cut(const double* __restrict__ x, int k, int64_t n, CutList cl,
                                                double* __restrict__ w) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    bool pass = true;
    for (int j = 0; j < k; ++j) {
        const double v = x[(int64_t)j * n + e];
        pass = pass && v >= cl.lo[j] && v < cl.hi[j];
    }
    if (!pass) w[e] = 0.0;
}

// Weighted histogram, deterministic: bin = floor((x - lo) * scale), events
// with x outside [lo, hi) or w = 0 skipped (they add nothing).  A workgroup
// takes a contiguous run of events; each group of lanes of its waves keeps a
// private (sum w, sum w^2) histogram in LDS and a wave adds its events 64 at a
// time: one ballot per bit of the bin number gives every lane the lanes of its
// group that share its bin, and the lanes then add in rounds, the r-th lane of
// every bin in round r, so no two lanes of a round write one entry and an
// entry's terms come in event order.  The histograms are added in order into the
// workgroup's partial, part[entry][workgroup], and k_hist_reduce sums every
// entry over the workgroups in a fixed order.
//
// The cost per 64 events is the ballots plus a round per event of the
// fullest bin (a dozen for the p_T and mass spectra of pp -> 4 jets in 50
// bins).  Before, every thread scanned the 2048 staged events of a workgroup
// for each of its bins: 600 us for 1e7 events and 50 bins, and 103 us more to
// add 4883 partials in two workgroups; with one histogram a wave 62 us and 5,
// with four 50 (eight: 47 to 50).
constexpr int kHistPer = 2048;    // events per workgroup at least
constexpr int kHistBlocks = 2048; // workgroups at most
constexpr int kHistSmall = 512;   // up to this many bins four waves have histograms (32 KiB of LDS), else one
// Beyond this many bins a workgroup's LDS leaves room for five, and three waves
// more clear and write out the one wave's histogram (4096 bins, one event: 18 us
// with a wave alone, 12 so).  Below, they would take the place of workgroups (513
// bins, 1e7 events in one of them: 1134 us without them, 1309 with).
constexpr int kHistLarge = 1024;

// Histograms of a wave: groups of neighbouring lanes have one each, as long as
// 32 KiB hold them, which shortens the rounds to the fullest bin of a group.
int hist_groups(int nb) { return nb <= kHistSmall / 4 ? 4 : nb <= kHistSmall / 2 ? 2 : 1; }

__global__ __launch_bounds__(kBlock) void k_hist_block(const double* __restrict__ x, const double* __restrict__ w,
                                                       int64_t n, int64_t chunk, int nb, int bits, int waves,
                                                       int groups, double lo, double hi, double scale,
                                                       double* __restrict__ part) {
    extern __shared__ double hs[];  // [waves][groups][nb][2]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, step = 64 * waves;
    for (int i = threadIdx.x; i < waves * groups * nb * 2; i += blockDim.x) hs[i] = 0.0;
    __syncthreads();
    const int wide = 64 / groups, group = lane / wide;  // lanes of a group
    volatile double* mine = hs + (size_t)(wave * groups + group) * nb * 2;
    const uint64_t peers = (~uint64_t(0) >> (64 - wide)) << (group * wide);
    const int64_t e0 = blockIdx.x * chunk, e1 = min(n, e0 + chunk);
    const uint64_t below = (uint64_t(1) << lane) - 1;
    constexpr int kFlight = 4;
    // waves without a histogram only clear and write out
    for (int64_t e = wave < waves ? e0 + wave * 64 : e1; e < e1; e += (int64_t)step * kFlight) {
        double xv[kFlight], wv[kFlight];
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
            const int64_t i = e + (int64_t)u * step + lane;
            xv[u] = i < e1 ? x[i] : 0.0;
            wv[u] = i < e1 ? w[i] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
            const bool in = xv[u] >= lo && xv[u] < hi && wv[u] != 0.0;
            int b = 0;
            if (in) {
                b = (int)floor((xv[u] - lo) * scale);
                b = b < 0 ? 0 : (b > nb - 1 ? nb - 1 : b);
            }
            uint64_t left = __ballot(in);
            uint64_t same = left & peers;
            for (int q = 0; q < bits; ++q) {
                const bool bit = (b >> q) & 1;
                const uint64_t set = __ballot(bit);
                same &= bit ? set : ~set;
            }
            const int rank = __popcll(same & below);
            for (int r = 0; left; ++r) {
                const bool turn = in && rank == r;
                if (turn) {
                    const double v = wv[u];
                    mine[2 * b] = mine[2 * b] + v;
                    mine[2 * b + 1] = mine[2 * b + 1] + v * v;
                }
                left &= ~__ballot(turn);
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nb * 2; i += blockDim.x) {
        double a = hs[i];
        for (int v = 1; v < waves * groups; ++v) a += hs[(size_t)v * nb * 2 + i];
        part[(int64_t)i * gridDim.x + blockIdx.x] = a;
    }
}

// Entry (bin, q) of the partials summed over the nz workgroups by one wave:
// out[q nb + bin].
__global__ __launch_bounds__(64) void k_hist_reduce(const double* __restrict__ part, int nz, int nb,
                                                    double* __restrict__ out) {
    const double* src = part + (int64_t)blockIdx.x * nz;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    int z = threadIdx.x;
    for (; z + 192 < nz; z += 256) {
        a0 += src[z];
        a1 += src[z + 64];
        a2 += src[z + 128];
        a3 += src[z + 192];
    }
    for (; z < nz; z += 64) a0 += src[z];
    const double s = wave_sum((a0 + a1) + (a2 + a3));
    if (threadIdx.x == 0) out[(int)(blockIdx.x & 1) * nb + (int)(blockIdx.x >> 1)] = s;
}

// Global multichannel density: g += alpha / J of a launch's channels, in order
// (first: from zero).  A channel whose chain cuts the event (J = 0)
// contributes nothing.
__global__ __launch_bounds__(kBlock) void k_density_add(double* __restrict__ g, const double* __restrict__ jac,
                                                        DensityAlpha alpha, int n_chans, int64_t n, int first) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double sum = first ? 0.0 : g[i];
    for (int c = 0; c < n_chans; ++c) {
        const double j = jac[c * n + i];
        sum += j > 0.0 ? alpha.a[c] / j : 0.0;
    }
    g[i] = sum;
}

// Device copy of a call table made on the host: one workgroup, a word per
// thread; it also clears n_clear accumulators for a
// caller whose statistics start with the call.  A launch of this size costs 4
// us whatever it does; written by one thread the table took 5, and clearing
// the accumulators by a memset 4 to 8 more (one fill kernel or two).
constexpr int kSetThreads = 256;
__global__ __launch_bounds__(kSetThreads) void k_set_call(SampleRanges call, SampleCall* __restrict__ dev,
                                                          double* __restrict__ clear, int n_clear) {
    constexpr int kWords = sizeof(SampleRanges) / 8;
    static_assert(sizeof(SampleRanges) % 8 == 0 && kWords + kMaxChannels <= kSetThreads, "a word per thread");
    const int i = threadIdx.x;
    if (i < kWords)
        reinterpret_cast<uint64_t*>(static_cast<SampleRanges*>(dev))[i] = reinterpret_cast<const uint64_t*>(&call)[i];
    else if (i < kWords + kMaxChannels)
        dev->slices_done[i - kWords] = 0;
    for (int k = i; k < n_clear; k += kSetThreads) clear[k] = 0.0;
}

__global__ __launch_bounds__(kSetThreads) void k_clear(double* __restrict__ x, int n) {
    for (int k = threadIdx.x; k < n; k += kSetThreads) x[k] = 0.0;
}

// VEGAS histograms of a fused sample: entry i of the context's histogram
// array (channel c from the offsets, i - hist_off[c] within its [dims][nb]
// block) gets the sum over c's tiles of the tiles' partials.  A workgroup
// takes 64 consecutive entries, its 16 waves the tiles w, w + 16, ... with
// four loads in flight each, and the 64 sums of an entry are added in a fixed
// order.  The kernel is bound by the latency of its loads: with one thread
// per entry walking all 391 tiles of 1e5 events it took 93 us, this way 5.
// The workgroups after those of the histograms do the call's statistics, which
// saves their launch (4.6 us).
constexpr int kVegasWaves = 16;
template <bool SLICED>
__global__ __launch_bounds__(64 * kVegasWaves) void k_vegas_tiles(const SampleCall* __restrict__ call,
                                                                  uint32_t* __restrict__ done,
                                                                  const int64_t* __restrict__ hist_off,
                                                                  int64_t hist_total, int vstride,
                                                                  const double* __restrict__ vpart,
                                                                  double* __restrict__ hist, int hist_blocks,
                                                                  int slices, double* tile_stats,
                                                                  double* __restrict__ stats,
                                                                  uint64_t* __restrict__ advance) {
    if ((int)blockIdx.x >= hist_blocks) {
        __shared__ double stat_red[4][kWaves];
        const int i = (int)blockIdx.x - hist_blocks;
        if (advance && threadIdx.x == 0 && i == 0) *advance += (uint64_t)call->ev_start[call->n_chan];
        channel_stats<SLICED>(i / slices, i % slices, call, done, tile_stats, stats, stat_red);
        return;
    }
    __shared__ double red[kVegasWaves][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * 64 + lane;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    if (i < hist_total) {
        const int n_chan = call->n_chan;
        int c = 0;
        while (c + 1 < n_chan && hist_off[c + 1] <= i) ++c;
        const double* src = vpart + (i - hist_off[c]);
        const int64_t t1 = call->tile_start[c + 1];
        int64_t t = call->tile_start[c] + wave;
        for (; t + 3 * kVegasWaves < t1; t += 4 * kVegasWaves) {
            a0 += src[t * vstride];
            a1 += src[(t + kVegasWaves) * vstride];
            a2 += src[(t + 2 * kVegasWaves) * vstride];
            a3 += src[(t + 3 * kVegasWaves) * vstride];
        }
        for (; t < t1; t += kVegasWaves) a0 += src[t * vstride];
    }
    red[wave][lane] = (a0 + a1) + (a2 + a3);
    __syncthreads();
    if (wave == 0 && i < hist_total) {
        double acc = red[0][lane];
#pragma unroll
        for (int v = 1; v < kVegasWaves; ++v) acc += red[v][lane];
        hist[i] += acc;
    }
}

// Call table from device-resident counts: lane c of one wave has channel c, the
// starts are prefix sums over the lanes (one thread walking 24 channels took
// 5.4 us, mostly its divisions).  A negative count or more events than the
// buffers hold make an empty call.
__global__ __launch_bounds__(64) void k_plan(const int64_t* __restrict__ counts, int n_chan, int64_t capacity, int ept,
                                             SampleCall* __restrict__ dev, int32_t* __restrict__ status) {
    static_assert(kMaxChannels <= 64, "one lane per channel");
    const int c = threadIdx.x;
    const int64_t T = (int64_t)kBlock * ept;
    const int64_t own = c < n_chan ? counts[c] : 0;
    const bool refused = own < 0 || own > capacity;
    const int64_t k = refused ? 0 : own;
    // sums that stop at the largest count, which no capacity exceeds
    constexpr uint64_t kMost = (uint64_t)INT64_MAX;
    uint64_t ev = (uint64_t)k;
    const int64_t mine = k / T + (k % T != 0);
    int64_t tiles = mine;
    for (int step = 1; step < n_chan; step *= 2) {
        const uint64_t e = __shfl_up((unsigned long long)ev, step);
        const int64_t t = __shfl_up((long long)tiles, step);
        if (c >= step) {
            ev = ev + e < kMost ? ev + e : kMost;
            tiles += t;
        }
    }
    const bool bad = __any(refused || ev > (uint64_t)capacity);
    if (c < n_chan) {
        dev->ev_start[c] = bad ? 0 : (int64_t)ev - k;
        dev->tile_start[c] = bad ? 0 : tiles - mine;
        dev->slices_done[c] = 0;
    }
    if (c == n_chan - 1) {
        dev->ev_start[n_chan] = bad ? 0 : (int64_t)ev;
        dev->tile_start[n_chan] = bad ? 0 : tiles;
        dev->n_tiles = bad ? 0 : tiles;
        dev->n_chan = n_chan;
        dev->ept = ept;
        dev->skip_mask = 0;
        if (status) *status = bad;
    }
}

// VEGAS histogram, pass 1: block (chunk, k) accumulates sum w^2 per bin of
// dimension k over its contiguous event chunk; each thread keeps a private
// row in LDS (visited in event order), rows are then summed in thread order.
__global__ __launch_bounds__(128) void k_vegas_partial(int64_t n, int nb, const double* __restrict__ y,
                                                       const double* __restrict__ w, int64_t chunk,
                                                       double* __restrict__ part) {
    extern __shared__ double rows[];  // [blockDim][nb]
    const int k = blockIdx.y;
    const int64_t b = blockIdx.x;
    const int tid = threadIdx.x;
    double* mine = rows + (int64_t)tid * nb;
    for (int i = 0; i < nb; ++i) mine[i] = 0.0;
    const int64_t lo = b * chunk, hi = min(n, lo + chunk);
    for (int64_t e = lo + tid; e < hi; e += blockDim.x) {
        double t = y[(int64_t)k * n + e] * nb;
        int i = (int)t;
        i = i < 0 ? 0 : (i > nb - 1 ? nb - 1 : i);
        double wv = w[e];
        mine[i] += wv * wv;
    }
    __syncthreads();
    for (int i = tid; i < nb; i += blockDim.x) {
        double acc = 0.0;
        for (int q = 0; q < (int)blockDim.x; ++q) acc += rows[(int64_t)q * nb + i];
        part[((int64_t)k * gridDim.x + b) * nb + i] = acc;
    }
}

// Pass 2: hist[k][i] += sum over chunks in order.
__global__ void k_vegas_reduce(int dims, int nb, int64_t nchunk, const double* __restrict__ part,
                               double* __restrict__ hist) {
    int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= dims * nb) return;
    int k = idx / nb, i = idx % nb;
    double acc = 0.0;
    for (int64_t b = 0; b < nchunk; ++b) acc += part[((int64_t)k * nchunk + b) * nb + i];
    hist[(int64_t)k * nb + i] += acc;
}

// x summed over the bins in ascending order, as one thread would add them
// (every lane gets the sum); lane b holds bins b (x0) and b + 64 (x1).
// incl0 / incl1 receive the running sum up to the lane's own bins.
__device__ __forceinline__ double ordered_sum(double x0, double x1, int nb, int lane, double& incl0, double& incl1) {
    double s = 0.0;
    for (int i = 0; i < min(nb, 64); ++i) {
        s += __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x0), i),
                              __builtin_amdgcn_readlane(__double2loint(x0), i));
        if (lane == i) incl0 = s;
    }
    for (int i = 64; i < nb; ++i) {
        s += __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x1), i - 64),
                              __builtin_amdgcn_readlane(__double2loint(x1), i - 64));
        if (lane == i - 64) incl1 = s;
    }
    return s;
}

// Grid refinement, one wave per (channel, dimension): smoothing (1,6,1)/8
// with (7,1)/8 at the ends, normalisation, damping
// omega_i = ((1 - d_i)/ln(1/d_i))^alpha, then new edges holding equal shares
// of sum(omega), linear inside old bins.  The histogram is cleared.  The
// logarithms and powers run one bin per lane and every lane finds its own
// edges by bisection in the running sums; those are added in bin order, so
// the edges are the ones a single thread computes (which took 152 us for 16
// rows of 64 bins, nearly all of it waiting for its own arrays in scratch
// memory; one wave per row takes 9 us).
__global__ __launch_bounds__(64) void k_vegas_refine(const int32_t* __restrict__ row_nb,
                                                     const int64_t* __restrict__ row_grid,
                                                     const int64_t* __restrict__ row_hist, double alpha,
                                                     double* __restrict__ grids, double* __restrict__ hist) {
    __shared__ double d[kMaxBins], om[kMaxBins], incl[kMaxBins], old[kMaxBins + 1];
    const int r = blockIdx.x, lane = threadIdx.x;
    const int nb = row_nb[r];
    double* e = grids + row_grid[r];
    double* h = hist + row_hist[r];
    double own = 0.0;
    for (int i = lane; i < nb; i += 64) {
        d[i] = h[i];
        own += d[i];
        old[i] = e[i];
        h[i] = 0.0;
    }
    if (lane == 0) old[nb] = e[nb];
    const double tot = wave_sum(own);
    __syncthreads();
    if (!(tot > 0.0)) return;
    double sm[2] = {0.0, 0.0}, w[2] = {0.0, 0.0}, in[2] = {0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int i = lane + 64 * q;
        if (i < nb) {
            if (nb == 1) sm[q] = d[0];
            else if (i == 0) sm[q] = (7.0 * d[0] + d[1]) / 8.0;
            else if (i == nb - 1) sm[q] = (d[nb - 2] + 7.0 * d[nb - 1]) / 8.0;
            else sm[q] = (d[i - 1] + 6.0 * d[i] + d[i + 1]) / 8.0;
        }
    }
    const double ssum = ordered_sum(sm[0], sm[1], nb, lane, in[0], in[1]);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        if (lane + 64 * q < nb) {
            const double v = sm[q] / ssum;
            if (v <= 0.0) w[q] = 0.0;
            else if (v >= 1.0) w[q] = 1.0;
            else w[q] = pow((1.0 - v) / log(1.0 / v), alpha);
        }
    }
    const double total = ordered_sum(w[0], w[1], nb, lane, in[0], in[1]);
    if (!(total > 0.0)) return;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int i = lane + 64 * q;
        if (i < nb) {
            om[i] = w[q];
            incl[i] = in[q];
        }
    }
    __syncthreads();
    const double share = total / nb;
    for (int j = lane + 1; j < nb; j += 64) {
        const double target = j * share;
        // the first bin whose running sum reaches the target (the last bin
        // if none does)
        int lo = 0, hi = nb - 1;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (incl[mid] < target) lo = mid + 1;
            else hi = mid;
        }
        const double acc = lo > 0 ? incl[lo - 1] : 0.0;
        double frac = om[lo] > 0.0 ? (target - acc) / om[lo] : 0.0;
        frac = fmin(fmax(frac, 0.0), 1.0);
        e[j] = old[lo] + (old[lo + 1] - old[lo]) * frac;
    }
    if (lane == 0) {
        e[0] = 0.0;
        e[nb] = 1.0;
    }
}

// Register-file class of a launch: momentum slots (2 per operation) and
// invariants per event.
int reg_class(int slots, int inv) {
    if (slots <= 6 && inv <= 4) return 0;
    if (slots <= 10 && inv <= 8) return 1;
    return 2;
}

// Map-kind class of a launch: 0 integer-root power laws only, 1 plus
// Breit-Wigner, 2 every tree kind; when the tree kinds fit class 1, 3 with
// Chili channels, 4 with 1 -> 3 decays; 5 for anything else and for (s~, t)
// blocks.
int kind_class(int kinds) {
    if (kinds & KIND_ST) return 5;
    if (kinds & (KIND_CHILI | KIND_DEC3)) {
        if (kinds & ~(KIND_POW_INT | KIND_BW | KIND_CHILI | KIND_DEC3)) return 5;
        if ((kinds & KIND_CHILI) && (kinds & KIND_DEC3)) return 5;
        return (kinds & KIND_CHILI) ? 3 : 4;
    }
    if ((kinds & ~KIND_POW_INT) == 0) return 0;
    if ((kinds & ~(KIND_POW_INT | KIND_BW)) == 0) return 1;
    return 2;
}

int grid_for(int64_t n, int cap) {
    int64_t g = (n + kBlock - 1) / kBlock;
    if (g > cap) g = cap;
    return (int)std::max<int64_t>(g, 1);
}

// Register class -> the instantiation unit compiled for it.
hipError_t launch_chain(int rc, int kc, int mixed, const ChainLaunch& a) {
    if (a.inverse) {
        if (rc == 0) return launch_inverse_class<6, 4>(kc, a);
        if (rc == 1) return launch_inverse_class<10, 8>(kc, a);
        return launch_inverse_class<14, 8>(kc, a);
    }
    if (mixed) {
        if (rc == 0) return launch_chain_class<6, 4, true>(kc, a);
        if (rc == 1) return launch_chain_class<10, 8, true>(kc, a);
        return launch_chain_class<14, 8, true>(kc, a);
    }
    if (rc == 0) return launch_chain_class<6, 4, false>(kc, a);
    if (rc == 1) return launch_chain_class<10, 8, false>(kc, a);
    return launch_chain_class<14, 8, false>(kc, a);
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

hipError_t launch_observables(const double* p, int np, int64_t n, const int32_t* spec, int k, double* out,
                              hipStream_t s) {
    if (n == 0) return hipSuccess;
    ObsList ol{};
    int reads = 0;  // particles of all sets
    for (int j = 0; j < k; ++j) {
        ol.o[j].kind = spec[4 * j];
        ol.o[j].set = (uint32_t)spec[4 * j + 1];
        ol.o[j].rank = spec[4 * j + 2];
        const int kind = ol.o[j].kind;
        const uint32_t set = ol.o[j].set;
        const bool ordered = kind == kObsPtRank || kind == kObsDrHardest;
        if (kind == kObsE || kind == kObsM) ol.need_e |= set;
        if (kind != kObsE) ol.need_xy |= set;
        if (kind == kObsEta || kind == kObsM || kind == kObsDrHardest) ol.need_z |= set;
        if (ordered) ol.need_pt |= set;
        reads += __builtin_popcount(set);
    }
    const dim3 b((unsigned)((n + kBlock - 1) / kBlock)), t(kBlock);
    static_assert(kMaxFinal == 8, "one instantiation per particle count");
    if (!ol.need_pt && reads <= np - 2) {
        k_observables_direct<<<b, t, 0, s>>>(p, np, n, ol, k, out);
        return hipGetLastError();
    }
    switch (np - 2) {
        case 2: k_observables<2><<<b, t, 0, s>>>(p, n, ol, k, out); break;
        case 3: k_observables<3><<<b, t, 0, s>>>(p, n, ol, k, out); break;
        case 4: k_observables<4><<<b, t, 0, s>>>(p, n, ol, k, out); break;
        case 5: k_observables<5><<<b, t, 0, s>>>(p, n, ol, k, out); break;
        case 6: k_observables<6><<<b, t, 0, s>>>(p, n, ol, k, out); break;
        case 7: k_observables<7><<<b, t, 0, s>>>(p, n, ol, k, out); break;
        case 8: k_observables<8><<<b, t, 0, s>>>(p, n, ol, k, out); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_cut(const double* x, int k, int64_t n, const double* lo, const double* hi, double* w, hipStream_t s) {
    if (n == 0) return hipSuccess;
    CutList cl{};
    for (int j = 0; j < k; ++j) {
        cl.lo[j] = lo[j];
        cl.hi[j] = hi[j];
    }
    const int64_t b = (n + kBlock - 1) / kBlock;
    k_cut<<<dim3((unsigned)b), dim3(kBlock), 0, s>>>(x, k, n, cl, w);
    return hipGetLastError();
}

int64_t histogram_blocks(int64_t n) {
    return std::max<int64_t>(1, std::min<int64_t>(kHistBlocks, (n + kHistPer - 1) / kHistPer));
}

hipError_t launch_histogram(const double* x, const double* w, int64_t n, int nb, double lo, double hi, double* part,
                            double* out, hipStream_t s) {
    const int64_t nz = histogram_blocks(n);
    const double scale = nb / (hi - lo);
    int bits = 0;
    while ((1 << bits) < nb) ++bits;
    const int waves = nb <= kHistSmall ? kWaves : 1, groups = hist_groups(nb);
    const size_t lds = sizeof(double) * 2 * (size_t)nb * waves * groups;
    const int threads = nb <= kHistLarge ? 64 * waves : kBlock;
    k_hist_block<<<dim3((unsigned)nz), dim3(threads), lds, s>>>(x, w, n, (n + nz - 1) / nz, nb, bits, waves, groups, lo, hi,
                                                                scale, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_hist_reduce<<<dim3((unsigned)(2 * nb)), dim3(64), 0, s>>>(part, (int)nz, nb, out);
    return hipGetLastError();
}

static int64_t unweight_blocks(int64_t n) { return (n + kUnwPer - 1) / kUnwPer; }
int64_t unweight_words(int64_t n) { return unweight_blocks(n) * (1 + kUnwMasks); }

hipError_t launch_unweight(const double* w, int64_t n, double w_max, uint64_t seed, uint64_t sid, uint64_t e0,
                           int64_t* blk, int64_t* keep, double* uw, int64_t* count, hipStream_t s) {
    const int64_t nb = unweight_blocks(n);
    if (nb == 0) {
        k_unw_scan<<<1, 1024, 0, s>>>(blk, 0, count);
        return hipGetLastError();
    }
    uint64_t* masks = (uint64_t*)(blk + nb);
    k_unw_count<<<dim3((unsigned)nb), dim3(kBlock), 0, s>>>(w, n, w_max, seed, sid, e0, blk, masks);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_unw_scan<<<1, 1024, 0, s>>>(blk, nb, count);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    k_unw_write<<<dim3((unsigned)nb), dim3(kBlock), 0, s>>>(w, w_max, blk, masks, keep, uw);
    return hipGetLastError();
}

hipError_t launch_density_add(double* g, const double* jac, const DensityAlpha& alpha, int n_chans, int64_t n, bool first,
                              hipStream_t s) {
    if (n == 0) return hipSuccess;
    const int64_t b = (n + kBlock - 1) / kBlock;
    k_density_add<<<dim3((unsigned)b), dim3(kBlock), 0, s>>>(g, jac, alpha, n_chans, n, first ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_uniform(uint64_t seed, uint64_t sid, uint64_t e0, int64_t n, int d, double* y, hipStream_t s) {
    if (n == 0) return hipSuccess;
    int64_t g = (n + kBlock - 1) / kBlock;
    k_uniform<<<dim3((unsigned)g), dim3(kBlock), 0, s>>>(seed, sid, e0, n, d, y);
    return hipGetLastError();
}

hipError_t launch_map(const LaunchChans& chans, const ProcessTab* pt, int dims, int nb, int n_slots, int n_inv, int kinds,
                      int mixed, double s_lab, int np, int64_t n, const double* y, double* p, double* x1x2, double* jac,
                      double* w, int cu_count, hipStream_t s) {
    if (n == 0) return hipSuccess;
    ChainLaunch a{};
    a.sample = false;
    a.lds = sizeof(double) * (size_t)dims * (nb + 1);
    a.grid = grid_for(n, cu_count * 8);
    a.stream = s;
    a.pts = pt;
    a.chans = chans;
    a.n_chans = 1;
    a.s_lab = s_lab;
    a.np = np;
    a.n = n;
    a.y = y;
    a.p = p;
    a.x1x2 = x1x2;
    a.jac = jac;
    a.w = w;
    return launch_chain(reg_class(n_slots, n_inv), kind_class(kinds), mixed, a);
}

bool same_chain_class(int n_slots_a, int n_inv_a, int kinds_a, int n_slots_b, int n_inv_b, int kinds_b) {
    return reg_class(n_slots_a, n_inv_a) == reg_class(n_slots_b, n_inv_b) && kind_class(kinds_a) == kind_class(kinds_b);
}

hipError_t launch_inverse(const LaunchChans& chans, int n_chans, int dims, int nb, int n_slots, int n_inv, int kinds,
                          double s_lab, int np, int64_t n, const double* p, const double* x1x2, double* y, double* jac,
                          int cu_count, hipStream_t s) {
    if (n == 0) return hipSuccess;
    ChainLaunch a{};
    a.inverse = true;
    a.lds = sizeof(double) * (size_t)dims * (nb + 1);
    a.grid = grid_for(n, cu_count * 8);
    a.stream = s;
    a.chans = chans;
    a.n_chans = n_chans;
    a.s_lab = s_lab;
    a.np = np;
    a.n = n;
    a.p_in = p;
    a.x1x2_in = x1x2;
    a.y_out = y;
    // always the FP64 units
    hipError_t err = launch_chain(reg_class(n_slots, n_inv), kind_class(kinds), 0, a);
    if (err != hipSuccess || !jac) return err;
    // the forward Jacobians at y: the map kernel without momentum stores
    ChainLaunch m{};
    m.lds = a.lds;
    m.grid = a.grid;
    m.stream = s;
    m.chans = chans;
    m.n_chans = n_chans;
    m.s_lab = s_lab;
    m.np = np;
    m.n = n;
    m.y = y;
    m.jac = jac;
    return launch_chain(reg_class(n_slots, n_inv), kind_class(kinds), 0, m);
}

hipError_t launch_weight(const ChannelTab* ct, const ProcessTab* pt, int mixed, int np, int64_t n, const double* p,
                         const double* x1x2, const double* jac, double* w, double* alpha, hipStream_t s) {
    if (n == 0) return hipSuccess;
    int64_t g = (n + kBlock - 1) / kBlock;
    if (mixed)
        k_weight<true><<<dim3((unsigned)g), dim3(kBlock), 0, s>>>(ct, pt, np, n, p, x1x2, jac, w, alpha);
    else
        k_weight<false><<<dim3((unsigned)g), dim3(kBlock), 0, s>>>(ct, pt, np, n, p, x1x2, jac, w, alpha);
    return hipGetLastError();
}

hipError_t launch_sample(const ChannelTab* cts, const ProcessTab* pts, const double* grids, const int64_t* grid_off,
                         const int32_t* chan_nb, SampleCall* call, int n_chan, int max_slots, int max_inv,
                         int kinds, int mixed, size_t lds_bytes, uint64_t seed, uint64_t sid, const uint64_t* ctr_dev,
                         uint64_t ctr_off, int np, int64_t ld, double* p, double* x1x2, double* w, int32_t* chan,
                         double* tile_stats, int64_t max_tiles, double* stats, int grid, hipStream_t s,
                         double* vpart, int vstride, const int64_t* hist_off, int64_t hist_total, double* hist,
                         const JitSampleSet* jit, uint64_t* advance) {
    if (jit && jit->n > 0) {
        int grid_doubles = (int)(lds_bytes / sizeof(double));
        void* args[] = {&cts, &pts, &grids, &grid_off, &chan_nb, &call, &seed, &sid, &ctr_dev, &ctr_off, &np, &ld,
                        &p, &x1x2, &w, &chan, &tile_stats, &grid_doubles, &vpart, &vstride};
        for (int g = 0; g < jit->n; ++g) {
            const size_t lds =
                lds_bytes + sizeof(double) * (size_t)jit->k[g].rows * kBlock + (vpart ? vegas_acc_lds(vstride) : 0);
            hipError_t err = hipModuleLaunchKernel(jit->k[g].fn, (unsigned)std::max(grid, 1), 1, 1, kBlock, 1, 1,
                                                   (unsigned)lds, s, args, nullptr);
            if (err != hipSuccess) return err;
        }
    } else {
        ChainLaunch a{};
        a.sample = true;
        a.lds = lds_bytes;
        a.grid = std::max(grid, 1);
        a.stream = s;
        a.cts = cts;
        a.pts = pts;
        a.grids = grids;
        a.grid_off = grid_off;
        a.chan_nb = chan_nb;
        a.call = call;
        a.seed = seed;
        a.sid = sid;
        a.ctr_dev = ctr_dev;
        a.ctr_off = ctr_off;
        a.np = np;
        a.n = ld;
        a.p = p;
        a.x1x2 = x1x2;
        a.w = w;
        a.chan = chan;
        a.tile_stats = tile_stats;
        a.vpart = vpart;
        a.vstride = vstride;
        hipError_t err = launch_chain(reg_class(max_slots, max_inv), kind_class(kinds), mixed, a);
        if (err != hipSuccess) return err;
    }
    const bool sliced = max_tiles > kStatTiles;
    const int slices = sliced ? kStatSlices : 1;
    if (vpart && hist_total > 0) {
        const int64_t g = (hist_total + 63) / 64;
        (sliced ? k_vegas_tiles<true> : k_vegas_tiles<false>)<<<dim3((unsigned)(g + (int64_t)n_chan * slices)),
                                                                dim3(64 * kVegasWaves), 0, s>>>(
            call, call->slices_done, hist_off, hist_total, vstride, vpart, hist, (int)g, slices, tile_stats, stats, advance);
    } else {
        (sliced ? k_stats_final<true> : k_stats_final<false>)<<<dim3((unsigned)slices, (unsigned)n_chan), kBlock, 0, s>>>(
            call, call->slices_done, tile_stats, stats, advance);
    }
    return hipGetLastError();
}

namespace {
// rows of the sample kernel's per-thread staging column (stage_rows of the
// chain kernels)
int stage_rows_host(int ns, int ni) { return (ns + ni + 1) > kQRows ? (ns + ni + 1) : kQRows; }
}  // namespace

size_t sample_lds_bytes(int max_slots, int max_inv, size_t lds_bytes, int vstride) {
    const int rc = reg_class(max_slots, max_inv);
    const int rows = rc == 0 ? stage_rows_host(6, 4) : (rc == 1 ? stage_rows_host(10, 8) : stage_rows_host(14, 8));
    return lds_bytes + sizeof(double) * (size_t)rows * kBlock + (vstride > 0 ? vegas_acc_lds(vstride) : 0);
}

hipError_t launch_set_call(const SampleRanges& host, SampleCall* dev, double* clear, int n_clear, hipStream_t s) {
    k_set_call<<<1, kSetThreads, 0, s>>>(host, dev, clear, clear ? n_clear : 0);
    return hipGetLastError();
}

hipError_t launch_clear(double* x, int n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    k_clear<<<1, kSetThreads, 0, s>>>(x, n);
    return hipGetLastError();
}

hipError_t launch_plan(const int64_t* counts, int n_chan, int64_t capacity, int ept, SampleCall* dev,
                       int32_t* status, hipStream_t s) {
    k_plan<<<1, 64, 0, s>>>(counts, n_chan, capacity, ept, dev, status);
    return hipGetLastError();
}

int sample_block() { return kBlock; }

// ---------------------------------------------------------------------------
// Fixed device scratch of the allocation-free sample entry point: the tile
// statistics of one launch (4 doubles per tile).  Each GPU that runs the
// library holds one copy for the life of the process; its device address is
// looked up once per device (hipGetSymbolAddress) and used from then on --
// the array's name in host code is only a host-side stand-in.
// ---------------------------------------------------------------------------
static __device__ __align__(256) double scratch[4 * kNoAllocTiles];

namespace {
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxScratchDevices] = {};
}  // namespace

hipError_t noalloc_scratch(int device, double** out) {
    *out = nullptr;
    if (device < 0 || device >= kMaxScratchDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        int cur = -1;
        hipError_t e = hipGetDevice(&cur);
        if (e != hipSuccess) return e;
        if (cur != device && (e = hipSetDevice(device)) != hipSuccess) return e;
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (cur != device) (void)hipSetDevice(cur);
        if (e != hipSuccess) return e;
        g_scratch_ptr[device] = ptr;
    }
    *out = (double*)g_scratch_ptr[device];
    return hipSuccess;
}

hipError_t launch_vegas_accumulate(int64_t n, int dims, int nb, const double* y, const double* w, double* part,
                                   int64_t nchunk, int64_t chunk, double* hist, hipStream_t s) {
    if (n == 0) return hipSuccess;
    // one private LDS row per thread, 64 KiB at most
    int threads = nb <= 64 ? 128 : 64;
    size_t lds = sizeof(double) * threads * (size_t)nb;
    k_vegas_partial<<<dim3((unsigned)nchunk, (unsigned)dims), dim3(threads), lds, s>>>(n, nb, y, w, chunk, part);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    int tot = dims * nb;
    k_vegas_reduce<<<(tot + 127) / 128, 128, 0, s>>>(dims, nb, nchunk, part, hist);
    return hipGetLastError();
}

hipError_t launch_vegas_refine(int n_rows, const int32_t* row_nb, const int64_t* row_grid, const int64_t* row_hist,
                               double alpha, double* grids, double* hist, hipStream_t s) {
    if (n_rows == 0) return hipSuccess;
    k_vegas_refine<<<n_rows, 64, 0, s>>>(row_nb, row_grid, row_hist, alpha, grids, hist);
    return hipGetLastError();
}

}  // namespace msx

// ---------------------------------------------------------------------------
// Unweighting efficiency: bucket histograms over the IEEE bit pattern, which
// orders non-negative doubles like their values.
// ---------------------------------------------------------------------------
namespace msx {
namespace {

constexpr int kUnwBuckets = 4096;
static_assert(kUnwBuckets == kUnwMaxBuckets, "bucket count");

// Counts and sums of the weights per bucket, with integer atomics only, so
// the result does not depend on the order of the additions: every weight of
// a bucket has the bucket's binary exponent (the buckets of every pass lie
// within one exponent), so its value is m 2^(e - 1075) with the integer
// significand m < 2^53, and the bucket sum is kept exactly as the sums of
// m's upper 27 and lower 26 bits (each < 2^63 for n < 2^36 weights).  In LDS
// the count rides in the upper sum's word, above bit 45 (a workgroup sees at
// most 2^17 weights, so that sum stays below 2^44).
//
// Eight weights are in flight per thread: with one the pass over 1e7 weights
// took 38 us (2.1 TB/s), bound by the latency of its loads.
constexpr int kUnwThreads = 512, kUnwFlight = 8;
constexpr int64_t kUnwPerBlock = 1 << 17;
__global__ __launch_bounds__(kUnwThreads) void k_unw_hist(int64_t n, int64_t chunk, const double* __restrict__ w,
                                                          int shift, int width, const UnwState* __restrict__ st,
                                                          int first, unsigned long long* __restrict__ counts,
                                                          unsigned long long* __restrict__ sum_hi,
                                                          unsigned long long* __restrict__ sum_lo) {
    const uint64_t prefix = st->prefix;
    __shared__ unsigned long long h_l[kUnwBuckets];
    __shared__ unsigned long long l_l[kUnwBuckets];
    const int nbk = 1 << width;
    for (int i = threadIdx.x; i < nbk; i += kUnwThreads) {
        h_l[i] = 0ull;
        l_l[i] = 0ull;
    }
    __syncthreads();
    const int64_t e0 = blockIdx.x * chunk, e1 = min(n, e0 + chunk);
    for (int64_t e = e0 + threadIdx.x; e < e1; e += kUnwThreads * kUnwFlight) {
        double v[kUnwFlight];
#pragma unroll
        for (int u = 0; u < kUnwFlight; ++u) {
            const int64_t i = e + u * kUnwThreads;
            v[u] = i < e1 ? w[i] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < kUnwFlight; ++u) {
            if (!(v[u] > 0.0)) continue;  // zero weights carry no excess
            const uint64_t bits = (uint64_t)__double_as_longlong(v[u]);
            if (!first && (bits >> (shift + width)) != prefix) continue;
            const int b = (int)((bits >> shift) & (uint64_t)(nbk - 1));
            const uint64_t ex = bits >> 52;
            const uint64_t m = (bits & ((1ull << 52) - 1)) | (ex ? (1ull << 52) : 0ull);
            atomicAdd(&h_l[b], (unsigned long long)((m >> 26) | (1ull << 45)));
            atomicAdd(&l_l[b], (unsigned long long)(m & ((1ull << 26) - 1)));
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nbk; i += kUnwThreads) {
        const unsigned long long h = h_l[i];
        if (h) {
            atomicAdd(&counts[i], h >> 45);
            atomicAdd(&sum_hi[i], h & ((1ull << 45) - 1));
            atomicAdd(&sum_lo[i], l_l[i]);
        }
    }
}

constexpr int kUnwScanWaves = 16;

// Running sums of S and N over the workgroup's threads (inclusive), in a
// fixed order.
__device__ __forceinline__ void scan_pairs(double& S, double& N, double (&red)[2][kUnwScanWaves]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double s = __shfl_up(S, o, 64), c = __shfl_up(N, o, 64);
        if (lane >= o) {
            S += s;
            N += c;
        }
    }
    if (lane == 63) {
        red[0][wave] = S;
        red[1][wave] = N;
    }
    __syncthreads();
    for (int v = 0; v < wave; ++v) {
        S += red[0][v];
        N += red[1][v];
    }
}

// The crossing bucket of one pass: the excess at the lower edge L_b of bucket
// b, S - L_b N over the weights in buckets >= b and above the earlier passes'
// crossing buckets, reaches the target first, from the top bucket down, at
// the crossing bucket; st gets the extended prefix and the sums above it.
// Every thread converts and sums a run of four buckets, the runs' sums are
// scanned over the workgroup, and each thread then looks for the crossing in
// its own run (a single thread walking the 4096 buckets took 155 us a pass,
// this way 10).  The bucket arrays are cleared for the next pass.
__global__ __launch_bounds__(64 * kUnwScanWaves) void k_unw_search(int shift, int width, double overweight,
                                                    const double* __restrict__ tot, UnwState* __restrict__ st,
                                                    unsigned long long* __restrict__ counts,
                                                    unsigned long long* __restrict__ sum_hi,
                                                    unsigned long long* __restrict__ sum_lo) {
    constexpr int kRun = kUnwBuckets / (64 * kUnwScanWaves);
    __shared__ double red[2][kUnwScanWaves];
    __shared__ int first;
    const int nbk = 1 << width;
    const uint64_t prefix = st->prefix;
    const double S_up = st->S_up, N_up = st->N_up;
    const double target = overweight * tot[0];
    if (threadIdx.x == 0) first = kUnwBuckets;
    // position q = 0, 1, ... from the top bucket down: bucket nbk - 1 - q
    const int q0 = threadIdx.x * kRun;
    double sv[kRun], nv[kRun], S = 0.0, N = 0.0;
#pragma unroll
    for (int u = 0; u < kRun; ++u) {
        const int b = nbk - 1 - (q0 + u);
        sv[u] = nv[u] = 0.0;
        if (b >= 0) {
            // the bucket's significand sum times 2^(e - 1075), e its biased
            // exponent (1 - 1075 for subnormals)
            const uint64_t lb_bits = ((prefix << width) | (uint64_t)b) << shift;
            const int ex = (int)(lb_bits >> 52);
            sv[u] = ldexp((double)sum_hi[b] * 67108864.0 + (double)sum_lo[b], (ex ? ex : 1) - 1075);
            nv[u] = (double)counts[b];
            counts[b] = 0ull;
            sum_hi[b] = 0ull;
            sum_lo[b] = 0ull;
        }
        S += sv[u];
        N += nv[u];
    }
    double Si = S, Ni = N;
    scan_pairs(Si, Ni, red);
    // the sums above this thread's run: the runs before it, added up the same
    // way on every thread
    double Sa = __shfl_up(Si, 1, 64), Na = __shfl_up(Ni, 1, 64);
    if ((threadIdx.x & 63) == 0) {
        Sa = Na = 0.0;
        for (int v = 0; v < (int)(threadIdx.x >> 6); ++v) {
            Sa += red[0][v];
            Na += red[1][v];
        }
    }
    Sa += S_up;
    Na += N_up;
    int found = kUnwBuckets;
    double S_above = 0.0, N_above = 0.0;
#pragma unroll
    for (int u = 0; u < kRun; ++u) {
        const int b = nbk - 1 - (q0 + u);
        if (b >= 0 && found == kUnwBuckets) {
            const uint64_t lb_bits = ((prefix << width) | (uint64_t)b) << shift;
            const double Sn = Sa + sv[u], Nn = Na + nv[u];
            // the last bucket stands in when none crosses: W then lies below
            // every positive weight
            if (Sn - __longlong_as_double((long long)lb_bits) * Nn >= target || b == 0) {
                found = q0 + u;
                S_above = Sa;
                N_above = Na;
            }
            Sa = Sn;
            Na = Nn;
        }
    }
    __syncthreads();
    if (found < kUnwBuckets) atomicMin(&first, found);
    __syncthreads();
    if (found == first && found < kUnwBuckets) {
        st->S_up = S_above;
        st->N_up = N_above;
        st->prefix = (prefix << width) | (uint64_t)(nbk - 1 - found);
    }
}

__global__ __launch_bounds__(256) void k_sum_max(int64_t n, const double* __restrict__ w, double* __restrict__ part) {
    double s = 0.0, m = 0.0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride) {
        double v = w[e];
        s += v;
        m = fmax(m, v);
    }
    __shared__ double rs[4], rm[4];
    double ws = wave_sum(s), wm = wave_max(m);
    if ((threadIdx.x & 63) == 0) {
        rs[threadIdx.x >> 6] = ws;
        rm[threadIdx.x >> 6] = wm;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = rs[0], b = rm[0];
        for (int i = 1; i < 4; ++i) {
            a += rs[i];
            b = fmax(b, rm[i]);
        }
        part[2 * blockIdx.x] = a;
        part[2 * blockIdx.x + 1] = b;
    }
}

__global__ __launch_bounds__(256) void k_sum_max_final(int nblk, const double* __restrict__ part,
                                                       double* __restrict__ out) {
    double a = 0.0, b = 0.0;
    for (int i = threadIdx.x; i < nblk; i += 256) {
        a += part[2 * i];
        b = fmax(b, part[2 * i + 1]);
    }
    __shared__ double rs[4], rm[4];
    const double ws = wave_sum(a), wm = wave_max(b);
    if ((threadIdx.x & 63) == 0) {
        rs[threadIdx.x >> 6] = ws;
        rm[threadIdx.x >> 6] = wm;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        out[0] = ((rs[0] + rs[1]) + rs[2]) + rs[3];
        out[1] = fmax(fmax(rm[0], rm[1]), fmax(rm[2], rm[3]));
    }
}

// Moments of a weight array: block b reduces its grid-stride share into
// part[b] = (sum w, sum w^2, n(w == 0), max w); the final pass sums blocks in
// order and adds to out = (sum w, sum w^2, n, n(w == 0), max w).
constexpr int kMomBlocks = 256;
__global__ __launch_bounds__(256) void k_moments(int64_t n, const double* __restrict__ w, double* __restrict__ part) {
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride) {
        const double v = w[e];
        a[0] += v;
        a[1] += v * v;
        a[2] += v == 0.0 ? 1.0 : 0.0;
        a[3] = fmax(a[3], v);
    }
    __shared__ double r[4][4];
    const double r0 = wave_sum(a[0]), r1 = wave_sum(a[1]), r2 = wave_sum(a[2]), r3 = wave_max(a[3]);
    if ((threadIdx.x & 63) == 0) {
        r[0][threadIdx.x >> 6] = r0;
        r[1][threadIdx.x >> 6] = r1;
        r[2][threadIdx.x >> 6] = r2;
        r[3][threadIdx.x >> 6] = r3;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const int q = threadIdx.x;
        double acc = r[q][0];
        for (int v = 1; v < 4; ++v) acc = q == 3 ? fmax(acc, r[q][v]) : acc + r[q][v];
        part[4 * blockIdx.x + q] = acc;
    }
}

__global__ void k_moments_final(int nblk, int64_t n, const double* __restrict__ part, double* __restrict__ out) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    double a = 0.0, b = 0.0, z = 0.0, m = 0.0;
    for (int i = 0; i < nblk; ++i) {
        a += part[4 * i];
        b += part[4 * i + 1];
        z += part[4 * i + 2];
        m = fmax(m, part[4 * i + 3]);
    }
    out[0] += a;
    out[1] += b;
    out[2] += (double)n;
    out[3] += z;
    out[4] = fmax(out[4], m);
}

__global__ void k_fill_i32(int32_t* __restrict__ x, int64_t n, int32_t v) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) x[i] = v;
}

}  // namespace

int64_t moments_blocks() { return kMomBlocks; }

hipError_t launch_moments_add(const double* w, int64_t n, double* part, double* out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int g = (int)std::min<int64_t>(kMomBlocks, (n + 255) / 256);
    k_moments<<<g, 256, 0, s>>>(n, w, part);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    k_moments_final<<<1, 64, 0, s>>>(g, n, part, out);
    return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t* x, int64_t n, int32_t v, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int g = (int)std::min<int64_t>(4096, (n + 255) / 256);
    k_fill_i32<<<g, 256, 0, s>>>(x, n, v);
    return hipGetLastError();
}

hipError_t launch_unw_search(int64_t n, const double* w, double overweight, const double* tot, UnwState* st,
                             uint64_t* counts, uint64_t* sum_hi, uint64_t* sum_lo, int cu_count, hipStream_t s) {
    // passes over the 63 value bits of non-negative doubles: buckets of 12
    // bits, the last pass 3
    const int shifts[6] = {51, 39, 27, 15, 3, 0};
    const int widths[6] = {12, 12, 12, 12, 12, 3};
    // contiguous chunks of at most kUnwPerBlock weights; two workgroups fill a
    // compute unit's LDS
    const int64_t g = std::max<int64_t>((n + kUnwPerBlock - 1) / kUnwPerBlock,
                                        std::min<int64_t>(2 * cu_count, (n + kUnwThreads - 1) / kUnwThreads));
    const int64_t chunk = (n + g - 1) / g;
    for (int pass = 0; pass < 6; ++pass) {
        k_unw_hist<<<(unsigned)g, kUnwThreads, 0, s>>>(n, chunk, w, shifts[pass], widths[pass], st, pass == 0, (unsigned long long*)counts,
                                     (unsigned long long*)sum_hi, (unsigned long long*)sum_lo);
        k_unw_search<<<1, 64 * kUnwScanWaves, 0, s>>>(shifts[pass], widths[pass], overweight, tot, st, (unsigned long long*)counts,
                                       (unsigned long long*)sum_hi, (unsigned long long*)sum_lo);
    }
    return hipGetLastError();
}

hipError_t launch_sum_max(int64_t n, const double* w, double* out, double* part, int nblk, hipStream_t s) {
    k_sum_max<<<nblk, 256, 0, s>>>(n, w, part);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    k_sum_max_final<<<1, 256, 0, s>>>(nblk, part, out);
    return hipGetLastError();
}

}  // namespace msx
