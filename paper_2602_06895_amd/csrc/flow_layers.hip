// Fused coupling layers of the flow on gfx950: conditioner on the matrix
// cores and spline in one kernel, for all layers of a pass.
#include <algorithm>

#include "flow_layers.h"

namespace msx {

namespace {

using namespace flow;

// LDS of a workgroup with tiles of EV = 16 NT events: the output layer's
// weights of `kept` coordinates, two activation tiles, two tiles of the
// conditioning inputs and of the d coordinates, the log-determinant terms of
// a tile.
template <int NT, class T>
constexpr size_t layers_lds(int d, int kept) {
    return sizeof(T) * ((size_t)kept * kOutElems + 2 * 16 * NT * (kHid + kCond)) +
           sizeof(float) * 16 * NT * (2 * (size_t)d + kWaves);
}

// All coupling layers of a pass, forward (sampling) or inverse (densities,
// and the first half of training).  Workgroup b owns tiles b, b + grid, ...
// of every layer and runs the layers one after the other over them, so the
// events never meet another workgroup and one launch does the whole flow;
// between layers z stays in memory (it comes back from the cache), within a
// layer the weights stay on chip: the hidden layers' in registers, the output
// layer's in LDS (KEEP: up to eight transformed coordinates).  A tile's
// coordinates are in flight a tile earlier, its running log-determinant from
// its start.
//
// What bounds it: per 64 events and layer each of the two waves of a SIMD
// issues 786 vector instructions, most of them in the splines (32
// exponentials, sums and knots per event and coordinate), 100 of them MFMAs, a
// quarter of those for the padding of 49 parameters to 64 rows; the vector
// units are busy 58% of the time, the matrix units 26%, and what is left is
// the latency of the three barriers and the LDS reads behind them.  Before, a
// wave read every weight of a layer from L2 for its own 64 events and walked
// each spline through LDS: 4583 us for eight layers of 2^20 events of 16
// dimensions, now 2580 us.  (Tried
// and slower: the output weights in registers, 2850 us; two workgroups of
// four waves per compute unit, 4240 us, and the splines of a tile interleaved
// with the next tile's hidden layers, 2840 us, which both spill.)
//
// FP32 conditioners are bound by the FP32 matrix instructions (16 of them for
// one in BF16): 4,097 events of 16 dimensions, inverse, 8 layers: 24 us each,
// of which 11 are products; they were 130 us as seven kernels.
template <bool INV, int NT, bool KEEP, int BINS, class T>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_flow_layers(FlowNet fn,
                                                                                                 FlowRun run) {
    constexpr int EV = 16 * NT;
    constexpr int ZR = 2;  // coordinates in flight per thread (all of a tile of 64 events up to 16 dimensions)
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int nh = fn.nh, d = 2 * nh, K = fn.K;
    T* const w4 = (T*)smem;                   // KEEP: [nh][kOutElems]
    T* const act = w4 + (KEEP ? nh * kOutElems : 0);  // [2][EV][kHid]
    T* const cond = act + 2 * EV * kHid;           // [2][EV][kCond]
    float* const zs = (float*)(cond + 2 * EV * kCond);  // [2][d][EV]
    float* const lds_ld = zs + 2 * d * EV;              // [kWaves][EV]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int e16 = lane & 15, q = lane >> 4;
    const int ev = lane & (EV - 1);        // this lane's event of a tile in the splines
    const bool mine = EV >= 64 || lane < EV;
    const int64_t n = run.n, step = gridDim.x;
    const int64_t tiles = (n + EV - 1) / EV;

    for (int i = tid; i < 2 * EV * kCond; i += kThreads) cond[i] = (T)0.0f;

    for (int li = 0; li < run.count; ++li) {
        const int layer = run.first + li * run.dir;
        const Mask mk = mask_of(layer, nh);
        const float* const zi = li == 0 ? run.zin : run.zout + (li - 1) * run.zstep;
        float* const zo = run.zout + li * run.zstep;
        HidW<T> hw = load_hidden<T>(fn, layer, wave, lane);
        const RegisterBias<KEEP> bias(fn, layer, wave, lane);
        if constexpr (KEEP) {
            __syncthreads();  // the previous layer's readers of w4
            load_out(fn, layer, w4, tid);
        }
        // staging of a tile: 64 / EV coordinates per wave and step, the lane's
        // event (the last one again beyond the end)
        float zr[ZR];
        auto row_of = [&](int i) { return (wave + i * kWaves) * (64 / EV) + (EV < 64 ? lane / EV : 0); };
        auto coord = [&](int i, uint32_t e) { return zi[(int64_t)min(row_of(i), d - 1) * n + e]; };
        auto event_of = [&](int64_t tile) { return (uint32_t)min(tile * EV + ev, n - 1); };
        auto put = [&](int buf, int i, float v) {
            const int c = row_of(i), k = cond_index(mk, nh, c);
            if (c >= d) return;
            zs[(buf * d + c) * EV + ev] = v;
            if (k >= 0) cond[cond_at<T>(buf * EV + ev, column<T>(k))] = (T)v;
        };
        auto fetch = [&](int64_t tile) {
            const uint32_t e = event_of(tile);
#pragma unroll
            for (int i = 0; i < ZR; ++i) zr[i] = coord(i, e);
        };
        auto stage = [&](int buf, int64_t tile) {
#pragma unroll
            for (int i = 0; i < ZR; ++i) put(buf, i, zr[i]);
            for (int i = ZR; i * kWaves * (64 / EV) < d; ++i) put(buf, i, coord(i, event_of(tile)));
        };
        // log-determinants: the sum over the layers before, and the new sum with
        // the coordinates' terms added in order
        auto before = [&](int64_t tile) {
            return li > 0 && tid < EV ? run.logdet[min(tile * EV + tid, n - 1)] : 0.0f;
        };
        auto flush = [&](int64_t tile, float old) {
            if (tid < EV && tile * EV + tid < n) {
                float s = 0.0f;
                for (int w = 0; w < min(kWaves, nh); ++w) s += lds_ld[w * EV + tid];
                run.logdet[tile * EV + tid] = old + s;
            }
        };
        // the previous layer's stores to z, and its last readers of LDS
        __syncthreads();
        fetch(blockIdx.x);
        stage(0, blockIdx.x);
        fetch(blockIdx.x + step);
        __syncthreads();
        int buf = 0, pa = 0;
        int64_t prev = -1;
        float old = 0.0f;
        for (int64_t tile = blockIdx.x; tile < tiles; tile += step) {
            const float* zt = zs + buf * d * EV;
            T* const a0 = act + pa * EV * kHid;
            T* const a1 = act + (pa ^ 1) * EV * kHid;
            const float old_next = before(tile);
            hw.per_tile();
#pragma unroll
            for (int t = 0; t < NT; ++t)
                store_act(mfma(hw.w1, cond8(cond, buf * EV + 16 * t + e16, 8 * q), zero4()),
                          bias.hidden(0), a0, 16 * t, wave, lane);
            __syncthreads();
            if (prev >= 0) flush(prev, old);
            old = old_next;
            hidden_layer<NT>(hw.w2, bias.hidden(1), a0, a1, wave, lane);
            __syncthreads();
            hidden_layer<NT>(hw.w3, bias.hidden(2), a1, a0, wave, lane);
            stage(buf ^ 1, tile + step);
            fetch(tile + 2 * step);
            __syncthreads();
            float ld_sum = 0.0f;
            for (int j = wave; j < nh; j += KEEP ? 2 * kFlowMaxHalf : kWaves) {
                const int tj = mk.t0 + mk.ts * j;
                Theta th = output_layer<NT, KEEP>(fn, layer, a0, w4, bias, j, K, lane);
                const float vin = zt[tj * EV + ev];
                float sw, sh, ld;
                spline_exp<BINS == 16>(th, BINS ? BINS : K, sw, sh);
                Bin b = spline_find<INV, BINS == 16>(th, BINS ? BINS : K, vin, sw, sh);
                spline_slopes(b);
                const float v = spline_value<INV>(b, vin, ld);
                const int64_t e = tile * EV + ev;
                if (mine && e < n) zo[(int64_t)tj * n + e] = v;
                ld_sum += ld;
            }
            if (mine) lds_ld[wave * EV + ev] = ld_sum;
            if (zi != zo) {
                // a new buffer: the conditioning coordinates go along
                const int64_t ec = tile * EV + ev;
                for (int i = 0; i * kWaves * (64 / EV) < nh; ++i) {
                    const int c = mk.c0 + mk.cs * row_of(i);
                    if (row_of(i) < nh && ec < n) zo[(int64_t)c * n + ec] = zt[c * EV + ev];
                }
            }
            prev = tile;
            buf ^= 1;
            pa ^= 1;
        }
        __syncthreads();
        flush(prev, old);
    }
}

// A pass over 16 events per workgroup (BF16, at most eight transformed
// coordinates): the coordinates stay in LDS over all layers, and a layer's
// weights are on their way while the layer before evaluates its splines, the
// hidden layers' to registers and the output layer's to LDS.
//
// What bounds it: a layer's 166 KB of weights come to the one compute unit at 28
// B/ns, 6 of the 7.4 us per layer (without them it takes 3); fewer events per
// tile would not change that, more take their splines' time.  1,000 events of 16
// dimensions, 8 layers: 60 us; with the weights loaded when a layer begins and
// the coordinates through memory (k_flow_layers with tiles of 16) 68.
template <bool INV, int BINS>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_flow_tile(FlowNet fn,
                                                                                               FlowRun run) {
    typedef __bf16 T;
    constexpr int EV = 16;
    __shared__ __attribute__((aligned(16))) T w4[kOutKept];  // [nh][kOutElems]
    __shared__ __attribute__((aligned(16))) T act[2][EV * kHid];
    __shared__ __attribute__((aligned(16))) T cond[EV * kCond];
    __shared__ float zs[2 * kWaves][EV];
    __shared__ float lds_ld[kWaves][EV];
    fn.K = BINS;
    const int nh = fn.nh, d = 2 * nh, K = fn.K;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ev = lane & 15, q = lane >> 4;
    const int64_t n = run.n, e0 = (int64_t)blockIdx.x * EV;
    const bool mine = tid < d * EV;  // thread tid moves coordinate tid / 16 of event tid % 16
    const int64_t em = e0 + (tid & 15);
    const float z0 = mine ? run.zin[(int64_t)(tid >> 4) * n + min(em, n - 1)] : 0.0f;
    HidW<T> hw = load_hidden<T>(fn, run.first, wave, lane);
    RegisterBias<true> bias(fn, run.first, wave, lane);
    const OutCopy copy_out(fn, wave, lane);
    copy_out(fn, run.first, w4, wave);
    for (int i = tid; i < EV * kCond; i += kThreads) cond[i] = (T)0.0f;
    if (mine) zs[tid >> 4][tid & 15] = z0;
    __syncthreads();
    float ld = 0.0f;
    for (int li = 0; li < run.count; ++li) {
        const int layer = run.first + li * run.dir, next = li + 1 < run.count ? layer + run.dir : layer;
        const Mask mk = mask_of(layer, nh);
        if (tid < nh * EV) {
            const int k = tid >> 4;
            cond[cond_at<T>(tid & 15, k)] = (T)zs[mk.c0 + mk.cs * k][tid & 15];
        }
        __syncthreads();
        store_act(mfma(hw.w1, cond8(cond, ev, 8 * q), zero4()), bias.hidden(0), act[0], 0, wave, lane);
        __syncthreads();
        hidden_layer<1>(hw.w2, bias.hidden(1), act[0], act[1], wave, lane);
        __syncthreads();
        hidden_layer<1>(hw.w3, bias.hidden(2), act[1], act[0], wave, lane);
        landed();  // this layer's w4
        __syncthreads();
        // the next layer's weights
        hw = load_hidden<T>(fn, next, wave, lane);
        Theta th;
        if (wave < nh) th = output_layer<1, true>(fn, layer, act[0], w4, bias, wave, K, lane);
        bias = RegisterBias<true>(fn, next, wave, lane);
        __syncthreads();  // w4 is read
        if (li + 1 < run.count) copy_out(fn, next, w4, wave);
        if (wave < nh) {
            const int tj = mk.t0 + mk.ts * wave;
            const float vin = zs[tj][ev];
            float sw, sh, l;
            spline_exp<BINS == 16>(th, K, sw, sh);
            Bin b = spline_find<INV, BINS == 16>(th, K, vin, sw, sh);
            spline_slopes(b);
            const float v = spline_value<INV>(b, vin, l);
            if (lane < EV) {
                zs[tj][ev] = v;
                lds_ld[wave][ev] = 0.0f + l;
            }
        }
        __syncthreads();
        if (tid < EV) {
            float s = 0.0f;
            for (int w = 0; w < nh; ++w) s += lds_ld[w][tid];
            ld = li > 0 ? ld + s : 0.0f + s;
        }
        if (mine && em < n && (run.zstep != 0 || li + 1 == run.count))
            run.zout[li * run.zstep + (int64_t)(tid >> 4) * n + em] = zs[tid >> 4][tid & 15];
    }
    if (tid < EV && e0 + tid < n) run.logdet[e0 + tid] = ld;
}

// The bins are a constant of the kernels of BF16 passes: with their number known
// at run time only, each bin's exponentials stand behind a branch of their own and
// wait for themselves (450,000 events of 10 dimensions, 6 layers, 8 bins, inverse:
// 1164 us, as a constant 805; 1,000 events of 10 dimensions, 8 layers, 2 bins 51 and
// 39, 5 bins 54 and 44, 12 bins 62 and 52), and small and large passes then do the
// same operations (one bin at run time gave other bits in tiles of 16).  In the
// others, bound by their weights or their products, only 16 bins are, whose knots
// are searched by halves.
template <bool INV, int BINS>
void launch_bins(const FlowNet& fn, const FlowRun& run, dim3 g, size_t lds, hipStream_t s) {
    if constexpr (BINS > 0) {
        if (fn.K == BINS)
            k_flow_layers<INV, 4, true, BINS, __bf16><<<g, dim3(kThreads), lds, s>>>(fn, run);
        else
            launch_bins<INV, BINS - 1>(fn, run, g, lds, s);
    }
}

template <bool INV, int BINS>
void launch_tile(const FlowNet& fn, const FlowRun& run, int64_t grid, hipStream_t s) {
    if constexpr (BINS > 0) {
        if (fn.K == BINS)
            k_flow_tile<INV, BINS><<<(unsigned)grid, kThreads, 0, s>>>(fn, run);
        else
            launch_tile<INV, BINS - 1>(fn, run, grid, s);
    }
}

template <bool INV, int NT, class T>
hipError_t launch_layers(const FlowNet& fn, const FlowRun& run, int64_t grid, hipStream_t s) {
    constexpr bool can_keep = sizeof(T) == 2 && NT == 4;
    const bool keep = can_keep && fn.nh <= kWaves;  // then W4 fits in LDS: at most 98 KiB
    const size_t lds = layers_lds<NT, T>(2 * fn.nh, keep ? fn.nh : 0);
    const dim3 g((unsigned)grid), t(kThreads);
    if (fn.K < 1 || fn.K > 16) return hipErrorInvalidValue;
    if (keep)
        launch_bins<INV, 16>(fn, run, g, lds, s);
    else if (fn.K == 16)
        k_flow_layers<INV, NT, false, 16, T><<<g, t, lds, s>>>(fn, run);
    else
        k_flow_layers<INV, NT, false, 0, T><<<g, t, lds, s>>>(fn, run);
    return hipGetLastError();
}

template <bool INV>
hipError_t launch_pass(const FlowNet& fn, const FlowRun& run, int cu_count, hipStream_t s) {
    const int64_t t16 = (run.n + 15) / 16;
    if (fn.f32) {
        // FP32 products take most of a tile's time (5 us per 16 events), so
        // the tile is the largest that does not leave more of the last round
        // empty than it saves in latencies (about 4 us per tile and layer)
        const int64_t r1 = (t16 + cu_count - 1) / cu_count, r2 = ((t16 + 1) / 2 + cu_count - 1) / cu_count,
                      r4 = ((t16 + 3) / 4 + cu_count - 1) / cu_count;
        if (r1 * 9 <= std::min(r2 * 14, r4 * 24))
            return launch_layers<INV, 1, float>(fn, run, std::min<int64_t>(t16, cu_count), s);
        if (r2 * 14 <= r4 * 24)
            return launch_layers<INV, 2, float>(fn, run, std::min<int64_t>((t16 + 1) / 2, cu_count), s);
        return launch_layers<INV, 4, float>(fn, run, std::min<int64_t>((t16 + 3) / 4, cu_count), s);
    }
    // up to one tile of 16 events for every compute unit the time is the
    // latency of a tile through the layers, which grows with the tile (8 layers
    // of 16 dimensions, 4,096 events: 60 us, one more 107; a second round of
    // tiles of 16 would take 118)
    if (t16 <= cu_count) {
        if (fn.nh > kWaves) return launch_layers<INV, 1, __bf16>(fn, run, t16, s);
        if (fn.K < 1 || fn.K > 16) return hipErrorInvalidValue;
        launch_tile<INV, 16>(fn, run, t16, s);
        return hipGetLastError();
    }
    return launch_layers<INV, 4, __bf16>(fn, run, std::min<int64_t>((t16 + 3) / 4, cu_count), s);
}

}  // namespace

hipError_t launch_flow_layers(bool inverse, const FlowNet& fn, const FlowRun& run, int cu_count, hipStream_t s) {
    if (run.n == 0) return hipSuccess;
    return inverse ? launch_pass<true>(fn, run, cu_count, s) : launch_pass<false>(fn, run, cu_count, s);
}

}  // namespace msx
