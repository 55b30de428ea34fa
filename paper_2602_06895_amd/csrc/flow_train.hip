// Reverse mode of the fused coupling layers (conditioner of hidden width 128 in
// BF16 or FP32, up to 16 spline bins) on gfx950: spline, conditioner and weight
// gradients of one layer in three kernels.  A layer of 8 + 8 coordinates and 16
// bins with 65,536 events took 490 us as 14 kernels (eight products, spline,
// four column sums over events, ...) with every operand through memory; the
// three take 56, 45 and 40 us.  FP32, 4,097 events: 440 us as 20 kernels (the
// products 65 workgroups each), now 29, 25 and 26 us, with 21 us of matrix
// instructions on the 129 compute units that have a tile, or 10 on all.
#include <algorithm>

#include "flow_adjoint.h"
#include "flow_layers.h"

namespace msx {

namespace {

using namespace flow;

// a / b with r = 1 / b: the quotient, corrected once by its exact remainder
// (as the division instruction sequence ends), so a shared reciprocal serves
// 16 quotients with the division's own results.
__device__ __forceinline__ float quotient(float a, float b, float r) {
    const float q = a * r;
    return __builtin_fmaf(__builtin_fmaf(-q, b, a), r, q);
}
__device__ __forceinline__ float sigmoid_f(float x) { return 1.0f / (1.0f + expf(-x)); }

// Gradients of one (event, coordinate): th as spline_exp leaves it, b the bin
// of v with the slopes applied, gp the adjoint of its quantities; put(p, g)
// takes the gradient of unconstrained parameter p.  Softmax of the widths and
// heights, softplus of the slopes.
template <bool K16, class Put>
__device__ __forceinline__ void spline_param_grads(const Theta& th, int K, const Bin& b, float t0, float t1, float sw,
                                                   float sh, const float (&gp)[7], Put&& put) {
    const float rw = 1.0f / sw, rh = 1.0f / sh;
    float pw[16], ph[16], below_w = 0.0f, below_h = 0.0f, pwk = 0.0f, phk = 0.0f, cw = 0.0f, ch = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        if (!(K16 || i < K)) continue;
        pw[i] = quotient(th.w[i], sw, rw);
        ph[i] = quotient(th.h[i], sh, rh);
        if (i == b.k) {
            pwk = pw[i];
            phk = ph[i];
            below_w = cw;
            below_h = ch;
        }
        cw += pw[i];
        ch += ph[i];
    }
    const float sumw = __builtin_fmaf(gp[1], below_w, gp[2] * pwk);
    const float sumh = __builtin_fmaf(gp[3], below_h, gp[4] * phk);
    const float Cw = 1.0f - (K16 ? 16 : K) * kMinW, Ch = 1.0f - (K16 ? 16 : K) * kMinH;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        if (!(K16 || i < K)) continue;
        const float dwi = i < b.k ? gp[1] : (i == b.k ? gp[2] : 0.0f);
        const float dhi = i < b.k ? gp[3] : (i == b.k ? gp[4] : 0.0f);
        put(i, Cw * pw[i] * (dwi - sumw));
        put((K16 ? 16 : K) + i, Ch * ph[i] * (dhi - sumh));
    }
    const float g0 = gp[5] * sigmoid_f(t0 + slope_shift()), g1 = gp[6] * sigmoid_f(t1 + slope_shift());
#pragma unroll
    for (int i = 0; i < 17; ++i) {
        if (!(K16 || i <= K)) continue;
        put(2 * (K16 ? 16 : K) + i, i == b.k ? g0 : (i == b.k + 1 ? g1 : 0.0f));
    }
}

// A tile's 16 NT x 128 activations (rows: events) from LDS to its blocks of out,
// each [384][32]: a thread packs eight events of a feature at a time.
template <int NT, class T>
__device__ __forceinline__ void store_blocks(const T* __restrict__ act, T* __restrict__ out, int tid) {
    static_assert(kThreads == 4 * kHid, "a block per round");
#pragma unroll
    for (int i = 0; i < NT / 2; ++i) {
        const int g = tid & 3, f = tid >> 2;
        Vec8<T> v;
#pragma unroll
        for (int x = 0; x < 8; ++x) v[x] = act[act_at<T>(32 * i + 8 * g + x, column<T>(f))];
        *(Vec8<T>*)&out[(i * 3 * kHid + f) * 32 + 8 * g] = v;
    }
}

// LDS: output weights of `kept` coordinates, two activation tiles, the
// conditioning inputs and the coordinates of a tile, the biases.
template <int NT, class T>
constexpr size_t reverse_lds(int d, int kept) {
    return sizeof(T) * ((size_t)kept * kOutElems + 16 * NT * (2 * kHid + kCond)) + sizeof(float) * (16 * NT * (size_t)d + kBiases);
}

// Rows of d that k_flow_wgrad reads: whole 16-row tiles of every chunk of eight
// coordinates.
constexpr int kGradTiles = 25;  // 8 x 49 parameters
__host__ __device__ constexpr int out_chunks(int nh) { return (nh + 7) / 8; }
__host__ __device__ constexpr int grad_rows(int nh, int K) {
    return (out_chunks(nh) - 1) * 8 * (3 * K + 1) + 16 * kGradTiles;
}

// Hidden activations and spline parameters of a layer recomputed from its
// input (as the inverse pass computes them), then the reverse mode of the
// inverse spline.  Waves and tiles as in the pass; the activations leave
// transposed through LDS, the spline gradients as rows of 32 events.
// Recomputing costs 100 MFMAs per wave and 64 events and saves writing and
// reading 1.6 KB of FP32 spline parameters per event and layer.  The biases
// come from LDS: in registers, the splines spill 28 (72 instead of 56 us per
// layer of 65,536 events).
template <int NT, bool KEEP, bool K16, class T>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_flow_spline_reverse(
    FlowNet fn, FlowRev r) {
    constexpr int EV = 16 * NT;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int nh = fn.nh, d = 2 * nh, K = K16 ? 16 : fn.K, P = 3 * K + 1;
    T* const w4 = (T*)smem;                                // KEEP: [nh][kOutElems]
    T* const a0 = w4 + (KEEP ? nh * kOutElems : 0);        // [EV][kHid]
    T* const a1 = a0 + EV * kHid;                          // [EV][kHid]
    T* const cond = a1 + EV * kHid;                        // [EV][kCond]
    float* const zs = (float*)(cond + EV * kCond);         // [d][EV]
    float* const lb = zs + d * EV;                         // [kBiases]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int e16 = lane & 15, q = lane >> 4;
    const int ev = lane & (EV - 1);  // this lane's event of a tile
    const bool mine = EV >= 64 || lane < EV;
    const int64_t n = r.n, tiles = (n + EV - 1) / EV;
    const int gr = grad_rows(nh, K);
    const Mask mk = mask_of(r.layer, nh);
    HidW<T> hw = load_hidden<T>(fn, r.layer, wave, lane);
    const LdsBias<KEEP> bias(fn, r.layer, wave, lane, lb);
    if constexpr (KEEP) load_out(fn, r.layer, w4, tid);
    for (int i = tid; i < EV * kCond; i += kThreads) cond[i] = (T)0.0f;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t e = tile * EV + ev, el = min(e, n - 1), block = tile * EV / 32;
        const int at = ev & 31, eb = ev >> 5;  // place and block of the lane's event
        T* const hb = (T*)r.h + block * 3 * kHid * 32;
        T* const xb = (T*)r.x0 + block * 32 * 32 + eb * 32 * 32 + at;
        T* const gb = (T*)r.d + block * gr * 32;
        uint16_t* const on = r.on + tile * 3 * kThreads + tid;
        hw.per_tile();
        __syncthreads();  // the previous tile's readers
        for (int i = 0; i * kWaves * (64 / EV) < d; ++i) {
            const int c = (wave + i * kWaves) * (64 / EV) + (EV < 64 ? lane / EV : 0);
            if (c >= d) continue;
            const float v = r.zin[c * n + el];
            const int k = cond_index(mk, nh, c);
            zs[c * EV + ev] = v;
            if (k >= 0) {
                cond[cond_at<T>(ev, column<T>(k))] = (T)v;
                xb[k * 32] = (T)v;
            }
        }
        const float ge = r.G[el];
        __syncthreads();
        uint32_t m = 0;
#pragma unroll
        for (int t = 0; t < NT; ++t)
            m |= store_act(mfma(hw.w1, cond8(cond, 16 * t + e16, 8 * q), zero4()), bias.hidden(0),
                           a0, 16 * t, wave, lane)
                 << (4 * t);
        on[0] = (uint16_t)m;
        __syncthreads();
        store_blocks<NT>(a0, hb, tid);
        on[kThreads] = (uint16_t)hidden_layer<NT>(hw.w2, bias.hidden(1), a0, a1, wave, lane);
        __syncthreads();
        store_blocks<NT>(a1, hb + kHid * 32, tid);
        on[2 * kThreads] = (uint16_t)hidden_layer<NT>(hw.w3, bias.hidden(2), a1, a0, wave, lane);
        __syncthreads();
        store_blocks<NT>(a0, hb + 2 * kHid * 32, tid);
        for (int j = wave; j < nh; j += KEEP ? 2 * kFlowMaxHalf : kWaves) {
            const int tj = mk.t0 + mk.ts * j;
            float* const aj = r.adj + tj * n + el;
            const float ax = r.first ? 0.0f : *aj;
            Theta th = output_layer<NT, KEEP>(fn, r.layer, a0, w4, bias, j, K, lane);
            const float vin = zs[tj * EV + ev];
            float sw, sh, gp[7];
            spline_exp<K16>(th, K, sw, sh);
            Bin b = spline_find<true, K16>(th, K, vin, sw, sh);
            const float t0 = b.d0, t1 = b.d1;
            spline_slopes(b);
            spline_inverse_adjoint(vin, b.w, b.y0, b.h, b.d0, b.d1, ge, ax, gp);
            if (mine && e < n) *aj = gp[0];
            if (e >= n) {
                // zeros beyond n, so that the sums over events need no mask
#pragma unroll
                for (int i = 0; i < 7; ++i) gp[i] = 0.0f;
            }
            T* const dj = gb + (eb * gr + j * P) * 32 + at;
            if (mine)
                spline_param_grads<K16>(th, K, b, t0, t1, sw, sh, gp, [&](int p, float g) { dj[p * 32] = (T)g; });
        }
    }
}

// Transposed weights of a layer: W4^T [chunks of 8 coordinates][128][kOutK]
// (columns beyond the chunk's parameters zero), W3^T, W2^T [128][128], W1^T
// [kFlowMaxHalf][128] (rows beyond nh zero).
constexpr int kOutK = 416;  // 8 x 49 parameters, padded to a multiple of 32
__host__ __device__ constexpr int off_w3t(int nh) { return out_chunks(nh) * kHid * kOutK; }
__host__ __device__ constexpr int off_w2t(int nh) { return off_w3t(nh) + kHid * kHid; }
__host__ __device__ constexpr int off_w1t(int nh) { return off_w2t(nh) + kHid * kHid; }
__host__ __device__ constexpr int transposed_elems(int nh) { return off_w1t(nh) + kFlowMaxHalf * kHid; }

template <class T>
__global__ __launch_bounds__(256) void k_flow_transpose(FlowNet fn, T* __restrict__ wt_t) {
    const int nh = fn.nh, P = 3 * fn.K + 1, layer = blockIdx.y;
    const float* W = fn.p + layer * fn.per;
    T* const o = wt_t + (int64_t)layer * transposed_elems(nh);
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= transposed_elems(nh)) return;
    float v = 0.0f;
    int k;
    if (i < off_w3t(nh)) {
        const int c = i / (kHid * kOutK), h = i / kOutK % kHid, row = c * 8 * P + i % kOutK;
        k = i % kOutK;
        if (k < 8 * P && row < nh * P) v = W[fn.off[6] + row * kHid + h];
    } else if (i < off_w1t(nh)) {
        const int l = i < off_w2t(nh) ? 4 : 2, j = i - (i < off_w2t(nh) ? off_w3t(nh) : off_w2t(nh));
        k = j % kHid;
        v = W[fn.off[l] + k * kHid + j / kHid];
    } else {
        const int j = i - off_w1t(nh);
        k = j % kHid;
        if (j / kHid < nh) v = W[fn.off[0] + k * nh + j / kHid];
    }
    o[i - k + column<T>(k)] = (T)v;
}

// The gradient of a hidden layer before its ReLU: kept where the activation is
// positive (four bits of `on`).
template <class T>
__device__ __forceinline__ void store_masked(const floatx4& acc, uint32_t on, T* __restrict__ act, int r0, int wave,
                                             int lane) {
    Vec4<T> v;
#pragma unroll
    for (int x = 0; x < 4; ++x) v[x] = on >> x & 1 ? (T)acc[x] : (T)0.0f;
    store4(v, act, r0 + (lane & 15), 16 * wave + 4 * (lane >> 4));
}

// LDS pitch of the spline-parameter gradients: the 16-byte operand reads of 16
// rows start at 16 (8 in BF16) different bank groups.
template <class T>
constexpr int kDPitch = kOutK + 16 / (int)sizeof(T);
template <int NT, class T>
constexpr size_t mlp_reverse_lds() {
    return sizeof(T) * 16 * NT * (kDPitch<T> + 2 * kHid);
}

// The conditioner's reverse mode for tiles of 16 NT events: dh3 = W4^T d, dh2
// = W3^T dh3, dh1 = W2^T dh2 (each masked by its ReLU), dx0 = W1^T dh1, the
// products as in the forward pass, with the transposed weights in registers:
// over all tiles in BF16 (W4^T where there is one chunk of coordinates: ONE),
// loaded ahead of their product in FP32.  The gradients of
// the spline parameters are turned to event-major in LDS.
template <int NT, bool ONE, class T>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_flow_mlp_reverse(
    FlowNet fn, FlowRev r, const T* __restrict__ wt_t) {
    constexpr int EV = 16 * NT, KB = kOutK / 32, PD = kDPitch<T>;
    constexpr bool REG = sizeof(T) == 2;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    T* const dt = (T*)smem;            // [EV][PD]
    T* const a0 = dt + EV * PD;        // [EV][kHid]
    T* const a1 = a0 + EV * kHid;      // [EV][kHid]
    const int nh = fn.nh, P = 3 * fn.K + 1, n_out = nh * P, chunks = out_chunks(nh), gr = grad_rows(nh, fn.K);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int e16 = lane & 15, q = lane >> 4, row = 16 * wave + e16;
    const int xt = wave % NT, xr = min(wave / NT, kFlowMaxHalf / 16 - 1);  // the inputs' gradients: event and row tile
    const int64_t n = r.n, tiles = (n + EV - 1) / EV;
    const Mask mk = mask_of(r.layer, nh);
    const T* const wl = wt_t + (int64_t)r.layer * transposed_elems(nh);
    Vec8<T> w4[KB], w3[4], w2[4], w1[4];
    auto load_w4 = [&](int c, int z) {
#pragma unroll
        for (int s = 0; s < KB; ++s) w4[s] = load8(&wl[z + (c * kHid + row) * kOutK + 32 * s + 8 * q]);
    };
    auto load_w3 = [&](int z) {
#pragma unroll
        for (int s = 0; s < 4; ++s) w3[s] = load8(&wl[z + off_w3t(nh) + row * kHid + 32 * s + 8 * q]);
    };
    auto load_w21 = [&](int z) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            w2[s] = load8(&wl[z + off_w2t(nh) + row * kHid + 32 * s + 8 * q]);
            w1[s] = load8(&wl[z + off_w1t(nh) + (16 * xr + e16) * kHid + 32 * s + 8 * q]);
        }
    };
    auto clear = [&] {
        for (int i = tid; i < EV * PD / 4; i += kThreads) *(Vec4<T>*)&dt[4 * i] = Vec4<T>{};
    };
    if (REG && ONE) load_w4(0, 0);
    if (REG) {
        load_w3(0);
        load_w21(0);
    }
    if (ONE) clear();
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const uint16_t* const on = r.on + tile * 3 * kThreads + tid;
        const uint32_t on1 = on[0], on2 = on[kThreads], on3 = on[2 * kThreads];
        const int64_t block = tile * EV / 32;
        T* const db = (T*)r.dh + block * 3 * kHid * 32;
        floatx4 acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = zero4();
        for (int c = 0; c < (ONE ? 1 : chunks); ++c) {
            const int rows = ONE ? n_out : min(8 * P, n_out - c * 8 * P), pairs = (rows + 1) >> 1;
            if (!REG || !ONE) load_w4(c, REG ? 0 : here());
            __syncthreads();  // readers of dt and a0
            if (!ONE) {
                clear();
                __syncthreads();
            }
            // two parameters of eight events per thread: neighbouring lanes
            // write neighbouring words
            for (int i = tid; i < pairs * (EV / 8); i += kThreads) {
                const int g = i / pairs, p = 2 * (i - g * pairs);
                const T* const src = (const T*)r.d + ((block + (g >> 2)) * gr + c * 8 * P + p) * 32 + 8 * (g & 3);
                const Vec8<T> u = load8(src), v = p + 1 < rows ? load8(src + 32) : zero8<T>();
#pragma unroll
                for (int x = 0; x < 8; ++x) {
                    T* const to = &dt[(8 * g + x) * PD];
                    if constexpr (REG) {
                        *(Vec2<T>*)&to[p] = Vec2<T>{u[x], v[x]};
                    } else {
                        to[column<T>(p)] = u[x];
                        to[column<T>(p + 1)] = v[x];
                    }
                }
            }
            __syncthreads();
            if (!REG) load_w3(here());
#pragma unroll
            for (int s = 0; s < KB; ++s)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    acc[t] = mfma(w4[s], load8(&dt[(16 * t + e16) * PD + 32 * s + 8 * q]), acc[t]);
        }
        if (!REG) load_w21(here());
        auto masked = [&](uint32_t on, T* to) {
#pragma unroll
            for (int t = 0; t < NT; ++t) store_masked(acc[t], on >> (4 * t), to, 16 * t, wave, lane);
        };
        masked(on3, a0);
        __syncthreads();
        store_blocks<NT>(a0, db + 2 * kHid * 32, tid);
        square<NT>(w3, a0, lane, acc);
        masked(on2, a1);
        __syncthreads();
        store_blocks<NT>(a1, db + kHid * 32, tid);
        square<NT>(w2, a1, lane, acc);
        masked(on1, a0);
        __syncthreads();
        store_blocks<NT>(a0, db, tid);
        if (wave / NT == xr && 16 * xr < nh) {
            floatx4 g = zero4();
#pragma unroll
            for (int s = 0; s < 4; ++s) g = mfma(w1[s], act8(a0, 16 * xt + e16, 32 * s + 8 * q), g);
            const int64_t e = tile * EV + 16 * xt + e16;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int k = 16 * xr + 4 * q + i;
                if (k < nh && e < n) {
                    float* const a = r.adj + (mk.c0 + mk.cs * k) * n + e;
                    *a = r.first ? g[i] : *a + g[i];
                }
            }
        }
    }
}

// Weight gradients of a layer over a run of 32-event blocks: d h3^T, dh3 h2^T,
// dh2 h1^T, dh1 x0^T, and the row sums of d, dh3, dh2, dh1 (the biases).  A
// workgroup holds all 84,000 sums in the accumulators of its eight waves (172
// registers each), so every element of the run is read from memory once.  A
// block's operands come to LDS as they lie in memory (an operand is 1 KiB
// without gaps), the next block's while this one is multiplied.  One launch
// (HIDDEN) takes the rows of d of eight coordinates and the hidden layers, a
// second one with a blockIdx.y for every eight more coordinates their rows.
// 65,536 events of 16 dimensions: 40 us, 157 MB at 3.9 TB/s (with every wave
// loading its operands from the caches itself, eight times the traffic and no
// load ahead of its use, 82 us).  The partial sums of 128 runs are 43 MB: more
// runs would fill more compute units, but write and add up as much again
// (flow_wgrad_splits).
constexpr int kBlockH = 3 * kHid * 32, kBlockD = 16 * kGradTiles * 32, kBlockX = 32 * 32;  // elements
constexpr int kBlockElems = 2 * kBlockH + kBlockD + kBlockX;

__device__ __forceinline__ void copy_to_lds(const __bf16* __restrict__ src, __bf16* __restrict__ dst, int chunks, int wave,
                                            int lane) {
    for (int c = wave; c < chunks; c += kWaves)
        copy16_to_lds(src + c * 512 + lane * 8, dst + c * 512);
}

template <bool HIDDEN>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_flow_wgrad(
    FlowNet fn, FlowRev r, int64_t blocks, int64_t chunk, float* __restrict__ part) {
    __shared__ __attribute__((aligned(16))) __bf16 smem[2 * kBlockElems];
    const int nh = fn.nh, P = 3 * fn.K + 1, n_out = nh * P, gr = grad_rows(nh, fn.K);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, q = lane >> 4;
    const int row0 = HIDDEN ? 0 : (blockIdx.y + 1) * 8 * P, rows = min(8 * P, n_out - row0);
    float* const out = part + (int64_t)blockIdx.x * fn.per;
    floatx4 a4[3][8], a24 = zero4(), a3[8], a2[8], a1[2];
    float s4[3] = {0.0f, 0.0f, 0.0f}, s24 = 0.0f, s3 = 0.0f, s2 = 0.0f, s1 = 0.0f;
#pragma unroll
    for (int c = 0; c < 8; ++c) a4[0][c] = a4[1][c] = a4[2][c] = a3[c] = a2[c] = zero4();
    a1[0] = a1[1] = zero4();
    const int mine = r16 * 32 + 8 * q;  // the lane's element of a 16-row operand
    auto frag = [&](const __bf16* m, int row) { return load8(m + row * 32 + mine); };
    auto sum8 = [](const Vec8<__bf16>& v) {
        return (((float)v[0] + (float)v[1]) + ((float)v[2] + (float)v[3])) +
               (((float)v[4] + (float)v[5]) + ((float)v[6] + (float)v[7]));
    };
    auto stage = [&](int64_t k, __bf16* __restrict__ to) {
        copy_to_lds((const __bf16*)r.d + (k * gr + row0) * 32, to, kBlockD / 512, wave, lane);
        copy_to_lds((const __bf16*)r.h + k * kBlockH, to + kBlockD, kBlockH / 512, wave, lane);
        if (!HIDDEN) return;
        copy_to_lds((const __bf16*)r.dh + k * kBlockH, to + kBlockD + kBlockH, kBlockH / 512, wave, lane);
        copy_to_lds((const __bf16*)r.x0 + k * kBlockX, to + kBlockD + 2 * kBlockH, kBlockX / 512, wave, lane);
    };
    // the copies of block k to `next` run under the products of `d`: restrict
    // tells the compiler that reading the one need not wait for the other
    auto step = [&](const __bf16* __restrict__ d, __bf16* __restrict__ next, int64_t k) {
        stage(k, next);
        const __bf16 *const h = d + kBlockD, *const dh = h + kBlockH, *const x0 = dh + kBlockH;
        Vec8<__bf16> b[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) b[c] = frag(h, 2 * kHid + 16 * c);
#pragma unroll
        for (int g = 0; g < 3; ++g) {
            const Vec8<__bf16> a = frag(d, 128 * g + 16 * wave);
            s4[g] += sum8(a);
#pragma unroll
            for (int c = 0; c < 8; ++c) a4[g][c] = mfma(a, b[c], a4[g][c]);
        }
        // the last row tile: one column tile per wave
        const Vec8<__bf16> al = frag(d, 384);
        s24 += sum8(al);
        a24 = mfma(al, frag(h, 2 * kHid + 16 * wave), a24);
        if (!HIDDEN) return;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < 8; ++c) b[c] = frag(h, kHid + 16 * c);
        const Vec8<__bf16> x3 = frag(dh, 2 * kHid + 16 * wave);
        s3 += sum8(x3);
#pragma unroll
        for (int c = 0; c < 8; ++c) a3[c] = mfma(x3, b[c], a3[c]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < 8; ++c) b[c] = frag(h, 16 * c);
        const Vec8<__bf16> x2 = frag(dh, kHid + 16 * wave);
        s2 += sum8(x2);
#pragma unroll
        for (int c = 0; c < 8; ++c) a2[c] = mfma(x2, b[c], a2[c]);
        const Vec8<__bf16> x1 = frag(dh, 16 * wave);
        s1 += sum8(x1);
#pragma unroll
        for (int c = 0; c < 2; ++c) a1[c] = mfma(x1, frag(x0, 16 * c), a1[c]);
    };
    const int64_t k0 = blockIdx.x * chunk, k1 = min(blocks, k0 + chunk);
    if (k0 < k1) stage(k0, smem);
    for (int64_t k = k0; k < k1; ++k) {
        landed();
        __syncthreads();  // block k is in LDS, the other buffer's readers are done
        const int cur = (int)(k - k0) & 1;
        step(smem + cur * kBlockElems, smem + (cur ^ 1) * kBlockElems, min(k + 1, k1 - 1));
    }
    landed();
    auto over_q = [](float v) {
        v += __shfl_xor(v, 16, 64);
        return v + __shfl_xor(v, 32, 64);
    };
    float* const w4 = out + fn.off[6] + row0 * kHid;
    float* const b4 = out + fn.off[7] + row0;
    const int my = 16 * wave + r16;
#pragma unroll
    for (int g = 0; g < 3; ++g) {
#pragma unroll
        for (int c = 0; c < 8; ++c)
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const int row = 128 * g + 16 * wave + 4 * q + x;
                if (row < rows) w4[row * kHid + 16 * c + r16] = a4[g][c][x];
            }
        const float s = over_q(s4[g]);
        if (q == 0 && 128 * g + my < rows) b4[128 * g + my] = s;
    }
#pragma unroll
    for (int x = 0; x < 4; ++x)
        if (384 + 4 * q + x < rows) w4[(384 + 4 * q + x) * kHid + my] = a24[x];
    const float sl = over_q(s24);
    if (wave == 0 && q == 0 && 384 + r16 < rows) b4[384 + r16] = sl;
    if (!HIDDEN) return;
    s3 = over_q(s3);
    s2 = over_q(s2);
    s1 = over_q(s1);
    if (q == 0) {
        out[fn.off[5] + my] = s3;
        out[fn.off[3] + my] = s2;
        out[fn.off[1] + my] = s1;
    }
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        const int row = 16 * wave + 4 * q + x;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            out[fn.off[4] + row * kHid + 16 * c + r16] = a3[c][x];
            out[fn.off[2] + row * kHid + 16 * c + r16] = a2[c][x];
        }
        if (r16 < nh) out[fn.off[0] + row * nh + r16] = a1[0][x];
        if (16 + r16 < nh) out[fn.off[0] + row * nh + 16 + r16] = a1[1][x];
    }
}

// The same in FP32, whose products take eight times as long and whose operands
// are twice as large: blockIdx.y takes 128 rows, a wave 16 of them (eight
// accumulators of 16 x 16) with operands straight from the caches.  Rows of d
// come first, then dh3, dh2 and dh1.
__global__ __launch_bounds__(kThreads) void k_flow_wgrad_f32(FlowNet fn, FlowRev r, int64_t blocks, int64_t chunk,
                                                             float* __restrict__ part) {
    const int nh = fn.nh, n_out = nh * (3 * fn.K + 1), gr = grad_rows(nh, fn.K);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, q = lane >> 4;
    const int out_groups = (n_out + kHid - 1) / kHid;
    const int g = (int)blockIdx.y, l = g < out_groups ? 3 : out_groups + 2 - g;  // layer: 3 the output, 0 the first
    const int row0 = (l == 3 ? g * kHid : 0) + 16 * wave, rows = l == 3 ? n_out : kHid;
    const int cols = l ? kHid : nh, tiles = l ? 8 : (nh + 15) / 16;
    if (row0 >= rows) return;
    const int64_t a_step = (l == 3 ? gr : 3 * kHid) * 32, b_step = (l ? 3 * kHid : 32) * 32;
    const float* A = (l == 3 ? (const float*)r.d + row0 * 32 : (const float*)r.dh + (l * kHid + row0) * 32) + r16 * 32 + 8 * q;
    const float* B = (l ? (const float*)r.h + (l - 1) * kHid * 32 : (const float*)r.x0) + r16 * 32 + 8 * q;
    const int64_t k0 = blockIdx.x * chunk, k1 = min(blocks, k0 + chunk);
    floatx4 acc[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] = zero4();
    float sum = 0.0f;
    for (int64_t k = k0; k < k1; ++k) {
        const Vec8<float> a = load8(A + k * a_step);
        sum += ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
        const float* const b = B + k * b_step;
        if (tiles == 8) {
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[c] = mfma(a, load8(b + c * 512), acc[c]);
        } else {
            acc[0] = mfma(a, load8(b), acc[0]);
            if (tiles == 2) acc[1] = mfma(a, load8(b + 512), acc[1]);
        }
    }
    float* const out = part + (int64_t)blockIdx.x * fn.per + fn.off[2 * l];
#pragma unroll
    for (int c = 0; c < 8; ++c)
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int row = row0 + 4 * q + x, col = 16 * c + r16;
            if (row < rows && col < cols) out[row * cols + col] = acc[c][x];
        }
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    if (q == 0 && row0 + r16 < rows) part[(int64_t)blockIdx.x * fn.per + fn.off[2 * l + 1] + row0 + r16] = sum;
}

template <int NT, class T>
hipError_t launch_spline_reverse(const FlowNet& fn, const FlowRev& r, int cu_count, hipStream_t s) {
    constexpr bool can_keep = sizeof(T) == 2;
    const bool keep = can_keep && fn.nh <= kWaves;
    const size_t lds = reverse_lds<NT, T>(2 * fn.nh, keep ? fn.nh : 0);
    const dim3 g((unsigned)std::min<int64_t>((r.n + 16 * NT - 1) / (16 * NT), cu_count)), t(kThreads);
    if (keep && fn.K == 16)
        k_flow_spline_reverse<NT, can_keep, true, T><<<g, t, lds, s>>>(fn, r);
    else if (keep)
        k_flow_spline_reverse<NT, can_keep, false, T><<<g, t, lds, s>>>(fn, r);
    else if (fn.K == 16)
        k_flow_spline_reverse<NT, false, true, T><<<g, t, lds, s>>>(fn, r);
    else
        k_flow_spline_reverse<NT, false, false, T><<<g, t, lds, s>>>(fn, r);
    return hipGetLastError();
}

template <int NT, class T>
hipError_t launch_mlp_reverse(const FlowNet& fn, const FlowRev& r, const void* wt_t, int cu_count, hipStream_t s) {
    const unsigned grid = (unsigned)std::min<int64_t>((r.n + 16 * NT - 1) / (16 * NT), cu_count);
    const size_t lds = mlp_reverse_lds<NT, T>();
    if (fn.nh <= 8)
        k_flow_mlp_reverse<NT, true, T><<<grid, kThreads, lds, s>>>(fn, r, (const T*)wt_t);
    else
        k_flow_mlp_reverse<NT, false, T><<<grid, kThreads, lds, s>>>(fn, r, (const T*)wt_t);
    return hipGetLastError();
}

// 16-event tiles per workgroup of the reverse kernels: 32 events in FP32 (of 64
// the 172 KiB would not fit in LDS), and while every compute unit gets at most
// one such tile (4,096 events of 16 dimensions: 569 us a gradient with tiles of
// 64, 512 with 32).
int reverse_tiles(const FlowNet& fn, int64_t n, int cu_count) { return fn.f32 || n <= 32 * (int64_t)cu_count ? 2 : 4; }

}  // namespace

int flow_grad_rows(int nh, int K) { return grad_rows(nh, K); }

hipError_t launch_flow_spline_reverse(const FlowNet& fn, const FlowRev& r, int cu_count, hipStream_t s) {
    if (fn.f32) return launch_spline_reverse<2, float>(fn, r, cu_count, s);
    return reverse_tiles(fn, r.n, cu_count) == 2 ? launch_spline_reverse<2, __bf16>(fn, r, cu_count, s)
                                                 : launch_spline_reverse<4, __bf16>(fn, r, cu_count, s);
}

int64_t flow_transposed_elems(int nh) { return transposed_elems(nh); }

hipError_t launch_flow_transpose(const FlowNet& fn, int layers, void* wt_t, hipStream_t s) {
    const dim3 grid((unsigned)((transposed_elems(fn.nh) + 255) / 256), (unsigned)layers);
    if (fn.f32)
        k_flow_transpose<<<grid, 256, 0, s>>>(fn, (float*)wt_t);
    else
        k_flow_transpose<<<grid, 256, 0, s>>>(fn, (__bf16*)wt_t);
    return hipGetLastError();
}

hipError_t launch_flow_mlp_reverse(const FlowNet& fn, const FlowRev& r, const void* wt_t, int cu_count,
                                   hipStream_t s) {
    if (fn.f32) return launch_mlp_reverse<2, float>(fn, r, wt_t, cu_count, s);
    return reverse_tiles(fn, r.n, cu_count) == 2 ? launch_mlp_reverse<2, __bf16>(fn, r, wt_t, cu_count, s)
                                                 : launch_mlp_reverse<4, __bf16>(fn, r, wt_t, cu_count, s);
}

// Runs of events of the weight gradients.  More of them fill more compute units,
// but each writes, and the reduction reads, all partial sums (336 KB for 8 + 8
// coordinates and 16 bins).  Their length is also the number of terms that one
// FP32 accumulator adds up, so the runs grow with n.
//
// BF16: runs of 64 events up to 64, from 8,192 events of 128, from 16,384 on 128
// runs (1,000 events, 8 layers: 515 us a gradient with runs of 256, 429 with 64;
// 8,192: 600, 580 with 64, 557 with 128), of 512 and more up to 256 runs (65,536
// events: 1449 us with 128 runs, 1559 with 256; 2^20 events, 2 layers: 4689 with
// 128, 4379 with 256, 4494 with 512).  The error against 64 bits is that of the
// BF16 operands (3e-3 to 2e-2), the same to four digits for 64 to 8,192 events a
// run.
//
// FP32: blockIdx.y gives seven workgroups per run of eight coordinates already, so
// up to 32 runs of at least 64, and from 8,192 events on runs of 256 up to 512
// runs.  With 32 runs whatever n is, the error of W4's gradient grew with n (2^18
// events: 9.0e-7, now 8.6e-7; 10 dimensions, 8 bins, 65,536 events: 3.4e-7, now
// 3.1e-7) and half of the chip waited (65,536 events, 4 layers: 3272 us, now 2943).
int flow_wgrad_splits(const FlowNet& fn, int64_t n) {
    if (fn.f32) return (int)std::max<int64_t>({1, std::min<int64_t>(n / 64, 32), std::min<int64_t>(n / 256, 512)});
    return (int)std::max<int64_t>({1, std::min<int64_t>(n / 64, 64), std::min<int64_t>(n / 128, 128),
                                   std::min<int64_t>(n / 512, 256)});
}

hipError_t launch_flow_wgrad(const FlowNet& fn, const FlowRev& r, int splits, float* part, int cu_count, hipStream_t s) {
    const int64_t ev = 16 * reverse_tiles(fn, r.n, cu_count), blocks = (r.n + ev - 1) / ev * ev / 32, chunk = (blocks + splits - 1) / splits;
    if (fn.f32) {
        const int groups = (fn.nh * (3 * fn.K + 1) + kHid - 1) / kHid + 3;
        k_flow_wgrad_f32<<<dim3((unsigned)splits, (unsigned)groups), kThreads, 0, s>>>(fn, r, blocks, chunk, part);
        return hipGetLastError();
    }
    k_flow_wgrad<true><<<(unsigned)splits, kThreads, 0, s>>>(fn, r, blocks, chunk, part);
    if (out_chunks(fn.nh) > 1)
        k_flow_wgrad<false><<<dim3((unsigned)splits, (unsigned)(out_chunks(fn.nh) - 1)), kThreads, 0, s>>>(fn, r, blocks,
                                                                                                        chunk, part);
    return hipGetLastError();
}

}  // namespace msx
