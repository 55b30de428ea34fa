// Reverse mode of the fused coupling layers (BF16 conditioner of hidden width
// 128, up to 16 spline bins) on gfx950: spline, conditioner and weight
// gradients of one layer in three kernels.  A layer of 8 + 8 coordinates and 16
// bins with 65,536 events took 490 us as 14 kernels (eight products, spline,
// four column sums over events, ...) with every operand through memory; the
// three take 63, 45 and 40 us.
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

// 64 x 128 activations (rows: events) from LDS to the tile's two blocks of out,
// each [384][32]: a thread packs eight events of two features.
__device__ __forceinline__ void store_blocks(const __bf16* __restrict__ act, __bf16* __restrict__ out, int tid) {
#pragma unroll
    for (int i = 0; i < kHid * 8 / kThreads; ++i) {
        const int c = tid + i * kThreads, g = (c & 3) + 4 * (c >> 9), f = (c >> 2) & (kHid - 1);
        bf16x8 v;
#pragma unroll
        for (int x = 0; x < 8; ++x) v[x] = act[act_chunk(8 * g + x, f >> 3) + (f & 7)];
        *(bf16x8*)&out[((g >> 2) * 3 * kHid + f) * 32 + 8 * (g & 3)] = v;
    }
}

// LDS: output weights of `kept` coordinates, two activation tiles, the
// conditioning inputs and the coordinates of a tile.
constexpr size_t reverse_lds(int d, int kept) {
    return sizeof(__bf16) * ((size_t)kept * kOutElems + 64 * (2 * kHid + kCond)) + sizeof(float) * 64 * (size_t)d;
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
// reading 1.6 KB of FP32 spline parameters per event and layer.
template <bool KEEP, bool K16>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_flow_spline_reverse(
    FlowNet fn, FlowRev r) {
    constexpr int NT = 4, EV = 64;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int nh = fn.nh, d = 2 * nh, K = K16 ? 16 : fn.K, P = 3 * K + 1;
    __bf16* const w4 = (__bf16*)smem;                      // KEEP: [nh][kOutElems]
    __bf16* const a0 = w4 + (KEEP ? nh * kOutElems : 0);   // [EV][kHid]
    __bf16* const a1 = a0 + EV * kHid;                     // [EV][kHid]
    __bf16* const cond = a1 + EV * kHid;                   // [EV][kCond]
    float* const zs = (float*)(cond + EV * kCond);         // [d][EV]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int e16 = lane & 15, q = lane >> 4;
    const int64_t n = r.n, tiles = (n + EV - 1) / EV;
    const int gr = grad_rows(nh, K);
    const Mask mk = mask_of(r.layer, nh);
    const HidW hw = load_hidden(fn, r.layer, wave, lane);
    OutBias ob;
    if (KEEP) {
        ob = load_out_bias(fn, r.layer, min(wave, nh - 1), lane);
        load_out(fn, r.layer, w4, tid);
    }
    for (int i = tid; i < EV * kCond; i += kThreads) cond[i] = (__bf16)0.0f;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t e = tile * EV + lane, el = min(e, n - 1);
        const int64_t block = 2 * tile + (lane >> 5);
        __bf16* const hb = r.h + 2 * tile * 3 * kHid * 32;
        uint16_t* const on = r.on + tile * 3 * kThreads + tid;
        __syncthreads();  // the previous tile's readers
        for (int c = wave; c < d; c += kWaves) {
            const float v = r.zin[c * n + el];
            const int k = cond_index(mk, nh, c);
            zs[c * EV + lane] = v;
            if (k >= 0) {
                cond[cond_chunk(lane, k >> 3) + (k & 7)] = (__bf16)v;
                r.x0[(block * 32 + k) * 32 + (lane & 31)] = (__bf16)v;
            }
        }
        const float ge = r.G[el];
        __syncthreads();
        uint32_t m = 0;
#pragma unroll
        for (int t = 0; t < NT; ++t)
            m |= store_act(mfma(hw.w1, *(const bf16x8*)&cond[cond_chunk(16 * t + e16, q)], zero4()), hw.b1, a0, 16 * t,
                           wave, lane)
                 << (4 * t);
        on[0] = (uint16_t)m;
        __syncthreads();
        store_blocks(a0, hb, tid);
        on[kThreads] = (uint16_t)hidden_layer<NT>(hw.w2, hw.b2, a0, a1, wave, lane);
        __syncthreads();
        store_blocks(a1, hb + kHid * 32, tid);
        on[2 * kThreads] = (uint16_t)hidden_layer<NT>(hw.w3, hw.b3, a1, a0, wave, lane);
        __syncthreads();
        store_blocks(a0, hb + 2 * kHid * 32, tid);
        for (int j = wave; j < nh; j += KEEP ? 2 * kFlowMaxHalf : kWaves) {
            const int tj = mk.t0 + mk.ts * j;
            float* const aj = r.adj + tj * n + el;
            const float ax = r.first ? 0.0f : *aj;
            Theta th = output_layer<NT, KEEP>(fn, r.layer, a0, w4, ob, j, K, lane);
            const float vin = zs[tj * EV + lane];
            float sw, sh, gp[7];
            spline_exp<K16>(th, K, sw, sh);
            Bin b = spline_find<true, K16>(th, K, vin, sw, sh);
            const float t0 = b.d0, t1 = b.d1;
            spline_slopes(b);
            spline_inverse_adjoint(vin, b.w, b.y0, b.h, b.d0, b.d1, ge, ax, gp);
            if (e < n) *aj = gp[0];
            if (e >= n) {
                // zeros beyond n, so that the sums over events need no mask
#pragma unroll
                for (int i = 0; i < 7; ++i) gp[i] = 0.0f;
            }
            __bf16* const dj = r.d + (block * gr + j * P) * 32 + (lane & 31);
            spline_param_grads<K16>(th, K, b, t0, t1, sw, sh, gp, [&](int p, float g) { dj[p * 32] = (__bf16)g; });
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

__global__ __launch_bounds__(256) void k_flow_transpose(FlowNet fn, __bf16* __restrict__ wt_t) {
    const int nh = fn.nh, P = 3 * fn.K + 1, layer = blockIdx.y;
    const __bf16* W = (const __bf16*)fn.wt + layer * fn.per_t;
    __bf16* const o = wt_t + (int64_t)layer * transposed_elems(nh);
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= transposed_elems(nh)) return;
    __bf16 v = (__bf16)0.0f;
    if (i < off_w3t(nh)) {
        const int c = i / (kHid * kOutK), h = i / kOutK % kHid, k = i % kOutK;
        const int row = c * 8 * P + k;
        if (k < 8 * P && row < nh * P) v = W[fn.off[6] + row * kHid + h];
    } else if (i < off_w1t(nh)) {
        const int l = i < off_w2t(nh) ? 4 : 2, j = i - (i < off_w2t(nh) ? off_w3t(nh) : off_w2t(nh));
        v = W[fn.off[l] + (j % kHid) * kHid + j / kHid];
    } else {
        const int j = i - off_w1t(nh);
        if (j / kHid < nh) v = W[fn.off[0] + (j % kHid) * nh + j / kHid];
    }
    o[i] = v;
}

// The gradient of a hidden layer before its ReLU: BF16 where the activation
// is positive (four bits of `on`).
__device__ __forceinline__ void store_masked(const floatx4& acc, uint32_t on, __bf16* __restrict__ act, int r0, int wave,
                                             int lane) {
    const int q = lane >> 4;
    bf16x4 v;
#pragma unroll
    for (int x = 0; x < 4; ++x) v[x] = on >> x & 1 ? (__bf16)acc[x] : (__bf16)0.0f;
    *(bf16x4*)&act[act_chunk(r0 + (lane & 15), 2 * wave + (q >> 1)) + 4 * (q & 1)] = v;
}

constexpr int kDPitch = kOutK + 8;  // LDS pitch of the spline-parameter gradients (odd in 16-byte units)

// The conditioner's reverse mode for tiles of 64 events: dh3 = W4^T d, dh2 =
// W3^T dh3, dh1 = W2^T dh2 (each masked by its ReLU), dx0 = W1^T dh1, the
// products as in the forward pass with the transposed weights in registers
// (ONE: all of W4^T, at most eight coordinates).  The gradients of the spline
// parameters are turned to event-major in LDS.
template <bool ONE>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_flow_mlp_reverse(
    FlowNet fn, FlowRev r, const __bf16* __restrict__ wt_t) {
    constexpr int EV = 64, NT = 4, KB = kOutK / 32;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __bf16* const dt = (__bf16*)smem;       // [EV][kDPitch]
    __bf16* const a0 = dt + EV * kDPitch;   // [EV][kHid]
    __bf16* const a1 = a0 + EV * kHid;      // [EV][kHid]
    const int nh = fn.nh, P = 3 * fn.K + 1, n_out = nh * P, chunks = out_chunks(nh), gr = grad_rows(nh, fn.K);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int e16 = lane & 15, q = lane >> 4, row = 16 * wave + e16;
    const int64_t n = r.n, tiles = (n + EV - 1) / EV;
    const Mask mk = mask_of(r.layer, nh);
    const __bf16* const wl = wt_t + (int64_t)r.layer * transposed_elems(nh);
    bf16x8 w4[KB], w3[4], w2[4], w1[4];
    auto load_w4 = [&](int c) {
#pragma unroll
        for (int s = 0; s < KB; ++s) w4[s] = *(const bf16x8*)&wl[(c * kHid + row) * kOutK + 32 * s + 8 * q];
    };
    auto clear = [&] {
        for (int i = tid; i < EV * kDPitch / 8; i += kThreads) *(bf16x8*)&dt[8 * i] = zero8();
    };
    if (ONE) load_w4(0);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        w3[s] = *(const bf16x8*)&wl[off_w3t(nh) + row * kHid + 32 * s + 8 * q];
        w2[s] = *(const bf16x8*)&wl[off_w2t(nh) + row * kHid + 32 * s + 8 * q];
        // the inputs' gradients: event tile wave % 4, rows 16 (wave / 4) ..
        w1[s] = *(const bf16x8*)&wl[off_w1t(nh) + (16 * (wave >> 2) + e16) * kHid + 32 * s + 8 * q];
    }
    if (ONE) clear();
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const uint16_t* const on = r.on + tile * 3 * kThreads + tid;
        const uint32_t on1 = on[0], on2 = on[kThreads], on3 = on[2 * kThreads];
        __bf16* const db = r.dh + 2 * tile * 3 * kHid * 32;
        floatx4 acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = zero4();
        for (int c = 0; c < (ONE ? 1 : chunks); ++c) {
            const int rows = ONE ? n_out : min(8 * P, n_out - c * 8 * P), pairs = (rows + 1) >> 1;
            __syncthreads();  // readers of dt and a0
            if (!ONE) {
                load_w4(c);
                clear();
                __syncthreads();
            }
            // two parameters of eight events per thread: neighbouring lanes
            // write neighbouring words
            for (int i = tid; i < pairs * 8; i += kThreads) {
                const int g = i / pairs, p = 2 * (i - g * pairs);
                const __bf16* const src = r.d + ((2 * tile + (g >> 2)) * gr + c * 8 * P + p) * 32 + 8 * (g & 3);
                const bf16x8 u = *(const bf16x8*)src, v = p + 1 < rows ? *(const bf16x8*)(src + 32) : zero8();
#pragma unroll
                for (int x = 0; x < 8; ++x) {
                    bf16x2 w;
                    w[0] = u[x];
                    w[1] = v[x];
                    *(bf16x2*)&dt[(8 * g + x) * kDPitch + p] = w;
                }
            }
            __syncthreads();
#pragma unroll
            for (int s = 0; s < KB; ++s)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    acc[t] = mfma(w4[s], *(const bf16x8*)&dt[(16 * t + e16) * kDPitch + 32 * s + 8 * q], acc[t]);
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) store_masked(acc[t], on3 >> (4 * t), a0, 16 * t, wave, lane);
        __syncthreads();
        store_blocks(a0, db + 2 * kHid * 32, tid);
        auto back = [&](const bf16x8 (&w)[4], const __bf16* in, uint32_t m, __bf16* out) {
            bf16x8 x[NT][4];
#pragma unroll
            for (int t = 0; t < NT; ++t) load_act(in, 16 * t, lane, x[t]);
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] = mfma(w[s], x[t][s], s ? acc[t] : zero4());
#pragma unroll
            for (int t = 0; t < NT; ++t) store_masked(acc[t], m >> (4 * t), out, 16 * t, wave, lane);
        };
        back(w3, a0, on2, a1);
        __syncthreads();
        store_blocks(a1, db + kHid * 32, tid);
        back(w2, a1, on1, a0);
        __syncthreads();
        store_blocks(a0, db, tid);
        if (16 * (wave >> 2) < nh) {
            const int t = wave & 3;
            bf16x8 x[4];
            load_act(a0, 16 * t, lane, x);
            floatx4 g = zero4();
#pragma unroll
            for (int s = 0; s < 4; ++s) g = mfma(w1[s], x[s], g);
            const int64_t e = tile * EV + 16 * t + e16;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int k = 16 * (wave >> 2) + 4 * q + i;
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
// runs would fill more compute units, but write and add up as much again.
constexpr int kBlockH = 3 * kHid * 32, kBlockD = 16 * kGradTiles * 32, kBlockX = 32 * 32;  // elements
constexpr int kBlockElems = 2 * kBlockH + kBlockD + kBlockX;

__device__ __forceinline__ void copy_to_lds(const __bf16* __restrict__ src, __bf16* __restrict__ dst, int chunks, int wave,
                                            int lane) {
    for (int c = wave; c < chunks; c += kWaves)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + c * 512 + lane * 8),
                                         (__attribute__((address_space(3))) void*)(dst + c * 512), 16, 0, 0);
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
    auto frag = [&](const __bf16* m, int row) { return *(const bf16x8*)(m + row * 32 + mine); };
    auto sum8 = [](const bf16x8& v) {
        return (((float)v[0] + (float)v[1]) + ((float)v[2] + (float)v[3])) +
               (((float)v[4] + (float)v[5]) + ((float)v[6] + (float)v[7]));
    };
    auto stage = [&](int64_t k, __bf16* __restrict__ to) {
        copy_to_lds(r.d + (k * gr + row0) * 32, to, kBlockD / 512, wave, lane);
        copy_to_lds(r.h + k * kBlockH, to + kBlockD, kBlockH / 512, wave, lane);
        if (!HIDDEN) return;
        copy_to_lds(r.dh + k * kBlockH, to + kBlockD + kBlockH, kBlockH / 512, wave, lane);
        copy_to_lds(r.x0 + k * kBlockX, to + kBlockD + 2 * kBlockH, kBlockX / 512, wave, lane);
    };
    // the copies of block k to `next` run under the products of `d`: restrict
    // tells the compiler that reading the one need not wait for the other
    auto step = [&](const __bf16* __restrict__ d, __bf16* __restrict__ next, int64_t k) {
        stage(k, next);
        const __bf16 *const h = d + kBlockD, *const dh = h + kBlockH, *const x0 = dh + kBlockH;
        bf16x8 b[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) b[c] = frag(h, 2 * kHid + 16 * c);
#pragma unroll
        for (int g = 0; g < 3; ++g) {
            const bf16x8 a = frag(d, 128 * g + 16 * wave);
            s4[g] += sum8(a);
#pragma unroll
            for (int c = 0; c < 8; ++c) a4[g][c] = mfma(a, b[c], a4[g][c]);
        }
        // the last row tile: one column tile per wave
        const bf16x8 al = frag(d, 384);
        s24 += sum8(al);
        a24 = mfma(al, frag(h, 2 * kHid + 16 * wave), a24);
        if (!HIDDEN) return;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < 8; ++c) b[c] = frag(h, kHid + 16 * c);
        const bf16x8 x3 = frag(dh, 2 * kHid + 16 * wave);
        s3 += sum8(x3);
#pragma unroll
        for (int c = 0; c < 8; ++c) a3[c] = mfma(x3, b[c], a3[c]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < 8; ++c) b[c] = frag(h, 16 * c);
        const bf16x8 x2 = frag(dh, kHid + 16 * wave);
        s2 += sum8(x2);
#pragma unroll
        for (int c = 0; c < 8; ++c) a2[c] = mfma(x2, b[c], a2[c]);
        const bf16x8 x1 = frag(dh, 16 * wave);
        s1 += sum8(x1);
#pragma unroll
        for (int c = 0; c < 2; ++c) a1[c] = mfma(x1, frag(x0, 16 * c), a1[c]);
    };
    const int64_t k0 = blockIdx.x * chunk, k1 = min(blocks, k0 + chunk);
    if (k0 < k1) stage(k0, smem);
    for (int64_t k = k0; k < k1; ++k) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();  // block k is in LDS, the other buffer's readers are done
        const int cur = (int)(k - k0) & 1;
        step(smem + cur * kBlockElems, smem + (cur ^ 1) * kBlockElems, min(k + 1, k1 - 1));
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
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

}  // namespace

int flow_grad_rows(int nh, int K) { return grad_rows(nh, K); }

hipError_t launch_flow_spline_reverse(const FlowNet& fn, const FlowRev& r, int cu_count, hipStream_t s) {
    const bool keep = fn.nh <= kWaves;
    const size_t lds = reverse_lds(2 * fn.nh, keep ? fn.nh : 0);
    const dim3 g((unsigned)std::min<int64_t>((r.n + 63) / 64, cu_count)), t(kThreads);
    if (keep && fn.K == 16)
        k_flow_spline_reverse<true, true><<<g, t, lds, s>>>(fn, r);
    else if (keep)
        k_flow_spline_reverse<true, false><<<g, t, lds, s>>>(fn, r);
    else if (fn.K == 16)
        k_flow_spline_reverse<false, true><<<g, t, lds, s>>>(fn, r);
    else
        k_flow_spline_reverse<false, false><<<g, t, lds, s>>>(fn, r);
    return hipGetLastError();
}

int64_t flow_transposed_elems(int nh) { return transposed_elems(nh); }

hipError_t launch_flow_transpose(const FlowNet& fn, int layers, void* wt_t, hipStream_t s) {
    k_flow_transpose<<<dim3((unsigned)((transposed_elems(fn.nh) + 255) / 256), (unsigned)layers), 256, 0, s>>>(
        fn, (__bf16*)wt_t);
    return hipGetLastError();
}

hipError_t launch_flow_mlp_reverse(const FlowNet& fn, const FlowRev& r, const void* wt_t, int cu_count,
                                   hipStream_t s) {
    const unsigned grid = (unsigned)std::min<int64_t>((r.n + 63) / 64, cu_count);
    const size_t lds = sizeof(__bf16) * 64 * (kDPitch + 2 * kHid);
    if (fn.nh <= 8)
        k_flow_mlp_reverse<true><<<grid, kThreads, lds, s>>>(fn, r, (const __bf16*)wt_t);
    else
        k_flow_mlp_reverse<false><<<grid, kThreads, lds, s>>>(fn, r, (const __bf16*)wt_t);
    return hipGetLastError();
}

int flow_wgrad_splits(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>(128, n / 256)); }

hipError_t launch_flow_wgrad(const FlowNet& fn, const FlowRev& r, int splits, float* part, hipStream_t s) {
    const int64_t blocks = (r.n + 63) / 64 * 2, chunk = (blocks + splits - 1) / splits;
    k_flow_wgrad<true><<<(unsigned)splits, kThreads, 0, s>>>(fn, r, blocks, chunk, part);
    if (out_chunks(fn.nh) > 1)
        k_flow_wgrad<false><<<dim3((unsigned)splits, (unsigned)(out_chunks(fn.nh) - 1)), kThreads, 0, s>>>(fn, r, blocks,
                                                                                                        chunk, part);
    return hipGetLastError();
}

}  // namespace msx
