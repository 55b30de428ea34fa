// Device side of the fused coupling layers (conditioner of hidden width 128 in
// BF16 or FP32, up to 16 spline bins): the layout that the kernels share.
//
// A workgroup of eight waves takes a tile of events.  Every product is formed
// with the weights as the left MFMA operand and the events as the right one
// (v_mfma_f32_16x16x32_bf16: lane l holds W[l % 16][8 (l / 16) + 0..7] and
// X[8 (l / 16) + 0..7][l % 16], and receives D[4 (l / 16) + 0..3][l % 16]; in
// FP32 eight v_mfma_f32_16x16x4_f32 take eight elements one by one, the
// columns of every 32 ordered so that a lane's eight stand together and the
// sum still runs over the columns in order), so a lane gets four neighbouring features of one event: an activation goes
// to LDS as one store, and the spline parameters of an event sit in
// the four lanes that share its column.  Wave w computes features 16 w .. 16 w
// + 15 of every hidden layer and the splines of transformed coordinates w, w +
// 8, ...
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "flow_launch.h"

namespace msx {
namespace flow {

template <class T>
using Vec8 = T __attribute__((ext_vector_type(8)));
template <class T>
using Vec4 = T __attribute__((ext_vector_type(4)));
template <class T>
using Vec2 = T __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 8;               // waves per workgroup
constexpr int kThreads = 64 * kWaves;
constexpr int kHid = kFusedHidden;      // hidden width: 16 features per wave
static_assert(kHid == 16 * kWaves, "one 16-feature tile per wave");

// Where column k of an operand stands.
template <class T>
__device__ __forceinline__ int column(int k) {
    return sizeof(T) == 2 ? k : f32_operand_index(k);
}

// Element c of row r of an activation tile in LDS, [events][128]: the 16-byte
// chunks of a row are permuted by chunk ^ (r mod 16), so the operand reads
// (one chunk column of many rows) and the stores (neighbouring chunks, or
// halves of one, of sixteen rows) each touch every bank once; with padded rows
// instead the reads took two passes.
template <class T>
__device__ __forceinline__ int act_at(int row, int c) {
    constexpr int L = sizeof(T) == 2 ? 3 : 2;  // log2 of the elements of a chunk
    return row * kHid + (((c >> L) ^ (row & 15)) << L) + (c & ((1 << L) - 1));
}
// The same for the conditioning inputs, [events][kCond] (zero beyond nh).
constexpr int kCond = kFlowMaxHalf;
template <class T>
__device__ __forceinline__ int cond_at(int row, int c) {
    if (sizeof(T) == 2) return row * kCond + (((c >> 3) ^ ((row >> 2) & 3)) << 3) + (c & 7);
    return row * kCond + (((c >> 2) ^ ((row >> 1) & 7)) << 2) + (c & 3);
}
// Eight elements from column c, a multiple of 8 (two chunks in FP32).
__device__ __forceinline__ Vec8<__bf16> act8(const __bf16* act, int row, int c) {
    return *(const Vec8<__bf16>*)&act[act_at<__bf16>(row, c)];
}
__device__ __forceinline__ Vec8<__bf16> cond8(const __bf16* cond, int row, int c) {
    return *(const Vec8<__bf16>*)&cond[cond_at<__bf16>(row, c)];
}
__device__ __forceinline__ Vec8<float> join(const floatx4& a, const floatx4& b) {
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}
__device__ __forceinline__ Vec8<float> act8(const float* act, int row, int c) {
    return join(*(const floatx4*)&act[act_at<float>(row, c)], *(const floatx4*)&act[act_at<float>(row, c + 4)]);
}
__device__ __forceinline__ Vec8<float> cond8(const float* cond, int row, int c) {
    return join(*(const floatx4*)&cond[cond_at<float>(row, c)], *(const floatx4*)&cond[cond_at<float>(row, c + 4)]);
}
// Eight elements from memory, 16-byte aligned.
__device__ __forceinline__ Vec8<__bf16> load8(const __bf16* p) { return *(const Vec8<__bf16>*)p; }
__device__ __forceinline__ Vec8<float> load8(const float* p) { return join(*(const floatx4*)p, *(const floatx4*)(p + 4)); }

constexpr float kMinW = 1e-3f, kMinH = 1e-3f, kMinD = 1e-3f;

// Coupling mask of a layer: conditioning coordinate k is c0 + cs k, the
// transformed coordinate j is t0 + ts j.
struct Mask {
    int c0, cs, t0, ts;
};
__device__ __forceinline__ Mask mask_of(int layer, int nh) {
    const int md = layer & 3;
    Mask m;
    m.cs = m.ts = md < 2 ? 1 : 2;
    m.t0 = md == 0 ? 0 : (md == 1 ? nh : md - 2);
    m.c0 = md == 0 ? nh : (md == 1 ? 0 : 3 - md);
    return m;
}

// The conditioning index of coordinate c, -1 if the layer transforms it.
__device__ __forceinline__ int cond_index(const Mask& m, int nh, int c) {
    const int r = c - m.c0;
    if (m.cs == 2) return r & 1 ? -1 : r >> 1;
    return r >= 0 && r < nh ? r : -1;
}

__device__ __forceinline__ floatx4 mfma(const Vec8<__bf16>& a, const Vec8<__bf16>& b, const floatx4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ floatx4 mfma(const Vec8<float>& a, const Vec8<float>& b, floatx4 c) {
#pragma unroll
    for (int i = 0; i < 8; ++i) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[i], c, 0, 0, 0);
    return c;
}
__device__ __forceinline__ floatx4 zero4() { return floatx4{0.0f, 0.0f, 0.0f, 0.0f}; }
template <class T>
__device__ __forceinline__ Vec8<T> zero8() {
    Vec8<T> r;
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = (T)0.0f;
    return r;
}

// 16 bytes per lane from memory to consecutive words of LDS from dst (the same
// for all lanes), without registers; there after landed().
__device__ __forceinline__ void copy16_to_lds(const __bf16* src, __bf16* dst) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                     (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}
__device__ __forceinline__ void landed() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// An offset of zero that the compiler takes for a new value wherever it is
// asked for: loads behind it stay where they are written.
__device__ __forceinline__ int here() {
    int z = 0;
    asm volatile("" : "+s"(z));
    return z;
}

// A wave's weights of the hidden layers.  BF16: in registers over all tiles of
// a layer.  FP32: the square layers' (64 registers) are
// loaded again at the start of every tile, which is little beside the FP32
// matrix rate (0.5 us of 20 us per 64 events).
template <class T>
struct HidW {
    Vec8<T> w1, w2[4], w3[4];
    const T *p2, *p3;
    __device__ __forceinline__ void load() {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            w2[s] = load8(p2 + 32 * s);
            w3[s] = load8(p3 + 32 * s);
        }
    }
    __device__ __forceinline__ void per_layer() {
        if (sizeof(T) == 2) load();
    }
    __device__ __forceinline__ void per_tile() {
        if (sizeof(T) == 2) return;
        const int z = here();
        p2 += z;
        p3 += z;
        load();
    }
};

template <class T>
__device__ __forceinline__ HidW<T> load_hidden(const FlowNet& fn, int layer, int wave, int lane) {
    const T* W = (const T*)fn.wt + layer * fn.per_t;
    const int r16 = lane & 15, q = lane >> 4, row = 16 * wave + r16;
    HidW<T> h;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int k = sizeof(T) == 2 ? 8 * q + i : 4 * i + q;
        const T v = W[fn.off[0] + row * fn.nh + min(k, fn.nh - 1)];
        h.w1[i] = k < fn.nh ? v : (T)0.0f;
    }
    h.p2 = &W[fn.off[2] + row * kHid + 8 * q];
    h.p3 = &W[fn.off[4] + row * kHid + 8 * q];
    h.per_layer();
    return h;
}

// The rows of W4 that 16-row tile m of a coordinate multiplies: tile 0 the
// widths, 1 the heights, 2 the slopes 0..15, 3 slope 16.  Rows without a
// parameter repeat an existing one; nothing reads their products.
__device__ __forceinline__ int param_row(int m, int r, int K) {
    if (m < 2) return m * K + min(r, K - 1);
    return min(2 * K + 16 * (m - 2) + r, 3 * K);
}
// W4 (BF16) in LDS, per coordinate: tiles 0..2 in fragment order (a wave's read is 64
// consecutive 16-byte words), then the row of slope 16, which all rows of
// tile 3 repeat.
constexpr int kOutElems = 48 * kHid + kHid;
__device__ __forceinline__ void load_out(const FlowNet& fn, int layer, __bf16* __restrict__ w4, int tid) {
    const __bf16* W = (const __bf16*)fn.wt + layer * fn.per_t + fn.off[6];
    const int P = 3 * fn.K + 1;
    for (int i = tid; i < fn.nh * 49 * 16; i += kThreads) {
        const int j = i / (49 * 16), c = i - j * (49 * 16);  // 16-byte word c of coordinate j
        const int m = c >> 8, s = (c >> 6) & 3, r = c & 15, q = (c >> 4) & 3;
        const int row = m < 3 ? param_row(m, r, fn.K) : param_row(3, 0, fn.K), k = m < 3 ? 32 * s + 8 * q : 8 * (c & 15);
        *(Vec8<__bf16>*)&w4[j * kOutElems + 8 * c] = load8(&W[(j * P + row) * kHid + k]);
    }
}
// The same copied straight to LDS, without registers and all words in flight at
// once; this wave's are there after landed(), the workgroup's after a barrier.
// The places that a lane copies from are the same in every layer.
constexpr int kOutRounds = (kWaves * kOutElems / 8 + kThreads - 1) / kThreads;
constexpr int kOutKept = kOutRounds * kThreads * 8;  // elements: up to eight coordinates, in whole rounds
struct OutCopy {
    int from[kOutRounds];
    __device__ __forceinline__ OutCopy(const FlowNet& fn, int wave, int lane) {
        const int words = fn.nh * (kOutElems / 8);
#pragma unroll
        for (int it = 0; it < kOutRounds; ++it) {
            const int i = min((it * kWaves + wave) * 64 + lane, words - 1);
            const int j = i / (kOutElems / 8), c = i - j * (kOutElems / 8);  // 16-byte word c of coordinate j
            const int m = c >> 8, s = (c >> 6) & 3, r = c & 15, q = (c >> 4) & 3;
            const int row = m < 3 ? param_row(m, r, fn.K) : param_row(3, 0, fn.K), k = m < 3 ? 32 * s + 8 * q : 8 * r;
            from[it] = (j * (3 * fn.K + 1) + row) * kHid + k;
        }
    }
    __device__ __forceinline__ void operator()(const FlowNet& fn, int layer, __bf16* w4, int wave) const {
        const __bf16* W = (const __bf16*)fn.wt + layer * fn.per_t + fn.off[6];
#pragma unroll
        for (int it = 0; it < kOutRounds; ++it) {
            const int base = (it * kWaves + wave) * 64;
            if (base < fn.nh * (kOutElems / 8)) copy16_to_lds(W + from[it], &w4[base * 8]);
        }
    }
};
__device__ __forceinline__ Vec8<__bf16> out_fragment(const __bf16* w4, int j, int m, int s, int lane) {
    const __bf16* c = w4 + j * kOutElems;
    return load8(m < 3 ? c + ((m * 4 + s) * 64 + lane) * 8 : c + 48 * kHid + 32 * s + 8 * (lane >> 4));
}

// The biases that a lane adds: hidden(l) to features 16 wave + 4 (lane / 16) ..
// + 3 of hidden layer l, out(j, m) to rows 4 (lane / 16) .. + 3 of tile m of
// coordinate j.  From memory:
struct MemoryBias {
    const float* P;
    int off1, off3, off5, off7, K, wave, q;
    __device__ __forceinline__ MemoryBias(const FlowNet& fn, int layer, int wave, int lane)
        : P(fn.p + layer * fn.per), off1(fn.off[1]), off3(fn.off[3]), off5(fn.off[5]), off7(fn.off[7]), K(fn.K),
          wave(wave), q(lane >> 4) {}
    __device__ __forceinline__ floatx4 hidden(int l) const {
        const float* b = P + (l == 0 ? off1 : (l == 1 ? off3 : off5)) + 16 * wave + 4 * q;
        return floatx4{b[0], b[1], b[2], b[3]};
    }
    __device__ __forceinline__ floatx4 out(int j, int m) const {
        const float* b = P + off7 + j * (3 * K + 1);
        floatx4 o;
#pragma unroll
        for (int x = 0; x < 4; ++x) o[x] = b[param_row(m, 4 * q + x, K)];
        return o;
    }
};
// From registers, a wave's hidden layers and (KEEP) its one coordinate; other
// coordinates from memory.
template <bool KEEP>
struct RegisterBias {
    MemoryBias mem;
    floatx4 h[3], o[4];
    __device__ __forceinline__ RegisterBias(const FlowNet& fn, int layer, int wave, int lane)
        : mem(fn, layer, wave, lane) {
#pragma unroll
        for (int l = 0; l < 3; ++l) h[l] = mem.hidden(l);
        if (KEEP) {
#pragma unroll
            for (int m = 0; m < 4; ++m) o[m] = mem.out(min(wave, fn.nh - 1), m);
        }
    }
    __device__ __forceinline__ floatx4 hidden(int l) const { return h[l]; }
    __device__ __forceinline__ floatx4 out(int j, int m) const { return KEEP ? o[m] : mem.out(j, m); }
};
// The same from LDS: 28 registers fewer over all tiles, for four or five more
// LDS reads.
constexpr int kBiases = 3 * kHid + kWaves * 64;  // floats
template <bool KEEP>
struct LdsBias {
    MemoryBias mem;
    const float* lb;
    __device__ __forceinline__ LdsBias(const FlowNet& fn, int layer, int wave, int lane, float* lds)
        : mem(fn, layer, wave, lane), lb(lds + 4 * (lane >> 4)) {
        const int tid = 64 * wave + lane;
        for (int i = tid; i < 3 * kHid; i += kThreads)
            lds[i] = mem.P[fn.off[2 * (i / kHid) + 1] + (i & (kHid - 1))];
        static_assert(kThreads == kWaves * 64, "one bias of a coordinate per thread");
        lds[3 * kHid + tid] =
            mem.P[fn.off[7] + min(wave, fn.nh - 1) * (3 * fn.K + 1) + param_row((tid >> 4) & 3, tid & 15, fn.K)];
    }
    __device__ __forceinline__ floatx4 hidden(int l) const {
        return *(const floatx4*)&lb[here() + l * kHid + 16 * mem.wave];
    }
    __device__ __forceinline__ floatx4 out(int j, int m) const {
        return KEEP ? *(const floatx4*)&lb[here() + 3 * kHid + j * 64 + m * 16] : mem.out(j, m);
    }
};

// Four neighbouring columns from c of an activation row.
__device__ __forceinline__ void store4(const Vec4<__bf16>& v, __bf16* __restrict__ act, int row, int c) {
    *(Vec4<__bf16>*)&act[act_at<__bf16>(row, c)] = v;
}
__device__ __forceinline__ void store4(const Vec4<float>& v, float* __restrict__ act, int row, int c) {
#pragma unroll
    for (int x = 0; x < 4; ++x) act[act_at<float>(row, column<float>(c + x))] = v[x];
}

// The activations of the wave's 16 features for the 16 events from row r0:
// bias, ReLU, conversion, one store per lane.  Returns which are positive.
template <class T>
__device__ __forceinline__ uint32_t store_act(const floatx4& acc, const floatx4& bias, T* __restrict__ act, int r0,
                                              int wave, int lane) {
    Vec4<T> v;
    uint32_t on = 0;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        v[x] = (T)fmaxf(acc[x] + bias[x], 0.0f);
        on |= (float)v[x] > 0.0f ? 1u << x : 0u;
    }
    store4(v, act, r0 + (lane & 15), 16 * wave + 4 * (lane >> 4));
    return on;
}

// The four right-hand fragments (128 features) of the 16 events from row r0.
template <class T>
__device__ __forceinline__ void load_act(const T* __restrict__ act, int r0, int lane, Vec8<T> (&b)[4]) {
#pragma unroll
    for (int s = 0; s < 4; ++s) b[s] = act8(act, r0 + (lane & 15), 32 * s + 8 * (lane >> 4));
}

// acc[t] = W X of the wave's 16 rows and the NT 16-event tiles of `in`.
template <int NT, class T>
__device__ __forceinline__ void square(const Vec8<T> (&w)[4], const T* in, int lane, floatx4 (&acc)[NT]) {
    Vec8<T> x[NT][4];
#pragma unroll
    for (int t = 0; t < NT; ++t) load_act(in, 16 * t, lane, x[t]);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = mfma(w[s], x[t][s], s ? acc[t] : zero4());
}

// x[t] of four 16-event tiles, where lane 16 q + e holds item q of event e, to
// items x[q] of lane 16 t + e's own event: the 4 x 4 transposition of (tile,
// row of 16 lanes).  A swap exchanges the halves (or alternate rows) of two
// registers, so four registers take four instructions.
__device__ __forceinline__ void transpose_rows(uint32_t (&x)[4]) {
    const auto a = __builtin_amdgcn_permlane32_swap(x[0], x[2], false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(x[1], x[3], false, false);
    const auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
    const auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
    x[0] = c[0];
    x[1] = c[1];
    x[2] = d[0];
    x[3] = d[1];
}

// The unconstrained spline parameters of one (event, coordinate) in a lane.
struct Theta {
    float w[16], h[16], s[17];
};
// From the accumulators of NT tiles (lane 16 q + e: parameters 4 q .. 4 q + 3
// of each 16-row tile, event e) to lane 16 t + e: all parameters of its event.
// With fewer than four tiles the remaining rows repeat them.
template <int NT>
__device__ __forceinline__ Theta gather_theta(const floatx4 (&acc)[NT][4]) {
    Theta th;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            uint32_t r[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) r[t] = __float_as_uint(acc[t % NT][m][x]);
            transpose_rows(r);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float v = __uint_as_float(r[q]);
                if (m == 0) th.w[4 * q + x] = v;
                if (m == 1) th.h[4 * q + x] = v;
                if (m == 2) th.s[4 * q + x] = v;
            }
        }
    }
    uint32_t r[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) r[t] = __float_as_uint(acc[t % NT][3][0]);
    transpose_rows(r);
    th.s[16] = __uint_as_float(r[0]);
    return th;
}

// One 128 -> 128 layer: the wave's 16 features of every event of the tile.
// Returns which are positive, four bits per 16-event tile.
template <int NT, class T>
__device__ __forceinline__ uint32_t hidden_layer(const Vec8<T> (&w)[4], const floatx4& bias, const T* in, T* out, int wave,
                                                 int lane) {
    floatx4 acc[NT];
    square<NT>(w, in, lane, acc);
    uint32_t on = 0;
#pragma unroll
    for (int t = 0; t < NT; ++t) on |= store_act(acc[t], bias, out, 16 * t, wave, lane) << (4 * t);
    return on;
}

// The spline parameters of coordinate j from the last activation; the output
// weights from LDS (KEEP) or from memory.
template <int NT, bool KEEP, class T, class B>
__device__ __forceinline__ Theta output_layer(const FlowNet& fn, int layer, const T* a, const T* w4, const B& bias,
                                              int j, int K, int lane) {
    const T* const w4g = (const T*)fn.wt + layer * fn.per_t + fn.off[6];
    floatx4 acc[NT][4];
    if constexpr (sizeof(T) == 2) {
        Vec8<T> x[NT][4];
#pragma unroll
        for (int t = 0; t < NT; ++t) load_act(a, 16 * t, lane, x[t]);
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int row = j * (3 * K + 1) + param_row(m, lane & 15, K);
            Vec8<T> w[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                if constexpr (KEEP)
                    w[s] = out_fragment(w4, j, m, s, lane);
                else
                    w[s] = load8(&w4g[row * kHid + 32 * s + 8 * (lane >> 4)]);
            }
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t][m] = mfma(w[s], x[t][s], s ? acc[t][m] : zero4());
        }
    } else {
        // the weights of a step are in flight during the step before
        const T* const wj = w4g + here() + 8 * (lane >> 4);
        auto weights = [&](int s, Vec8<T>(&w)[4]) {
#pragma unroll
            for (int m = 0; m < 4; ++m) w[m] = load8(&wj[(j * (3 * K + 1) + param_row(m, lane & 15, K)) * kHid + 32 * s]);
        };
        Vec8<T> w[2][4];
        weights(0, w[0]);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (s < 3) weights(s + 1, w[(s + 1) & 1]);
            Vec8<T> x[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) x[t] = act8(a, 16 * t + (lane & 15), 32 * s + 8 * (lane >> 4));
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t][m] = mfma(w[s & 1][m], x[t], s ? acc[t][m] : zero4());
        }
    }
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const floatx4 b = bias.out(j, m);
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t][m] += b;
    }
    return gather_theta<NT>(acc);
}

// softplus(x) = max(x, 0) + log(1 + e^-|x|) through the hardware's exp2 and
// log2: absolute error about 1e-7, against knot slopes of at least kMinD
__device__ __forceinline__ float softplus_f(float x) {
    return x > 20.0f ? x : fmaxf(x, 0.0f) + __logf(1.0f + __expf(-fabsf(x)));
}
__device__ __forceinline__ float slope_shift() { return logf(expm1f(1.0f - kMinD)); }

// The bin that a value falls in: left knot, width, height and the slopes on
// both sides.
struct Bin {
    int k;
    float x0, w, y0, h, d0, d1;
};

// The largest of 16 values (v_max3: the compiler's own maxima first quiet
// every operand that it cannot prove to be a number).
__device__ __forceinline__ float max16(const float (&x)[16]) {
    auto max3 = [](float a, float b, float c) {
        float r;
        asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
        return r;
    };
    const float a = max3(x[0], x[1], x[2]), b = max3(x[3], x[4], x[5]), c = max3(x[6], x[7], x[8]);
    const float d = max3(x[9], x[10], x[11]), e = max3(x[12], x[13], x[14]);
    return max3(max3(a, b, c), max3(d, e, x[15]), x[15]);
}

// Exponentials of the widths / heights in place of their parameters, and
// their sums.  Sixteen bins (K16) use the hardware's exp2: the sums
// normalise, so its ulp-level error cancels to first order; other counts keep
// expf.
template <bool K16>
__device__ __forceinline__ void spline_exp(Theta& th, int K, float& sw, float& sh) {
    float mw = th.w[0], mh = th.h[0];
    if (K16) {
        mw = max16(th.w);
        mh = max16(th.h);
    } else {
#pragma unroll
        for (int i = 1; i < 16; ++i) {
            if (i < K) {
                mw = fmaxf(mw, th.w[i]);
                mh = fmaxf(mh, th.h[i]);
            }
        }
    }
    sw = 0.0f;
    sh = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        if (K16 || i < K) {
            th.w[i] = K16 ? __expf(th.w[i] - mw) : expf(th.w[i] - mw);
            th.h[i] = K16 ? __expf(th.h[i] - mh) : expf(th.h[i] - mh);
            sw += th.w[i];
            sh += th.h[i];
        } else {
            th.w[i] = th.h[i] = 0.0f;
        }
    }
}

// Keeps the upper or the lower half of 2 HALF bins, the one that v lies in.
template <bool BY_Y, int HALF>
__device__ __forceinline__ void halve(float v, float (&X)[17], float (&Y)[17], float (&S)[17], int& k) {
    const bool up = v >= (BY_Y ? Y[HALF] : X[HALF]);
    k += up ? HALF : 0;
#pragma unroll
    for (int i = 0; i <= HALF; ++i) {
        X[i] = up ? X[i + HALF] : X[i];
        Y[i] = up ? Y[i + HALF] : Y[i];
        S[i] = up ? S[i + HALF] : S[i];
    }
}

// The bin of v among the x knots (or, BY_Y, the y knots) after spline_exp;
// d0 and d1 are still the unconstrained slopes.
template <bool BY_Y, bool K16>
__device__ __forceinline__ Bin spline_find(const Theta& th, int K, float v, float sw, float sh) {
    const float cw = (1.0f - (K16 ? 16 : K) * kMinW) / sw, ch = (1.0f - (K16 ? 16 : K) * kMinH) / sh;
    Bin b{};
    if (K16) {
        // knots, then the bin by four halvings: the knots increase strictly
        // (every bin is at least kMinW wide), so the last knot at or below v
        // is the one a scan would keep
        float X[17], Y[17], S[17];
        X[0] = Y[0] = 0.0f;
#pragma unroll
        for (int i = 0; i < 15; ++i) {
            X[i + 1] = X[i] + (kMinW + cw * th.w[i]);
            Y[i + 1] = Y[i] + (kMinH + ch * th.h[i]);
        }
        X[16] = Y[16] = 1.0f;
#pragma unroll
        for (int i = 0; i < 17; ++i) S[i] = th.s[i];
        b.k = 0;
        halve<BY_Y, 8>(v, X, Y, S, b.k);
        halve<BY_Y, 4>(v, X, Y, S, b.k);
        halve<BY_Y, 2>(v, X, Y, S, b.k);
        halve<BY_Y, 1>(v, X, Y, S, b.k);
        b.x0 = X[0];
        b.w = X[1] - X[0];
        b.y0 = Y[0];
        b.h = Y[1] - Y[0];
        b.d0 = S[0];
        b.d1 = S[1];
    } else {
        float cx = 0.0f, cy = 0.0f;
        b.d0 = th.s[0];
        b.d1 = th.s[1];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            if (i >= K) continue;
            const float xl = cx, yl = cy;
            cx = i == K - 1 ? 1.0f : cx + (kMinW + cw * th.w[i]);
            cy = i == K - 1 ? 1.0f : cy + (kMinH + ch * th.h[i]);
            if (i == 0 || v >= (BY_Y ? yl : xl)) {
                b.k = i;
                b.x0 = xl;
                b.w = cx - xl;
                b.y0 = yl;
                b.h = cy - yl;
                b.d0 = th.s[i];
                b.d1 = th.s[i + 1];
            }
        }
    }
    return b;
}
__device__ __forceinline__ void spline_slopes(Bin& b) {
    const float s0 = slope_shift();
    b.d0 = kMinD + softplus_f(b.d0 + s0);
    b.d1 = kMinD + softplus_f(b.d1 + s0);
}

__device__ __forceinline__ float spline_slope(const Bin& b, float xi) {
    const float s = b.h / b.w;
    const float om = xi * (1.0f - xi);
    const float den = s + (b.d1 + b.d0 - 2.0f * s) * om;
    return s * s * (b.d1 * xi * xi + 2.0f * s * om + b.d0 * (1.0f - xi) * (1.0f - xi)) / (den * den);
}

// The rational-quadratic spline (or its inverse) of one (event, coordinate):
// the new value; ld receives log |d out / d v|.
template <bool INV>
__device__ __forceinline__ float spline_value(const Bin& b, float v, float& ld) {
    const float sl = b.h / b.w;
    const float kap = b.d1 + b.d0 - 2.0f * sl;
    if (!INV) {
        const float xi = (v - b.x0) / b.w;
        const float om = xi * (1.0f - xi);
        ld = logf(spline_slope(b, xi));
        return b.y0 + b.h * (sl * xi * xi + b.d0 * om) / (sl + kap * om);
    }
    const float dy = v - b.y0;
    const float qa = b.h * (sl - b.d0) + dy * kap;
    const float qb = b.h * b.d0 - dy * kap;
    const float qc = -sl * dy;
    const float disc = fmaxf(qb * qb - 4.0f * qa * qc, 0.0f);
    const float xi = 2.0f * qc / (-qb - sqrtf(disc));
    ld = -logf(spline_slope(b, xi));
    return b.x0 + xi * b.w;
}

}  // namespace flow
}  // namespace msx
