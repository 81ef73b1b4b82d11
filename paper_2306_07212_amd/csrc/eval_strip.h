// The evaluation of one narrow layer by one workgroup (the batched and the
// small-network kernel).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device.h"

namespace pcx {

// Step 1 (Sec. 4.2) for one layer of at most 64 neurons, by the whole
// workgroup on the matrix cores: each wave takes strips of 16 vertex rows and
// computes all 16 CT >= N columns of a strip with FP64 16x16x4 MFMAs (A lane l:
// row l%16, k l/16; B lane l: k l/16, column l%16; result lane l, value i:
// row l/16 + 4i, column l%16), its inputs and the weights read straight from
// memory (no LDS, no barrier: a wave reads every input of its rows before it
// writes them, so the evaluation can be in place). A chain of these MFMAs
// rounds as the sequential FMA chain over k from zero does (the padding of k
// adds a zero, which leaves any sum other than -0 unchanged, and a sum started
// at +0 becomes -0 only if a product underflows), and then + bias: the values
// are those of every other evaluation kernel, bit for bit.
// (Not inlined, and given plain pointers rather than the workgroup's Bufs, so
// that its registers and the Bufs stay out of the split's register allocation.)
// (The pointers are taken as global memory, so that the loads are global
// loads whose completion is counted in order, and every operand load is made
// unconditional, from a clamped in-bounds address, with the value selected
// after it: the loads of a round are all in flight together.)
typedef const __attribute__((address_space(1))) double gcdouble;
typedef const __attribute__((address_space(1))) uint64_t gcuint64;
typedef __attribute__((address_space(1))) double gdouble;
typedef __attribute__((address_space(1))) uint64_t guint64;

template <int CT, int T = kThreads>
__device__ __noinline__ void eval_mfma(double *Zo_, uint64_t *SGo_, int *ctr, int ZS,
                                       const double *in_, int in_stride, int relu, int V, int K, int N,
                                       const double *Wt_, const double *bias_, int Wd, int lw0) {
    gdouble *Zo = (gdouble *)Zo_;
    guint64 *SGo = (guint64 *)SGo_;
    gcuint64 *in = (gcuint64 *)in_, *Wt = (gcuint64 *)Wt_;
    gcdouble *bias = (gcdouble *)bias_;
    const int l = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = l & 15, q = l >> 4;
    double bv[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) bv[ct] = ct * 16 + r < N ? bias[ct * 16 + r] : 0.0;
    int zero = 0;
    for (int v0 = wave * 16; v0 < V; v0 += 16 * (T / 64)) {
        const bool arow = v0 + r < V;
        gcuint64 *hp = in + (size_t)(arow ? v0 + r : 0) * in_stride;
        dbl4 acc[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[ct] = dbl4{0.0, 0.0, 0.0, 0.0};
        // four k-steps of 4 per round, each with its own operand registers: a
        // step's operands for the next round are loaded right after its MFMAs
        // issue, three steps ahead of their use, as raw bits from clamped
        // in-bounds addresses; the zeros past K and the ReLU are applied when the
        // step is used, so no load waits on a condition
        uint64_t ar[4], br[4][CT];
        auto load = [&](int k0, uint64_t &a, uint64_t *bw) {
            const int k = k0 + q, kc = k < K ? k : K - 1;
            a = hp[kc];
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const int col = ct * 16 + r;
                bw[ct] = Wt[(size_t)kc * N + (col < N ? col : N - 1)];
            }
        };
#pragma unroll
        for (int st = 0; st < 4; ++st) load(4 * st, ar[st], br[st]);
        // (every round is whole: a step past K has zero weights, adding a zero
        // to the sum)
        for (int k0 = 0; k0 < K; k0 += 16) {
#pragma unroll
            for (int st = 0; st < 4; ++st) {
                const bool kin = k0 + 4 * st + q < K;
                const double h = __builtin_bit_cast(double, ar[st]);
                // (0 past K also here: an input that is infinite would make the zero weights' products NaN)
                const double af = relu ? (kin && h > 0.0 ? h : 0.0) : h;
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    const uint64_t m = (kin && ct * 16 + r < N) ? ~0ull : 0ull;
                    const double bf = __builtin_bit_cast(double, br[st][ct] & m);
                    acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(af, bf, acc[ct], 0, 0, 0);
                }
                load(k0 + 16 + 4 * st, ar[st], br[st]);
                // (keeps the loads here, in flight, rather than moved next to their use)
                asm volatile("" ::: "memory");
            }
        }
        // bias, store, and the layer's sign words (word p from tiles 2p and 2p+1)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int v = v0 + q + 4 * i;
            uint64_t pb[CT], nb[CT];
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const int col = ct * 16 + r;
                const bool ok = v < V && col < N;
                double z = 0.0;
                if (ok) {
                    z = acc[ct][i] + bv[ct];
                    Zo[(size_t)v * ZS + col] = z;
                    zero |= (z == 0.0);
                }
                pb[ct] = __ballot(ok && z > 0.0);
                nb[ct] = __ballot(ok && z < 0.0);
            }
            const int sh = 16 * q;
#pragma unroll
            for (int p = 0; p < (CT + 1) / 2; ++p) {
                if (r == p && v < V) {
                    uint32_t pos = (uint32_t)((pb[2 * p] >> sh) & 0xFFFFu);
                    uint32_t neg = (uint32_t)((nb[2 * p] >> sh) & 0xFFFFu);
                    if (2 * p + 1 < CT) {
                        pos |= (uint32_t)((pb[2 * p + 1] >> sh) & 0xFFFFu) << 16;
                        neg |= (uint32_t)((nb[2 * p + 1] >> sh) & 0xFFFFu) << 16;
                    }
                    SGo[(size_t)v * Wd + lw0 + p] = codes_of(pos, neg);
                }
            }
        }
    }
    if (zero) raise_flag(ctr, FLAG_ZERO_SIGN);
}

// a layer of N <= 64 neurons
template <int T>
__device__ __forceinline__ void eval_strips(const Bufs &b, int ZS, const double *in, int ins, int relu, int V, int K,
                                            int N, const double *Wt, const double *bias, int Wd, int lw0) {
    if (N <= 16) eval_mfma<1, T>(b.Z, b.SG, b.CTR, ZS, in, ins, relu, V, K, N, Wt, bias, Wd, lw0);
    else if (N <= 32) eval_mfma<2, T>(b.Z, b.SG, b.CTR, ZS, in, ins, relu, V, K, N, Wt, bias, Wd, lw0);
    else if (N <= 48) eval_mfma<3, T>(b.Z, b.SG, b.CTR, ZS, in, ins, relu, V, K, N, Wt, bias, Wd, lw0);
    else eval_mfma<4, T>(b.Z, b.SG, b.CTR, ZS, in, ins, relu, V, K, N, Wt, bias, Wd, lw0);
}

}  // namespace pcx
