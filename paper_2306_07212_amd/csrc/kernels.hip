// Device kernels of libpcx.so: edge subdivision (Berzins 2023, Sec. 4.2) on
// gfx950. One neuron step is: the split of its list of splitting edges
// (interpolation, new vertices, 2-face keys into the hash table; steps 4-5), then
// the pairing into intersecting edges (step 5), which also lists the next neuron's
// splitting edges (step 3): two launches, three in large steps. With sort pairing
// the list is compacted, the keys sorted and the pairs grouped in launches of their
// own. Each layer starts with the pre-activation evaluation (step 1) and a scan that
// records, per edge, the first neuron of the layer whose sign differs at its
// endpoints (steps 2-3), and compacts the first neuron's list.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>

#include "device.h"
#include "internal.h"

namespace pcx {

// A per-step kernel of global step `step` does nothing while a hard failure is
// flagged or an earlier step's pairing failed (the host redoes that pairing
// exactly, then queues the later steps again). A step's own pairing failure
// does not stop its split, which the exact pass needs whole.
__device__ __forceinline__ bool step_blocked(const int *ctr, int step) {
    return ctr[CTR_FLAGS] != 0 || ctr[CTR_PFAIL] < step;
}

// The counters a per-step kernel starts from, read at once: a test of the flags
// before the other loads would put another round trip to memory on the chain of
// every launch. (The empty asm keeps the loads together, before the test.)
struct StepCounters {
    int flags, pfail, V0, E0, S;
    __device__ __forceinline__ StepCounters(const int *ctr, int par)
        : flags(ctr[CTR_FLAGS]), pfail(ctr[CTR_PFAIL]), V0(ctr[CTR_V + par]), E0(ctr[CTR_E + par]), S(ctr[CTR_S]) {
        flags = __builtin_amdgcn_readfirstlane(flags);
        pfail = __builtin_amdgcn_readfirstlane(pfail);
        V0 = __builtin_amdgcn_readfirstlane(V0);
        E0 = __builtin_amdgcn_readfirstlane(E0);
        S = __builtin_amdgcn_readfirstlane(S);
        asm volatile("" : "+s"(flags), "+s"(pfail), "+s"(V0), "+s"(E0), "+s"(S));
    }
};

// --------------------------------------------------------- step 0: the box

// 2^D corners (bit j of the corner id picks hi_j) and D 2^(D-1) edges between
// corners at Hamming distance one. Box entries: 2j is x_j - lo_j (zero at
// lo_j), 2j+1 is hi_j - x_j (zero at hi_j).
__global__ void k_init_box(Bufs b, int D, int Wd, const double *__restrict__ lo, const double *__restrict__ hi) {
    const int nc = 1 << D;
    const int ne = D << (D - 1);
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nc + ne; i += gridDim.x * blockDim.x) {
        if (i < nc) {
            uint64_t w0 = 0;
            for (int j = 0; j < D; ++j) {
                const int up = (i >> j) & 1;
                b.X[(size_t)i * D + j] = up ? hi[j] : lo[j];
                w0 |= (uint64_t)(up ? 1 : 0) << (4 * j);      // entry 2j:   + unless at lo
                w0 |= (uint64_t)(up ? 0 : 1) << (4 * j + 2);  // entry 2j+1: + unless at hi
            }
            b.SG[(size_t)i * Wd] = w0;
            for (int w = 1; w < Wd; ++w) b.SG[(size_t)i * Wd + w] = 0;
        } else {
            const int e = i - nc;
            const int j = e >> (D - 1);
            const int r = e & ((1 << (D - 1)) - 1);
            const int c = ((r >> j) << (j + 1)) | (r & ((1 << j) - 1));
            b.EDG[e] = make_int2(c, c | (1 << j));
        }
    }
}

void launch_init_box(const Bufs &b, int D, int Wd, const double *lo, const double *hi, hipStream_t st) {
    const int n = (1 << D) + (D << (D - 1));
    const int grid = (n + kThreads - 1) / kThreads;
    hipLaunchKernelGGL(k_init_box, dim3(grid), dim3(kThreads), 0, st, b, D, Wd, lo, hi);
}

// ------------------------------------------------- step 1: pre-activations
//
// Z[v] = W h(v) + b with h(v) = ReLU(in[v]) (or in[v] itself for the first
// layer). A workgroup owns kGemmRows vertex rows and all N <= 256 outputs, so
// with in == Z the evaluation runs in place: every read of the workgroup's
// rows happens before its first write. Thread (tv, tc) holds 4 rows x 8
// columns {tc, tc+32, ..., tc+224}; this lane order makes the LDS reads of W
// conflict-free and builds each 32-entry sign word from two wave ballots. The
// epilogue writes the layer's sign entries (Sec. 3.4: the sign of the
// pre-activation) into the layer's own words of each row.
__global__ __launch_bounds__(kThreads) void k_gemm(Bufs b, int ZS, const double *in, int in_stride, int relu,
                                                    int V, int K, int N, const double *__restrict__ Wt,
                                                    const double *__restrict__ bias, int Wd, int lw0) {
    __shared__ double hs[kGemmRows][kGemmK + 1];
    __shared__ double ws[kGemmK][kMaxWidth];
    gemm_tile(b, ZS, in, in_stride, relu, V, K, N, Wt, bias, Wd, lw0, blockIdx.x * kGemmRows, hs, ws);
}

// ---- rows of an evaluation in spatial order
//
// Vertices that lie close together share most of the previous layer's dead
// neurons (h = 0): in 64 neighbouring rows of the 768-neuron network about 45%
// of the columns are zero in all of them, and the matrix-core kernel below
// skips those. The rows are binned by a grid of 2^12 cells over the domain's
// bounding box (12 bits of the coordinates shared out over the axes); the order
// inside a bin does not matter, since every row's result is its own. Bound:
// one read of the coordinates a pass, two passes and 4 B a row written
// (0.35 ms over the 768-neuron network's two layers, 14.2M rows). In their own
// order 64 rows there leave 78 to 90% of the columns, by this grid 55 to 57%,
// by one of 2^15 cells 54 to 55%. From kBinRows rows and kBinWork products on:
// below, the four launches cost more than they save.
constexpr int kBins = 4096, kBinThreads = 1024;

__device__ __forceinline__ int bin_of(const double *__restrict__ x, const EvalGrid &g, int D) {
    int key = 0;
    for (int d = 0; d < D; ++d) {
        const int n = 1 << g.bits[d];
        const int i = (int)((x[d] - g.lo[d]) * g.scale[d]);  // (out of range, also NaN: an end cell)
        key = key * n + min(max(i, 0), n - 1);
    }
    return key;
}

// rows of workgroup blk
__device__ __forceinline__ void bin_rows(int V, int &v0, int &v1) {
    const int per = (V + (int)gridDim.x - 1) / (int)gridDim.x;
    v0 = min(V, (int)blockIdx.x * per);
    v1 = min(V, v0 + per);
}

__global__ __launch_bounds__(kBinThreads) void k_bin_count(const double *__restrict__ X, EvalGrid g, int D, int V,
                                                           int *__restrict__ cnt) {
    __shared__ int h[kBins];
    const int t = threadIdx.x;
    for (int i = t; i < kBins; i += kBinThreads) h[i] = 0;
    __syncthreads();
    int v0, v1;
    bin_rows(V, v0, v1);
    for (int v = v0 + t; v < v1; v += kBinThreads) atomicAdd(&h[bin_of(X + (size_t)v * D, g, D)], 1);
    __syncthreads();
    for (int i = t; i < kBins; i += kBinThreads)
        if (h[i]) atomicAdd(&cnt[i], h[i]);
}

// counts -> first places (exclusive prefix sums), by one workgroup
__global__ __launch_bounds__(kBinThreads) void k_bin_scan(int *cnt) {
    __shared__ int s_w[kBinThreads / 64];
    constexpr int per = kBins / kBinThreads;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    int x[per], mine = 0;
#pragma unroll
    for (int i = 0; i < per; ++i) {
        x[i] = cnt[t * per + i];
        mine += x[i];
    }
    int incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    if (lane == 63) s_w[wave] = incl;
    __syncthreads();
    int run = incl - mine;
    for (int w = 0; w < wave; ++w) run += s_w[w];
#pragma unroll
    for (int i = 0; i < per; ++i) {
        cnt[t * per + i] = run;
        run += x[i];
    }
}

__global__ __launch_bounds__(kBinThreads) void k_bin_scatter(const double *__restrict__ X, EvalGrid g, int D, int V,
                                                             int *__restrict__ next, int *__restrict__ perm) {
    __shared__ int h[kBins];
    const int t = threadIdx.x;
    for (int i = t; i < kBins; i += kBinThreads) h[i] = 0;
    __syncthreads();
    int v0, v1;
    bin_rows(V, v0, v1);
    for (int v = v0 + t; v < v1; v += kBinThreads) atomicAdd(&h[bin_of(X + (size_t)v * D, g, D)], 1);
    __syncthreads();
    for (int i = t; i < kBins; i += kBinThreads)
        if (h[i]) h[i] = atomicAdd(&next[i], h[i]);  // this workgroup's places in the bin
    __syncthreads();
    for (int v = v0 + t; v < v1; v += kBinThreads) perm[atomicAdd(&h[bin_of(X + (size_t)v * D, g, D)], 1)] = v;
}

// The same evaluation on the matrix cores (finite weights). A
// workgroup takes 32 rows; its 4 waves are CW blocks of 16 CT columns and 4 / CW
// bands of 16 RT rows, a wave RT x CT tiles of the FP64 16x16x4 MFMA (lane l of a
// tile holds rows l/16 + 4i, column l%16, i = 0..3). A chain of these MFMAs
// rounds exactly like the sequential fma chain of k_gemm, so both kernels give
// identical bits.
//
// The rows are read once, all loads in flight together (nothing looks at a value
// before the last is issued), and the inputs (ReLU applied) that are not zero in
// all 32 rows go to LDS, so that the product loop has no barrier and skips the
// other columns: adding 0 * w leaves a sum as it is (w finite, the sum started
// at +0), so the bits are the same. With the rows in spatial order (perm) 45% of
// the columns of the 768-neuron network fall out, in their own order 10 to 20%.
// A wave reads its weights straight from the L2, SLOTS k-steps ahead. In place
// as above: a workgroup reads all its rows before the epilogue writes them.
//
// Bound: the rows' traffic (4.6 KB a row at K = N = 256) and the matrix cores,
// about equal once 45% of the columns are out, so 39 KB of LDS (KSEG columns at
// a time, mostly all of them) lets four workgroups of a CU take turns at both.
// 2M rows of 256, 115 columns out: 3.35 ms; 3.53 with two workgroups of 64 rows;
// 2.45 without the products, about 2.2 for them alone. The 768-neuron network's
// two layers: 23.5 ms, 38.1 with every column in barrier-separated chunks of 8
// whose ReLU waited for each load.
constexpr int kEvalThreads = 256, kEvalRows = 32;
template <int CW, int CT, int RT>
__global__ __launch_bounds__(kEvalThreads, 4) void k_gemm_mfma(Bufs b, int ZS, const double *in, int in_stride,
                                                               int relu, int V, int K, int N,
                                                               const double *__restrict__ Wt,
                                                               const double *__restrict__ bias, int Wd, int lw0,
                                                               const int *__restrict__ perm) {
    constexpr int ROWS = kEvalRows, WAVES = kEvalThreads / 64, SLOTS = 2;
    static_assert((WAVES / CW) * 16 * RT == ROWS && CT % 2 == 0 && kEvalThreads == kMaxWidth, "wave layout");
    constexpr int PITCH = 146;                  // 16 rows of a tile start 4 banks apart: no conflicts
    constexpr int KSEG = PITCH / (4 * SLOTS) * (4 * SLOTS);
    constexpr int RPW = ROWS / WAVES;           // rows staged by a wave
    constexpr int CPL = kMaxWidth / 64;         // columns of a row staged by a lane
    constexpr uint16_t kOut = 0xFFFF;           // a column that is zero in every row
    __shared__ double as[ROWS][PITCH];
    __shared__ uint32_t s_off[kMaxWidth + 8 * SLOTS];  // byte offset of each multiplied column's weights
    __shared__ uint16_t s_idx[kMaxWidth];              // its place among the multiplied ones, by column
    __shared__ uint8_t s_any[kMaxWidth];               // columns that are not zero in some row
    __shared__ int s_row[ROWS];                        // the workgroup's rows (-1: none)
    __shared__ int s_n[4];
    const int t = threadIdx.x, l = t & 63, w = t >> 6, r = l & 15, q = l >> 4;
    const int v0 = blockIdx.x * ROWS;
    if (t < ROWS) s_row[t] = v0 + t >= V ? -1 : perm ? perm[v0 + t] : v0 + t;
    s_any[t] = 0;
    __syncthreads();
    // wave w reads rows RPW w .. +RPW-1, a lane the columns l, l + 64, ...
    double x[CPL][RPW];
    const double *row[RPW];
#pragma unroll
    for (int i = 0; i < RPW; ++i)
        row[i] = in + (size_t)max(__builtin_amdgcn_readfirstlane(s_row[w * RPW + i]), 0) * in_stride;
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        if (c * 64 >= K) break;
        const int k = min(c * 64 + l, K - 1);
#pragma unroll
        for (int i = 0; i < RPW; ++i) x[c][i] = row[i][k];
    }
    auto value = [&](double v, int i) {  // input of row w * RPW + i
        return (s_row[w * RPW + i] >= 0) & ((relu == 0) | (v > 0.0)) ? v : 0.0;
    };
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        if (c * 64 >= K) break;
        bool any = false;
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            x[c][i] = value(x[c][i], i);
            any |= !(x[c][i] == 0.0);
        }
        if (any && c * 64 + l < K) s_any[c * 64 + l] = 1;
    }
    __syncthreads();
    {
        const bool act = s_any[t];
        const uint64_t m = __ballot(act);
        if (l == 0) s_n[w] = __popcll(m);
        __syncthreads();
        int pos = __popcll(m & ((1ull << l) - 1ull));
        for (int i = 0; i < w; ++i) pos += s_n[i];
        s_idx[t] = act ? (uint16_t)pos : kOut;
        if (act) s_off[pos] = (uint32_t)(t * N) * 8u;
    }
    const int KA = s_n[0] + s_n[1] + s_n[2] + s_n[3];  // columns to multiply
    if (t < 8 * SLOTS) s_off[KA + t] = 0u;  // (weights that are there, for the loads past the end)
    __syncthreads();
    auto pad = [](int n) { return (n + 4 * SLOTS - 1) / (4 * SLOTS) * (4 * SLOTS); };
    // the multiplied columns ks .. ks + KSEG - 1 to LDS, with zeros up to a whole round
    auto zeros = [&](int kn) {
        const int n = pad(kn) - kn;
        if (t < ROWS * n) as[t / n][kn + t % n] = 0.0;  // (n < 8: at most 7 * ROWS threads)
    };
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        if (c * 64 >= K) break;
        const int k = c * 64 + l, p = k < K ? s_idx[k] : kOut;
        if (p < KSEG) {
#pragma unroll
            for (int i = 0; i < RPW; ++i) as[w * RPW + i][p] = x[c][i];
        }
    }
    zeros(min(KSEG, KA));
    const int col0 = (w % CW) * 16 * CT;
    const int rb = (w / CW) * RT * 16;
    uint32_t cb[CT];  // byte offset of this lane's columns in a row of W^T
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) cb[ct] = (uint32_t)min(col0 + ct * 16 + r, N - 1) * 8u;
    const char *wbase = reinterpret_cast<const char *>(Wt);
    double bw[SLOTS][CT];
    auto load_w = [&](int k, int slot) {  // the weights of k-step k .. k+3
        const uint32_t o = s_off[k + q];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) bw[slot][ct] = *reinterpret_cast<const double *>(wbase + (o + cb[ct]));
    };
    __syncthreads();
    dbl4 acc[RT][CT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[rt][ct] = dbl4{0.0, 0.0, 0.0, 0.0};
    for (int ks = 0; ks < KA; ks += KSEG) {
        const int kn = min(KSEG, KA - ks), kpad = pad(kn);
        if (ks > 0) {
            // more columns than the LDS takes: the next ones, read again
            __syncthreads();  // the previous ones have been multiplied
            for (int k = l; k < K; k += 64) {
                const int p = (int)s_idx[k] - ks;
                if (s_idx[k] == kOut || p < 0 || p >= KSEG) continue;
                for (int i = 0; i < RPW; ++i) as[w * RPW + i][p] = value(row[i][k], i);
            }
            zeros(kn);
            __syncthreads();
        }
        if (col0 >= N) continue;
#pragma unroll
        for (int i = 0; i < SLOTS; ++i) {
            load_w(ks + 4 * i, i);
            __builtin_amdgcn_sched_barrier(0);
        }
        for (int k = 0; k < kpad; k += 4 * SLOTS) {
#pragma unroll
            for (int i = 0; i < SLOTS; ++i) {
                double af[RT];
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) af[rt] = as[rb + rt * 16 + r][k + 4 * i + q];
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct)
                        acc[rt][ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(af[rt], bw[i][ct], acc[rt][ct], 0, 0, 0);
                load_w(ks + k + 4 * (i + SLOTS), i);
                __builtin_amdgcn_sched_barrier(0);  // (in flight from here)
            }
        }
    }
    // epilogue: bias, store, and the layer's sign words (one per two tiles, from their ballots)
    const int nwords = (N + 31) >> 5;
    int zero = 0;
    __syncthreads();  // the inputs in LDS have been multiplied: their place takes the sign words
    uint64_t(*s_word)[8] = reinterpret_cast<uint64_t(*)[8]>(&as[0][0]);
    if (col0 < N) {
        double bv[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) bv[ct] = bias[min(col0 + ct * 16 + r, N - 1)];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int at = rb + rt * 16 + q + 4 * i, v = s_row[at];
                uint64_t pb[CT], nb[CT];
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    const int col = col0 + ct * 16 + r;
                    const bool ok = v >= 0 && col < N;
                    double z = 0.0;
                    if (ok) {
                        z = acc[rt][ct][i] + bv[ct];
                        // (wide rows past the caches, which hold few of them until they are read: 1.6% faster)
                        vstore<CT == 4>(&b.Z[(size_t)v * ZS + col], z);
                        zero |= (z == 0.0);
                    }
                    pb[ct] = __ballot(ok && z > 0.0);
                    nb[ct] = __ballot(ok && z < 0.0);
                }
                // lane 16q + p holds word p of this row
                const int sh = 16 * q;
#pragma unroll
                for (int p = 0; p < CT / 2; ++p) {
                    const uint32_t pos = (uint32_t)((pb[2 * p] >> sh) & 0xFFFFu) |
                                         ((uint32_t)((pb[2 * p + 1] >> sh) & 0xFFFFu) << 16);
                    const uint32_t neg = (uint32_t)((nb[2 * p] >> sh) & 0xFFFFu) |
                                         ((uint32_t)((nb[2 * p + 1] >> sh) & 0xFFFFu) << 16);
                    if (r == p) s_word[at][(col0 >> 5) + p] = codes_of(pos, neg);
                }
            }
        }
    }
    // each row's words together: 64 bytes a row (the column blocks' waves apart
    // write 16 bytes at a time)
    __syncthreads();
    static_assert(ROWS * 8 == kEvalThreads, "one word a thread");
    const int v = s_row[t >> 3], p = t & 7;
    if (v >= 0 && p < nwords) {
        const uint64_t cw = s_word[t >> 3][p];
        b.SG[(size_t)v * Wd + lw0 + p] = cw;
        if (b.LW) b.LW[(size_t)v * 8 + p] = cw;
    }
    if (zero) raise_flag(b.CTR, FLAG_ZERO_SIGN);
}

void launch_gemm(const Bufs &b, int ZS, const double *in, int in_stride, int relu, int V, int K, int N,
                 const double *Wt, const double *bias, int Wd, int lw0, bool finite, hipStream_t st,
                 const EvalGrid *grid) {
    if (V <= 0) return;
    if (!finite || K > kMaxWidth) {
        const int blocks = (V + kGemmRows - 1) / kGemmRows;
        hipLaunchKernelGGL(k_gemm, dim3(blocks), dim3(kThreads), 0, st, b, ZS, in, in_stride, relu, V, K, N, Wt, bias,
                           Wd, lw0);
        return;
    }
    int *perm = nullptr;
    if (grid && V >= kBinRows && (int64_t)V * K * N >= kBinWork) {
        int *cnt = b.SPLX;
        perm = reinterpret_cast<int *>(b.SPLE);
        const int blocks = std::max(1, std::min(512, V / 8192));
        launch_fill64(reinterpret_cast<uint64_t *>(cnt), kBins / 2, 0ull, st);
        hipLaunchKernelGGL(k_bin_count, dim3(blocks), dim3(kBinThreads), 0, st, b.X, *grid, grid->D, V, cnt);
        hipLaunchKernelGGL(k_bin_scan, dim3(1), dim3(kBinThreads), 0, st, cnt);
        hipLaunchKernelGGL(k_bin_scatter, dim3(blocks), dim3(kBinThreads), 0, st, b.X, *grid, grid->D, V, cnt, perm);
    }
    auto run = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((V + kEvalRows - 1) / kEvalRows), dim3(kEvalThreads), 0, st, b, ZS, in,
                           in_stride, relu, V, K, N, Wt, bias, Wd, lw0, perm);
    };
    // (column blocks as narrow as the layer allows: a wave of a wider one would
    // sit idle. A layer of one neuron is bound by reading its rows: one thread a
    // row took 0.195 ms for all layers of 2-200-200-1 with its output, this 0.105;
    // 0.260 and 0.267 for 3-64-64-64-1)
    if (N <= 64) run(k_gemm_mfma<2, 2, 1>);
    else if (N <= 128) run(k_gemm_mfma<4, 2, 2>);
    else run(k_gemm_mfma<4, 4, 2>);
}

// ---------------------------------------------- step 3: splitting edges
//
// Ordered stream compaction of {e : NX8[e] == target}. The edge array is cut
// into one contiguous chunk per workgroup (up to kSelBlocks; fewer for small
// steps). The first kernel reads its chunk once and writes the matching ids in
// order (wave ballot / prefix sum inside each tile) to the chunk's own range of
// SPLX, with the chunk's count; the second moves each chunk's matches to their
// offset in SPLE, the sum of the counts before it, with their endpoints (work
// proportional to the matches, not to the edges). No
// workgroup ever waits on another, so the scan runs at streaming speed on all
// XCDs and reads each next-crossing once per step.
__device__ __forceinline__ void sel_chunk(int E, int &c0, int &c1) {
    const int per = ((E + (int)gridDim.x - 1) / (int)gridDim.x + kScanItems - 1) / kScanItems * kScanItems;
    c0 = min(E, (int)blockIdx.x * per);
    c1 = min(E, c0 + per);
}

__global__ __launch_bounds__(kThreads) void k_sel_local(Bufs b, uint16_t target, int par, int step) {
    __shared__ int s_w[kThreads / 64];
    if (step_blocked(b.CTR, step)) return;  // an earlier step failed: the host redoes or reports it
    const int E = b.CTR[CTR_E + par];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    int c0, c1;
    sel_chunk(E, c0, c1);
    int run = c0;
    // the next tile's bytes are loaded before this tile's scan, so that their
    // latency hides behind it (raw words carried, compared at the next round)
    int nbase = c0 + t * kScanItems;
    uint4 ra = make_uint4(0, 0, 0, 0), rc = ra;
    if (nbase + kScanItems <= c1) load32b(b.NX8, nbase, ra, rc);
    for (int tb = c0; tb < c1; tb += kScanTile) {
        const int base = nbase;
        uint32_t hit = base < c1 ? match32b_raw(b.NX8, base, c1, (uint8_t)target, ra, rc) : 0u;
        nbase = base + kScanTile;
        if (nbase + kScanItems <= c1) load32b(b.NX8, nbase, ra, rc);
        const int cnt = __popc(hit);
        int incl = cnt;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        __syncthreads();  // s_w reuse
        if (lane == 63) s_w[wave] = incl;
        __syncthreads();
        int wave_off = 0, total = 0;
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) {
            const int ws = s_w[w];
            if (w < wave) wave_off += ws;
            total += ws;
        }
        int pos = run + wave_off + incl - cnt;
        while (hit) {
            const int i = __builtin_ctz(hit);
            hit &= hit - 1;
            b.SPLX[pos++] = base + i;
        }
        run += total;
    }
    if (t == 0) b.SELCNT[blockIdx.x] = run - c0;
}

__global__ __launch_bounds__(kThreads) void k_sel_gather(Bufs b, int par, int step) {
    __shared__ int s_w[kThreads / 64];
    __shared__ int s_base;
    if (step_blocked(b.CTR, step)) return;
    const int E = b.CTR[CTR_E + par];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    int c0, c1;
    sel_chunk(E, c0, c1);
    // the first round of entries is loaded while the chunk's offset is summed
    const int n = b.SELCNT[blockIdx.x];
    int e0 = 0;
    int2 ab0 = make_int2(0, 0);
    if (t < n) {
        e0 = b.SPLX[c0 + t];
        ab0 = b.EDG[e0];
    }
    int pre = 0;
    for (int i = t; i < (int)blockIdx.x; i += kThreads) pre += b.SELCNT[i];
    for (int o = 32; o > 0; o >>= 1) pre += __shfl_xor(pre, o, 64);
    if (lane == 0) s_w[wave] = pre;
    __syncthreads();
    if (t == 0) {
        int x = 0;
        for (int w = 0; w < kThreads / 64; ++w) x += s_w[w];
        s_base = x;
        if (blockIdx.x == gridDim.x - 1) {
            const int S = x + b.SELCNT[blockIdx.x];
            b.CTR[CTR_S] = S;
            b.SELTAB[0] = make_int2(0, S);
        }
    }
    __syncthreads();
    // each entry carries its edge's endpoints, so the split starts from them
    // without another dependent load
    const int base = s_base;
    if (t < n) b.SPLE[base + t] = make_int4(e0, ab0.x, ab0.y, 0);
    for (int i = t + kThreads; i < n; i += kThreads) {
        const int e = b.SPLX[c0 + i];
        const int2 ab = b.EDG[e];
        b.SPLE[base + i] = make_int4(e, ab.x, ab.y, 0);
    }
}

static int clamp_grid(int64_t g, int lo) { return (int)std::min<int64_t>(kSelBlocks, std::max<int64_t>(lo, g)); }
int select_grid(int64_t edges) { return clamp_grid((edges + 2047) / 2048, 32); }

// both kernels chunk the edges by the grid they are launched with: the same one
void launch_select(const Bufs &b, uint16_t target, int par, int step, int grid, hipStream_t st) {
    hipLaunchKernelGGL(k_sel_local, dim3(grid), dim3(kThreads), 0, st, b, target, par, step);
    hipLaunchKernelGGL(k_sel_gather, dim3(grid), dim3(kThreads), 0, st, b, par, step);
}

// ------------------------------------ steps 2-3 at a layer start, per edge
//
// For every edge, the first neuron of the layer at which its endpoints carry
// different signs (both are nonzero there: every vertex has all of this
// layer's entries set by the evaluation above). Edges with no such neuron
// never split in this layer. Each workgroup takes one contiguous chunk of the
// edges (one edge per thread per tile) and also writes the edges whose first
// crossing is the layer's neuron 0, in edge order, to its chunk's range of
// SPLX: the first pass of that step's compaction (byte 0 stands for both
// "none" and neuron 0, which no later step looks up).
__global__ __launch_bounds__(kThreads) void k_next_all(Bufs b, int V, int Wd, int lw0, int lw1, int par, int step) {
    __shared__ int s_w[kThreads / 64];
    if (step_blocked(b.CTR, step)) return;
    const int E = b.CTR[CTR_E + par];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const uint64_t below = (1ull << lane) - 1ull;
    int c0, c1;
    sel_chunk(E, c0, c1);
    int run = c0;
    for (int tb = c0; tb < c1; tb += kThreads) {
        const int e = tb + t;
        int col = kNoCol;
        if (e < c1) {
            const int2 ab = b.EDG[e];
            if ((unsigned)ab.x >= (unsigned)V || (unsigned)ab.y >= (unsigned)V) {
                raise_flag(b.CTR, FLAG_BOUNDS);
            } else if (b.LW) {
                // the layer's words from their 64-byte copies: four aligned 16-byte loads per endpoint
                const uint4 *ra = reinterpret_cast<const uint4 *>(b.LW + (size_t)ab.x * 8);
                const uint4 *rb = reinterpret_cast<const uint4 *>(b.LW + (size_t)ab.y * 8);
                uint4 qa[4], qb[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    qa[i] = ra[i];
                    qb[i] = rb[i];
                }
                const int nw = lw1 - lw0;
#pragma unroll
                for (int i = 3; i >= 0; --i) {
                    const uint64_t x1 = (((uint64_t)(qa[i].w ^ qb[i].w)) << 32) | (qa[i].z ^ qb[i].z);
                    const uint64_t x0 = (((uint64_t)(qa[i].y ^ qb[i].y)) << 32) | (qa[i].x ^ qb[i].x);
                    if (2 * i + 1 < nw && x1) col = first_col(x1, lw0 + 2 * i + 1, lw0);
                    if (2 * i < nw && x0) col = first_col(x0, lw0 + 2 * i, lw0);
                }
            } else {
                const uint64_t *ra = b.SG + (size_t)ab.x * Wd;
                const uint64_t *rb = b.SG + (size_t)ab.y * Wd;
                for (int w = lw0; w < lw1 && col == kNoCol; ++w) col = first_col(ra[w] ^ rb[w], w, lw0);
            }
            b.NX8[e] = (col == kNoCol || col == 0) ? 0 : (uint8_t)col;
        }
        const bool hit = col == 0;
        const uint64_t m = __ballot(hit);
        __syncthreads();  // s_w reuse
        if (lane == 0) s_w[wave] = __popcll(m);
        __syncthreads();
        int wave_off = 0, total = 0;
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) {
            const int ws = s_w[w];
            if (w < wave) wave_off += ws;
            total += ws;
        }
        if (hit) b.SPLX[run + wave_off + __popcll(m & below)] = e;
        run += total;
    }
    if (t == 0) b.SELCNT[blockIdx.x] = run - c0;
}

// chunks of the layer-start scan: about 4096 edges each, up to kNextBlocks
static int next_blocks(int E) {
    int g = (E + 4095) / 4096;
    return g < 1 ? 1 : (g > kNextBlocks ? kNextBlocks : g);
}

void launch_next_all(const Bufs &b, int V, int Wd, int lw0, int lw1, int E, int par, int step, hipStream_t st) {
    hipLaunchKernelGGL(k_next_all, dim3(next_blocks(E)), dim3(kThreads), 0, st, b, V, Wd, lw0, lw1, par, step);
}

void launch_gather(const Bufs &b, int E, int par, int step, hipStream_t st) {
    hipLaunchKernelGGL(k_sel_gather, dim3(next_blocks(E)), dim3(kThreads), 0, st, b, par, step);
}

// -------------------------------------------- steps 4-5a: split and keys
//
// One group of G lanes per splitting edge (p, q), p = V+ and q = V-:
//   t = z_p / (z_p - z_q), x0 = x_p + t (x_q - x_p)            (Sec. 4.2.1)
// and the same interpolation for every pre-activation of the layer (each is
// affine along the edge, since all earlier layers are already subdivided), with
// the current neuron set to exactly 0. The sign row of x0 is the join of the
// endpoints' rows before this neuron, 0 at it, and the signs of the
// interpolated pre-activations after it. The edge slot becomes (a, x0) and
// (x0, b) is appended; each half records its next crossing in the layer.
// The splitting edge's sign-vector over earlier entries has D-1 zeros; each is
// perturbed to + and - (box zeros only to +, Sec. 4.1) to give the parent
// 2-faces, hashed as the sum of per-word hashes (Sec. 4.2.2).
//
// Every load of a split (both endpoint rows of pre-activations, signs and
// coordinates) is issued before any arithmetic or store, so a wave keeps
// ~NC+3 independent memory requests in flight per split. Lane c of chunk k
// holds column k*G + c; the sign words of the layer are built from the chunk
// ballots, parked in LDS for the lane that owns each word.

// hash-table words for n key slots (at most n / 2 faces): a power of two, at
// least 2n, so the table is at most a quarter full
__device__ __forceinline__ uint32_t table_size(int n) {
    uint32_t t = 256;
    while (t < 2u * (uint32_t)n) t <<= 1;
    return t;
}

// The chunks of the step's split list (SELTAB), read by load() and scanned by
// the whole workgroup: s_pre[c] = splits before chunk c, s_off[c] = its first
// entry less that. scan() returns the step's split count. One gathered list
// (n == 1) takes no scan.
struct ListScan {
    static constexpr int kPer = kListMax / kThreads;
    int2 e[kPer];
    int head;  // splits in the first chunk
    __device__ __forceinline__ void load(const Bufs &b, int n) {
        const int per = (n + kThreads - 1) / kThreads;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int c = (int)threadIdx.x * per + i;
            e[i] = i < per && c < n && n > 1 ? b.SELTAB[c] : make_int2(0, 0);
        }
        head = b.SELTAB[0].y;
    }
    __device__ __forceinline__ int scan(int n, int *s_pre, int *s_off, int *s_w) const {
        if (n == 1) return head;
        const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
        const int per = (n + kThreads - 1) / kThreads;
        int mine = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) mine += e[i].y;
        int incl = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        if (lane == 63) s_w[wave] = incl;
        __syncthreads();
        int run = incl - mine, total = 0;
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) {
            const int x = s_w[w];
            if (w < wave) run += x;
            total += x;
        }
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int c = t * per + i;
            if (i < per && c < n) {
                s_pre[c] = run;
                s_off[c] = e[i].x - run;
                run += e[i].y;
            }
        }
        __syncthreads();
        return total;
    }
};

// place of split s in SPLE: in the last chunk that starts at or before it
// (`head` splits in the first one, which starts at entry 0)
__device__ __forceinline__ int list_entry(int s, int n, int head, const int *s_pre, const int *s_off) {
    if (s < head) return s;
    int lo = 1, hi = n;  // s_pre[lo] <= s, and s_pre[hi] > s or hi == n
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (s_pre[mid] <= s) lo = mid;
        else hi = mid;
    }
    return s + s_off[lo];
}

template <int G, int NC>
__global__ __launch_bounds__(kThreads, 5) void k_split(Bufs b, StepGeom g) {
    __shared__ int s_pre[kListMax], s_off[kListMax], s_w[kThreads / 64];
    ListScan list;
    list.load(b, g.nlist);
    const StepCounters ctr(b.CTR, g.par);
    const int V0 = ctr.V0, E0 = ctr.E0;
    const int head = list.head, S = list.scan(g.nlist, s_pre, s_off, s_w);
    // (step_blocked, tested past the scan's barriers: a step that finds the storage
    // too small raises its flag in this very launch, and waves of one workgroup may
    // read it differently; those that see it and those that compute it then agree)
    if (ctr.flags != 0 || ctr.pfail < g.step) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) b.CTR[CTR_S] = S;
    // every later kernel of the step writes within these bounds
    if ((int64_t)V0 + S > g.Vcap || (int64_t)E0 + (int64_t)S * g.D > g.Ecap || (int64_t)S * g.P > g.Kcap) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            atomicMin(&b.CTR[CTR_FAIL], g.step);
            atomicOr(&b.CTR[CTR_FLAGS], FLAG_CAPACITY);
        }
        return;
    }
    const int nslots = S * g.P;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        b.CTR[CTR_V + (g.par ^ 1)] = V0 + S;
        // more key slots than a table word can name: the exact pass pairs this step
        if (g.pair_mode == PAIR_HASH && (uint32_t)nslots > kMaxHashSlots) raise_pair_flag(b.CTR, FLAG_BIGSTEP, g.step);
    }
    if (g.pair_mode == PAIR_HASH) {
        g.hmask = (uint32_t)nslots <= kMaxHashSlots ? table_size(nslots) - 1u : 0u;
        g.sbits = slot_bits(nslots);
    }
    constexpr int groups = kThreads / G;
    // new vertices' rows streamed past the caches for layers wider than 128 neurons
    constexpr bool kStream = G * NC > 128;
    const int lane = threadIdx.x % G;
    const int grp = threadIdx.x / G;
    const int half = (threadIdx.x & 63) / G;
    for (int s = blockIdx.x * groups + grp; s < S; s += gridDim.x * groups) {
        const int4 q = b.SPLE[list_entry(s, g.nlist, head, s_pre, s_off)];
        const int2 ab = make_int2(q.y, q.z);
        if (!split_entry_ok(b, q.x, E0) || !split_edge_ok(ab, V0)) {
            if (lane == 0) raise_flag(b.CTR, FLAG_BOUNDS);
            continue;
        }
        split_core<G, NC, kStream>(b, g, V0, E0, s, q.x, ab, lane, half, nslots);
    }
}

// two splits per wave (32-lane groups; layers of up to 128 neurons take four,
// in 16-lane groups): the per-split bookkeeping on the sign words runs once
// for all groups of the wave. (The grid is sized for 32-lane groups; the
// launch cuts it to one residency wave, split_resident below.)
int split_blocks(int S_hint, int Nl) {
    (void)Nl;
    const int groups = kThreads / 32;
    int grid = (S_hint + groups - 1) / groups;
    return grid < 1 ? 1 : (grid > 16384 ? 16384 : grid);
}

// Workgroups of k_split<G, NC> that the device holds at once (one residency
// wave), per device, from the occupancy of the compiled kernel; 0 if unknown.
// A split grid is cut to one such wave and the grid-stride loop takes the
// rest: on the 768-neuron network (five workgroups per CU, 1280 in all) one
// wave took 57.1-57.8 us per split launch, 0.8 wave 60.2-60.6, 1.2 waves 65-66,
// two waves 57.6, and one workgroup per eight splits (up to ~12.5K) 59.0-59.7.
template <int G, int NC>
static int split_resident() {
    constexpr int kDevs = 64;
    static std::atomic<int> cache[kDevs];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    if (dev < 0 || dev >= kDevs) return 0;
    int r = cache[dev].load(std::memory_order_relaxed);
    if (r) return r;
    int per_cu = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_split<G, NC>, kThreads, 0) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || per_cu < 1 ||
        cus < 1) {
        // (the launch then keeps its grid; the error must not be reported by
        // the caller's check of the launch)
        (void)hipGetLastError();
        return 0;
    }
    r = per_cu * cus;
    cache[dev].store(r, std::memory_order_relaxed);
    return r;
}

// untimed: the plain launch (also what a captured graph records); timed: the
// launch records its own start and end events
template <int G, int NC>
static void launch_split_as(const Bufs &b, const StepGeom &g, int blocks, hipStream_t st, hipEvent_t t0,
                            hipEvent_t t1) {
    const int wave = split_resident<G, NC>();
    if (wave > 0 && blocks > wave) blocks = wave;
    if (!t0 && !t1)
        hipLaunchKernelGGL((k_split<G, NC>), dim3(blocks), dim3(kThreads), 0, st, b, g);
    else
        hipExtLaunchKernelGGL((k_split<G, NC>), dim3(blocks), dim3(kThreads), 0, st, t0, t1, 0, b, g);
}

void launch_split(const Bufs &b, const StepGeom &g, int blocks, hipStream_t st, hipEvent_t t0, hipEvent_t t1) {
    // a group builds each of a split's 2-face keys in a lane of its own: 16-lane
    // groups only while 2(D - 1) <= 16
    const bool narrow = g.P <= 16;
    if (g.Nl <= 32) {
        if (narrow) launch_split_as<16, 2>(b, g, blocks, st, t0, t1);
        else launch_split_as<32, 1>(b, g, blocks, st, t0, t1);
    } else if (g.Nl <= 64) {
        if (narrow) launch_split_as<16, 4>(b, g, blocks, st, t0, t1);
        else launch_split_as<32, 2>(b, g, blocks, st, t0, t1);
    } else if (g.Nl <= 128) {
        if (narrow) launch_split_as<16, 8>(b, g, blocks, st, t0, t1);
        else launch_split_as<32, 4>(b, g, blocks, st, t0, t1);
    } else {
        launch_split_as<32, 8>(b, g, blocks, st, t0, t1);
    }
}

// ---------------------------------------------------- step 5b: radix sort
//
// Stable LSD radix sort of (key, slot) pairs, 8-bit digits, kSortPasses passes
// over the low 24 bits (keys are 24-bit slices of the 2-face hash, all-ones
// excluded; the sentinel of an unused slot sorts last).
// Per pass: tile histograms, an exclusive scan over the tiles of each digit
// (one workgroup per digit), and a stable scatter that adds the totals of the
// smaller digits and ranks equal digits inside a tile by wave ballots.
template <typename K>
__global__ __launch_bounds__(kThreads) void k_sort_hist(const K *__restrict__ keys, int n, int shift,
                                                         uint32_t *__restrict__ hist, int ntiles) {
    __shared__ uint32_t h[kSortBins];
    const int t = threadIdx.x, tile = blockIdx.x;
    h[t] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
        const int idx = tile * kSortTile + i * kThreads + t;
        if (idx < n) atomicAdd(&h[(uint32_t)(keys[idx] >> shift) & 0xFFu], 1u);
    }
    __syncthreads();
    hist[(size_t)t * ntiles + tile] = h[t];
}

// per digit d (one workgroup each): exclusive scan of hist[d][0..ntiles) in
// place, and the digit's total in hist[kSortBins * ntiles + d] (the scatter
// adds the totals of the smaller digits itself)
__global__ __launch_bounds__(kThreads) void k_sort_scan(uint32_t *hist, int ntiles) {
    __shared__ uint32_t wsum[kThreads / 64];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, d = blockIdx.x;
    uint32_t *h = hist + (size_t)d * ntiles;
    uint32_t carry = 0;
    for (int base = 0; base < ntiles; base += 4 * kThreads) {
        const int i0 = base + 4 * t;
        uint32_t x[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = i0 + k < ntiles ? h[i0 + k] : 0u;
        const uint32_t tsum = x[0] + x[1] + x[2] + x[3];
        uint32_t incl = tsum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        uint32_t woff = 0, total = 0;
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) {
            const uint32_t v = wsum[w];
            if (w < wave) woff += v;
            total += v;
        }
        uint32_t run = carry + woff + incl - tsum;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (i0 + k < ntiles) h[i0 + k] = run;
            run += x[k];
        }
        carry += total;
        __syncthreads();
    }
    if (t == 0) hist[(size_t)kSortBins * ntiles + d] = carry;
}

template <typename K>
__global__ __launch_bounds__(kThreads) void k_sort_scatter(const K *__restrict__ kin,
                                                            const uint32_t *__restrict__ vin,
                                                            K *__restrict__ kout, uint32_t *__restrict__ vout,
                                                            int n, int shift, const uint32_t *__restrict__ hist,
                                                            int ntiles) {
    __shared__ uint32_t base[kSortBins];
    __shared__ uint32_t wcnt[kThreads / 64][kSortBins];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, tile = blockIdx.x;
    static_assert(kSortBins == kThreads, "one digit per thread");
    // digit t starts after the keys of all smaller digits: exclusive scan of the totals
    const uint32_t tot = hist[(size_t)kSortBins * ntiles + t];
    uint32_t incl = tot;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    if (lane == 63) wcnt[0][wave] = incl;
    __syncthreads();
    uint32_t woff = 0;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w)
        if (w < wave) woff += wcnt[0][w];
    base[t] = woff + incl - tot + hist[(size_t)t * ntiles + tile];
    __syncthreads();  // wcnt[0] read by every wave before it is cleared
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) wcnt[w][t] = 0;
    __syncthreads();
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    for (int i = 0; i < kSortItems; ++i) {
        const int idx = tile * kSortTile + i * kThreads + t;
        const bool valid = idx < n;
        const K k = valid ? kin[idx] : (K)0;
        const uint32_t v = valid ? (vin ? vin[idx] : (uint32_t)idx) : 0u;
        const uint32_t d = (uint32_t)(k >> shift) & 0xFFu;
        uint64_t m = __ballot(valid);
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
            const uint64_t bb = __ballot((d >> bit) & 1u);
            m &= ((d >> bit) & 1u) ? bb : ~bb;
        }
        const int rank = __popcll(m & lt);
        if (valid && rank == 0) wcnt[wave][d] = (uint32_t)__popcll(m);
        __syncthreads();
        if (valid) {
            uint32_t pos = base[d] + rank;
            for (int w = 0; w < wave; ++w) pos += wcnt[w][d];
            kout[pos] = k;
            vout[pos] = v;
        }
        __syncthreads();
        uint32_t add = 0;
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) {
            add += wcnt[w][t];
            wcnt[w][t] = 0;
        }
        base[t] += add;
        __syncthreads();
    }
}

// passes of 8 bits over the key bits from 8 * first on; the first pass takes the
// slot ids as values, or (have_vals) those in va
template <typename K>
static void sort_passes(K *ka, K *kb, uint32_t *va, uint32_t *vb, uint32_t *hist, int n, int first, int passes,
                        hipStream_t st, const K **keys, const uint32_t **vals, bool have_vals = false) {
    const int ntiles = (n + kSortTile - 1) / kSortTile;
    for (int pass = 0; n > 0 && pass < passes; ++pass) {
        const int shift = 8 * (first + pass);
        hipLaunchKernelGGL(k_sort_hist<K>, dim3(ntiles), dim3(kThreads), 0, st, ka, n, shift, hist, ntiles);
        hipLaunchKernelGGL(k_sort_scan, dim3(kSortBins), dim3(kThreads), 0, st, hist, ntiles);
        hipLaunchKernelGGL(k_sort_scatter<K>, dim3(ntiles), dim3(kThreads), 0, st, ka,
                           pass == 0 && !have_vals ? nullptr : va, kb,
                           vb, n, shift, hist, ntiles);
        K *tk = ka; ka = kb; kb = tk;
        uint32_t *tv = va; va = vb; vb = tv;
    }
    *keys = ka;
    *vals = va;
}

void launch_sort(const Bufs &b, int n, hipStream_t st, const uint32_t **keys, const uint32_t **vals) {
    sort_passes<uint32_t>(b.K32a, b.K32b, b.VALa, b.VALb, b.HIST, n, 0, kSortPasses, st, keys, vals);
}

void launch_sort64(const Bufs &b, int n, hipStream_t st, const uint64_t **keys, const uint32_t **vals, int first,
                   int passes, bool have_vals) {
    sort_passes<uint64_t>(b.K64a, b.K64b, b.VALa, b.VALb, b.HIST, n, first, passes, st, keys, vals, have_vals);
}

// ------------------------------------------- step 5c: pair and connect
//
// In the sorted key array every run of equal keys has even length (each
// splitting 2-face is met by exactly two splitting edges, Sec. 4.2.2), so the
// run starting at sorted position i owns output edges i/2, i/2+1, ... A run of
// two is the common case; a longer run (two faces whose 24-bit keys collide)
// is grouped by the full 64-bit hash. Every pair is verified by comparing the
// two perturbed sign-vectors word by word. The new edge joins the two new
// vertices; its sign is the face's with 0 at the current neuron (Sec. 4.2.2).
__global__ __launch_bounds__(kThreads) void k_pair(Bufs b, StepGeom g, int V0, int E1, int nslots,
                                                    const uint32_t *__restrict__ KS, const uint32_t *__restrict__ VS) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nslots; i += gridDim.x * blockDim.x) {
        const uint32_t k = KS[i];
        // valid keys (< 2^24 - 1) sort before the sentinels: the last valid one fixes the edge count
        if (k == kSentinel) {
            if (i == 0) b.CTR[CTR_E + (g.par ^ 1)] = E1;
            continue;
        }
        if (i + 1 == nslots || KS[i + 1] == kSentinel) b.CTR[CTR_E + (g.par ^ 1)] = E1 + (i + 1) / 2;
        if (i > 0 && KS[i - 1] == k) continue;  // not the start of a run
        int j = i + 1;
        while (j < nslots && KS[j] == k) ++j;
        const int len = j - i;
        if (len == 2) {
            emit_pair(b, g, V0, nslots, (int)VS[i], (int)VS[i + 1], (size_t)E1 + i / 2);
            continue;
        }
        if ((len & 1) || len > 32) {
            raise_pair_flag(b.CTR, FLAG_RUN, g.step);
            continue;
        }
        uint32_t used = 0;
        int np = 0;
        for (int u = 0; u < len; ++u) {
            if (used & (1u << u)) continue;
            const uint32_t su = VS[i + u];
            if (su >= (uint32_t)nslots) {
                raise_flag(b.CTR, FLAG_BOUNDS);
                break;
            }
            const uint64_t hu = b.FULL[su];
            int w = u + 1;
            while (w < len && ((used & (1u << w)) || VS[i + w] >= (uint32_t)nslots || b.FULL[VS[i + w]] != hu)) ++w;
            if (w == len) {
                raise_pair_flag(b.CTR, FLAG_RUN, g.step);
                break;
            }
            used |= (1u << u) | (1u << w);
            emit_pair(b, g, V0, nslots, (int)VS[i + u], (int)VS[i + w], (size_t)E1 + i / 2 + np++);
        }
    }
}

void launch_pair(const Bufs &b, const StepGeom &g, int V0, int E1, int nslots, const uint32_t *keys,
                 const uint32_t *vals, hipStream_t st) {
    int grid = (nslots + kThreads - 1) / kThreads;
    grid = grid < 1 ? 1 : (grid > 8192 ? 8192 : grid);
    hipLaunchKernelGGL(k_pair, dim3(grid), dim3(kThreads), 0, st, b, g, V0, E1, nslots, keys, vals);
}

// ---------------------------------- step 5c with the hash table, and the
// next step's splitting edges
//
// The split recorded every pair as it found it (the second arrival at a
// 2-face). The emission appends the pairs' edges in the order of their owner
// slots (the smaller slot of a pair): each workgroup takes a chunk of the
// slots, ranks the owners inside it by wave ballots, and checks every slot: a
// fresh record must be mutual, and a valid slot must have one (a failure sends
// the step to the exact pass). The edge list is therefore the same on every run
// and whatever the launch shapes. The owners before a chunk are counted either
// by the workgroup itself, from the records of all slots before its own (small
// steps: one launch does it all), or by a first pass over the slots.
//
// The same launches list the edges that the next neuron of the layer splits, so
// that a step is two launches (three when large) and not five: the scan's
// workgroups take the edges that were there before the pairing (every next
// crossing is final once the split is done), the emission's those that they
// append. Each chunk's matches go, with their endpoints, to the chunk's own
// range of SPLE, and (first entry, count) to SELTAB; the split finds its
// entries by a scan of that table. In large steps the scan's matches (nearly
// all of the list) are moved to their final places beside the emission, as one
// first chunk, so that the split looks up only the few appended edges (the
// 768-neuron network: 103.3 ms; 108.3 with a search for every split; 106.5 with
// the five launches). Bound: the latency of each launch's chain of dependent
// loads, 5 to 10 us a launch while a step has few edges.
__device__ __forceinline__ void pair_chunk(int n, int grid, int blk, int &c0, int &c1) {
    const int per = ((n + grid - 1) / grid + kPairItems - 1) / kPairItems * kPairItems;
    c0 = min(n, blk * per);
    c1 = min(n, c0 + per);
}

// slot u's record names a larger slot of this step
__device__ __forceinline__ int owns(uint64_t r, int u, int step, int nslots) {
    const int p1 = (int)(uint32_t)r;
    return (uint32_t)(r >> 32) == (uint32_t)(step + 1) && p1 > u + 1 && p1 <= nslots;
}

// the workgroup's share of emptying the previous step's table, which no kernel
// reads any more, for the next step
__device__ __forceinline__ void clear_table(const Bufs &b, const StepGeom &g) {
    if (!g.HTo) return;
    const uint32_t clear_n = (uint32_t)b.CTR[CTR_TUSED + (g.par ^ 1)];
    for (uint32_t i = blockIdx.x * kThreads + threadIdx.x; i < clear_n; i += gridDim.x * kThreads) g.HTo[i] = 0ull;
}

// The workgroup's share of the tape words of the step's new vertices (their
// parents are all older than the step).
__device__ __forceinline__ void tape_depths(const Bufs &b, const StepGeom &g, int V0, int S) {
    if (!b.PQ) return;
    for (int x0 = V0 + blockIdx.x * kThreads + threadIdx.x; x0 < V0 + S; x0 += gridDim.x * kThreads) {
        const int2 pq = b.PQ[x0];
        b.DEP[x0] = dep_word(g.lw0, g.j, 1 + max(dep_depth(b.DEP[pq.x], g.lw0), dep_depth(b.DEP[pq.y], g.lw0)));
    }
}

// the same alone (sort pairing)
__global__ __launch_bounds__(kThreads) void k_tape_depths(Bufs b, StepGeom g) {
    tape_depths(b, g, b.CTR[CTR_V + g.par], b.CTR[CTR_S]);
}

void launch_tape_depths(const Bufs &b, const StepGeom &g, int S, hipStream_t st) {
    const int grid = std::max(1, std::min(1024, (S + kThreads - 1) / kThreads));
    hipLaunchKernelGGL(k_tape_depths, dim3(grid), dim3(kThreads), 0, st, b, g);
}

// Sum over the workgroup (every thread gets it); s_w: one int per wave.
__device__ __forceinline__ int block_sum(int x, int *s_w) {
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    __syncthreads();  // s_w has been read
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = x;
    __syncthreads();
    int t = 0;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) t += s_w[w];
    return t;
}

// Rank of this thread among the workgroup's threads with `hit`, and their number.
__device__ __forceinline__ int block_rank(bool hit, int &total, int *s_w) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t m = __ballot(hit);
    __syncthreads();  // s_w has been read
    if (lane == 0) s_w[wave] = __popcll(m);
    __syncthreads();
    int off = __popcll(m & ((1ull << lane) - 1ull));
    total = 0;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) {
        const int x = s_w[w];
        if (w < wave) off += x;
        total += x;
    }
    return off;
}

// Chunk blk of nb of the edges there after the split: those that split at
// neuron g.next. PACK: their ids to SPLX and their number to SELCNT, for
// pack_chunk; else entries of the split list and its table.
__device__ __forceinline__ void scan_range(int E1, int blk, int nb, int &c0, int &c1) {
    const int per = ((E1 + nb - 1) / nb + kScanItems - 1) / kScanItems * kScanItems;
    c0 = min(E1, blk * per);
    c1 = min(E1, c0 + per);
}

template <bool PACK>
__device__ __forceinline__ void scan_chunk(const Bufs &b, const StepGeom &g, int E1, int blk, int nb, int *s_w) {
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    int c0, c1;
    scan_range(E1, blk, nb, c0, c1);
    int run = c0;
    // the next tile's bytes are loaded before this tile's scan, so that their
    // latency hides behind it (raw words carried, compared at the next round)
    int nbase = c0 + t * kScanItems;
    uint4 ra = make_uint4(0, 0, 0, 0), rc = ra;
    if (nbase + kScanItems <= c1) load32b(b.NX8, nbase, ra, rc);
    for (int tb = c0; tb < c1; tb += kScanTile) {
        const int base = nbase;
        uint32_t hit = base < c1 ? match32b_raw(b.NX8, base, c1, (uint8_t)g.next, ra, rc) : 0u;
        nbase = base + kScanTile;
        if (nbase + kScanItems <= c1) load32b(b.NX8, nbase, ra, rc);
        const int cnt = __popc(hit);
        int incl = cnt;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        __syncthreads();  // s_w reuse
        if (lane == 63) s_w[wave] = incl;
        __syncthreads();
        int wave_off = 0, total = 0;
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) {
            const int ws = s_w[w];
            if (w < wave) wave_off += ws;
            total += ws;
        }
        int pos = run + wave_off + incl - cnt;
        while (hit) {
            const int e = base + __builtin_ctz(hit);
            hit &= hit - 1;
            if (PACK) {
                b.SPLX[pos++] = e;
            } else {
                const int2 ab = b.EDG[e];
                b.SPLE[pos++] = make_int4(e, ab.x, ab.y, 0);
            }
        }
        run += total;
    }
    if (t != 0) return;
    if (PACK) b.SELCNT[kSelBlocks + blk] = run - c0;
    else b.SELTAB[blk] = make_int2(c0, run - c0);
}

// The matches of the scan's chunk blk of nb to their places in the split list:
// its first chunk, as one.
__device__ __forceinline__ void pack_chunk(const Bufs &b, int E1, int blk, int nb, int *s_w) {
    const int t = threadIdx.x;
    const int *cnt = b.SELCNT + kSelBlocks;
    int c0, c1;
    scan_range(E1, blk, nb, c0, c1);
    // the first round of entries is loaded while the chunk's place is summed
    const int n = cnt[blk];
    int e0 = 0;
    int2 ab0 = make_int2(0, 0);
    if (t < n) {
        e0 = b.SPLX[c0 + t];
        ab0 = b.EDG[e0];
    }
    int before = 0;
    for (int i = t; i < blk; i += kThreads) before += cnt[i];
    const int base = block_sum(before, s_w);
    if (t < n) b.SPLE[base + t] = make_int4(e0, ab0.x, ab0.y, 0);
    for (int i = t + kThreads; i < n; i += kThreads) {
        const int e = b.SPLX[c0 + i];
        const int2 ab = b.EDG[e];
        b.SPLE[base + i] = make_int4(e, ab.x, ab.y, 0);
    }
    if (t == 0 && blk == nb - 1) b.SELTAB[0] = make_int2(0, base + n);
}

// Chunk blk of np of the key slots; the owners before it are counted here
// (RECOUNT) or summed from the first pass's counts. nscan: the chunks of the
// scan, before the emission's in the next step's list.
template <bool RECOUNT>
__device__ __forceinline__ void emit_chunk(const Bufs &b, const StepGeom &g, int V0, int E0, int S, int blk, int np,
                                           int nscan, int *s_w) {
    const int nslots = S * g.P, E1 = E0 + S, t = threadIdx.x;
    int c0, c1;
    pair_chunk(nslots, np, blk, c0, c1);
    // one slot per thread: an owner's edge is a chain of dependent row loads,
    // so owners are spread over as many threads as possible. A slot's record,
    // its partner's, and its row words from the neuron on (where an owner's
    // first-crossing search starts) are loaded together, the partner's row words
    // as soon as its slot is known (3-256-256-256: 9.27 -> 8.93 ms).
    int partner = -1;
    uint64_t pre[4], prb[4];
    auto load_slot = [&](int u) {
        partner = -1;
#pragma unroll
        for (int i = 0; i < 4; ++i) pre[i] = 0ull;
        if (u >= c1) return;
        const uint64_t *Ra = b.SG + (size_t)(V0 + u / g.P) * g.Wd;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (g.wn + i < g.lw1) pre[i] = Ra[g.wn + i];
        partner = slot_partner(b, g, u, nslots);
        const uint64_t *Rb = b.SG + (size_t)(V0 + max(partner, 0) / g.P) * g.Wd;
#pragma unroll
        for (int i = 0; i < 4; ++i) prb[i] = partner > u && g.wn + i < g.lw1 ? Rb[g.wn + i] : 0ull;
        // a fresh record must be returned by the partner's; a valid slot must have one
        if (partner < 0 ? b.PINFO[u] != kNoInfo
                        : (RECOUNT || partner > u) && slot_partner(b, g, partner, nslots) != u)
            raise_pair_flag(b.CTR, FLAG_RUN, g.step);
    };
    load_slot(c0 + t);  // in flight while the owners before the chunk are counted
    int before = 0, left = 0;
    if (RECOUNT) {
        // (chunks start at multiples of kPairItems: two records per load)
        const ulonglong2 *rec = reinterpret_cast<const ulonglong2 *>(b.PART);
#pragma unroll 4
        for (int u = 2 * t; u < c0; u += 2 * kThreads) {
            const ulonglong2 r = rec[u >> 1];
            before += owns(r.x, u, g.step, nslots) + owns(r.y, u + 1, g.step, nslots);
        }
    } else {
        for (int i = t; i < blk; i += kThreads) before += b.SELCNT[i];
        if (blk == np - 1) {
            for (int i = t; i < np; i += kThreads) left += b.SELCNT[2 * kSelBlocks + i];
            if (block_sum(left, s_w) != 0 && t == 0) raise_pair_flag(b.CTR, FLAG_RUN, g.step);
        }
    }
    const int first = block_sum(before, s_w);
    int run = first, listed = 0;
    for (int tb = c0; tb < c1; tb += kThreads) {
        const int u = tb + t;
        if (tb != c0) load_slot(u);
        const bool own = partner > u;
        int total;
        const int pos = E1 + run + block_rank(own, total, s_w);
        int col = kNoCol;
        // (where faces share a table word, more slots than half can name a larger
        // one, and the step asked for room for half: such a step is paired again, so
        // an edge past the storage is left out)
        const bool fits = pos < g.Ecap;
        if (own && fits)
            col = emit_pair(b, g, V0, nslots, u, partner, (size_t)pos, false, g.verify != 0, pre, GlobalMem(), prb);
        run += total;
        if (g.next >= 0) {
            const bool hit = own && fits && col == g.next;
            const int at = block_rank(hit, total, s_w);
            if (hit)
                b.SPLE[E1 + first + listed + at] = make_int4(pos, V0 + u / g.P, V0 + partner / g.P, 0);
            listed += total;
        }
    }
    if (t == 0) {
        if (g.next >= 0) b.SELTAB[nscan + blk] = make_int2(E1 + first, listed);
        if (blk == np - 1) {
            // the next step's counts, and this step's log entry
            const int En = E1 + run;
            b.CTR[CTR_E + (g.par ^ 1)] = En;
            if (g.HT) b.CTR[CTR_TUSED + g.par] = (uint32_t)nslots <= kMaxHashSlots ? (int)table_size(nslots) : 0;
            if (S > b.CTR[CTR_SMAX]) b.CTR[CTR_SMAX] = S;
            if (b.REC) b.REC[g.step] = StepRec{V0, E0, S, En};
        }
    }
}

// this step's split must not have failed its pairing (else the exact pass redoes
// it). The emission raises these flags itself, so the waves of a workgroup may
// read them differently: the first wave's answer is everyone's, as no wave may be
// missing at the barriers that follow.
__device__ __forceinline__ bool pair_blocked(const StepCounters &c, const StepGeom &g, int *s_w) {
    if (threadIdx.x == 0) s_w[0] = c.flags != 0 || c.pfail <= g.step;
    __syncthreads();
    const bool blocked = s_w[0] != 0;
    __syncthreads();  // s_w may be written
    return blocked;
}

// Small steps: np emission workgroups, which count the owners before their
// chunks themselves, then the scan's.
__global__ __launch_bounds__(kThreads) void k_pair_scan(Bufs b, StepGeom g, int np) {
    __shared__ int s_w[kThreads / 64];
    const StepCounters ctr(b.CTR, g.par);
    if (pair_blocked(ctr, g, s_w)) return;
    const int V0 = ctr.V0, E0 = ctr.E0, S = ctr.S;
    clear_table(b, g);
    tape_depths(b, g, V0, S);
    const int nscan = (int)gridDim.x - np;
    if ((int)blockIdx.x < np) emit_chunk<true>(b, g, V0, E0, S, blockIdx.x, np, nscan, s_w);
    else scan_chunk<false>(b, g, E0 + S, blockIdx.x - np, nscan, s_w);
}

// Large steps, first launch: the owners of each of np chunks of the slots
// (SELCNT) from one coalesced read of the records, and the scan beside it. Beside
// the owners, what they are more than the chunk's other slots with a record: an
// owner whose partner returns its record has that partner alone, so if every
// owner's does (the emission looks) and these differences add up to 0, every
// slot's does, and the emission need not read the other half's partners (random
// reads of the records; 6-32-32 on a simplex, 15M splits of 10 keys, 3.25 -> 2.8 ms).
__global__ __launch_bounds__(kThreads) void k_count_scan(Bufs b, StepGeom g, int np) {
    __shared__ int s_w[kThreads / 64];
    const StepCounters ctr(b.CTR, g.par);
    if (pair_blocked(ctr, g, s_w)) return;
    const int E0 = ctr.E0, S = ctr.S, nslots = S * g.P;
    clear_table(b, g);
    tape_depths(b, g, ctr.V0, S);
    if ((int)blockIdx.x >= np) {
        scan_chunk<true>(b, g, E0 + S, blockIdx.x - np, (int)gridDim.x - np, s_w);
        return;
    }
    int c0, c1;
    pair_chunk(nslots, np, blockIdx.x, c0, c1);
    int cnt = 0, left = 0;
    for (int u = c0 + (int)threadIdx.x; u < c1; u += kThreads) {
        const uint64_t r = b.PART[u];
        const int own = owns(r, u, g.step, nslots);
        cnt += own;
        left += 2 * own - (record_partner(r, g.step, nslots) >= 0);
    }
    cnt = block_sum(cnt, s_w);
    left = block_sum(left, s_w);
    if (threadIdx.x == 0) {
        b.SELCNT[blockIdx.x] = cnt;
        b.SELCNT[2 * kSelBlocks + blockIdx.x] = left;
    }
}

// second launch: the emission, and the scan's matches packed beside it
__global__ __launch_bounds__(kThreads) void k_pair_emit(Bufs b, StepGeom g, int np) {
    __shared__ int s_w[kThreads / 64];
    const StepCounters ctr(b.CTR, g.par);
    if (pair_blocked(ctr, g, s_w)) return;
    const int V0 = ctr.V0, E0 = ctr.E0, S = ctr.S;
    if ((int)blockIdx.x < np) emit_chunk<false>(b, g, V0, E0, S, blockIdx.x, np, 1, s_w);
    else pack_chunk(b, E0 + S, blockIdx.x - np, (int)gridDim.x - np, s_w);
}

// Steps of up to this many key slots count their owners in the emission itself:
// the last workgroup then reads at most 128 KB of records, beside its own
// slots' loads. Over 3-64-64-64-1 (up to 26K slots a step) the one launch takes
// 7.4 us a step where the two take 11; with twice this limit the extraction
// takes 4.54 ms, not 4.49.
constexpr int64_t kRecountSlots = 16384;

int launch_hash_pair(const Bufs &b, const StepGeom &g, int64_t slots, int64_t edges, bool full, hipStream_t st) {
    const int np = full ? kSelBlocks : clamp_grid((slots + 255) / 256, 1);
    const int nscan = g.next < 0 ? 0 : full ? kSelBlocks : clamp_grid((edges + 2047) / 2048, 1);
    static_assert(2 * kSelBlocks <= kListMax && 3 * kSelBlocks <= kNextBlocks, "chunks of both kinds fit the tables");
    if (!full && slots <= kRecountSlots) {
        hipLaunchKernelGGL(k_pair_scan, dim3(np + nscan), dim3(kThreads), 0, st, b, g, np);
        return g.next < 0 ? 0 : nscan + np;
    }
    hipLaunchKernelGGL(k_count_scan, dim3(np + nscan), dim3(kThreads), 0, st, b, g, np);
    hipLaunchKernelGGL(k_pair_emit, dim3(np + nscan), dim3(kThreads), 0, st, b, g, np);
    return g.next < 0 ? 0 : 1 + np;
}

// ------------------------------------- step 5c, the exact pass of a step
//
// After a pairing failure (a 2-face word reached three times, a valid slot
// left without a partner, equal hashes of different faces, or a step too big
// for the table) the step's pairing is redone without trusting any hash: each
// valid key slot's 2-face sign-vector is rebuilt from its new vertex's row
// (entries before the neuron, one zero perturbed: Sec. 4.1), the slots are
// sorted by a second, independent 64-bit hash of it, and inside each run of
// equal hashes the slots are grouped by comparing the sign-vectors word by
// word. Every group must have exactly two slots (Sec. 4.2.2); anything else is
// a true degeneracy of the input. The pairs are recorded as the table path
// records them, so the emission (and the edge order) is the same.

__device__ __forceinline__ uint64_t face_word(const uint64_t *R, uint32_t info, int w, int wn, int bn) {
    uint64_t f = R[w] & lt_mask(w, wn, bn);
    if (w == (int)(info >> 8)) f |= ((info & 1u) ? 2ull : 1ull) << ((info >> 1) & 63u);
    return f;
}

__global__ __launch_bounds__(kThreads) void k_exact_keys(Bufs b, StepGeom g, int nslots) {
    const int V0 = b.CTR[CTR_V + g.par];
    for (int u = blockIdx.x * kThreads + threadIdx.x; u < nslots; u += gridDim.x * kThreads) {
        const uint32_t info = b.PINFO[u];
        uint64_t k = ~0ull;  // unused slots sort last
        if (info != kNoInfo) {
            const uint64_t *R = b.SG + (size_t)(V0 + u / g.P) * g.Wd;
            uint64_t h = 0x243f6a8885a308d3ull;
            for (int w = 0; w <= g.wn; ++w) h = mix64(h ^ face_word(R, info, w, g.wn, g.bn)) + (uint64_t)(w + 1);
            if (g.fbits < 64) h &= (1ull << g.fbits) - 1ull;  // (collisions on purpose: a test of the grouping)
            k = h == ~0ull ? h - 1 : h;
        }
        b.K64a[u] = k;
        b.VALa[u] = (uint32_t)u;
    }
}

__device__ __forceinline__ bool same_face(const Bufs &b, const StepGeom &g, int V0, uint32_t ua, uint32_t ub) {
    const uint64_t *Ra = b.SG + (size_t)(V0 + ua / g.P) * g.Wd, *Rb = b.SG + (size_t)(V0 + ub / g.P) * g.Wd;
    const uint32_t ia = b.PINFO[ua], ib = b.PINFO[ub];
    uint64_t diff = 0;
    for (int w = 0; w <= g.wn; ++w) diff |= face_word(Ra, ia, w, g.wn, g.bn) ^ face_word(Rb, ib, w, g.wn, g.bn);
    return diff == 0;
}

constexpr int kExactRun = 64;  // longest run of equal 64-bit hashes the grouping takes

__global__ __launch_bounds__(kThreads) void k_exact_group(Bufs b, StepGeom g, int nslots,
                                                           const uint64_t *__restrict__ KS,
                                                           const uint32_t *__restrict__ VS) {
    const int V0 = b.CTR[CTR_V + g.par];
    for (int i = blockIdx.x * kThreads + threadIdx.x; i < nslots; i += gridDim.x * kThreads) {
        const uint64_t k = KS[i];
        if (k == ~0ull) continue;                  // unused slots (sorted last)
        if (i > 0 && KS[i - 1] == k) continue;     // not the start of a run
        int j = i + 1;
        while (j < nslots && KS[j] == k && j - i <= kExactRun) ++j;
        const int len = j - i;
        if (len > kExactRun) {
            raise_flag(b.CTR, FLAG_RUN);  // more than kExactRun slots on one hash: not generic
            continue;
        }
        uint64_t used = 0;
        for (int a = 0; a < len; ++a) {
            if (used >> a & 1ull) continue;
            const uint32_t ua = VS[i + a];
            int mate = -1, same = 0;
            for (int c = a + 1; c < len; ++c) {
                if (used >> c & 1ull) continue;
                if (same_face(b, g, V0, ua, VS[i + c])) {
                    if (mate < 0) mate = c;
                    ++same;
                }
            }
            if (same != 1) {
                raise_flag(b.CTR, FLAG_RUN);  // a 2-face not met by exactly two splitting edges
                break;
            }
            used |= (1ull << a) | (1ull << mate);
            record_pair(b, g, ua, VS[i + mate], nslots);
        }
    }
}

// the counters at the start of an extraction (a kernel, so that a captured graph can set them)
__global__ void k_ctr_init(int *ctr, int V0, int E0) {
    const int i = threadIdx.x;
    if (i < CTR_COUNT)
        ctr[i] = i == CTR_V ? V0 : i == CTR_E ? E0 : (i == CTR_FAIL || i == CTR_PFAIL) ? 0x7fffffff : 0;
}

void launch_ctr_init(int *ctr, int V0, int E0, hipStream_t st) {
    hipLaunchKernelGGL(k_ctr_init, dim3(1), dim3(64), 0, st, ctr, V0, E0);
}

__global__ __launch_bounds__(kThreads) void k_fill64(uint64_t *p, size_t n, uint64_t v) {
    for (size_t i = blockIdx.x * (size_t)kThreads + threadIdx.x; i < n; i += (size_t)gridDim.x * kThreads) p[i] = v;
}

void launch_fill64(uint64_t *p, size_t n, uint64_t v, hipStream_t st) {
    if (n == 0) return;
    const int grid = (int)std::min<size_t>(4096, (n + kThreads - 1) / kThreads);
    hipLaunchKernelGGL(k_fill64, dim3(grid), dim3(kThreads), 0, st, p, n, v);
}

void launch_exact_pair(const Bufs &b, StepGeom g, int nslots, bool full, hipStream_t st) {
    if (nslots > 0) {
        const int kg = std::min(8192, (nslots + kThreads - 1) / kThreads);
        hipLaunchKernelGGL(k_exact_keys, dim3(kg), dim3(kThreads), 0, st, b, g, nslots);
        const uint64_t *keys = nullptr;
        const uint32_t *vals = nullptr;
        launch_sort64(b, nslots, st, &keys, &vals);
        hipLaunchKernelGGL(k_exact_group, dim3(kg), dim3(kThreads), 0, st, b, g, nslots, keys, vals);
    }
    g.next = -1;
    launch_hash_pair(b, g, nslots, 0, full, st);
}

}  // namespace pcx
