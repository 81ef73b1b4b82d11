// Backward pass of edge subdivision: gradients of a loss on the vertex
// coordinates with respect to the weights and biases (the differentiability
// used in Sec. 5.3 of Berzins 2023).
//
// The forward pass computed every value along a graph that is recorded in the
// tape: the box corners' pre-activations by the layer evaluation
//   Z^(l)[v] = W^(l) h(v) + b^(l),  h(v) = ReLU(Z^(l-1)[v])  (x_v for l = 1),
// and each new vertex x0 of step (l, j) from its splitting edge (p, q), p = V+:
//   t = z_p / (z_p - z_q),  x0 = x_p + t (x_q - x_p),
//   Z(x0)[c] = Z_p[c] + t (Z_q[c] - Z_p[c])  (c != j),   Z(x0)[j] = 0.
// Reverse mode walks it back, a layer at a time: children before their parents,
// then the layer start. Within a layer the tape gives every new vertex its depth
// (longest chain of parents made in the layer), and the vertices of one depth
// are independent: one launch a depth, the deepest first, in which each vertex
// sums the contributions of its children itself, youngest child first (no
// atomics: the gradients are the same bits on every run). A layer of 64 neurons
// has some 20 depths, so that is 20 launches and not two for each of 64 steps:
// launches bound the pass (3-64-64-64-1: 2.8 ms in 364 launches of the steps,
// now 1.3 in 54). Every
// parent's children come from one sort of (parent, child) records per backward
// call. T is the arithmetic type of the
// gradients (double, or float for the throughput mode); the recorded values
// are FP64.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "internal.h"

namespace pcx {

template <typename T>
__global__ __launch_bounds__(kThreads) void k_bwd_init(const double *__restrict__ grad, T *__restrict__ gx, size_t n,
                                                        T *__restrict__ gz, size_t nz) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        gx[i] = (T)grad[i];
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < nz; i += (size_t)gridDim.x * blockDim.x)
        gz[i] = (T)0;
}

// Records of the creation graph, one per (new vertex, parent): key = parent
// << 32 | child << 1 | side (side 0: the child's V+ parent, 1: its V- parent),
// record index 2 (child - Vb) + side. Sorted, they list each parent's
// children in increasing order.
__global__ __launch_bounds__(kThreads) void k_bwd_records(const int2 *__restrict__ PQ, int Vb, int V,
                                                           uint64_t *__restrict__ keys, int *flag) {
    for (int x0 = Vb + blockIdx.x * kThreads + threadIdx.x; x0 < V; x0 += gridDim.x * kThreads) {
        const int2 pq = PQ[x0];
        if ((unsigned)pq.x >= (unsigned)x0 || (unsigned)pq.y >= (unsigned)x0) atomicOr(flag, 1);
        const uint64_t c2 = (uint64_t)(uint32_t)x0 << 1;
        keys[2 * (size_t)(x0 - Vb)] = ((uint64_t)(uint32_t)pq.x << 32) | c2;
        keys[2 * (size_t)(x0 - Vb) + 1] = ((uint64_t)(uint32_t)pq.y << 32) | c2 | 1u;
    }
}

// range of every parent's records in the sorted order (the others keep (0, 0))
__global__ __launch_bounds__(kThreads) void k_bwd_ranges(const uint64_t *__restrict__ skey, int nrec, int V,
                                                         int2 *__restrict__ range) {
    for (int i = blockIdx.x * kThreads + threadIdx.x; i < nrec; i += gridDim.x * kThreads) {
        const uint32_t P = (uint32_t)(skey[i] >> 32);
        if (P >= (uint32_t)V) continue;
        if (i == 0 || (uint32_t)(skey[i - 1] >> 32) != P) range[P].x = i;
        if (i == nrec - 1 || (uint32_t)(skey[i + 1] >> 32) != P) range[P].y = i + 1;
    }
}

// Depths of a layer's new vertices: counts, and the vertices grouped by depth
// (their order inside a depth does not matter).
__global__ __launch_bounds__(kThreads) void k_bwd_depth_count(const uint32_t *__restrict__ DEP, int lw0, int Vs, int Ve,
                                                              int *__restrict__ count, int *flag) {
    __shared__ int h[kMaxDepth + 1];
    for (int i = threadIdx.x; i <= kMaxDepth; i += kThreads) h[i] = 0;
    __syncthreads();
    for (int v = Vs + blockIdx.x * kThreads + threadIdx.x; v < Ve; v += gridDim.x * kThreads) {
        const int d = dep_depth(DEP[v], lw0);
        if (d < 1 || d > kMaxDepth) atomicOr(flag, 1);
        else atomicAdd(&h[d], 1);
    }
    __syncthreads();
    for (int i = threadIdx.x; i <= kMaxDepth; i += kThreads)
        if (h[i]) atomicAdd(&count[i], h[i]);
}

__global__ __launch_bounds__(kThreads) void k_bwd_depth_order(const uint32_t *__restrict__ DEP, int lw0, int Vs, int Ve,
                                                              int *__restrict__ next, int *__restrict__ order) {
    __shared__ int h[kMaxDepth + 1];
    const int per = (Ve - Vs + (int)gridDim.x - 1) / (int)gridDim.x;
    const int v0 = min(Ve, Vs + (int)blockIdx.x * per), v1 = min(Ve, v0 + per);
    for (int i = threadIdx.x; i <= kMaxDepth; i += kThreads) h[i] = 0;
    __syncthreads();
    for (int v = v0 + threadIdx.x; v < v1; v += kThreads) {
        const int d = dep_depth(DEP[v], lw0);
        if (d >= 1 && d <= kMaxDepth) atomicAdd(&h[d], 1);
    }
    __syncthreads();
    for (int i = threadIdx.x; i <= kMaxDepth; i += kThreads)
        if (h[i]) h[i] = atomicAdd(&next[i], h[i]);  // this workgroup's places of the depth
    __syncthreads();
    for (int v = v0 + threadIdx.x; v < v1; v += kThreads) {
        const int d = dep_depth(DEP[v], lw0);
        if (d >= 1 && d <= kMaxDepth) order[atomicAdd(&h[d], 1)] = v;
    }
}

// One group of G lanes per vertex v of one depth (lane c of chunk k holds column
// k G + c). First what its children of the layer add, youngest first:
//   dL/dx_v += s dL/dx0,  dL/dZ_v[c] += s dL/dZ0[c]  (c != j),
// s = 1 - t for the V+ parent and t for the V- parent, and to dL/dz_v of the
// child's neuron j its share of dL/dt, f dL/dt, with f = dt/dz:
//   -z_q / (z_p - z_q)^2 for the V+ parent, z_p / (z_p - z_q)^2 for the V- parent.
// Every term is one fused multiply-add in T (the two factors are selected, not
// the product: a rounded product put the FP32 gradients half as far again from
// FP64). The vertex's gradients are then complete (its children's were: they are
// deeper), so a new vertex gets its record as a child: dL/dt from its coordinates and
// every carried pre-activation but its own neuron's, and (s, f) of either parent.
// Bound: the latency of the chain list -> child's record and row, so kAhead
// children's loads are in flight at once, and of a record only the one parent's pair
// is loaded (a whole record took 82 registers instead of 69 and a depth of
// 3-64-64-64-1 in FP64 26 us instead of 24).
template <typename T, int G, int NC>
__global__ __launch_bounds__(kThreads) void k_bwd_pull(BwdLayer<T> L, const int *__restrict__ order, int n) {
    constexpr int kAhead = 4;
    const int lane = threadIdx.x % G;
    const int groups = gridDim.x * (kThreads / G);
    for (int i = (blockIdx.x * kThreads + threadIdx.x) / G; i < n; i += groups) {
        const int v = order ? order[i] : i;
        const int2 own = L.range[v];
        T ax = 0, az[NC];
        bool any = false;
        T *gzv = L.gz + (size_t)v * L.ZS, *gxv = L.gx + (size_t)v * L.D;
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            const int c = k * G + lane;
            az[k] = c < L.N ? gzv[c] : (T)0;
        }
        if (lane < L.D) ax = gxv[lane];
        // (youngest first: later layers' children, which have been summed, are passed
        // over, and an earlier layer's ends the list)
        bool more = true;
        for (int r = own.y - 1; r >= own.x && more; r -= kAhead) {
            int child[kAhead], jn[kAhead];
            T s[kAhead], f[kAhead], gt[kAhead], cx[kAhead], cz[kAhead][NC];
            bool live[kAhead];
#pragma unroll
            for (int a = 0; a < kAhead; ++a) {
                const uint32_t key = (uint32_t)L.skey[max(r - a, own.x)];
                child[a] = (int)(key >> 1);
                live[a] = r - a >= own.x && child[a] >= L.Vs && child[a] < L.Ve;
                more = more && child[a] >= L.Vs;
                if (!live[a]) child[a] = L.Ve - 1;  // (a new vertex that is there; not used)
                const int side = (int)(key & 1u);
                const BwdChild<T> &rec = L.child[child[a] - L.Vb];
                s[a] = rec.sf[side][0];
                f[a] = rec.sf[side][1];
                gt[a] = rec.gt;
                jn[a] = dep_neuron(L.DEP[child[a]]);
            }
#pragma unroll
            for (int a = 0; a < kAhead; ++a) {
                const T *gzc = L.gz + (size_t)child[a] * L.ZS;
#pragma unroll
                for (int k = 0; k < NC; ++k) cz[a][k] = gzc[min(k * G + lane, L.N - 1)];
                cx[a] = L.gx[(size_t)child[a] * L.D + min(lane, L.D - 1)];
            }
#pragma unroll
            for (int a = 0; a < kAhead; ++a) {
                if (!live[a]) continue;
                any = true;
                ax = fma(s[a], cx[a], ax);
#pragma unroll
                for (int k = 0; k < NC; ++k) {
                    const bool own_col = k * G + lane == jn[a];
                    az[k] = fma(own_col ? f[a] : s[a], own_col ? gt[a] : cz[a][k], az[k]);
                }
            }
        }
        if (any) {
#pragma unroll
            for (int k = 0; k < NC; ++k)
                if (k * G + lane < L.N) gzv[k * G + lane] = az[k];
            if (lane < L.D) gxv[lane] = ax;
        }
        if (v < L.Vs) continue;
        const int j = dep_neuron(L.DEP[v]);
        const int2 pq = L.PQ[v];
        const size_t p = pq.x, q = pq.y;
        const double zp = L.Z[p * L.ZS + j], zq = L.Z[q * L.ZS + j], den = zp - zq;
        T gt = 0;
        if (lane < L.D) gt = ax * (T)(L.X[q * L.D + lane] - L.X[p * L.D + lane]);
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            const int c = k * G + lane;
            if (c < L.N && c != j) gt = fma(az[k], (T)(L.Z[q * L.ZS + c] - L.Z[p * L.ZS + c]), gt);
        }
#pragma unroll
        for (int o = G / 2; o > 0; o >>= 1) gt += __shfl_xor(gt, o, G);
        if (lane == 0) {
            const double inv = 1.0 / (den * den);
            const double t = zp / den;
            L.child[v - L.Vb] = BwdChild<T>{{{(T)(1.0 - t), (T)(-zq * inv)}, {(T)t, (T)(zp * inv)}}, gt};
        }
    }
}

// Partial sums of the weight and bias gradients over one chunk of vertices:
// part[chunk][c][k] = sum_v gz[v][c] h[v][k], h = ReLU of the previous layer's
// pre-activations (the coordinates for layer 1), and k == K is the bias
// (h = 1; summed by the tiles of k = 0). A workgroup takes a 64 x 64 tile of the (c, k) entries and its
// chunk, stages 32 vertices' gz and h values of the tile through LDS at a time,
// and each thread accumulates 4 x 4 entries. Every entry sums its chunk's
// vertices in order, one fused multiply-add each, and k_bwd_wreduce adds the
// chunks in order: the gradients are the same bits on every run.
constexpr int kWgTile = 64, kWgRows = 32;
template <typename T>
__global__ __launch_bounds__(256) void k_bwd_wgrad_tiled(const T *__restrict__ gz, int ZS,
                                                         const double *__restrict__ hin, int hstride, int relu, int Vs,
                                                         int N, int K, int tiles_k, double *__restrict__ part) {
    __shared__ T gs[kWgRows][kWgTile + 1];
    __shared__ T hs[kWgRows][kWgTile + 1];
    const int t = threadIdx.x, tc = t & 15, tk = t >> 4;
    const int c0 = (blockIdx.x / tiles_k) * kWgTile, k0 = (blockIdx.x % tiles_k) * kWgTile;
    const int chunk = (Vs + gridDim.y - 1) / gridDim.y;
    const int v0 = blockIdx.y * chunk, v1 = min(Vs, v0 + chunk);
    T acc[4][4], accb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        accb[i] = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = 0;
    }
    for (int vb = v0; vb < v1; vb += kWgRows) {
        const int nv = min(kWgRows, v1 - vb);
        for (int idx = t; idx < kWgRows * kWgTile; idx += 256) {
            const int r = idx / kWgTile, q = idx % kWgTile;
            const int v = vb + r, c = c0 + q, k = k0 + q;
            T g = 0, h = 0;
            if (r < nv) {
                if (c < N) g = gz[(size_t)v * ZS + c];
                if (k < K) {
                    double x = hin[(size_t)v * hstride + k];
                    if (relu) x = x > 0.0 ? x : 0.0;
                    h = (T)x;
                }
            }
            gs[r][q] = g;
            hs[r][q] = h;
        }
        __syncthreads();
        for (int r = 0; r < nv; ++r) {
            T a[4], bb[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = gs[r][tc + 16 * i];
#pragma unroll
            for (int j = 0; j < 4; ++j) bb[j] = hs[r][tk + 16 * j];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_fma(a[i], bb[j], acc[i][j]);
            if (k0 == 0 && tk == 0) {
#pragma unroll
                for (int i = 0; i < 4; ++i) accb[i] += a[i];
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = c0 + tc + 16 * i;
        if (c >= N) continue;
        if (k0 == 0 && tk == 0) part[(size_t)blockIdx.y * N * (K + 1) + (size_t)c * (K + 1) + K] = (double)accb[i];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = k0 + tk + 16 * j;
            if (k < K) part[(size_t)blockIdx.y * N * (K + 1) + (size_t)c * (K + 1) + k] = (double)acc[i][j];
        }
    }
}

// the chunks' sums, 32 entries a workgroup: thread (i, y) adds the chunks y, y + 8,
// ... of entry i in order, and the eight sums are added in order
__global__ __launch_bounds__(kThreads) void k_bwd_wreduce(const double *__restrict__ part, int chunks, int N, int K,
                                                           double *__restrict__ gW, double *__restrict__ gb) {
    __shared__ double sums[8][33];
    const int i = threadIdx.x & 31, y = threadIdx.x >> 5;
    const int entry = blockIdx.x * 32 + i, total = N * (K + 1);
    double s = 0.0;
    if (entry < total) {
#pragma unroll 4
        for (int c = y; c < chunks; c += 8) s += part[(size_t)c * total + entry];
    }
    sums[y][i] = s;
    __syncthreads();
    if (y != 0 || entry >= total) return;
#pragma unroll
    for (int k = 1; k < 8; ++k) s += sums[k][i];
    const int c = entry / (K + 1), k = entry % (K + 1);
    if (k == K) gb[c] = s;
    else gW[(size_t)c * K + k] = s;
}

// gz_prev[v][k] = (sum_c W[c][k] gz[v][c]) * [Z_prev[v][k] > 0] for the
// vertices present at the layer start. A workgroup takes 64 vertices x 64
// columns k, stages 32 neurons c of gz and W at a time through LDS, and each
// thread accumulates 4 x 4 entries, summing over c in order.
template <typename T>
__global__ __launch_bounds__(256) void k_bwd_prev(const T *__restrict__ gz, int ZS, const double *__restrict__ W,
                                                  const double *__restrict__ Zprev, int ZSp, int Vs, int N, int K,
                                                  T *__restrict__ gzp) {
    __shared__ T gs[kWgTile][kWgRows + 1];
    __shared__ T ws[kWgRows][kWgTile + 1];
    const int t = threadIdx.x, tv = t & 15, tk = t >> 4;
    const int v0 = blockIdx.x * kWgTile, k0 = blockIdx.y * kWgTile;
    T acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = 0;
    for (int cb = 0; cb < N; cb += kWgRows) {
        const int nc = min(kWgRows, N - cb);
        for (int idx = t; idx < kWgTile * kWgRows; idx += 256) {
            const int r = idx / kWgRows, q = idx % kWgRows;  // gz: vertex r, neuron q
            const int v = v0 + r;
            gs[r][q] = (v < Vs && q < nc) ? gz[(size_t)v * ZS + cb + q] : (T)0;
            const int cr = idx / kWgTile, kq = idx % kWgTile;  // W: neuron cr, column kq
            ws[cr][kq] = (cr < nc && k0 + kq < K) ? (T)W[(size_t)(cb + cr) * K + k0 + kq] : (T)0;
        }
        __syncthreads();
        for (int c = 0; c < nc; ++c) {
            T a[4], bb[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = gs[tv + 16 * i][c];
#pragma unroll
            for (int j = 0; j < 4; ++j) bb[j] = ws[c][tk + 16 * j];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_fma(bb[j], a[i], acc[i][j]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int v = v0 + tv + 16 * i;
        if (v >= Vs) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = k0 + tk + 16 * j;
            if (k < K) gzp[(size_t)v * ZSp + k] = Zprev[(size_t)v * ZSp + k] > 0.0 ? acc[i][j] : (T)0;
        }
    }
}

// ------------------------------------------------------------- launchers

template <typename T>
void bwd_init(const double *grad, T *gx, size_t n, T *gz, size_t nz, hipStream_t st) {
    hipLaunchKernelGGL(k_bwd_init<T>, dim3(1024), dim3(kThreads), 0, st, grad, gx, n, gz, nz);
}
void bwd_records(const int2 *PQ, int Vb, int V, uint64_t *keys, int *flag, hipStream_t st) {
    if (V <= Vb) return;
    const int grid = std::min(8192, (V - Vb + kThreads - 1) / kThreads);
    hipLaunchKernelGGL(k_bwd_records, dim3(grid), dim3(kThreads), 0, st, PQ, Vb, V, keys, flag);
}
void bwd_ranges(const uint64_t *skey, int nrec, int V, int2 *range, hipStream_t st) {
    launch_fill64(reinterpret_cast<uint64_t *>(range), V, 0ull, st);
    if (nrec <= 0) return;
    const int grid = std::min(8192, (nrec + kThreads - 1) / kThreads);
    hipLaunchKernelGGL(k_bwd_ranges, dim3(grid), dim3(kThreads), 0, st, skey, nrec, V, range);
}
static int depth_grid(int n) { return std::max(1, std::min(512, n / 2048)); }
void bwd_depth_count(const uint32_t *DEP, int lw0, int Vs, int Ve, int *count, int *flag, hipStream_t st) {
    if (Ve <= Vs) return;
    hipLaunchKernelGGL(k_bwd_depth_count, dim3(depth_grid(Ve - Vs)), dim3(kThreads), 0, st, DEP, lw0, Vs, Ve, count,
                       flag);
}
void bwd_depth_order(const uint32_t *DEP, int lw0, int Vs, int Ve, int *next, int *order, hipStream_t st) {
    if (Ve <= Vs) return;
    hipLaunchKernelGGL(k_bwd_depth_order, dim3(depth_grid(Ve - Vs)), dim3(kThreads), 0, st, DEP, lw0, Vs, Ve, next,
                       order);
}
template <typename T, int G, int NC>
static void pull_as(const BwdLayer<T> &L, const int *order, int n, hipStream_t st) {
    const int per = kThreads / G, grid = std::min(8192, (n + per - 1) / per);
    hipLaunchKernelGGL((k_bwd_pull<T, G, NC>), dim3(grid), dim3(kThreads), 0, st, L, order, n);
}
template <typename T>
void bwd_pull(const BwdLayer<T> &L, const int *order, int n, hipStream_t st) {
    if (n <= 0) return;
    // (a group also holds the D <= 16 coordinates)
    if (L.N <= 16) pull_as<T, 16, 1>(L, order, n, st);
    else if (L.N <= 32) pull_as<T, 32, 1>(L, order, n, st);
    else if (L.N <= 64) pull_as<T, 64, 1>(L, order, n, st);
    else if (L.N <= 128) pull_as<T, 64, 2>(L, order, n, st);
    else pull_as<T, 64, 4>(L, order, n, st);
}
static int wg_tiles(int n) { return (n + kWgTile - 1) / kWgTile; }
// Enough workgroups to fill the card (a chunk of 2048 vertices left 12 of them
// to 25K vertices: 0.37 ms a layer), a chunk of at least two rounds of rows; and,
// as a chunk's rows are summed in the gradient's own arithmetic and only the
// chunks in FP64, no longer chunks than that for layers of many tiles: 2048 rows
// up to half a million vertices, then a 256th of them.
int bwd_chunks(int Vs, int N, int K) {
    const int tiles = wg_tiles(N) * wg_tiles(K);
    const int fill = std::min((1024 + tiles - 1) / tiles, Vs / (2 * kWgRows));
    return std::max({1, fill, std::min(256, Vs / 2048)});
}
template <typename T>
void bwd_layer(const T *gz, int ZS, const double *hin, int hstride, int relu, int Vs, int N, int K, const double *W,
               double *part, int chunks, double *gW, double *gb, T *gzp, int ZSp, hipStream_t st) {
    const int gx = (N * (K + 1) + 31) / 32;
    const int tiles_c = wg_tiles(N), tiles_k = wg_tiles(K);
    hipLaunchKernelGGL(k_bwd_wgrad_tiled<T>, dim3(tiles_c * tiles_k, chunks), dim3(256), 0, st, gz, ZS, hin, hstride,
                       relu, Vs, N, K, tiles_k, part);
    hipLaunchKernelGGL(k_bwd_wreduce, dim3(gx), dim3(kThreads), 0, st, part, chunks, N, K, gW, gb);
    if (gzp && Vs > 0) {
        const dim3 grid((Vs + kWgTile - 1) / kWgTile, (K + kWgTile - 1) / kWgTile);
        hipLaunchKernelGGL(k_bwd_prev<T>, grid, dim3(256), 0, st, gz, ZS, W, hin, hstride, Vs, N, K, gzp);
    }
}

template void bwd_init<double>(const double *, double *, size_t, double *, size_t, hipStream_t);
template void bwd_init<float>(const double *, float *, size_t, float *, size_t, hipStream_t);
template void bwd_pull<double>(const BwdLayer<double> &, const int *, int, hipStream_t);
template void bwd_pull<float>(const BwdLayer<float> &, const int *, int, hipStream_t);
template void bwd_layer<double>(const double *, int, const double *, int, int, int, int, int, const double *, double *,
                                int, double *, double *, double *, int, hipStream_t);
template void bwd_layer<float>(const float *, int, const double *, int, int, int, int, int, const double *, double *,
                               int, double *, double *, float *, int, hipStream_t);

}  // namespace pcx
