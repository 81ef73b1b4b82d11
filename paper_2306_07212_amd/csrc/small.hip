// Batched edge subdivision of networks with narrow layers (at most 64 neurons):
// one workgroup per network at a time, as in batch.hip, but of 512 threads, one
// a CU, and with the structures of a step in LDS.
//
// Bound: the chain of dependent accesses and instructions of a neuron step, not
// its work. With everything in global memory one 256-thread workgroup took 8 us
// for the smallest step (2-8-8-1: 16 steps, 127 us) and 19 us for one of 50
// splits (2-50-50-1 with output: 1.93 ms). Here the next crossings (one byte an
// edge), the split list, the 2-face table and the key slots sit in LDS, so that
// of a step's chain only the endpoint rows and the new rows go to the caches,
// and a step's splits, slots and edges mostly fit one round of the workgroup:
// 84 us and 1.01 ms. 512 threads because two waves a SIMD leave each 256
// registers: 1024 threads, or two workgroups a CU, spill 100 of their 128 in
// every step (133 us and 1.28 ms; 101 us and 1.22 ms), and 256 threads take more
// rounds (82 us and 1.36 ms).
//
// What does not fit goes on in the arena: edges from NEXT on keep their
// crossings there, a step of more than KEYS key slots its table and records,
// a split list its entries from LIST on. The same device functions in the same
// order as every other path: the complexes are bit-identical.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "batch.h"
#include "device.h"
#include "eval_strip.h"

namespace pcx {

// LDS of the workgroup
template <int T>
struct SmallLds {
    static constexpr int KEYS = 2048, LIST = 1024, TABLE = 2 * KEYS, NEXT = 88 << 10;
    unsigned long long table[TABLE];  // face hash (52 bits) | 1 + key slot (12 bits); 0 = empty
    int4 list[LIST];
    uint64_t valid[kBatchMaxWords];
    uint32_t info[KEYS];
    int ctr[CTR_COUNT];
    int wsum[T / 64];
    int misc[4];
    uint16_t part[KEYS];  // 1 + the partner slot; 0 = none
    uint8_t next[NEXT];   // 1 + first crossing in the layer; 0 = none
    static_assert(KEYS < 1 << 12, "slot field");
};

// The step's structures; KEYS: its key slots and table are in LDS too.
template <int T, bool KEYS>
struct LdsMem {
    SmallLds<T> *s;
    uint32_t mask;   // table words - 1
    uint8_t *rest;   // next crossings of the edges from NEXT on
    __device__ __forceinline__ void next(const Bufs &, const StepGeom &, size_t e, int col) const {
        const uint8_t c = col == kNoCol ? 0 : (uint8_t)(col + 1);
        if (e < (size_t)SmallLds<T>::NEXT) s->next[e] = c;
        else rest[e - SmallLds<T>::NEXT] = c;
    }
    __device__ __forceinline__ uint32_t info(const Bufs &b, size_t slot) const {
        return KEYS ? s->info[slot] : b.PINFO[slot];
    }
    __device__ __forceinline__ void key(const Bufs &b, const StepGeom &g, size_t slot, uint32_t info, uint64_t H,
                                        int nslots) const {
        if (!KEYS) {
            GlobalMem().key(b, g, slot, info, H, nslots);
            return;
        }
        s->info[slot] = info;
        const unsigned long long key = H & ~0xFFFull, mine = key | (unsigned long long)(slot + 1);
        uint32_t h = (uint32_t)(H >> 52 ^ H) & mask;
        for (uint32_t probe = 0; probe <= mask; ++probe) {
            const unsigned long long old = atomicCAS(&s->table[h], 0ull, mine);
            if (old == 0ull) return;  // first arrival: the second records the pair
            if ((old & ~0xFFFull) == key) {
                const uint32_t p = (uint32_t)(old & 0xFFFull) - 1u;
                if (p >= (uint32_t)nslots || p == (uint32_t)slot) break;
                s->part[slot] = (uint16_t)(p + 1);
                s->part[p] = (uint16_t)(slot + 1);
                return;
            }
            h = (h + 1) & mask;
        }
        raise_flag(b.CTR, FLAG_BOUNDS);  // table full: cannot happen at load factor <= 1/2
    }
    __device__ __forceinline__ void unused(const Bufs &b, const StepGeom &, size_t slot) const {
        if (KEYS) s->info[slot] = kNoInfo;
        else b.PINFO[slot] = kNoInfo;
    }
    __device__ __forceinline__ int partner(const Bufs &b, const StepGeom &g, int u, int nslots) const {
        if (!KEYS) return slot_partner(b, g, u, nslots);
        const int p = s->part[u];
        return p > 0 && p <= nslots ? p - 1 : -1;
    }
};

// rank of this thread's first of cnt items among the workgroup's, and their number
template <int T>
__device__ __forceinline__ int small_scan(int cnt, int &total, int *s_w) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int incl = cnt;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    if (lane == 63) s_w[wave] = incl;
    __syncthreads();
    int at = incl - cnt;
    total = 0;
#pragma unroll
    for (int w = 0; w < T / 64; ++w) {
        const int x = s_w[w];
        if (w < wave) at += x;
        total += x;
    }
    __syncthreads();  // s_w may be written again
    return at;
}

// Splitting edges of neuron j among the E edges, in edge order: 16 edges a thread a round.
template <int T>
__device__ __forceinline__ int small_select(const Bufs &b, SmallLds<T> &s, const uint8_t *rest, int E, int j) {
    const uint32_t t4 = 0x01010101u * (uint32_t)(j + 1);
    int run = 0;
    for (int tb = 0; tb < E; tb += 16 * T) {
        const int base = tb + 16 * (int)threadIdx.x;
        uint32_t hit = 0;
        if (base < E) {
            // (NEXT and the arena's share are multiples of 16: a thread's edges are in one of them)
            const uint4 x = base < SmallLds<T>::NEXT
                                ? *reinterpret_cast<const uint4 *>(s.next + base)
                                : *reinterpret_cast<const uint4 *>(rest + (base - SmallLds<T>::NEXT));
            hit = eq_bytes4(x.x, t4) | eq_bytes4(x.y, t4) << 4 | eq_bytes4(x.z, t4) << 8 | eq_bytes4(x.w, t4) << 12;
            if (base + 16 > E) hit &= (1u << (E - base)) - 1u;
        }
        int total;
        int pos = run + small_scan<T>(__popc(hit), total, s.wsum);
        while (hit) {
            const int e = base + __builtin_ctz(hit);
            hit &= hit - 1;
            const int2 ab = b.EDG[e];
            const int4 q = make_int4(e, ab.x, ab.y, 0);
            if (pos < SmallLds<T>::LIST) s.list[pos] = q;
            else b.SPLE[pos] = q;
            ++pos;
        }
        run += total;
    }
    return run;
}

template <int T, int NC, bool KEYS>
__device__ __forceinline__ void small_split(const Bufs &b, const StepGeom &g, SmallLds<T> &s,
                                            const LdsMem<T, KEYS> &m, int V0, int E0, int S) {
    constexpr int G = 16;
    const int lane = threadIdx.x % G, half = (threadIdx.x & 63) / G;
    for (int i = threadIdx.x / G; i < S; i += T / G) {
        const int4 q = i < SmallLds<T>::LIST ? s.list[i] : b.SPLE[i];
        const int2 ab = make_int2(q.y, q.z);
        if (split_entry_ok(b, q.x, E0) && split_edge_ok(ab, V0))
            split_core<G, NC, false, T>(b, g, V0, E0, i, q.x, ab, lane, half, S * g.P, m);
        else if (lane == 0)
            raise_flag(b.CTR, FLAG_BOUNDS);
    }
}

// The pairs' edges in owner slot order, one slot a thread a round.
template <int T, bool KEYS>
__device__ __forceinline__ int small_pair(const Bufs &b, const StepGeom &g, SmallLds<T> &s, const LdsMem<T, KEYS> &m,
                                          int V0, int E1, int nslots) {
    int run = 0;
    for (int tb = 0; tb < nslots; tb += T) {
        const int u = tb + (int)threadIdx.x;
        int partner = -1, total;
        const bool own = u < nslots && slot_owner(b, g, u, nslots, partner, m);
        const int pos = run + small_scan<T>(own, total, s.wsum);
        if (own) emit_pair(b, g, V0, nslots, u, partner, (size_t)E1 + pos, false, g.verify != 0, nullptr, m);
        run += total;
    }
    return run;
}

template <int T>
__device__ void run_small(const BatchArgs &A, const BatchNet &net, int ni, SmallLds<T> &s) {
    const int t = threadIdx.x;
    const int D = net.D, nsub = net.nsub;
    int lw[kBatchMaxLayers + 1];
    lw[0] = 1;
    int ZS = 1;
    for (int l = 0; l < nsub; ++l) {
        lw[l + 1] = lw[l] + (net.widths[l + 1] + 31) / 32;
        ZS = max(ZS, net.widths[l + 1]);
    }
    const int Wd = lw[nsub];
    const int P = D >= 2 ? 2 * (D - 1) : 0;
    // the arena, carved as in batch.hip
    char *base = A.arena + (size_t)blockIdx.x * A.arena_bytes;
    const size_t per_v = 8ull * (D + Wd + ZS);
    const int Vcap = (int)min((size_t)0x7fffffff, A.vbytes / per_v);
    const int Ecap = A.ecap, Kcap = A.kcap;
    Bufs b{};
    b.X = (double *)base;
    b.SG = (uint64_t *)(base + (size_t)Vcap * 8 * D);
    b.Z = (double *)(base + (size_t)Vcap * 8 * (D + Wd));
    char *eb = base + A.vbytes;
    b.EDG = (int2 *)eb;
    uint8_t *rest = (uint8_t *)(eb + (size_t)Ecap * 8);
    b.SPLE = (int4 *)(eb + (size_t)Ecap * 16);
    char *kb = eb + (size_t)Ecap * 32;
    b.PART = (uint64_t *)kb;
    b.PINFO = (uint32_t *)(kb + (size_t)Kcap * 8);
    unsigned long long *table = (unsigned long long *)(kb + (size_t)Kcap * 12 + 256 - ((size_t)Kcap * 12) % 256);
    b.CTR = s.ctr;
    b.VALID = s.valid;

    int status = BATCH_OK;
    const int V0 = 1 << D, E0 = D << (D - 1);
    if (V0 > Vcap || E0 > Ecap || Wd > kBatchMaxWords) status = BATCH_OVERFLOW;
    if (status == BATCH_OK) {
        for (int w = t; w < Wd; w += T) {
            uint64_t v = 0;
            if (w == 0)
                for (int e = 0; e < 2 * D; ++e) v |= 1ull << (2 * e);
            for (int l = 0; l < nsub; ++l)
                if (w >= lw[l] && w < lw[l + 1]) {
                    const int c0 = (w - lw[l]) * 32, n = min(32, net.widths[l + 1] - c0);
                    for (int c = 0; c < n; ++c) v |= 1ull << (2 * c);
                }
            s.valid[w] = v;
        }
        if (t < CTR_COUNT) s.ctr[t] = t == CTR_PFAIL ? 0x7fffffff : 0;
        for (int i = t; i < SmallLds<T>::TABLE; i += T) s.table[i] = 0ull;
        for (int i = t; i < SmallLds<T>::KEYS; i += T) s.part[i] = 0;
        // step 0: the box
        for (int i = t; i < V0 + E0; i += T) {
            if (i < V0) {
                uint64_t w0 = 0;
                for (int j = 0; j < D; ++j) {
                    const int up = (i >> j) & 1;
                    b.X[(size_t)i * D + j] = up ? net.hi[j] : net.lo[j];
                    w0 |= (uint64_t)(up ? 1 : 0) << (4 * j);
                    w0 |= (uint64_t)(up ? 0 : 1) << (4 * j + 2);
                }
                b.SG[(size_t)i * Wd] = w0;
                for (int w = 1; w < Wd; ++w) b.SG[(size_t)i * Wd + w] = 0;
            } else {
                const int e = i - V0;
                const int j = e >> (D - 1);
                const int r = e & ((1 << (D - 1)) - 1);
                const int c = ((r >> j) << (j + 1)) | (r & ((1 << j) - 1));
                b.EDG[e] = make_int2(c, c | (1 << j));
            }
        }
        __syncthreads();
    }
    int V = V0, E = E0;
    long long splits = 0, pairs = 0;
    int step = 0;
    bool untagged = false;  // the arena's partner records
    for (int l = 0; l < nsub && status == BATCH_OK; ++l) {
        const int N = net.widths[l + 1], K = net.widths[l];
        eval_strips<T>(b, ZS, l == 0 ? b.X : b.Z, l == 0 ? D : ZS, l > 0, V, K, N, net.Wt[l], net.b[l], Wd, lw[l]);
        __syncthreads();
        // each edge's first crossing in the layer (at most two words a row)
        for (int e = t; e < E; e += T) {
            const int2 ab = b.EDG[e];
            const uint64_t *ra = b.SG + (size_t)ab.x * Wd + lw[l], *rb = b.SG + (size_t)ab.y * Wd + lw[l];
            int col = first_col(ra[0] ^ rb[0], 0, 0);
            if (N > 32) {
                const uint64_t x1 = ra[1] ^ rb[1];
                if (col == kNoCol) col = first_col(x1, 1, 0);
            }
            LdsMem<T, true>{&s, 0u, rest}.next(b, StepGeom{}, e, col);
        }
        __syncthreads();
        const int lflags = s.ctr[CTR_FLAGS];
        if (lflags) {  // a vertex on one of this layer's hyperplanes
            status = (lflags & FLAG_BOUNDS) ? BATCH_INTERNAL : BATCH_DEGENERATE;
            break;
        }
        for (int j = 0; j < N; ++j, ++step) {
            const int S = small_select<T>(b, s, rest, E, j);
            if (S == 0) {
                if (t == 0 && net.rec) net.rec[step] = StepRec{V, E, 0, E};
                continue;
            }
            const int nslots = S * P;
            if (V + S > Vcap || E + S * D > Ecap || nslots > Kcap) {
                status = BATCH_OVERFLOW;
                break;
            }
            uint32_t tsz = 256;  // (nslots <= Kcap: the doubling ends)
            while (tsz < 2u * (uint32_t)nslots) tsz <<= 1;
            if (tsz > A.tcap) {
                status = BATCH_OVERFLOW;
                break;
            }
            StepGeom g{};
            g.D = D;
            g.Wd = Wd;
            g.ZS = ZS;
            g.Nl = N;
            g.lw0 = lw[l];
            g.lw1 = lw[l + 1];
            g.j = j;
            g.wn = lw[l] + (j >> 5);
            g.bn = 2 * (j & 31);
            g.P = P;
            g.pair_mode = PAIR_HASH;
            g.HT = table;
            g.hmask = tsz - 1;
            g.sbits = kSlotBits;  // (a network's steps have far fewer key slots than 2^24)
            g.step = step;
            g.hkeep = A.hbits < 64 ? (1ull << A.hbits) - 1ull : ~0ull;
            g.fbits = 64;
            g.verify = A.verify;
            int np = 0;
            if (nslots <= SmallLds<T>::KEYS) {
                __syncthreads();  // the list is complete
                const LdsMem<T, true> m{&s, tsz - 1, rest};
                if (N <= 32) small_split<T, 2>(b, g, s, m, V, E, S);
                else small_split<T, 4>(b, g, s, m, V, E, S);
                __syncthreads();
                if (P > 0) np = small_pair(b, g, s, m, V, E + S, nslots);
                // (the table's last reader was the split, the records' the pairing's last scan)
                for (uint32_t i = t; i < tsz && P > 0; i += T) s.table[i] = 0ull;
                for (int i = t; i < nslots; i += T) s.part[i] = 0;
            } else {
                const LdsMem<T, false> m{&s, 0u, rest};
                // (before the network's first such step: partner records of an earlier
                // network in this arena untagged again)
                for (int i = t; i < Kcap && !untagged; i += T) b.PART[i] = 0ull;
                untagged = true;
                for (uint32_t i = t; i < tsz; i += T) table[i] = 0ull;
                __syncthreads();
                if (N <= 32) small_split<T, 2>(b, g, s, m, V, E, S);
                else small_split<T, 4>(b, g, s, m, V, E, S);
                __syncthreads();
                // the pairing reads partner records other waves of this workgroup stored: past the L1
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                np = small_pair(b, g, s, m, V, E + S, nslots);
            }
            if (t == 0 && net.rec) net.rec[step] = StepRec{V, E, S, E + S + np};
            V += S;
            E += S + np;
            splits += S;
            pairs += np;
            __syncthreads();  // the step's edges, rows and flags are written
            const int flags = s.ctr[CTR_FLAGS], pflags = s.ctr[CTR_PFLAGS];
            if (flags) {
                status = (flags & FLAG_BOUNDS) ? BATCH_INTERNAL : BATCH_DEGENERATE;
                break;
            }
            if (pflags) {
                // a hash collision or a face not met twice: the per-step path decides exactly
                status = BATCH_RETRY;
                break;
            }
        }
    }
    __syncthreads();
    // hand the complex over to the pool
    if (t == 0) {
        long long ov = -1, osg = -1, oe = -1;
        if (status == BATCH_OK) {
            ov = (long long)atomicAdd(&A.pool[0], (unsigned long long)V * D);  // doubles: D differs per network
            osg = (long long)atomicAdd(&A.pool[1], (unsigned long long)V * Wd);
            oe = (long long)atomicAdd(&A.pool[2], (unsigned long long)E);
            if ((unsigned long long)ov + (unsigned long long)V * D > A.capV ||
                (unsigned long long)osg + (unsigned long long)V * Wd > A.capSG || (unsigned long long)oe + E > A.capE)
                status = BATCH_POOL;
        }
        A.res[ni] = BatchResult{status, V, E, Wd, ov, osg, oe, splits, pairs};
        s.misc[0] = status;
    }
    __syncthreads();
    if (s.misc[0] == BATCH_OK) {
        const size_t ov = (size_t)A.res[ni].offV, osg = (size_t)A.res[ni].offSG, oe = (size_t)A.res[ni].offE;
        for (size_t i = t; i < (size_t)V * D; i += T) A.oX[ov + i] = b.X[i];
        for (size_t i = t; i < (size_t)V * Wd; i += T) A.oSG[osg + i] = b.SG[i];
        for (size_t i = t; i < (size_t)E; i += T) A.oE[oe + i] = b.EDG[i];
    }
    __syncthreads();
}

template <int T>
__global__ __launch_bounds__(T, 2) void k_small(BatchArgs A) {
    __shared__ SmallLds<T> s;
    for (;;) {
        if (threadIdx.x == 0) s.misc[1] = atomicAdd(A.ticket, 1);
        __syncthreads();
        const int k = s.misc[1];
        __syncthreads();
        if (k >= A.n) break;
        const int ni = A.order[k];
        run_small<T>(A, A.nets[ni], ni, s);
    }
}

void launch_small(const BatchArgs &A, int grid, hipStream_t st) {
    hipLaunchKernelGGL(k_small<512>, dim3(grid), dim3(512), 0, st, A);
}

}  // namespace pcx
