// C ABI of the batched extraction (one persistent launch for many networks).
#include <hip/hip_runtime.h>

#include <chrono>
#include <cmath>
#include <cstring>
#include <numeric>

#include "batch.h"
#include "host.h"

using namespace pcx;

struct pcx_batch {
    int n = 0;
    std::vector<int> D, Wd, M, nsteps;
    std::vector<BatchResult> res;
    std::vector<pcx_complex *> fallback;  // networks extracted on the per-step path
    double *oX = nullptr;
    uint64_t *oSG = nullptr;
    int2 *oE = nullptr;
    double time_ms = 0.0, kernel_ms = 0.0;
    int workgroups = 0, wg_per_cu = 0, n_fallback = 0;
    bool outgrown = false;                    // a network did not fit its room
    int sched = 0;                            // schedule bits of the launch (kSched*)
    std::vector<int> sig;                     // size signature of the batched networks
    std::vector<std::vector<int64_t>> steps;  // per-step counters of each batched network (kStepsNow)
    StepRec *rec_dev = nullptr;               // the same, still on the device (kStepsLater)
    std::vector<size_t> rec_off;              //   network i's first record
    std::vector<int> nsub, ZS;
    std::vector<std::vector<uint64_t>> valid;
};

namespace {

// the autotuner's choices: batch size signature -> (workgroups per CU, schedule bits)
std::mutex g_tune_mu;
std::map<std::vector<int>, std::pair<int, int>> g_tuned;

// size signature of a batch: the sorted (subdivided neurons, D) of its batched networks
std::vector<int> signature(const std::vector<int> &nsteps, const std::vector<int> &D, const std::vector<int> &idx) {
    std::vector<int> sig;
    for (int i : idx) sig.push_back(nsteps[i] * 16 + D[i]);
    std::sort(sig.begin(), sig.end());
    return sig;
}

// This thread's pinned staging buffer of at least `bytes` bytes, kept for its
// later calls (every caller synchronizes its stream before it returns, so no
// copy through the old buffer is pending when it grows). Like the thread's
// other pinned buffers and events it is never released: the runtime may be
// gone at thread exit.
int staging(size_t bytes, char *&out) {
    thread_local char *buf = nullptr;
    thread_local size_t cap = 0;
    if (bytes > cap) {
        std::shared_lock<std::shared_mutex> gate(capture_gate());
        if (buf) (void)hipHostFree(buf);
        buf = nullptr;
        cap = 0;
        const size_t nc = std::max<size_t>(bytes, 64 << 10);
        if (hipHostMalloc((void **)&buf, nc, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            buf = nullptr;
            return fail(PCX_ERR_OOM, "pinned staging buffer");
        }
        cap = nc;
    }
    out = buf;
    return PCX_OK;
}

// this thread's pair of timing events on the current device (created once)
int launch_events(hipEvent_t &a, hipEvent_t &b) {
    thread_local std::map<int, std::pair<hipEvent_t, hipEvent_t>> ev;
    int dev = 0;
    HIPCHK(hipGetDevice(&dev));
    auto it = ev.find(dev);
    if (it == ev.end()) {
        std::shared_lock<std::shared_mutex> gate(capture_gate());
        hipEvent_t x = nullptr, y = nullptr;
        HIPCHK(hipEventCreate(&x));
        HIPCHK(hipEventCreate(&y));
        it = ev.emplace(dev, std::make_pair(x, y)).first;
    }
    a = it->second.first;
    b = it->second.second;
    return PCX_OK;
}

// Storage of a batched launch: one arena per workgroup, for its largest network,
// and the output pool.
struct BatchRoom {
    size_t vbytes, abytes;
    int ecap, kcap;
    uint32_t tcap;
    unsigned long long capV, capSG, capE;
};

// Vertices and key slots that a batched network gets room for. The least is a
// quarter above the prediction, and key slots for steps of a twelfth of that. The
// prediction falls short from D = 4 on and the last steps of a network of few
// neurons split more of it, and a network that does not fit is extracted a second
// time, so with `spare` both are sized by D. Largest over 2,554 He networks of 1 to
// 4 layers (V above 512 over the prediction; S, the largest step, over V):
//   D = 3: 0.9, 0.17;  4: 1.6, 0.26;  5: 4.4, 0.32;  6: 14, 0.35;  8: 76, 0.44.
// (The 256-thread kernel clears its key slots for every network: no more spare of
// them than 24K or twice the least.)
size_t least_vertices(double pred) { return (size_t)(pred * 1.25) + 64; }
size_t vertex_room(int D, double pred, bool spare) {
    const size_t least = least_vertices(pred);
    if (!spare) return least;
    const double grown = pred * (D <= 3 ? 1.25 : std::pow(2.5, D - 3)) + 512.0;
    return D <= 3 ? (size_t)grown : std::max<size_t>(least, (size_t)std::min(grown, 12288.0));
}
size_t key_room(int D, double pred, bool spare) {
    const size_t P = std::max(1, 2 * (D - 1));
    const size_t least = P * std::max<size_t>(256, least_vertices(pred) / 12);
    if (!spare || D <= 2) return least;
    const size_t grown = P * std::max<size_t>(256, vertex_room(D, pred, true) * D / 14);
    return std::max(least, std::min(grown, std::max<size_t>(24576, 2 * least)));
}

// idx: the batched networks among those of Ds, Wds and pred
BatchRoom batch_room(const std::vector<int> &Ds, const std::vector<int> &Wds, const std::vector<double> &pred,
                     const std::vector<int> &idx, int maxD, int maxWd, int maxZS, bool spare) {
    BatchRoom r{};
    size_t vcap = 0, kcap = 1024;
    double largest = 0;
    for (int i : idx) {
        vcap = std::max(vcap, vertex_room(Ds[i], pred[i], spare));
        kcap = std::max(kcap, key_room(Ds[i], pred[i], spare));
        largest = std::max(largest, pred[i]);
    }
    r.vbytes = (vcap * 8 * (size_t)(maxD + maxWd + maxZS) + 255) / 256 * 256;
    r.ecap = (int)((vcap * (maxD + 1) + 15) / 16 * 16);
    r.kcap = (int)std::max(kcap, key_room(maxD, largest, false));
    r.tcap = 256;
    while ((uint64_t)r.tcap < 2ull * (uint64_t)r.kcap && r.tcap < (1u << 31)) r.tcap <<= 1;
    r.abytes = (batch_arena_bytes(r.vbytes, r.ecap, r.kcap, r.tcap) + 255) / 256 * 256;
    double sv = 0, ssg = 0, se = 0;
    for (int i : idx) {
        const double v = std::min(spare ? (double)vertex_room(Ds[i], pred[i], true) : 1.1 * pred[i], (double)vcap);
        sv += v * Ds[i];
        ssg += v * Wds[i];
        se += v * (Ds[i] + 1);
    }
    r.capV = (unsigned long long)sv + 1024;
    r.capSG = (unsigned long long)ssg + 1024;
    r.capE = (unsigned long long)se + 1024;
    return r;
}

size_t align16(size_t x) { return (x + 15) / 16 * 16; }

}  // namespace

namespace {

// The batched extraction. steps: kStepsNow copies every batched network's
// per-step counters to the host at once (the batch of one behind small
// pcx_extract calls); kStepsLater keeps them on the device for
// pcx_batch_steps to copy one network's on request; kStepsNone logs nothing.
enum { kStepsNone = 0, kStepsNow = 1, kStepsLater = 2 };
int batch_run(int32_t n, const pcx_mlp *const *mlps, const double *lo, const double *hi, const pcx_opts *opts,
              int steps_mode, pcx_batch **out, int force_sched = -1) {
    const bool keep_steps = steps_mode != kStepsNone;
    if (!out) return fail(PCX_ERR_INVALID, "out is NULL");
    *out = nullptr;
    if (n < 0 || (n > 0 && (!mlps || !lo || !hi))) return fail(PCX_ERR_INVALID, "NULL argument");
    pcx_opts o{};
    if (opts) o = *opts;
    if (o.prune || o.record_tape) return fail(PCX_ERR_INVALID, "batched extraction supports neither prune nor record_tape");
    hipStream_t st = (hipStream_t)o.stream;
    auto t_start = std::chrono::steady_clock::now();
    auto *bt = new pcx_batch();
    bt->n = n;
    bt->res.assign(n, BatchResult{});
    bt->fallback.assign(n, nullptr);
    bt->D.resize(n);
    bt->Wd.resize(n);
    bt->M.resize(n);
    bt->nsteps.resize(n);
    bt->nsub.resize(n);
    bt->ZS.resize(n);
    bt->valid.resize(n);
    bt->steps.resize(n);
    std::vector<BatchNet> nets(n);
    std::vector<double> pred(n);
    std::vector<int> batched, direct;
    size_t box_off = 0;
    int maxD = 1, maxWd = 1, maxZS = 1;
    bool narrow = true;  // every batched network has layers of at most kSmallWidth neurons
    for (int i = 0; i < n; ++i) {
        const pcx_mlp *m = mlps[i];
        if (!m) {
            pcx_batch_free(bt);
            return fail(PCX_ERR_INVALID, "NULL network");
        }
        const int D = m->D, L = m->L, nsub = o.include_output ? L : L - 1;
        for (int j = 0; j < D; ++j)
            if (!(lo[box_off + j] < hi[box_off + j])) {
                pcx_batch_free(bt);
                return fail(PCX_ERR_INVALID, "box must have lo < hi in every coordinate");
            }
        int Wd = 1, M = 2 * D, N = 0, ZS = 1;
        bool fits = D <= kBatchMaxD && L <= kBatchMaxLayers;
        for (int l = 1; l <= nsub; ++l) {
            if (m->widths[l] > kMaxWidth) fits = false;
            Wd += (m->widths[l] + 31) / 32;
            M += m->widths[l];
            N += m->widths[l];
            ZS = std::max(ZS, m->widths[l]);
        }
        if (Wd > kBatchMaxWords) fits = false;
        bt->D[i] = D;
        bt->Wd[i] = Wd;
        bt->M[i] = M;
        bt->nsteps[i] = N;
        bt->nsub[i] = nsub;
        bt->ZS[i] = ZS;
        if (steps_mode == kStepsNow) {
            std::vector<uint64_t> v(Wd, 0);
            for (int e = 0; e < 2 * D; ++e) v[0] |= 1ull << (2 * e);
            int w0 = 1;
            for (int l = 1; l <= nsub; ++l) {
                for (int c = 0; c < m->widths[l]; ++c) v[w0 + (c >> 5)] |= 1ull << (2 * (c & 31));
                w0 += (m->widths[l] + 31) / 32;
            }
            bt->valid[i] = v;
        }
        pred[i] = predict_vertices(D, N);
        if (pred[i] > 65536.0) fits = false;  // larger networks use the per-step path
        if (fits) {
            BatchNet &bn = nets[i];
            std::memset(&bn, 0, sizeof bn);
            for (int l = 0; l < L; ++l) {
                bn.Wt[l] = m->Wt[l];
                bn.b[l] = m->b[l];
            }
            for (int l = 0; l <= L; ++l) bn.widths[l] = m->widths[l];
            bn.L = L;
            bn.nsub = nsub;
            bn.D = D;
            for (int j = 0; j < D; ++j) {
                bn.lo[j] = lo[box_off + j];
                bn.hi[j] = hi[box_off + j];
            }
            batched.push_back(i);
            maxD = std::max(maxD, D);
            maxWd = std::max(maxWd, Wd);
            maxZS = std::max(maxZS, ZS);
            narrow = narrow && ZS <= kSmallWidth;
        } else {
            direct.push_back(i);
        }
        box_off += D;
    }
    // largest predicted work first (the queue of the persistent kernel)
    std::sort(batched.begin(), batched.end(), [&](int a, int b) {
        return pred[a] * bt->nsteps[a] > pred[b] * bt->nsteps[b] || (pred[a] * bt->nsteps[a] == pred[b] * bt->nsteps[b] && a < b);
    });
    int rc = PCX_OK;
    Arena ar;
    ar.cap = o.max_bytes;
    float kms = 0.f;
    StepRec *rec_dev = nullptr;
    size_t rec_tot = 0;
    std::vector<size_t> rec_off(n, 0);
    size_t in_bytes = 0, out_bytes = 0, res_bytes = 0;
    char *in_dev = nullptr, *out_dev = nullptr;
    if (!batched.empty()) {
        int dev = 0, cus = 256;
        (void)hipGetDevice(&dev);
        (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        // schedule and workgroups per CU: as asked, else from the autotuner's cache,
        // else the default ones. Narrow networks under the default schedule run on the
        // small-network kernel where one workgroup a CU is asked for or nothing is;
        // two and more are the 256-thread kernel's.
        bt->sig = signature(bt->nsteps, bt->D, batched);
        bt->sig.push_back(narrow);
        int wpc = 0, sched = force_sched;
        bool hook = false;
        if (sched < 0) {
            // test hook: one schedule of the 256-thread kernel for every launch (0 .. kSchedCount-1)
            const char *v = getenv("PCX_BATCH_SCHED");
            hook = v && *v;
            if (hook) sched = std::max(0, std::min(kSchedCount - 1, atoi(v)));
        }
        if (sched < 0) {
            std::lock_guard<std::mutex> lk(g_tune_mu);
            auto it = g_tuned.find(bt->sig);
            if (it != g_tuned.end()) {
                wpc = it->second.first;
                sched = it->second.second;
            }
        }
        if (sched < 0) sched = kSchedDefault;
        if (o.batch_wg_per_cu > 0) wpc = o.batch_wg_per_cu;
        if (wpc == 0) wpc = narrow && sched == kSchedDefault && !hook ? 1 : 2;
        const bool small = narrow && sched == kSchedDefault && wpc == 1 && !hook;
        bt->sched = sched;
        const int grid = std::min<int>((int)batched.size(), cus * wpc);
        BatchArgs A{};
        // the inputs in one block (the pool counters, zero; the order; the network
        // descriptors) and the outputs in one block (the results, and the step
        // log with kStepsNow), each moved by one copy through pinned memory
        in_bytes = 8 * sizeof(unsigned long long) + align16(batched.size() * sizeof(int)) + (size_t)n * sizeof(BatchNet);
        res_bytes = align16((size_t)n * sizeof(BatchResult));
        {
            size_t tot = 0;
            if (keep_steps)
                for (int i : batched) tot += (size_t)bt->nsteps[i];
            out_bytes = res_bytes + (steps_mode == kStepsNow ? std::max<size_t>(tot, 1) * sizeof(StepRec) : 0);
        }
        // Room for the networks' complexes: with spare if that can be had, else
        // (a byte cap, or no memory) a quarter above the predictions, and the
        // networks that outgrow it fall back to the per-step path.
        BatchRoom room;
        {
            for (const bool spare : {true, false}) {
                room = batch_room(bt->D, bt->Wd, pred, batched, maxD, maxWd, maxZS, spare);
                void *q[6] = {};
                const size_t bytes[6] = {(size_t)grid * room.abytes, room.capV * sizeof(double),
                                         room.capSG * sizeof(uint64_t), room.capE * sizeof(int2),
                                         in_bytes, out_bytes};
                size_t total = 0;
                for (size_t x : bytes) total += Pool::size_class(std::max<size_t>(x, 1));
                if (spare && o.max_bytes && total > o.max_bytes) continue;
                rc = PCX_OK;
                for (int k = 0; k < 6 && !rc; ++k) rc = ar.alloc(&q[k], bytes[k]);
                if (rc) {
                    for (void *x : q) ar.release(x);
                    continue;
                }
                A.arena = (char *)q[0];
                bt->oX = (double *)q[1];
                bt->oSG = (uint64_t *)q[2];
                bt->oE = (int2 *)q[3];
                in_dev = (char *)q[4];
                out_dev = (char *)q[5];
                for (int k = 1; k <= 3; ++k) ar.forget(q[k]);  // owned by the batch from here on
                break;
            }
            if (rc) goto fail_out;
        }
        A.pool = (unsigned long long *)in_dev;
        A.ticket = (int *)(A.pool + 4);
        A.order = (const int *)(in_dev + 8 * sizeof(unsigned long long));
        A.nets = (const BatchNet *)(in_dev + 8 * sizeof(unsigned long long) + align16(batched.size() * sizeof(int)));
        A.res = (BatchResult *)out_dev;
        if (keep_steps) {
            size_t tot = 0;
            for (int i : batched) tot += (size_t)bt->nsteps[i];
            if (steps_mode == kStepsLater) {
                // kept by the batch (returned to the pool by pcx_batch_free)
                size_t got = 0;
                rec_dev = (StepRec *)pool().get(std::max<size_t>(tot, 1) * sizeof(StepRec), &got, ~(size_t)0);
                if (!rec_dev) {
                    rc = fail(PCX_ERR_OOM, "step log of the batch");
                    goto fail_out;
                }
                bt->rec_dev = rec_dev;
            } else {
                rec_dev = (StepRec *)(out_dev + res_bytes);
            }
            size_t off = 0;
            for (int i : batched) {
                nets[i].rec = rec_dev + off;
                rec_off[i] = off;
                off += (size_t)bt->nsteps[i];
            }
            rec_tot = tot;
            if (steps_mode == kStepsLater) bt->rec_off = rec_off;
        }
        A.n = (int)batched.size();
        A.arena_bytes = room.abytes;
        A.vbytes = room.vbytes;
        A.ecap = room.ecap;
        A.kcap = room.kcap;
        A.tcap = room.tcap;
        A.oX = bt->oX;
        A.oSG = bt->oSG;
        A.oE = bt->oE;
        A.capV = room.capV;
        A.capSG = room.capSG;
        A.capE = room.capE;
        {
            // (PCX_DEBUG_HASH_BITS: as in pcx_extract, collisions on purpose for tests)
            const char *v = getenv("PCX_DEBUG_HASH_BITS");
            const int hb = v ? atoi(v) : 64;
            A.hbits = hb >= 1 && hb < 64 ? hb : 64;
            A.verify = o.verify_pairs ? 1 : 0;
        }
        {
            char *stg = nullptr;
            if ((rc = staging(std::max(in_bytes, out_bytes), stg))) goto fail_out;
            std::memset(stg, 0, 8 * sizeof(unsigned long long));
            std::memcpy(stg + 8 * sizeof(unsigned long long), batched.data(), batched.size() * sizeof(int));
            std::memcpy(stg + 8 * sizeof(unsigned long long) + align16(batched.size() * sizeof(int)), nets.data(),
                        (size_t)n * sizeof(BatchNet));
            HIPCHK(hipMemcpyAsync(in_dev, stg, in_bytes, hipMemcpyHostToDevice, st));
            hipEvent_t e0, e1;
            if ((rc = launch_events(e0, e1))) goto fail_out;
            HIPCHK(hipEventRecord(e0, st));
            if (small) launch_small(A, grid, st);
            else launch_batch(A, grid, sched, st);
            HIPCHK(hipGetLastError());
            HIPCHK(hipEventRecord(e1, st));
            // (stream order: the input copy out of the staging buffer is done before this one lands there)
            HIPCHK(hipMemcpyAsync(stg, out_dev, out_bytes, hipMemcpyDeviceToHost, st));
            HIPCHK(hipStreamSynchronize(st));
            std::memcpy(bt->res.data(), stg, (size_t)n * sizeof(BatchResult));
            std::vector<StepRec> rec(steps_mode == kStepsNow ? rec_tot : 0);
            if (!rec.empty()) std::memcpy(rec.data(), stg + res_bytes, rec_tot * sizeof(StepRec));
            for (int i : batched) {
                if (steps_mode != kStepsNow || bt->res[i].status != BATCH_OK) continue;
                auto &sv = bt->steps[i];
                sv.resize((size_t)bt->nsteps[i] * 4);
                for (int k = 0; k < bt->nsteps[i]; ++k) {
                    const StepRec &q = rec[rec_off[i] + k];
                    sv[(size_t)k * 4 + 0] = q.V0;
                    sv[(size_t)k * 4 + 1] = q.E0;
                    sv[(size_t)k * 4 + 2] = q.S;
                    sv[(size_t)k * 4 + 3] = 2 * ((int64_t)q.E1 - q.E0 - q.S);
                }
            }
            HIPCHK(hipEventElapsedTime(&kms, e0, e1));
        }
        bt->workgroups = grid;
        bt->wg_per_cu = wpc;
        for (int i : batched) {
            const int s = bt->res[i].status;
            if (s == BATCH_OVERFLOW || s == BATCH_POOL) bt->outgrown = true;
            if (s == BATCH_OVERFLOW || s == BATCH_POOL || s == BATCH_RETRY) direct.push_back(i);
            else if (s == BATCH_INTERNAL) {
                rc = fail(PCX_ERR_DEVICE, "internal error in the batched kernel");
                goto fail_out;
            }
        }
    }
    bt->kernel_ms = kms;
    // networks that do not fit the batched kernel: the per-step path
    box_off = 0;
    {
        std::vector<size_t> offs(n);
        for (int i = 0; i < n; ++i) {
            offs[i] = box_off;
            box_off += bt->D[i];
        }
        pcx_opts od = o;
        for (int i : direct) {
            pcx_complex *cx = nullptr;
            int r = extract_ordinary(mlps[i], lo + offs[i], hi + offs[i], &od, &cx);
            BatchResult &br = bt->res[i];
            std::memset(&br, 0, sizeof br);
            if (r == PCX_ERR_DEGENERATE) {
                br.status = BATCH_DEGENERATE;
                continue;
            }
            if (r != PCX_OK) {
                rc = r;
                goto fail_out;
            }
            bt->fallback[i] = cx;
            br.status = BATCH_OK;
            br.V = (int)cx->V;
            br.E = (int)cx->E;
            br.Wd = cx->Wd;
            br.splits = cx->total_splits;
            br.pairs = cx->total_pairs;
            bt->n_fallback++;
        }
    }
    bt->time_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t_start).count();
    *out = bt;
    return PCX_OK;
fail_out:
    pcx_batch_free(bt);
    return rc;
}

}  // namespace

extern "C" int pcx_extract_batch(int32_t n, const pcx_mlp *const *mlps, const double *lo, const double *hi,
                                 const pcx_opts *opts, pcx_batch **out) {
    return batch_run(n, mlps, lo, hi, opts, kStepsLater, out);
}

namespace pcx {

// A small network's pcx_extract as a batch of one: one launch of the batched
// kernel (one workgroup runs every step) instead of several launches per
// neuron step. The complex, its numbering and its per-step counters are those
// of the per-step path (the same device functions in the same order).
int tiny_extract(const pcx_mlp *mlp, const double *lo, const double *hi, const pcx_opts &o, pcx_complex **out) {
    *out = nullptr;
    pcx_batch *bt = nullptr;
    const pcx_mlp *const one[1] = {mlp};
    int rc = batch_run(1, one, lo, hi, &o, kStepsNow, &bt);
    if (rc) return rc;
    const BatchResult &r = bt->res[0];
    if (r.status == BATCH_DEGENERATE) {
        pcx_batch_free(bt);
        return fail(PCX_ERR_DEGENERATE, "input is not generic");
    }
    if (bt->fallback[0]) {  // too large for the kernel's arena: the per-step path ran, and will at once from now on
        if (bt->outgrown) const_cast<pcx_mlp *>(mlp)->outgrew.store(true);
        *out = bt->fallback[0];
        bt->fallback[0] = nullptr;
        pcx_batch_free(bt);
        return PCX_OK;
    }
    auto *cx = new pcx_complex();
    cx->D = bt->D[0];
    cx->M = bt->M[0];
    cx->Wd = bt->Wd[0];
    cx->n_steps = bt->nsteps[0];
    cx->V = r.V;
    cx->E = r.E;
    cx->valid = bt->valid[0];
    // the output pools hold this network alone, from offset 0: they become its arrays
    cx->X = bt->oX;
    cx->SG = bt->oSG;
    cx->EDG = bt->oE;
    bt->oX = nullptr;
    bt->oSG = nullptr;
    bt->oE = nullptr;
    cx->steps = bt->steps[0];
    cx->total_splits = r.splits;
    cx->total_pairs = r.pairs;
    cx->time_ms = bt->kernel_ms;
    cx->ZS = bt->ZS[0];
    cx->nsub = bt->nsub[0];
    pcx_batch_free(bt);
    *out = cx;
    return PCX_OK;
}

}  // namespace pcx

extern "C" {

int pcx_batch_info(const pcx_batch *bt, int32_t i, pcx_info *info) {
    if (!bt || !info || i < 0 || i >= bt->n) return fail(PCX_ERR_INVALID, "bad argument");
    const BatchResult &r = bt->res[i];
    if (r.status == BATCH_DEGENERATE) return fail(PCX_ERR_DEGENERATE, "network is not generic");
    std::memset(info, 0, sizeof *info);
    info->V = r.V;
    info->E = r.E;
    info->D = bt->D[i];
    info->M = bt->M[i];
    info->Wd = bt->Wd[i];
    info->n_steps = bt->nsteps[i];
    info->total_splits = r.splits;
    info->total_pairs = r.pairs;
    return PCX_OK;
}

int pcx_batch_copy(const pcx_batch *bt, int32_t i, double *coords, uint64_t *signs, int32_t *edges) {
    if (!bt || i < 0 || i >= bt->n) return fail(PCX_ERR_INVALID, "bad argument");
    const BatchResult &r = bt->res[i];
    if (r.status == BATCH_DEGENERATE) return fail(PCX_ERR_DEGENERATE, "network is not generic");
    if (bt->fallback[i]) return pcx_complex_copy(bt->fallback[i], coords, signs, edges);
    const int D = bt->D[i];
    int rc;
    if (coords &&
        (rc = copy_sync(coords, bt->oX + (size_t)r.offV, (size_t)r.V * D * sizeof(double), hipMemcpyDeviceToHost)))
        return rc;
    if (signs &&
        (rc = copy_sync(signs, bt->oSG + r.offSG, (size_t)r.V * r.Wd * sizeof(uint64_t), hipMemcpyDeviceToHost)))
        return rc;
    if (edges && (rc = copy_sync(edges, bt->oE + r.offE, (size_t)r.E * sizeof(int2), hipMemcpyDeviceToHost)))
        return rc;
    return PCX_OK;
}

int pcx_batch_steps(const pcx_batch *bt, int32_t i, int64_t *steps) {
    if (!bt || !steps || i < 0 || i >= bt->n) return fail(PCX_ERR_INVALID, "bad argument");
    const BatchResult &r = bt->res[i];
    if (r.status == BATCH_DEGENERATE) return fail(PCX_ERR_DEGENERATE, "network is not generic");
    if (bt->fallback[i]) return pcx_complex_steps(bt->fallback[i], steps);
    if (!bt->steps[i].empty()) {
        std::memcpy(steps, bt->steps[i].data(), bt->steps[i].size() * sizeof(int64_t));
        return PCX_OK;
    }
    if (!bt->rec_dev) return fail(PCX_ERR_INVALID, "the batch kept no step log");
    // this network's records, from the device
    const int ns = bt->nsteps[i];
    std::vector<StepRec> rec(ns);
    int rc;
    if ((rc = copy_sync(rec.data(), bt->rec_dev + bt->rec_off[i], (size_t)ns * sizeof(StepRec), hipMemcpyDeviceToHost)))
        return rc;
    for (int k = 0; k < ns; ++k) {
        steps[(size_t)k * 4 + 0] = rec[k].V0;
        steps[(size_t)k * 4 + 1] = rec[k].E0;
        steps[(size_t)k * 4 + 2] = rec[k].S;
        steps[(size_t)k * 4 + 3] = 2 * ((int64_t)rec[k].E1 - rec[k].E0 - rec[k].S);
    }
    return PCX_OK;
}

int pcx_batch_summary(const pcx_batch *bt, pcx_batch_stats *s) {
    if (!bt || !s) return fail(PCX_ERR_INVALID, "NULL argument");
    std::memset(s, 0, sizeof *s);
    s->n = bt->n;
    for (int i = 0; i < bt->n; ++i) {
        const BatchResult &r = bt->res[i];
        if (r.status == BATCH_DEGENERATE) {
            s->degenerate++;
            continue;
        }
        s->total_V += r.V;
        s->total_E += r.E;
        s->total_splits += r.splits;
    }
    s->fallbacks = bt->n_fallback;
    s->workgroups = bt->workgroups;
    s->wg_per_cu = bt->wg_per_cu;
    s->split_lanes = sched_split_lanes(bt->sched);
    s->select_items = (bt->sched & kSchedSelect8) ? 8 : 16;
    s->kernel_ms = bt->kernel_ms;
    s->time_ms = bt->time_ms;
    return PCX_OK;
}

void pcx_batch_free(pcx_batch *bt) {
    if (!bt) return;
    pool().put(bt->oX);
    pool().put(bt->oSG);
    pool().put(bt->oE);
    pool().put(bt->rec_dev);
    for (auto *c : bt->fallback) pcx_complex_free(c);
    delete bt;
}

int pcx_batch_tune(int32_t n, const pcx_mlp *const *mlps, const double *lo, const double *hi, const pcx_opts *opts,
                   pcx_batch_tuning *result) {
    // time the batch's launch under the default schedule as an untuned batch runs
    // it, under each other one at two workgroups per CU, then the other occupancies
    // of 1, 2 and 4 under the best schedule (best of two launches each)
    std::vector<int> sig;
    int ran_wpc = 2;
    auto measure = [&](int wpc, int sched, double *ms) -> int {
        *ms = 1e300;
        for (int rep = 0; rep < 2; ++rep) {
            pcx_opts o{};
            if (opts) o = *opts;
            o.batch_wg_per_cu = wpc;
            pcx_batch *bt = nullptr;
            int rc = batch_run(n, mlps, lo, hi, &o, kStepsNone, &bt, sched);
            if (rc) return rc;
            *ms = std::min(*ms, bt->kernel_ms);
            sig = bt->sig;
            if (bt->wg_per_cu) ran_wpc = bt->wg_per_cu;  // (0: no network was batched)
            pcx_batch_free(bt);
        }
        return PCX_OK;
    };
    int rc, best_sched = kSchedDefault, best_wpc = 2, tried = 0;
    double ms_default = 0, best = 1e300, ms;
    for (int i = 0; i < kSchedCount; ++i) {
        // the default first, then the others in order
        const int sc = i == 0 ? kSchedDefault : (i <= kSchedDefault ? i - 1 : i);
        if ((rc = measure(i == 0 ? 0 : 2, sc, &ms))) return rc;
        ++tried;
        if (i == 0) ms_default = ms;
        if (ms < best) {
            best = ms;
            best_sched = sc;
            best_wpc = ran_wpc;
        }
    }
    const int timed_wpc = best_wpc;
    for (int w : {1, 2, 4}) {
        if (w == timed_wpc) continue;
        if ((rc = measure(w, best_sched, &ms))) return rc;
        ++tried;
        if (ms < best) {
            best = ms;
            best_wpc = w;
        }
    }
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        g_tuned[sig] = {best_wpc, best_sched};
    }
    if (result) {
        result->wg_per_cu = best_wpc;
        result->split_lanes = sched_split_lanes(best_sched);
        result->select_items = (best_sched & kSchedSelect8) ? 8 : 16;
        result->candidates = tried;
        result->ms_default = ms_default;
        result->ms_best = best;
    }
    return PCX_OK;
}

}  // extern "C"
