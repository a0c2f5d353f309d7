// spk_runtime.hip -- host runtime and C ABI of libspk (declared in spk.h).
//
// A network owns its device memory and orders all work on one HIP stream.
// Creation expands the connectivity parameters on the GPU (paper Sec. III-B:
// the layout description is expanded on the device) into one row per source
// neuron, grouped by target tile (Sec. III-A keeps rows sorted by target),
// with each synapse carrying its delay (Sec. V), and records where every row
// crosses the tile or XCD-group boundaries.  Steps run either as one
// persistent cooperative launch per spk_step call (spk_run.hip), or as the
// tile kernel (delivery into LDS + update + spike list), then for binned
// delivery the push kernel (the new spikes' events into per-arrival pages),
// then the optional raster record, batches of steps captured once into a HIP
// graph and replayed.  Spike counts stay on the device, so stepping never
// waits for the host.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "spk_internal.h"

using namespace spk;

namespace {

thread_local std::string g_err;

spk_status fail(spk_status st, const std::string &msg)
{
    g_err = msg;
    return st;
}

#define SPK_HIP(expr)                                                                   \
    do {                                                                                \
        hipError_t e_ = (expr);                                                         \
        if (e_ != hipSuccess)                                                           \
            return fail(e_ == hipErrorOutOfMemory ? SPK_ENOMEM : SPK_EHIP,              \
                        std::string(#expr) + ": " + hipGetErrorString(e_));             \
    } while (0)

#define SPK_TRY(expr)                   \
    do {                                \
        spk_status s_ = (expr);         \
        if (s_ != SPK_OK) return s_;    \
    } while (0)

constexpr uint32_t kPoisCap = 256;
constexpr uint32_t kBatch = 32;                    // steps per captured graph
constexpr uint64_t kPageBudget = 256ull << 20;     // page records across all pages (2 GiB)
constexpr uint64_t kDebugPageCap = 4096;           // records per page for spk_debug_deliver
constexpr uint64_t kRunMaxSteps = 1ull << 24;      // steps per persistent launch (barrier epochs fit u32)
constexpr uint64_t kRingPlainBatches = 3;          // batches of a call launched one by one (resident kernel)
constexpr uint32_t kFlagRunStopped = 4u;           // device flag: a persistent launch stopped early

// Scratch of spk_deliver_noalloc: two fixed areas per device, held until the
// process ends, shared by every call on that device (the caller orders
// them).  `scratch` holds pages; `scratch_zero` the fill counters, overflow
// flags and accumulators, which are zero between calls: the tile kernel puts
// back to zero what the push kernel used, so that no call clears 4 or 8
// bytes per neuron first (1e6 neurons, 1,000 spikes: 20.3 -> 17.2 us per call).
// In host code the arrays' names stand for host-side shadows, not device
// addresses: kernels get the addresses hipGetSymbolAddress returned for
// the device, looked up once per device when a network is created there.
constexpr uint64_t kNoAllocScratchBytes = SPK_NOALLOC_SCRATCH_BYTES;
__device__ __align__(256) uint8_t scratch[kNoAllocScratchBytes];
__device__ __align__(256) uint8_t scratch_zero[kNoAllocScratchBytes];
constexpr int kMaxDevices = 64;
struct Scratch {
    uint8_t *pages = nullptr, *zero = nullptr;
    ScratchFlag flag;  // a call's kernels were not all launched: the zero area is cleared by the next
};
std::mutex g_scratch_mu;
Scratch g_scratch[kMaxDevices];

// Addresses of this device's scratch (the device is current); looked up once.
spk_status scratch_lookup(int device)
{
    if (device < 0 || device >= kMaxDevices) return fail(SPK_EINVAL, "device index beyond the scratch table");
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch[device].pages) return SPK_OK;
    void *p = nullptr, *z = nullptr;
    SPK_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    SPK_HIP(hipGetSymbolAddress(&z, HIP_SYMBOL(scratch_zero)));
    if (!p || !z) return fail(SPK_EHIP, "hipGetSymbolAddress returned no address for the scratch area");
    g_scratch[device].zero = (uint8_t *)z;
    g_scratch[device].pages = (uint8_t *)p;
    return SPK_OK;
}

// Pinned host blocks for the readers, one per network while it lives; a few
// are kept for the next networks (allocating one takes as long as creating a
// small network).
constexpr size_t kStageKeep = 4;
std::mutex g_stage_mu;
std::vector<uint32_t *> g_stage_free;

uint32_t *stage_take()
{
    {
        std::lock_guard<std::mutex> lock(g_stage_mu);
        if (!g_stage_free.empty()) {
            uint32_t *p = g_stage_free.back();
            g_stage_free.pop_back();
            return p;
        }
    }
    void *p = nullptr;  // (mapped into every device's address space)
    if (hipHostMalloc(&p, kStageBytes, hipHostMallocPortable | hipHostMallocMapped) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    return (uint32_t *)p;
}

void stage_give(uint32_t *p)
{
    if (!p) return;
    {
        std::lock_guard<std::mutex> lock(g_stage_mu);
        if (g_stage_free.size() < kStageKeep) {
            g_stage_free.push_back(p);
            return;
        }
    }
    (void)hipHostFree(p);
}

// The device's scratch for one call (ScratchFlag): *clear = its zero area has
// to be cleared first.
Scratch scratch_take(int device, bool capturing, bool *clear)
{
    *clear = false;
    if (device < 0 || device >= kMaxDevices) return Scratch{};
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    *clear = g_scratch[device].flag.begin(capturing);
    return g_scratch[device];
}

void scratch_done(int device, bool capturing, bool zero)
{
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    g_scratch[device].flag.end(capturing, zero);
}

uint64_t prob_threshold(double p)
{
    if (!(p > 0.0)) return 0;
    if (p >= 1.0) return 4294967296ull;
    return (uint64_t)std::floor(p * 4294967296.0);
}

// Poisson(lambda) thresholds on a 32-bit uniform draw: T_k = floor(CDF(k)*2^32)
// with the CDF summed in double from p_0 = exp(-lambda), p_k = p_{k-1}*lambda/k;
// the table ends with 2^32 once the CDF reaches 1 - 2^-32.
int poisson_thresholds(double lambda, std::vector<uint64_t> &thr)
{
    thr.clear();
    if (!(lambda > 0.0) || lambda > 100.0) return -1;
    double pk = std::exp(-lambda), cdf = pk;
    for (uint32_t k = 0;; k++) {
        const double T = std::floor(cdf * 4294967296.0);
        if (T >= 4294967295.0 || k == kPoisCap - 1) {
            thr.push_back(4294967296ull);
            return (int)thr.size();
        }
        thr.push_back((uint64_t)T);
        pk = (pk * lambda) / (double)(k + 1);
        cdf = cdf + pk;
    }
}

// Guide table of the indexed search (Chen & Asau 1974): for the 256 ranges of
// the top 8 bits of the draw, the first k whose threshold exceeds the range
// start; the search for K = min{k : h < T_k} starts there.
std::vector<uint16_t> poisson_guide(const std::vector<uint64_t> &thr)
{
    std::vector<uint16_t> g(256, 0);
    uint32_t k = 0;
    for (uint32_t b = 0; b < 256; b++) {
        const uint64_t lo = (uint64_t)b << 24;
        while (k + 1 < thr.size() && thr[k] <= lo) k++;
        g[b] = (uint16_t)k;
    }
    return g;
}

bool quantise(float w, int S, int32_t *out)
{
    const float x = std::rint(std::ldexp(w, S));
    if (!(std::fabs(x) < 2147483648.0f)) return false;
    *out = (int32_t)x;
    return true;
}

// Tiles of W neurons (a power of two, at most kMaxTileW), 8 groups of T8
// tiles; the smallest W that keeps T8 <= max_t8 (default 32: one tile per
// compute unit).  SPK_TILES_PER_XCD overrides max_t8 (a tuning knob).
Tiling tiling_of(uint32_t n, uint32_t W)
{
    Tiling tl{};
    tl.W = W;
    while ((1u << tl.logW) < W) tl.logW++;
    tl.T8 = (uint32_t)((n + 8ull * W - 1) / (8ull * W));
    tl.T = kGroups * tl.T8;
    tl.Gw = tl.T8 * W;
    tl.T8inv = tl.T8 > 1 ? (uint32_t)(((1ull << 32) + tl.T8 - 1) / tl.T8) : 0u;
    return tl;
}

uint32_t tiles_per_xcd_cap()
{
    if (const char *e = std::getenv("SPK_TILES_PER_XCD")) {
        const long v = std::strtol(e, nullptr, 10);
        if (v >= 1 && v <= (long)kMaxT8) return (uint32_t)v;
    }
    return 32;
}

Tiling make_tiling(uint32_t n)
{
    const uint32_t max_t8 = tiles_per_xcd_cap();
    uint32_t W = 64;
    while (W < kMaxTileW && (n + 8ull * W - 1) / (8ull * W) > max_t8) W <<= 1;
    return tiling_of(n, W);
}

}  // namespace

struct spk_net {
    spk_params P{};
    // derived constants
    uint32_t n = 0, n_exc = 0, lists = 1, dmin = 1, dmax = 1, ref_steps = 0;
    uint32_t pois_len = 0, max_row = 0;
    float k = 0.f;
    uint64_t conn_thr = 0, src_thr = 0, nnz = 0;
    int32_t ext_wq = 0, bias_q = 0, shift64 = 0;
    Keys keys{};
    std::vector<uint64_t> pois;
    std::vector<uint16_t> guide;
    Tiling tl{};   // rows are grouped by; tiles of the step paths but the resident kernel
    Tiling rtl{};  // tiles of the resident kernel: one or several of tl's each
    bool direct = false;
    uint32_t spk_slots = 1, pslots = 1, pg1 = 1, page_cap = 0;
    // device
    hipStream_t stream = nullptr, cap_stream = nullptr;
    bool own_stream = false;
    int device = 0;
    uint64_t *row_ptr = nullptr;
    // synapses: full (int2) or compact (u32 with a weight class)
    bool compact = false;
    bool proc = false;  // procedural synapses: generated when their source fires, not stored
    bool proc_once = false;  // ... each fired row generated once (pages of every group per push block)
    uint32_t n_cls = 0;
    float cls_w[kMaxClasses] = {};
    ClassTab ctab{};
    long long wval[kMaxClasses] = {};
    int2 *syn = nullptr;
    uint32_t *syn32 = nullptr;
    RowDesc *desc = nullptr;
    uint16_t *toff = nullptr;
    uint16_t *rtoff = nullptr;  // resident kernel: the offsets of its tiles (toff itself where they are the same)
    uint32_t *outdeg = nullptr;
    float *V = nullptr;
    uint8_t *ref = nullptr;
    uint32_t *spk_ids = nullptr, *spk_cnt = nullptr, *counts8 = nullptr, *flags = nullptr;
    uint64_t *events8 = nullptr, *delivered8 = nullptr, *pois_dev = nullptr, *t_base = nullptr;
    uint16_t *guide_dev = nullptr;
    int2 *pages = nullptr;
    uint16_t *pages16 = nullptr;
    uint32_t *pfill = nullptr, *ovf_flag = nullptr;
    void *acc_ovf = nullptr;
    uint32_t *raster = nullptr;
    uint64_t *raster_offs = nullptr;
    void *dbg_out = nullptr;
    uint32_t *stage = nullptr;  // pinned host block of the readers (null: none could be had)
    uint64_t t = 0;
    uint64_t device_bytes = 0;
    std::vector<void *> allocs;
    std::map<uint32_t, hipGraphExec_t> graphs;
    // persistent step kernel
    bool persistent = false;
    uint32_t run_R = 0;
    uint32_t run_D = 1;  // persistent kernel, binned delivery: steps per batch
    bool run_counts = false;  // persistent kernel: accumulators are packed event counts
    RunCtl *ctl = nullptr;
    // resident step kernel: planned before the rows are laid out (the tiling
    // and the per-tile row offsets depend on it), used if it can be launched
    bool ring = false;
    bool ring_counts = false;   // accumulators are packed event counts
    uint32_t ring_epoch = 0;    // batches published so far
    uint32_t ring_pending = 0;  // steps of the last batch, if its spikes are still to be gathered
    uint32_t seg_cap = 0;
    RingCtl *rctl = nullptr;
    void *ring_buf = nullptr;
    uint32_t *ring_seg = nullptr, *ring_cnts = nullptr;
    // profiling
    bool profiling = false;
    std::vector<hipEvent_t> ev_free;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> ev_push, ev_tile, ev_run;
    double ms_push = 0, ms_tile = 0, ms_run = 0;
    uint64_t launches = 0, run_launches = 0;
    // setup timing
    double setup_ms = 0, gen_ms = 0, range_ms = 0;
};

namespace {

// GPU time of the work enqueued on a stream between start() and stop(),
// added to *acc by stop() (which waits for the work).
struct SegTimer {
    hipEvent_t e0 = nullptr, e1 = nullptr;
    SegTimer() = default;
    SegTimer(const SegTimer &) = delete;
    SegTimer &operator=(const SegTimer &) = delete;
    ~SegTimer()
    {
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
    }
    hipError_t start(hipStream_t s)
    {
        hipError_t e = e0 ? hipSuccess : hipEventCreate(&e0);
        if (e == hipSuccess && !e1) e = hipEventCreate(&e1);
        return e == hipSuccess ? hipEventRecord(e0, s) : e;
    }
    hipError_t stop(hipStream_t s, double *acc)
    {
        hipError_t e = hipEventRecord(e1, s);
        if (e == hipSuccess) e = hipEventSynchronize(e1);
        float t = 0.f;
        if (e == hipSuccess) e = hipEventElapsedTime(&t, e0, e1);
        if (e == hipSuccess) *acc += t;
        return e;
    }
};

template <class T>
spk_status dalloc(spk_net *net, T **p, size_t count)
{
    *p = nullptr;
    const size_t bytes = (count ? count : 1) * sizeof(T);
    void *q = nullptr;
    hipError_t e = hipMalloc(&q, bytes);
    if (e != hipSuccess)
        return fail(SPK_ENOMEM, "hipMalloc of " + std::to_string(bytes) + " bytes: " +
                                    hipGetErrorString(e));
    net->allocs.push_back(q);
    net->device_bytes += bytes;
    *p = (T *)q;
    return SPK_OK;
}

void dfree(spk_net *net, void *p)
{
    if (!p) return;
    auto it = std::find(net->allocs.begin(), net->allocs.end(), p);
    if (it != net->allocs.end()) net->allocs.erase(it);
    (void)hipFree(p);
}

ModelArgs model_args(const spk_net *net)
{
    ModelArgs m{};
    m.n = net->n;
    m.kind = net->P.neuron_kind;
    m.fixed = net->P.acc_mode == SPK_ACC_FIXED;
    m.shift = net->P.fixed_shift;
    m.shift64 = net->shift64;
    m.k = net->k;
    m.v_rest = net->P.v_rest;
    m.v_th = net->P.v_th;
    m.v_reset = net->P.v_reset;
    m.i_bias = net->P.i_bias;
    m.ext_w = net->P.ext_w;
    m.ext_wq = net->ext_wq;
    m.bias_q = net->bias_q;
    m.ref_steps = net->ref_steps;
    m.pois_len = net->pois_len;
    m.src_thr = net->src_thr;
    m.keys = net->keys;
    return m;
}

StepArgs step_args(const spk_net *net)
{
    StepArgs a{};
    a.m = model_args(net);
    a.tl = net->tl;
    a.n = net->n;
    a.lists = net->lists;
    a.dmin = net->dmin;
    a.direct = net->direct ? 1u : 0u;
    a.row_ptr = net->row_ptr;
    a.compact = net->compact ? 1u : 0u;
    a.proc = net->proc ? 1u : 0u;
    a.pr.k_out = net->P.k_out;
    a.pr.once = net->proc_once ? 1u : 0u;
    a.pr.n_exc = net->n_exc;
    a.pr.w_uniform = net->P.w_uniform;
    a.pr.w_lo = net->P.w_lo;
    a.pr.w_hi = net->P.w_hi;
    a.pr.w_exc = net->P.w_exc;
    a.pr.w_inh = net->P.w_inh;
    a.pr.qscale = std::ldexp(1.0f, net->P.fixed_shift);
    for (uint32_t k = 0; k < kMaxClasses; k++) a.wval[k] = net->wval[k];
    a.syn = net->syn;
    a.syn32 = net->syn32;
    a.desc = net->desc;
    a.toff = net->toff;
    a.row_len = net->P.conn_kind == SPK_CONN_FIXED_OUT ? net->P.k_out : 0u;
    a.outdeg = net->outdeg;
    a.V = net->V;
    a.ref = net->ref;
    a.spk_slots = net->spk_slots;
    a.spk_ids = net->spk_ids;
    a.spk_cnt = net->spk_cnt;
    a.counts8 = net->counts8;
    a.events8 = net->events8;
    a.delivered8 = net->delivered8;
    a.pages = net->pages;
    a.pages16 = net->pages16;
    a.pfill = net->pfill;
    a.page_cap = net->page_cap;
    a.pslots = net->pslots;
    a.pg1 = net->pg1;
    a.acc_ovf = net->acc_ovf;
    a.ovf_flag = net->ovf_flag;
    a.pois = net->pois_dev;
    a.pois_guide = net->guide_dev;
    a.flags = net->flags;
    a.raster = net->raster;
    a.raster_offs = net->raster_offs;
    a.raster_cap = net->P.raster_capacity;
    a.t_base = net->t_base;
    a.dbg_j = -1;
    return a;
}

ConnArgs conn_args(const spk_net *net)
{
    ConnArgs c{};
    c.n = net->n;
    c.n_exc = net->n_exc;
    c.kind = net->P.conn_kind;
    c.lists = net->lists;
    c.dmin = net->dmin;
    c.k_out = net->P.k_out;
    c.k_in_exc = net->P.k_in_exc;
    c.k_in_inh = net->P.k_in_inh;
    c.conn_thr = net->conn_thr;
    c.w_uniform = net->P.w_uniform;
    c.w_exc = net->P.w_exc;
    c.w_inh = net->P.w_inh;
    c.w_lo = net->P.w_lo;
    c.w_hi = net->P.w_hi;
    c.fixed = net->P.acc_mode == SPK_ACC_FIXED;
    c.qscale = std::ldexp(1.0f, net->P.fixed_shift);
    c.compact = net->compact ? 1u : 0u;
    for (uint32_t k = 0; k < kMaxClasses; k++) {
        float w = net->cls_w[k < net->n_cls ? k : 0];
        std::memcpy(&c.cls_w[k], &w, 4);
    }
    c.keys = net->keys;
    c.tl = net->tl;
    return c;
}

// Synapse format.  classes = the distinct weights (null: per-synapse weights).
// Class k stores its weight bits (fp32, or the quantised int32 in fixed mode)
// and the |weight| term of the accumulator-range bound, both as the full
// format would per synapse.
spk_status choose_format(spk_net *net, const float *classes, uint32_t n_cls)
{
    const uint32_t f = net->P.syn_format;
    const bool ok = classes && n_cls >= 1 && n_cls <= kMaxClasses;
    if (f == SPK_FORMAT_COMPACT && !ok)
        return fail(SPK_EINVAL, "the compact synapse format needs at most 4 distinct weights");
    net->compact = ok && f != SPK_FORMAT_FULL;
    net->n_cls = 0;
    net->ctab = ClassTab{};
    if (!net->compact) return SPK_OK;
    const bool fixed = net->P.acc_mode == SPK_ACC_FIXED;
    net->n_cls = n_cls;
    for (uint32_t k = 0; k < kMaxClasses; k++) {
        const float w = classes[k < n_cls ? k : 0];
        net->cls_w[k] = w;
        if (fixed) {
            int32_t q = 0;
            if (!quantise(w, net->P.fixed_shift, &q))
                return fail(SPK_EOVERFLOW, "a weight does not fit int32 at this fixed_shift");
            net->ctab.bits[k] = (uint32_t)q;
            net->ctab.abs[k] = (uint64_t)std::llabs((long long)q);
        } else {
            std::memcpy(&net->ctab.bits[k], &w, 4);
            net->ctab.abs[k] = (uint64_t)std::ceil(std::ldexp((double)std::fabs(w), 24));
        }
    }
    return SPK_OK;
}

// How the accumulator range of a generated Bernoulli network is found: per
// target from the pair predicate (n^2 hashes, ~1.7e12 per s) when that costs
// less than one global atomic per synapse (~2.4e10 per s).
// SPK_RANGE_PASS=targets / atomics forces either (a tuning knob, for tests).
bool range_by_targets(const spk_net *net)
{
    if (net->P.conn_kind != SPK_CONN_BERNOULLI) return false;
    if (const char *e = std::getenv("SPK_RANGE_PASS")) return std::strcmp(e, "targets") == 0;
    return (double)net->nnz * 70.0 > (double)net->n * (double)net->n;
}

// Fixed out-degree networks with population weights (generated, compact
// classes = source populations): the range from the synapses drawn again and
// filed by target tile, counted per class in LDS (no global atomic per
// synapse).  SPK_RANGE_PASS=atomics forces the per-synapse atomic pass.
bool range_by_tiles(const spk_net *net)
{
    if (net->P.conn_kind != SPK_CONN_FIXED_OUT || !net->compact || net->n_cls > 2) return false;
    if (const char *e = std::getenv("SPK_RANGE_PASS")) return std::strcmp(e, "atomics") != 0;
    return !net->toff;  // (rows grouped by tile are summed as they are)
}

// Largest in_abs_sum of a fixed out-degree network by tiles (range_by_tiles);
// *ok = false (and nothing changed) when its temporary buckets (2 bytes per
// synapse) cannot be allocated.
spk_status fo_range(spk_net *net, uint64_t *m, bool *ok)
{
    hipStream_t s = net->stream;
    const ConnArgs c = conn_args(net);
    const uint32_t T = net->tl.T, nb = fo_blocks(net->n);
    *ok = false;
    uint16_t *entries = nullptr;
    if (dalloc(net, &entries, (size_t)std::max<uint64_t>(net->nnz, 1)) != SPK_OK) {
        (void)hipGetLastError();  // the failed allocation is not an error of a later call
        return SPK_OK;
    }
    uint32_t *base = nullptr, *tot = nullptr;
    uint64_t *start = nullptr, *mx = nullptr;
    SPK_TRY(dalloc(net, &base, (size_t)nb * T));
    SPK_TRY(dalloc(net, &tot, T));
    SPK_TRY(dalloc(net, &start, T + 1));
    SPK_TRY(dalloc(net, &mx, 1));
    SPK_HIP(hipMemsetAsync(tot, 0, (size_t)T * 4, s));
    SPK_HIP(hipMemsetAsync(mx, 0, 8, s));
    SegTimer tm;
    SPK_HIP(tm.start(s));
    SPK_HIP(fo_count(c, base, tot, s));
    std::vector<uint32_t> ht(T);
    SPK_HIP(hipMemcpyAsync(ht.data(), tot, (size_t)T * 4, hipMemcpyDeviceToHost, s));
    SPK_HIP(hipStreamSynchronize(s));
    std::vector<uint64_t> hs(T + 1, 0);
    for (uint32_t k = 0; k < T; k++) hs[k + 1] = hs[k] + ht[k];
    if (hs[T] != net->nnz) return fail(SPK_EHIP, "range pass: filed synapses do not add up to nnz");
    SPK_HIP(hipMemcpyAsync(start, hs.data(), (size_t)(T + 1) * 8, hipMemcpyHostToDevice, s));
    SPK_HIP(fo_file(c, base, start, entries, s));
    SPK_HIP(fo_max(c, start, entries, net->ctab, mx, s));
    SPK_HIP(tm.stop(s, &net->range_ms));
    SPK_HIP(hipMemcpyAsync(m, mx, 8, hipMemcpyDeviceToHost, s));
    SPK_HIP(hipStreamSynchronize(s));  // (hs is host memory read by the copy above)
    dfree(net, entries); dfree(net, base); dfree(net, tot); dfree(net, start); dfree(net, mx);
    *ok = true;
    return SPK_OK;
}

// The term of one synapse of weight w in the accumulator-range bound, as the
// range pass computes it: |quantised w| (fixed mode) or |w| in units of
// 2^-24 rounded up (fp32 mode).
spk_status abs_term(const spk_net *net, float w, uint64_t *out)
{
    if (net->P.acc_mode == SPK_ACC_FIXED) {
        int32_t q = 0;
        if (!quantise(w, net->P.fixed_shift, &q))
            return fail(SPK_EOVERFLOW, "a weight does not fit int32 at this fixed_shift");
        *out = (uint64_t)std::llabs((long long)q);
    } else {
        *out = (uint64_t)std::ceil(std::ldexp((double)std::fabs(w), 24));
    }
    return SPK_OK;
}

// Per-class accumulator units, once the unit is known.
void class_units(spk_net *net)
{
    const bool fixed = net->P.acc_mode == SPK_ACC_FIXED;
    for (uint32_t k = 0; k < kMaxClasses; k++) {
        if (!net->compact) {
            net->wval[k] = 0;
        } else if (fixed) {
            net->wval[k] = (long long)(int32_t)net->ctab.bits[k];
        } else {
            // exact: every weight is a multiple of the unit 2^-S64 (as the
            // per-event conversion of the full format, rounded to nearest)
            net->wval[k] = std::llrint(std::ldexp((double)net->cls_w[k], net->shift64));
        }
    }
}

// Whether the resident step kernel serves the network, its tiling, and the
// one that rows are grouped by (called once the synapse format is known,
// before rows are laid out).
// in_max: the largest in-degree per class where it is known (explicit
// adjacency), else null.
void plan_ring(spk_net *net, uint64_t nnz_expected, const uint64_t *in_max)
{
    net->ring = net->ring_counts = false;
    const spk_params &P = net->P;
    if (net->proc || P.step_mode == SPK_STEP_GRAPH || P.delivery == SPK_DELIVERY_BINNED) return;
    if (P.delivery == SPK_DELIVERY_DIRECT && net->lists > 1) return;
    uint32_t knob = 0;  // tile width asked for
    if (const char *e = std::getenv("SPK_RING")) {
        const long v = std::strtol(e, nullptr, 10);
        if (e[0] == '0') return;
        if (v >= 64 && v <= (long)kMaxTileW && (v & (v - 1)) == 0) knob = (uint32_t)v;
    }
    const double n = (double)net->n, ne = (double)net->n_exc, ni = n - ne;
    // Packed counts: at most two classes, and no neuron may receive 2^16
    // events of one class in one step (each in-synapse delivers at most one).
    // Checked against the range pass once it has run (finish_rows); here
    // only where that check is sure to hold.
    bool counts = net->compact && net->n_cls <= 2;
    if (counts) {
        const double a0 = (double)net->ctab.abs[0], a1 = (double)net->ctab.abs[1];
        if (in_max) {
            counts = in_max[0] < 65536 && in_max[1] < 65536;
        } else {
            const double per = (double)nnz_expected / n / n;  // synapses per (source, target)
            double me = ne * per, mi = ni * per;
            if (P.conn_kind == SPK_CONN_FIXED_IN) {
                me = P.k_in_exc;
                mi = P.k_in_inh;
            }
            const double sum = (me + 12.0 * std::sqrt(me) + 64.0) * a0 + (mi + 12.0 * std::sqrt(mi) + 64.0) * a1;
            counts = a0 > 0 && a1 > 0 && sum / std::min(a0, a1) < 65000.0;
        }
    }
    if (!counts && net->lists > 1) return;
    const uint32_t acc = ring_acc_bytes(P.acc_mode == SPK_ACC_FIXED, counts);
    // Tile width (microseconds per step on one MI355X):
    //   One tile has no hand-off, but one compute unit delivers every event:
    //   1,000 neurons with 1,000 events per step 2.6, against 3.4 on 16 tiles;
    //   600 sources with 5,900 events 4.0 and 3.9, with 36,000 13.1 and 5.0
    //   (page kernel 10.3); 1,500 sources (a tile of 2,048) with 1,500 events
    //   3.5 and 3.5, with 7,300 5.0 and 3.8.  Sources fire at a known rate.
    //   Neurons fire at most as often as their refractory time lets them,
    //   and then one tile is to be no slower than the page kernel (2,040
    //   neurons at 17,800 events 8.8 against 10.3; at 2,400 3.8 against 9.1).
    //   Batches share their hand-offs: several tiles are as fast from the
    //   start (700 neurons with delay 15 0.9 against 1.1, 2,040 0.9 against
    //   2.5 and, driven hard, 1.3 against 6.5).
    //   Several: narrow ones, up to 48, spread the events over more compute
    //   units (2,500 sources at 10 / 50 / 300 Hz 4.0 / 4.7 / 10.0 on 40 tiles
    //   of 64, 7.2 / 18.8 / 44 on 5 of 512, 9.9 / 10.5 / 19.8 in the page
    //   kernel); more mailboxes to poll cost more than that gives at ordinary
    //   rates (4,000 neurons 3.8 on 32 tiles, 4.0 on 63; 30,000 4.8 on 59
    //   tiles of 512, 5.2 on 118, 6.6 on 235), and fewer do where tiles twice
    //   as wide would have few events in a step (300 of sources: 2,500 at 2 Hz
    //   3.6 on 20 tiles, 3.7 on 10, 4.4 on 5 with 820 each; 1,000 of neurons at
    //   their most, a tenth of that as a rule: 4,852 neurons with fan-out 68
    //   4.1 on 10 tiles, 4.3 on 38), batches apart;
    //   from 512 on at most 128 tiles (120,000 neurons: 6.2 on 118 tiles of
    //   1,024, 7.0 on 235 of 512), but not wider than 2,048 for it (300,000:
    //   7.9 on 147 tiles of 2,048, 8.6 on 74 of 4,096);
    //   from 7e8 synapses on the gather decides, on as many compute units as
    //   there are (120,000 neurons on 235 / 118 tiles: 4e8 synapses 6.4 / 5.9,
    //   7e8 6.8 / 6.9; 250,000 on 245 / 123: 4e8 7.3 / 6.7, 7e8 7.7 / 7.3,
    //   1.25e9 8.8 / 10.0), in batches, whose polling is shared, from 4e8 on
    //   (delay 15: 120,000 neurons, 4e8 1.9 / 2.4; 100,000, 1e9 2.0 on 196, 2.6
    //   on 98).
    //   Where a tile would deliver more than 8,000 events per step, narrower
    //   ones (sources, 5,100 per tile: 60,000 at 10 Hz 7.7 on 118 tiles, 9.0
    //   on 235; 12,700: 20,000 at 50 Hz 10.0 on 79, 8.6 on 157); neurons, which
    //   rarely fire that often, up to 80 tiles (20,000: 4.5 on 40 and on 79).
    const uint64_t nnz = nnz_expected;
    const bool fixed_cap = std::getenv("SPK_TILES_PER_XCD") != nullptr;
    auto fits = [&](uint32_t W) {
        return (uint64_t)net->dmax * W * acc <= (W >= net->n && W <= kRingW1 ? kRingBytes1 : kRingBytes);
    };
    auto tiles = [&](uint32_t W) { return (net->n + W - 1) / W; };
    const bool source = P.neuron_kind == SPK_SOURCE;
    const double ev = source ? (double)nnz * (double)net->src_thr * 0x1p-32  // events per step
                             : (double)nnz / (net->ref_steps + 1.0);         // ... at most, sustained
    const uint32_t W1 = net->n <= 1024 ? 1024 : 2048;
    const double ev1 = !source ? 20000.0 : W1 == 1024 ? 5000.0 : 2000.0;
    const bool batches = net->dmin > 1 && P.delivery != SPK_DELIVERY_DIRECT;
    uint32_t W = 0;
    if (knob) {
        W = knob;
    } else if (fixed_cap) {
        W = make_tiling(net->n).W;
    } else if (net->n <= 2048 && !batches && ev <= ev1 && fits(W1)) {
        W = W1;
    } else {
        const uint32_t most = nnz >= (batches ? 400000000ull : 700000000ull) ? kRingMaxT : 128;
        const double few = batches ? 0.0 : source ? 300.0 : 1000.0;
        for (W = 64; W < 512 && (tiles(W) > 48 || ev <= few * tiles(2 * W)); W <<= 1) {}
        for (; W < kMaxTileW; W <<= 1)
            if (tiles(W) <= most || (W >= 2048 && tiles(W) <= kRingMaxT)) break;
        while (W > 64 && ev > 8000.0 * tiles(W) && tiles(W >> 1) <= (source ? kRingMaxT : 80u)) W >>= 1;
        while (W > 64 && !fits(W)) W >>= 1;  // (narrower tiles hold more arrival steps)
    }
    if (!fits(W)) return;
    const Tiling tl = tiling_of(net->n, W);
    if (tl.T > kRingMaxT) return;
    // the rows' tile offsets: 64 MB, or half the full synapses' size
    auto room = [&](const Tiling &x) { return (double)net->n * (x.T + 1) * 2.0 <= std::max(64e6, 4.0 * (double)nnz); };
    if (!room(tl)) return;
    net->ring = true;
    net->ring_counts = counts;
    net->rtl = tl;
    // Rows are grouped by the general tiling, as for the other step paths,
    // where its narrower tiles' offsets have room: deliveries of a given
    // spike list (k_tile) then run on as many compute units as there
    // (1,000 spikes through 20,000 neurons with fan-out 700: 10.7 us, on
    // this kernel's 40 tiles 19.3).
    if (net->tl.W > W || !room(net->tl)) net->tl = tl;
}

// Synapse storage of the chosen format.
spk_status alloc_syn(spk_net *net, void **p, uint64_t nnz)
{
    uint8_t *q = nullptr;
    SPK_TRY(dalloc(net, &q, (size_t)nnz * (net->compact ? 4 : 8)));
    *p = q;
    return SPK_OK;
}

// The rows' tile offsets, and the resident kernel's beside them where its
// tiles are wider.
spk_status alloc_toff(spk_net *net)
{
    const size_t m = (size_t)net->n * (net->tl.T + 1);
    const bool two = net->ring && net->rtl.W != net->tl.W;
    SPK_TRY(dalloc(net, &net->toff, m + (two ? (size_t)net->n * (net->rtl.T + 1) : 0)));
    net->rtoff = two ? net->toff + m : net->toff;
    return SPK_OK;
}

const void *syn_ptr(const spk_net *net)
{
    return net->compact ? (const void *)net->syn32 : (const void *)net->syn;
}

// Largest in-degree over neurons of the compact records syn, of each of two
// weight classes: counted together first, apart only where both together
// could pass the bound that plan_ring puts on each.  (On the device: 1e7
// synapses counted in the host's pass over them took 6 ms of a creation of 18.)
spk_status in_degrees(spk_net *net, const void *syn, uint64_t nnz, uint64_t in_max[2])
{
    hipStream_t s = net->stream;
    uint64_t *cnt = nullptr, *mx = nullptr;
    SPK_TRY(dalloc(net, &cnt, net->n));
    SPK_TRY(dalloc(net, &mx, 1));
    auto largest = [&](uint64_t a0, uint64_t a1, uint64_t *out) -> spk_status {
        ClassTab one{};
        one.abs[0] = a0;
        one.abs[1] = a1;
        SPK_HIP(hipMemsetAsync(cnt, 0, (size_t)net->n * 8, s));
        SPK_HIP(hipMemsetAsync(mx, 0, 8, s));
        SPK_HIP(in_abs_sum(syn, nnz, false, true, one, cnt, s));
        SPK_HIP(max_u64(cnt, net->n, mx, s));
        SPK_HIP(hipMemcpyAsync(out, mx, 8, hipMemcpyDeviceToHost, s));
        SPK_HIP(hipStreamSynchronize(s));
        return SPK_OK;
    };
    SPK_TRY(largest(1, 1, &in_max[0]));
    in_max[1] = in_max[0];
    if (in_max[0] > 65535) {
        SPK_TRY(largest(1, 0, &in_max[0]));
        SPK_TRY(largest(0, 1, &in_max[1]));
    }
    dfree(net, cnt);
    dfree(net, mx);
    return SPK_OK;
}

// Validate parameters and compute the derived constants.
spk_status derive(spk_net *net, bool explicit_csr)
{
    const spk_params &P = net->P;
    if (P.abi_version != SPK_ABI_VERSION) return fail(SPK_EINVAL, "abi_version mismatch");
    if (P.n == 0 || P.n > (1u << kTargetBits))
        return fail(SPK_EINVAL, "n must be in [1, 2^24]");
    if (!(P.dt_ms > 0.0) || !(P.tau_m_ms > 0.0) || !(P.t_ref_ms >= 0.0))
        return fail(SPK_EINVAL, "dt_ms, tau_m_ms must be > 0 and t_ref_ms >= 0");
    if (P.delay_min < 1 || P.delay_max < P.delay_min || P.delay_max > 253)
        return fail(SPK_EINVAL, "delays must satisfy 1 <= delay_min <= delay_max <= 253");
    if (P.delay_max - P.delay_min + 1 > kMaxLists)
        return fail(SPK_EINVAL, "at most 64 distinct delays");
    if (!(P.frac_exc >= 0.0 && P.frac_exc <= 1.0)) return fail(SPK_EINVAL, "frac_exc in [0,1]");
    if (P.neuron_kind > SPK_SOURCE) return fail(SPK_EINVAL, "neuron_kind");
    if (P.acc_mode > SPK_ACC_FIXED) return fail(SPK_EINVAL, "acc_mode");
    if (P.delivery > SPK_DELIVERY_BINNED) return fail(SPK_EINVAL, "delivery");
    if (P.syn_format > SPK_FORMAT_PROCEDURAL) return fail(SPK_EINVAL, "syn_format");
    if (P.syn_format == SPK_FORMAT_PROCEDURAL) {
        if (explicit_csr || P.conn_kind != SPK_CONN_FIXED_OUT || P.k_out == 0)
            return fail(SPK_EINVAL, "procedural synapses need a generated fixed out-degree network (k_out >= 1)");
        if (P.delivery == SPK_DELIVERY_DIRECT)
            return fail(SPK_EINVAL, "procedural synapses are delivered binned (each fired row generated once)");
        if (P.step_mode == SPK_STEP_PERSISTENT)
            return fail(SPK_EINVAL, "procedural synapses run as graphs of steps, not in the persistent kernel");
        net->proc = true;
    }
    if (P.step_mode > SPK_STEP_PERSISTENT) return fail(SPK_EINVAL, "step_mode");
    if (!explicit_csr && P.conn_kind > SPK_CONN_FIXED_IN) return fail(SPK_EINVAL, "conn_kind");
    if (!(P.p >= 0.0 && P.p <= 1.0)) return fail(SPK_EINVAL, "p in [0,1]");
    if (P.max_steps == 0) return fail(SPK_EINVAL, "max_steps must be >= 1");
    if (!(P.ext_lambda >= 0.0) || P.ext_lambda > 100.0) return fail(SPK_EINVAL, "ext_lambda in [0,100]");
    if (!explicit_csr && P.conn_kind == SPK_CONN_FIXED_OUT && P.k_out > kMaxRow)
        return fail(SPK_EINVAL, "k_out exceeds the longest supported row (65535)");
    net->n = P.n;
    net->n_exc = (uint32_t)std::llround(P.frac_exc * (double)P.n);
    net->k = (float)(P.dt_ms / P.tau_m_ms);
    const long long rs = std::llround(P.t_ref_ms / P.dt_ms);
    if (rs < 0 || rs > 255) return fail(SPK_EINVAL, "t_ref/dt must round to 0..255 steps");
    net->ref_steps = (uint32_t)rs;
    net->dmin = P.delay_min;
    net->dmax = P.delay_max;
    net->lists = P.delay_max - P.delay_min + 1;
    net->conn_thr = prob_threshold(P.p);
    net->src_thr = prob_threshold(P.src_rate_hz * P.dt_ms * 1e-3);
    net->tl = make_tiling(P.n);
    if (!explicit_csr && P.conn_kind == SPK_CONN_FIXED_IN &&
        ((P.k_in_exc > 0 && net->n_exc == 0) || (P.k_in_inh > 0 && net->n_exc == P.n)))
        return fail(SPK_EINVAL, "fixed in-degree needs a non-empty source population");
    if (P.ext_lambda > 0.0) {
        const int L = poisson_thresholds(P.ext_lambda, net->pois);
        if (L < 0) return fail(SPK_EINVAL, "ext_lambda");
        net->pois_len = (uint32_t)L;
        net->guide = poisson_guide(net->pois);
    }
    if (P.acc_mode == SPK_ACC_FIXED) {
        if (P.fixed_shift < 0 || P.fixed_shift > 30) return fail(SPK_EINVAL, "fixed_shift in 0..30");
        int32_t dummy;
        const int S = P.fixed_shift;
        if (!quantise(P.ext_w, S, &net->ext_wq) || !quantise(P.i_bias, S, &net->bias_q) ||
            !quantise(P.w_exc, S, &dummy) || !quantise(P.w_inh, S, &dummy) ||
            !quantise(P.w_lo, S, &dummy) || !quantise(P.w_hi, S, &dummy))
            return fail(SPK_EOVERFLOW, "a weight does not fit int32 at this fixed_shift");
    }
    if (!explicit_csr) {  // population weights: class 0 excitatory, 1 inhibitory
        const float w[2] = {P.w_exc, P.w_inh};
        SPK_TRY(choose_format(net, P.w_uniform ? nullptr : w, 2));
        const double nn = (double)P.n;
        plan_ring(net, (uint64_t)(P.conn_kind == SPK_CONN_BERNOULLI ? nn * nn * P.p
                                  : P.conn_kind == SPK_CONN_FIXED_OUT ? nn * P.k_out
                                                                      : nn * ((double)P.k_in_exc + P.k_in_inh)),
                  nullptr);
    }
    const uint64_t seed = P.seed;
    net->keys.conn = stream_key(seed, TAG_CONN);
    net->keys.tgt = stream_key(seed, TAG_TGT);
    net->keys.src_e = stream_key(seed, TAG_SRC_E);
    net->keys.src_i = stream_key(seed, TAG_SRC_I);
    net->keys.w = stream_key(seed, TAG_W);
    net->keys.delay = stream_key(seed, TAG_DELAY);
    net->keys.v0 = stream_key(seed, TAG_V0);
    net->keys.pois = stream_key(seed, TAG_POIS);
    net->keys.bern = stream_key(seed, TAG_BERN);
    return SPK_OK;
}

spk_status setup_stream(spk_net *net, void *stream)
{
    SPK_HIP(hipGetDevice(&net->device));
    SPK_TRY(scratch_lookup(net->device));
    if (stream) {
        net->stream = (hipStream_t)stream;
    } else {
        SPK_HIP(hipStreamCreateWithFlags(&net->stream, hipStreamNonBlocking));
        net->own_stream = true;
    }
    SPK_HIP(hipStreamCreateWithFlags(&net->cap_stream, hipStreamNonBlocking));
    net->stage = stage_take();
    return SPK_OK;
}

// Row offsets from per-row counts.
spk_status finish_counts(spk_net *net, const uint32_t *cnt)
{
    hipStream_t s = net->stream;
    const uint64_t n = net->n;
    uint64_t *bsum = nullptr;
    uint32_t *maxp = nullptr;
    SPK_TRY(dalloc(net, &net->row_ptr, n + 1));
    SPK_TRY(dalloc(net, &bsum, scan_scratch_elems(n) + 1));
    SPK_TRY(dalloc(net, &maxp, 1));
    SPK_HIP(hipMemsetAsync(maxp, 0, 4, s));
    SegTimer tm;
    SPK_HIP(tm.start(s));
    SPK_HIP(scan_counts(cnt, n, net->row_ptr, bsum, maxp, s));
    SPK_HIP(tm.stop(s, &net->gen_ms));
    uint64_t nnz = 0;
    uint32_t mr = 0;
    SPK_HIP(hipMemcpyAsync(&nnz, net->row_ptr + n, 8, hipMemcpyDeviceToHost, s));
    SPK_HIP(hipMemcpyAsync(&mr, maxp, 4, hipMemcpyDeviceToHost, s));
    SPK_HIP(hipStreamSynchronize(s));
    dfree(net, bsum);
    dfree(net, maxp);
    net->nnz = nnz;
    net->max_row = mr;
    return SPK_OK;
}

// Delivery strategy and the row index it needs.  Direct: every tile reads
// its run of each due row (rows long compared with the tile count, one
// delay, offsets small next to the synapses).  Binned: the push kernel sorts
// each fired row's events by (arrival step, tile) into pages.
spk_status choose_delivery(spk_net *net, RowIndex *ix)
{
    if (net->max_row > kMaxRow)
        return fail(SPK_EINVAL, "a source row of " + std::to_string(net->max_row) +
                                    " synapses exceeds the supported " + std::to_string(kMaxRow));
    const Tiling &tl = net->tl;
    const double mean_row = (double)net->nnz / (double)net->n;
    const double toff_bytes = (double)net->n * (tl.T + 1) * 2.0;
    const bool binned_ok = (uint64_t)net->lists * tl.T8 <= kMaxBuckets;
    bool direct = net->lists == 1 && mean_row >= 2.0 * tl.T && toff_bytes <= 0.5 * 8.0 * (double)net->nnz;
    // With a smallest delay of two steps or more, no event filed at t is
    // needed at t + 1: binned delivery lets the persistent kernel run steps
    // in batches and file a whole batch's events at once (or file them beside
    // the updates), which beats reading the due rows at arrival.
    if (direct && net->dmin >= 2 && net->P.step_mode != SPK_STEP_GRAPH && binned_ok) direct = false;
    if (!binned_ok || net->P.delivery == SPK_DELIVERY_DIRECT) direct = true;
    if (net->P.delivery == SPK_DELIVERY_BINNED) {
        if (!binned_ok)
            return fail(SPK_EINVAL, "binned delivery supports at most 2048 (delay, tile) buckets per "
                                    "XCD group; use fewer delays or direct delivery");
        direct = false;
    }
    if (net->ring) direct = true;  // (its rows are read by tile)
    net->direct = direct;
    *ix = RowIndex{};
    if (direct) {
        SPK_TRY(alloc_toff(net));
        ix->toff = net->toff;
    } else {
        SPK_TRY(dalloc(net, &net->desc, net->n));
        ix->desc = net->desc;
    }
    return SPK_OK;
}

// Out-degrees, accumulator range, delivery buffers.
spk_status finish_rows(spk_net *net)
{
    hipStream_t s = net->stream;
    const bool have_deg = net->outdeg != nullptr;
    if (!have_deg) SPK_TRY(dalloc(net, &net->outdeg, net->n));
    if (have_deg) {
        // (written with the rows)
    } else if (net->proc) {  // every row has k_out synapses
        const std::vector<uint32_t> deg(net->n, net->P.k_out);
        SPK_HIP(hipMemcpyAsync(net->outdeg, deg.data(), (size_t)net->n * 4, hipMemcpyHostToDevice, s));
        SPK_HIP(hipStreamSynchronize(s));
    } else {
        SPK_HIP(out_degree(net->row_ptr, net->n, net->outdeg, s));
    }

    if (net->rtoff != net->toff)
        SPK_HIP(coarse_toff(net->toff, net->n, net->tl.T, net->rtl.W / net->tl.W, net->rtl.T, net->rtoff, s));

    // Accumulator range.  Fixed mode: all in-synapses of one neuron at once,
    // plus the largest Poisson count and the bias, must fit in int32.  fp32
    // mode: choose the 64-bit fixed-point unit 2^-S64 as fine as the largest
    // possible sum allows.
    const bool fixed = net->P.acc_mode == SPK_ACC_FIXED;
    uint64_t m = 0;
    bool done = false;
    if (range_by_tiles(net)) SPK_TRY(fo_range(net, &m, &done));
    if (done) {
        // (the range is known)
    } else if (net->P.conn_kind == SPK_CONN_FIXED_IN && !net->P.w_uniform) {
        // every neuron has exactly k_in_exc excitatory and k_in_inh
        // inhibitory in-synapses, each with its population's weight: the
        // largest sum is every neuron's, no pass over the synapses needed
        uint64_t te = 0, ti = 0;
        SPK_TRY(abs_term(net, net->P.w_exc, &te));
        SPK_TRY(abs_term(net, net->P.w_inh, &ti));
        m = (uint64_t)net->P.k_in_exc * te + (uint64_t)net->P.k_in_inh * ti;
    } else if (net->toff && !std::getenv("SPK_RANGE_PASS")) {
        // rows grouped by tile: summed tile by tile in LDS (the resident
        // kernel's tiles, whose runs are longer)
        ConnArgs c = conn_args(net);
        if (net->ring) c.tl = net->rtl;
        uint64_t *insum = nullptr, *mx = nullptr;
        SPK_TRY(dalloc(net, &insum, net->n));
        SPK_TRY(dalloc(net, &mx, 1));
        SPK_HIP(hipMemsetAsync(insum, 0, (size_t)net->n * 8, s));
        SPK_HIP(hipMemsetAsync(mx, 0, 8, s));
        SegTimer tm;
        SPK_HIP(tm.start(s));
        SPK_HIP(rows_abs_sum(c, net->row_ptr, syn_ptr(net), net->ring ? net->rtoff : net->toff, net->ctab, insum, s));
        SPK_HIP(max_u64(insum, net->n, mx, s));
        SPK_HIP(tm.stop(s, &net->range_ms));
        SPK_HIP(hipMemcpyAsync(&m, mx, 8, hipMemcpyDeviceToHost, s));
        SPK_HIP(hipStreamSynchronize(s));
        dfree(net, insum);
        dfree(net, mx);
    } else if (range_by_targets(net)) {
        // Bernoulli: the pair predicate evaluated per target (n^2 hashes)
        // costs less than a global atomic per synapse above ~1.4 % density
        uint64_t *mx = nullptr, *insum = nullptr;
        SPK_TRY(dalloc(net, &mx, 1));
        SPK_HIP(hipMemsetAsync(mx, 0, 8, s));
        if (bern_src_ranges(net->n) > 1) {
            SPK_TRY(dalloc(net, &insum, net->n));
            SPK_HIP(hipMemsetAsync(insum, 0, (size_t)net->n * 8, s));
        }
        SegTimer tm;
        SPK_HIP(tm.start(s));
        SPK_HIP(bern_in_abs_max(conn_args(net), mx, insum, s));
        SPK_HIP(tm.stop(s, &net->range_ms));
        SPK_HIP(hipMemcpyAsync(&m, mx, 8, hipMemcpyDeviceToHost, s));
        SPK_HIP(hipStreamSynchronize(s));
        dfree(net, mx);
        if (insum) dfree(net, insum);
    } else {
        uint64_t *insum = nullptr, *mx = nullptr;
        SPK_TRY(dalloc(net, &insum, net->n));
        SPK_TRY(dalloc(net, &mx, 1));
        SPK_HIP(hipMemsetAsync(insum, 0, (size_t)net->n * 8, s));
        SPK_HIP(hipMemsetAsync(mx, 0, 8, s));
        SegTimer tm;
        SPK_HIP(tm.start(s));
        if (net->proc) SPK_HIP(proc_in_abs_sum(step_args(net), insum, s));
        else SPK_HIP(in_abs_sum(syn_ptr(net), net->nnz, fixed, net->compact, net->ctab, insum, s));
        SPK_HIP(max_u64(insum, net->n, mx, s));
        SPK_HIP(tm.stop(s, &net->range_ms));
        SPK_HIP(hipMemcpyAsync(&m, mx, 8, hipMemcpyDeviceToHost, s));
        SPK_HIP(hipStreamSynchronize(s));
        dfree(net, insum);
        dfree(net, mx);
    }
    if (fixed) {
        const uint64_t kmax = net->pois_len ? net->pois_len - 1 : 0;
        const uint64_t extra = kmax * (uint64_t)std::llabs((long long)net->ext_wq) +
                               (uint64_t)std::llabs((long long)net->bias_q);
        if (m + extra > 2147483647ull)
            return fail(SPK_EOVERFLOW, "fixed-point inputs could exceed int32; lower fixed_shift");
    } else {
        // every reachable |sum| stays below 2^52 (M <= 2^e): exact in double
        const double M = std::ldexp((double)m, -24);
        const int e = M > 0.0 ? (int)std::ceil(std::log2(M)) : 0;
        net->shift64 = std::max(0, std::min(100, 52 - e));
    }
    class_units(net);
    // no neuron can receive 2^16 events of a class in one step (an in-synapse
    // delivers at most one): m bounds each class's count times its |weight|
    const uint64_t abs_min = net->compact && net->n_cls <= 2 ? std::min(net->ctab.abs[0], net->ctab.abs[1]) : 0;
    const bool counts_fit = abs_min && m / abs_min <= 65535;
    if (net->ring_counts && net->P.conn_kind != SPK_CONN_EXPLICIT && !counts_fit) {
        // a neuron could receive 2^16 events of a class: sums, where they fit
        net->ring_counts = false;
        if (net->lists > 1 || (uint64_t)net->dmax * net->rtl.W * ring_acc_bytes(fixed, false) > kRingBytes) net->ring = false;
    }

    // Steps per batch of the persistent kernel (binned delivery): up
    // to the smallest delay, so that nothing a batch files arrives within it,
    // and within the bucket, slot and LDS limits.
    const Tiling &tl = net->tl;
    // (fixed-point sums are 32 bits wide already)
    net->run_counts = counts_fit && !fixed && !net->direct && !net->proc;
    net->run_D = 1;
    if (!net->direct || (net->ring && net->P.delivery != SPK_DELIVERY_DIRECT)) {
        // Default at most 8 steps: longer batches save hand-offs but give a
        // push block more events than one 16K-event sorting window holds
        // (measured on the delay-15 network: 7.3 us per step at 8, 7.4 at
        // 10, 7.6 at 12, 7.9 at 15).  SPK_BATCH_STEPS sets the cap (1..16).
        uint32_t cap = 8;
        if (const char *e = std::getenv("SPK_BATCH_STEPS")) {
            const long v = std::strtol(e, nullptr, 10);
            if (v >= 1) cap = (uint32_t)std::min<long>(v, kRunMaxD);
        }
        uint32_t D = std::min<uint32_t>(net->dmin, cap);
        // the tile keeps one accumulator array per step of the batch in LDS
        const uint32_t W = net->ring ? net->rtl.W : tl.W;
        while (D > 1 && ((!net->ring && (uint64_t)(D + net->lists - 1) * tl.T8 > kRunMaxBuckets) || D * W > kMaxTileW)) D--;
        net->run_D = D;
    }
    // Spike lists: direct delivery reads the lists of steps t - dmax .. t - dmin
    // while writing that of t; binned delivery consumes the list of t within t,
    // but in the persistent kernel one XCD may publish t + 1 while another
    // still reads t, so there are three; with batches of
    // D steps, one XCD may publish the next batch while another reads this one.
    net->spk_slots = net->direct ? net->dmax + 1 : std::max<uint32_t>(3, 2 * net->run_D);
    if (net->ring) net->pslots = net->dmax;
    if (!net->direct) {
        // Pages: (group, push block, arrival slot, tile).  A page never holds
        // more than nnz records (each synapse arrives at most once per slot),
        // so small networks never overflow; large ones get an equal share of
        // the budget and fall back to global atomics beyond it.
        net->pslots = net->dmax;
        net->pg1 = push_blocks_per_group();
        // procedural rows are generated once, by one push block per compute
        // unit, whose pages cover every group (graph path: the kernel boundary
        // makes them visible on every XCD), where its buckets fit
        net->proc_once = net->proc && (uint64_t)net->lists * tl.T <= kOnceMaxB;
        if (const char *e = std::getenv("SPK_PROC_ONCE"))  // 0: the per-group push (tests)
            if (e[0] == '0') net->proc_once = false;
        if (net->proc_once) net->pg1 *= kGroups;
        const uint64_t n_pages = (uint64_t)kGroups * net->pg1 * net->pslots * tl.T8;
        uint64_t cap = std::min<uint64_t>(kPageBudget / n_pages, std::max<uint64_t>(net->nnz, 1));
        if (const char *e = std::getenv("SPK_PAGE_CAP")) {
            const long long v = std::strtoll(e, nullptr, 10);
            if (v >= 1 && v <= (1ll << 30)) cap = (uint64_t)v;
        }
        cap = std::max<uint64_t>(16, (cap + 15) / 16 * 16);
        if (n_pages * cap >= (1ull << 32))  // page records are addressed with 32-bit indices
            return fail(SPK_EINVAL, "page capacity too large: pages x records must stay below 2^32");
        net->page_cap = (uint32_t)cap;
        const size_t acc_elems = (size_t)net->pslots * tl.T * tl.W;
        if (net->compact) SPK_TRY(dalloc(net, &net->pages16, n_pages * cap));
        else SPK_TRY(dalloc(net, &net->pages, n_pages * cap));
        SPK_TRY(dalloc(net, &net->pfill, n_pages));
        SPK_TRY(dalloc(net, &net->ovf_flag, (size_t)net->pslots * tl.T));
        SPK_TRY(dalloc(net, (uint64_t **)&net->acc_ovf, acc_elems));
        SPK_HIP(hipMemsetAsync(net->pfill, 0, n_pages * 4, s));
        SPK_HIP(hipMemsetAsync(net->ovf_flag, 0, (size_t)net->pslots * tl.T * 4, s));
        SPK_HIP(hipMemsetAsync(net->acc_ovf, 0, acc_elems * 8, s));
    }
    SPK_HIP(hipStreamSynchronize(s));
    return SPK_OK;
}

// Procedural synapses: nothing is generated or stored at creation; every
// row has k_out synapses, drawn when its source fires (binned delivery).
spk_status generate_proc(spk_net *net)
{
    net->nnz = (uint64_t)net->n * net->P.k_out;
    net->max_row = net->P.k_out;
    if ((uint64_t)net->lists * net->tl.T8 > kMaxBuckets)
        return fail(SPK_EINVAL, "binned delivery supports at most 2048 (delay, tile) buckets per XCD group");
    net->direct = false;
    return finish_rows(net);
}

// Bernoulli rows of a network of the resident kernel, drawn once: *ok =
// false (and nothing left behind) where they do not suit or did not fit.
spk_status generate_bern_once(spk_net *net, bool *ok)
{
    *ok = false;
    const double p = net->P.p, nn = (double)net->n, sd = std::sqrt(nn * p * (1.0 - p));
    // (the stage has a part for each of four waves, a quarter of the targets)
    if (!net->ring || net->P.conn_kind != SPK_CONN_BERNOULLI || nn * p / 4 + 5.0 * sd + 64.0 > (double)kBernStage / 4)
        return SPK_OK;
    hipStream_t s = net->stream;
    const uint64_t room = (uint64_t)(nn * nn * p + 10.0 * std::sqrt(nn) * sd) + 64;
    void *syn = nullptr;
    uint64_t *cursor = nullptr;
    uint32_t *mx = nullptr;
    SPK_TRY(dalloc(net, &net->row_ptr, (size_t)net->n + 1));
    SPK_TRY(dalloc(net, &net->outdeg, net->n));
    SPK_TRY(alloc_toff(net));
    SPK_TRY(alloc_syn(net, &syn, room));
    SPK_TRY(dalloc(net, &cursor, 1));
    SPK_TRY(dalloc(net, &mx, 1));
    SPK_HIP(hipMemsetAsync(cursor, 0, 8, s));
    SPK_HIP(hipMemsetAsync(mx, 0, 4, s));
    SegTimer tm;
    SPK_HIP(tm.start(s));
    SPK_HIP(gen_bern_once(conn_args(net), room, cursor, mx, net->row_ptr, net->outdeg, net->toff, syn, s));
    SPK_HIP(tm.stop(s, &net->gen_ms));
    uint64_t nnz = 0;
    uint32_t mr = 0;
    SPK_HIP(hipMemcpyAsync(&nnz, cursor, 8, hipMemcpyDeviceToHost, s));
    SPK_HIP(hipMemcpyAsync(&mr, mx, 4, hipMemcpyDeviceToHost, s));
    SPK_HIP(hipStreamSynchronize(s));
    dfree(net, cursor);
    dfree(net, mx);
    if (nnz > room) {
        dfree(net, syn);
        dfree(net, net->row_ptr);
        dfree(net, net->outdeg);
        dfree(net, net->toff);
        net->row_ptr = nullptr;
        net->outdeg = nullptr;
        net->toff = net->rtoff = nullptr;
        return SPK_OK;
    }
    if (net->compact) net->syn32 = (uint32_t *)syn;
    else net->syn = (int2 *)syn;
    net->nnz = nnz;
    net->max_row = mr;
    net->direct = true;
    *ok = true;
    return SPK_OK;
}

spk_status generate(spk_net *net)
{
    if (net->proc) return generate_proc(net);
    bool once = false;
    SPK_TRY(generate_bern_once(net, &once));
    if (once) return finish_rows(net);
    hipStream_t s = net->stream;
    uint32_t *cnt = nullptr;
    SPK_TRY(dalloc(net, &cnt, net->n));
    SPK_HIP(hipMemsetAsync(cnt, 0, (size_t)net->n * 4, s));
    ConnArgs c = conn_args(net);
    const bool in_rows = net->P.conn_kind == SPK_CONN_FIXED_IN;
    // Bernoulli rows: the count pass keeps every row's bucket counts (u16,
    // both deliveries' buckets), so the placement pass draws each row once
    // (SPK_GEN_HIST=0 skips it, as when it cannot be allocated: a test knob)
    uint16_t *hist = nullptr;
    const uint64_t hist_elems = (uint64_t)net->n * (net->tl.T + 2 * kGroups);
    const char *gh = std::getenv("SPK_GEN_HIST");
    const bool want_hist = !(gh && std::strcmp(gh, "0") == 0);
    if (net->P.conn_kind == SPK_CONN_BERNOULLI && want_hist && hist_elems * 2 <= (4ull << 30) &&
        dalloc(net, &hist, hist_elems) != SPK_OK) {
        hist = nullptr;          // (then the placement pass counts for itself)
        (void)hipGetLastError();  // the failed allocation is not an error of the launches below
    }
    // ... and keeps each row's synapses, up to cap = mean + 10 sd + 64 per
    // row, so that the placement pass need not draw the rows again (unless a
    // row turns out longer, or the keys would take more than 32 GB; small
    // networks are drawn again sooner than the keys are allocated: creation
    // of 5,000 neurons at 10 % 0.98 ms with keys, 0.69 without, of 20,000 at
    // 2 % 1.97 and 2.07, with 20 delays 2.14 and 2.40).  SPK_GEN_KEYS=0 / 1
    // never / always keeps them (a test knob).
    uint32_t *keys = nullptr;
    uint32_t cap = 0;
    const char *gk = std::getenv("SPK_GEN_KEYS");
    if (hist && (gk ? std::strcmp(gk, "0") != 0 : (uint64_t)net->n * net->n >= 200000000ull)) {
        const double p = net->P.p, nn = (double)net->n;
        const double capd = std::ceil(p * nn + 10.0 * std::sqrt(nn * p * (1.0 - p)) + 64.0);
        if (capd <= (double)kMaxRow && (double)net->n * capd * 4.0 <= (double)(32ull << 30)) {
            cap = (uint32_t)capd;
            if (dalloc(net, &keys, (size_t)net->n * cap) != SPK_OK) {
                keys = nullptr;
                (void)hipGetLastError();
            }
        }
    }
    SegTimer tm;
    SPK_HIP(tm.start(s));
    if (in_rows) SPK_HIP(gen_in_count(c, cnt, s));
    else SPK_HIP(gen_count_rows(c, cnt, hist, keys, cap, s));
    SPK_HIP(tm.stop(s, &net->gen_ms));
    SPK_TRY(finish_counts(net, cnt));
    if (keys && net->max_row > cap) {  // a row did not fit: placement draws the rows again
        dfree(net, keys);
        keys = nullptr;
    }
    RowIndex ix{};
    SPK_TRY(choose_delivery(net, &ix));
    void *syn = nullptr;
    SPK_TRY(alloc_syn(net, &syn, net->nnz));
    if (net->compact) net->syn32 = (uint32_t *)syn;
    else net->syn = (int2 *)syn;
    if (in_rows) {  // drawn per target: regroup by source, then bucket
        void *tmp = nullptr;
        SPK_TRY(alloc_syn(net, &tmp, net->nnz));
        SPK_HIP(hipMemsetAsync(cnt, 0, (size_t)net->n * 4, s));
        SPK_HIP(tm.start(s));
        SPK_HIP(gen_in_fill(c, net->row_ptr, cnt, tmp, s));
        SPK_HIP(bucket_rows(c, net->row_ptr, tmp, syn, ix, s));
        SPK_HIP(tm.stop(s, &net->gen_ms));
        dfree(net, tmp);
    } else {        // drawn per source, bucketed while drawn
        SPK_HIP(tm.start(s));
        SPK_HIP(gen_fill_rows(c, net->row_ptr, syn, ix, hist, keys, cap, s));
        SPK_HIP(tm.stop(s, &net->gen_ms));
    }
    SPK_HIP(hipStreamSynchronize(s));
    dfree(net, cnt);
    dfree(net, hist);
    dfree(net, keys);
    return finish_rows(net);
}

// State, spike lists and per-step records.
spk_status alloc_state(spk_net *net)
{
    const uint32_t n = net->n;
    const uint64_t T = net->P.max_steps;
    const Tiling &tl = net->tl;
    hipStream_t s = net->stream;
    const uint64_t segs = (uint64_t)net->spk_slots * tl.T;
    SPK_TRY(dalloc(net, &net->V, n));
    SPK_TRY(dalloc(net, &net->ref, n));
    SPK_TRY(dalloc(net, &net->spk_ids, segs * tl.W));
    SPK_TRY(dalloc(net, &net->spk_cnt, segs));
    SPK_TRY(dalloc(net, &net->counts8, T * kGroups));
    SPK_TRY(dalloc(net, &net->events8, T * kGroups));
    SPK_TRY(dalloc(net, &net->delivered8, T * kGroups));
    SPK_TRY(dalloc(net, &net->flags, 1));
    SPK_TRY(dalloc(net, (uint32_t **)&net->dbg_out, n));
    SPK_TRY(dalloc(net, &net->t_base, 1));
    SPK_TRY(dalloc(net, &net->raster_offs, T + 1));
    SPK_TRY(dalloc(net, &net->raster, net->P.raster_capacity));
    SPK_TRY(dalloc(net, &net->pois_dev, net->pois_len ? net->pois_len : 1));
    SPK_TRY(dalloc(net, &net->guide_dev, 256));
    SPK_HIP(hipMemsetAsync(net->spk_cnt, 0, segs * 4, s));
    SPK_HIP(hipMemsetAsync(net->counts8, 0, T * kGroups * 4, s));
    SPK_HIP(hipMemsetAsync(net->events8, 0, T * kGroups * 8, s));
    SPK_HIP(hipMemsetAsync(net->delivered8, 0, T * kGroups * 8, s));
    SPK_HIP(hipMemsetAsync(net->flags, 0, 4, s));
    SPK_HIP(hipMemsetAsync(net->t_base, 0, 8, s));
    SPK_HIP(hipMemsetAsync(net->raster_offs, 0, (T + 1) * 8, s));
    SPK_HIP(hipMemsetAsync(net->guide_dev, 0, 512, s));
    if (net->pois_len) {
        SPK_HIP(hipMemcpyAsync(net->pois_dev, net->pois.data(), net->pois_len * 8,
                               hipMemcpyHostToDevice, s));
        SPK_HIP(hipMemcpyAsync(net->guide_dev, net->guide.data(), 512, hipMemcpyHostToDevice, s));
    }
    ModelArgs m = model_args(net);
    SPK_HIP(init_state(m, net->P.v0_lo, net->P.v0_hi, net->V, net->ref, s));
    SPK_HIP(hipStreamSynchronize(s));  // host tables above are stack/vector memory
    return SPK_OK;
}

spk_status check_ready(spk_net *net)
{
    if (!net) return fail(SPK_EINVAL, "null network");
    return SPK_OK;
}

// What the device flags say.
spk_status check_flags(spk_net *net, uint32_t f, uint32_t *flags_out)
{
    if (flags_out) *flags_out = f;
    if (f & kFlagRunStopped)
        return fail(SPK_EHIP, "a persistent step launch stopped early (a barrier wait exceeded its "
                              "bound); the network state is undefined");
    if (f & kFlagBadSpike) {  // reported once, then cleared: the network is unchanged
        const uint32_t g = f & ~kFlagBadSpike;
        SPK_HIP(hipMemcpy(net->flags, &g, 4, hipMemcpyHostToDevice));
        return fail(SPK_EINVAL, "a spike ID given to spk_deliver_noalloc was >= n; those spikes "
                                "delivered nothing");
    }
    return SPK_OK;
}

spk_status sync_flags(spk_net *net, uint32_t *flags_out)
{
    uint32_t f = 0;
    if (net->stage) {
        SPK_HIP(read_records(nullptr, nullptr, 0, 0, net->flags, net->stage, net->stream));
        SPK_HIP(hipStreamSynchronize(net->stream));
        f = net->stage[0];
    } else {
        SPK_HIP(hipStreamSynchronize(net->stream));
        SPK_HIP(hipMemcpy(&f, net->flags, 4, hipMemcpyDeviceToHost));
    }
    return check_flags(net, f, flags_out);
}

RunArgs run_args(const spk_net *net, uint64_t t0, uint64_t n_steps)
{
    RunArgs ra{};
    ra.s = step_args(net);
    ra.ctl = net->ctl;
    ra.t0 = t0;
    ra.n_steps = n_steps;
    ra.R = net->run_R;
    ra.D = net->direct ? 1u : net->run_D;
    if (net->run_counts) {
        ra.counts = 1u;
        ra.w0 = std::ldexp((double)net->wval[0], -net->shift64);
        ra.w1 = std::ldexp((double)net->wval[1], -net->shift64);
        for (uint32_t k = 0; k < kMaxClasses; k++) ra.s.wval[k] = k == 0 ? 1 : k == 1 ? 65536 : 0;
    }
    return ra;
}

RingArgs ring_args(const spk_net *net, uint64_t t0, uint64_t n_steps)
{
    RingArgs ra{};
    ra.s = step_args(net);
    ra.s.tl = net->rtl;
    ra.s.toff = net->rtoff;
    ra.ctl = net->rctl;
    ra.ring = net->ring_buf;
    ra.seg = net->ring_seg;
    ra.cnts = net->ring_cnts;
    ra.t0 = t0;
    ra.n_steps = n_steps;
    ra.Tn = (net->n + net->rtl.W - 1) / net->rtl.W;
    ra.D = net->run_D;
    ra.seg_cap = net->seg_cap;
    ra.e0 = net->ring_epoch;
    ra.counts = net->ring_counts ? 1u : 0u;
    ra.w0 = std::ldexp((double)net->wval[0], -net->shift64);
    ra.w1 = std::ldexp((double)net->wval[1], -net->shift64);
    ra.pending = net->ring_pending;
    // the raster positions of a batch need every tile's count, so a recorded
    // run waits for its last batch too
    ra.defer = ra.Tn > 1 && !net->P.raster_capacity ? 1u : 0u;
    ra.waits = ra.Tn > 1 && (n_steps == 0 || n_steps > ra.D || !ra.defer) ? 1u : 0u;
    return ra;
}

hipError_t launch_persistent(spk_net *net, uint64_t t0, uint64_t n_steps, hipStream_t s)
{
    if (net->ring) {
        // A few batches are launched one by one: such a launch waits for
        // nothing inside and is an ordinary one.
        const uint64_t D = net->run_D;
        const bool single = n_steps > 0 && n_steps <= kRingPlainBatches * D && !net->P.raster_capacity;
        do {
            const uint64_t B = single ? std::min<uint64_t>(D, n_steps) : n_steps;
            const RingArgs ra = ring_args(net, t0, B);
            const hipError_t e = launch_ring(ra, s);
            if (e != hipSuccess) return e;
            net->ring_epoch += (uint32_t)((B + D - 1) / D);
            if (B) net->ring_pending = ra.defer ? (uint32_t)((B - 1) % D + 1) : 0u;
            t0 += B;
            n_steps -= B;
        } while (n_steps);
        return hipSuccess;
    }
    return launch_run(run_args(net, t0, n_steps), s);
}

// The control words of the next launch start at zero (the resident kernel's
// carry on from launch to launch).
hipError_t reset_control(const spk_net *net, hipStream_t s)
{
    return net->ring ? hipSuccess : hipMemsetAsync(net->ctl, 0, sizeof(RunCtl), s);
}

// A zero-step launch of the persistent kernel: checks that the workgroups
// were placed evenly over the XCDs (it only loads and stores back state).
spk_status probe_persistent(spk_net *net, bool *ok)
{
    hipStream_t s = net->stream;
    *ok = false;
    hipError_t e = reset_control(net, s);
    if (e == hipSuccess) e = launch_persistent(net, net->t, 0, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    uint32_t abort_flag = 1;
    const uint32_t *af = net->ring ? &net->rctl->abort_flag : &net->ctl->abort_flag;
    if (e == hipSuccess) e = hipMemcpy(&abort_flag, af, 4, hipMemcpyDeviceToHost);
    if (e == hipSuccess && abort_flag == 0) {
        *ok = true;
        return SPK_OK;
    }
    (void)hipGetLastError();
    (void)hipStreamSynchronize(s);
    SPK_HIP(hipMemsetAsync(net->flags, 0, 4, s));  // the probe's stop flag
    SPK_HIP(hipStreamSynchronize(s));
    return SPK_OK;
}

// Step mode.  The persistent kernel needs a cooperative launch of one
// workgroup per compute unit spread evenly over the XCDs; a launch of zero
// steps checks that once (it only loads and stores back the state).
spk_status choose_step_mode(spk_net *net)
{
    net->persistent = false;
    const uint32_t mode = net->P.step_mode;
    if (mode == SPK_STEP_GRAPH) return SPK_OK;
    int coop = 0;
    SPK_HIP(hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, net->device));
    const int cus = cu_count();
    net->run_R = cus > 0 && cus % (int)kGroups == 0 ? (uint32_t)(cus / (int)kGroups) : 0u;
    if (net->ring) {
        // one workgroup per tile, all resident at once
        const Tiling &tl = net->rtl;
        const uint32_t Tn = (net->n + tl.W - 1) / tl.W;
        const size_t bytes = (size_t)Tn * net->pslots * tl.W * ring_acc_bytes(net->P.acc_mode == SPK_ACC_FIXED, net->ring_counts);
        net->seg_cap = net->run_D * tl.W;
        bool ok = (Tn == 1 || (coop && (int)tl.T <= cus)) && ring_supported(ring_args(net, 0, 0));
        if (ok) {
            SPK_TRY(dalloc(net, (uint8_t **)&net->ring_buf, bytes));
            SPK_TRY(dalloc(net, &net->ring_seg, (size_t)2 * Tn * net->seg_cap));
            SPK_TRY(dalloc(net, &net->ring_cnts, (size_t)2 * kRunMaxD * Tn));
            SPK_TRY(dalloc(net, &net->rctl, 1));
            SPK_HIP(hipMemsetAsync(net->ring_buf, 0, bytes, net->stream));
            SPK_HIP(hipMemsetAsync(net->rctl, 0, sizeof(RingCtl), net->stream));
            SPK_TRY(probe_persistent(net, &ok));
        }
        if (ok) {
            net->persistent = true;
            return SPK_OK;
        }
        net->ring = false;  // (the rows serve direct delivery)
    }
    const StepArgs a = step_args(net);
    const bool run_fits = coop && run_supported(a, net->run_R) && run_batch_supported(a, net->direct ? 1u : net->run_D);
    if (!run_fits) {
        if (mode == SPK_STEP_PERSISTENT)
            return fail(SPK_EINVAL, "the persistent step kernel does not apply to this network or device "
                                    "(tiles per XCD, delays, or cooperative launch)");
        return SPK_OK;
    }
    SPK_TRY(dalloc(net, &net->ctl, 1));
    bool ok = false;
    SPK_TRY(probe_persistent(net, &ok));
    if (ok) {
        net->persistent = true;
        return SPK_OK;
    }
    dfree(net, net->ctl);
    net->ctl = nullptr;
    if (mode == SPK_STEP_PERSISTENT)
        return fail(SPK_EHIP, "the persistent step kernel could not be placed evenly over the XCDs");
    return SPK_OK;
}

spk_status collect_profile(spk_net *net)
{
    SPK_HIP(hipStreamSynchronize(net->stream));
    for (int which = 0; which < 3; which++) {
        auto &v = which == 2 ? net->ev_run : which ? net->ev_tile : net->ev_push;
        double &acc = which == 2 ? net->ms_run : which ? net->ms_tile : net->ms_push;
        for (auto &pr : v) {
            float ms = 0;
            SPK_HIP(hipEventElapsedTime(&ms, pr.first, pr.second));
            acc += ms;
            net->ev_free.push_back(pr.first);
            net->ev_free.push_back(pr.second);
        }
        v.clear();
    }
    return SPK_OK;
}

spk_status get_event(spk_net *net, hipEvent_t *e)
{
    if (!net->ev_free.empty()) {
        *e = net->ev_free.back();
        net->ev_free.pop_back();
        return SPK_OK;
    }
    SPK_HIP(hipEventCreate(e));
    return SPK_OK;
}

// One step's kernels on stream s (step i of a batch, or explicit t).
spk_status enqueue_step(spk_net *net, const StepArgs &a, hipStream_t s, uint32_t i, int64_t t_explicit)
{
    SPK_HIP(launch_tile(a, i, t_explicit, s));
    if (!net->direct) SPK_HIP(launch_push(a, i, t_explicit, s));
    if (net->P.raster_capacity) SPK_HIP(launch_record(a, i, t_explicit, s));
    return SPK_OK;
}

// A graph of B steps followed by the step-counter advance, built once.
spk_status batch_graph(spk_net *net, uint32_t B, hipGraphExec_t *out)
{
    auto it = net->graphs.find(B);
    if (it != net->graphs.end()) {
        *out = it->second;
        return SPK_OK;
    }
    const StepArgs a = step_args(net);
    hipStream_t cs = net->cap_stream;
    SPK_HIP(hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal));
    spk_status st = SPK_OK;
    for (uint32_t i = 0; i < B && st == SPK_OK; i++) st = enqueue_step(net, a, cs, i, -1);
    if (st == SPK_OK && launch_advance(net->t_base, B, cs) != hipSuccess)
        st = fail(SPK_EHIP, "advance launch");
    hipGraph_t g = nullptr;
    hipError_t e = hipStreamEndCapture(cs, &g);
    if (st != SPK_OK) {
        if (g) (void)hipGraphDestroy(g);
        return st;
    }
    SPK_HIP(e);
    hipGraphExec_t ge = nullptr;
    e = hipGraphInstantiate(&ge, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    SPK_HIP(e);
    net->graphs[B] = ge;
    *out = ge;
    return SPK_OK;
}

void destroy_net(spk_net *net)
{
    if (!net) return;
    if (net->stream) (void)hipStreamSynchronize(net->stream);
    for (auto &kv : net->graphs) (void)hipGraphExecDestroy(kv.second);
    for (auto *v : {&net->ev_push, &net->ev_tile, &net->ev_run})
        for (auto &pr : *v) {
            (void)hipEventDestroy(pr.first);
            (void)hipEventDestroy(pr.second);
        }
    for (auto e : net->ev_free) (void)hipEventDestroy(e);
    for (void *p : net->allocs) (void)hipFree(p);
    if (net->cap_stream) (void)hipStreamDestroy(net->cap_stream);
    if (net->own_stream && net->stream) (void)hipStreamDestroy(net->stream);
    stage_give(net->stage);
    delete net;
}

// Whether the resident kernel's network counts as binned: its events are
// filed by arrival step right after their spike, as binned delivery does; with
// one delay of one step, or where direct delivery was asked for, a tile reads
// the due rows.
bool ring_binned(const spk_net *net)
{
    return net->ring && net->P.delivery != SPK_DELIVERY_DIRECT && net->dmax > 1;
}

// Whether a given spike list is delivered faster through pages than by each
// tile reading its runs, on a resident network's rows.  Microseconds of
// spk_deliver_noalloc, E = 1e6 events, T tiles, about: by tile 8.5 + 900 E / T
// (fan-out 1,500, 20,000 neurons on 157 tiles: 9.5 at 300 spikes, 21.9 at
// 1,500, 45 at 4,000; 60,000 on 235: 9.5, 15.1, 28.8), through pages 14 + 4.3 E,
// or 1.6 E where only one of several delays is filed (20,000: 39.3 at 4,000;
// one delay of 20 16.4 at 1,500, 23.1 at 4,000; 60,000 23.3 at 4,000).  Not on
// networks that count as direct: those use no scratch, and their callers need
// not order such calls.
bool binned_pays(const spk_net *net, uint64_t n_spikes, uint32_t delay)
{
    if (!ring_binned(net) || !net->compact) return false;
    const Tiling &tl = net->tl;
    const double E = 1e-6 * (double)n_spikes * (double)net->nnz / (double)net->n;
    const double T = (double)((net->n + tl.W - 1) / tl.W);
    // (its accumulators and pages of the least size have to fit the scratch)
    const uint64_t need = (uint64_t)tl.T * tl.W * 8 + (uint64_t)kGroups * push_blocks_per_group() * tl.T8 * (4 + 16 * 2);
    return E * (900.0 / T - (delay && net->lists > 1 ? 1.6 : 4.3)) > 5.5 && need + 65536 <= kNoAllocScratchBytes;
}

// Records of n steps, summed over the groups, after the enqueued work.
spk_status read_groups(spk_net *net, const void *dev, size_t elem, uint64_t t0, uint64_t n, void *out)
{
    if (net->stage && n * elem <= kStageBytes - kStageWords * 4) {
        SPK_HIP(read_records(elem == 4 ? (const uint32_t *)dev : nullptr, elem == 8 ? (const uint64_t *)dev : nullptr, t0,
                             (uint32_t)n, net->flags, net->stage, net->stream));
        SPK_HIP(hipStreamSynchronize(net->stream));
        SPK_TRY(check_flags(net, net->stage[0], nullptr));
        if (n) std::memcpy(out, net->stage + kStageWords, n * elem);
        return SPK_OK;
    }
    SPK_TRY(sync_flags(net, nullptr));
    std::vector<uint8_t> buf(n * kGroups * elem);
    if (n) SPK_HIP(hipMemcpy(buf.data(), (const uint8_t *)dev + t0 * kGroups * elem, buf.size(),
                             hipMemcpyDeviceToHost));
    for (uint64_t k = 0; k < n; k++) {
        uint64_t sum = 0;
        for (uint32_t x = 0; x < kGroups; x++) {
            if (elem == 4) {
                uint32_t v;
                std::memcpy(&v, &buf[(k * kGroups + x) * 4], 4);
                sum += v;
            } else {
                uint64_t v;
                std::memcpy(&v, &buf[(k * kGroups + x) * 8], 8);
                sum += v;
            }
        }
        if (elem == 4) ((uint32_t *)out)[k] = (uint32_t)sum;
        else ((uint64_t *)out)[k] = sum;
    }
    return SPK_OK;
}

}  // namespace

// ===================================================================== ABI

extern "C" {

uint32_t spk_abi_version(void) { return SPK_ABI_VERSION; }

const char *spk_last_error(void) { return g_err.c_str(); }

spk_status spk_preset(int index, int driven, double rate_hz, uint64_t seed, spk_params *out)
{
    if (!out) return fail(SPK_EINVAL, "null output");
    spk_params p{};
    p.abi_version = SPK_ABI_VERSION;
    p.seed = seed;
    p.neuron_kind = SPK_LIF;
    p.frac_exc = 0.8;
    p.dt_ms = 0.1;
    p.tau_m_ms = 20.0;
    p.t_ref_ms = 5.0;
    p.v_rest = -60.0f;
    p.v_th = -50.0f;
    p.v_reset = -60.0f;
    p.v0_lo = -60.0f;
    p.v0_hi = -50.0f;
    p.delay_min = p.delay_max = 1;
    p.acc_mode = SPK_ACC_F32;
    p.fixed_shift = 20;
    switch (index) {
    case 0:
        p.n = 1000; p.conn_kind = SPK_CONN_BERNOULLI; p.p = 0.02;
        p.w_exc = 0.27f; p.w_inh = -4.5f; p.max_steps = 1000;
        break;
    case 1: {
        p.n = 250000; p.conn_kind = SPK_CONN_BERNOULLI; p.p = 0.02;
        const double sc = 80.0 / (0.02 * p.n);
        p.w_exc = (float)(0.27 * sc); p.w_inh = (float)(-4.5 * sc); p.max_steps = 10000;
        break;
    }
    case 2:
        p.n = 100000; p.conn_kind = SPK_CONN_FIXED_IN; p.k_in_exc = 8000; p.k_in_inh = 2000;
        p.w_exc = 0.1f; p.w_inh = -0.5f; p.delay_min = p.delay_max = 15;
        p.ext_lambda = 1.0; p.ext_w = 0.1f; p.max_steps = 10000;
        break;
    case 3:
        p.n = 1000000; p.neuron_kind = SPK_SOURCE; p.frac_exc = 1.0; p.dt_ms = 1.0;
        p.conn_kind = SPK_CONN_FIXED_OUT; p.k_out = 1000; p.w_uniform = 1; p.w_lo = 0.0f;
        p.w_hi = 1e-3f; p.src_rate_hz = rate_hz; p.max_steps = 1000;
        break;
    case 4: {
        p.n = 2000000; p.conn_kind = SPK_CONN_FIXED_OUT; p.k_out = 1500;
        const double sc = 80.0 / 1500.0;
        p.w_exc = (float)(0.27 * sc); p.w_inh = (float)(-4.5 * sc);
        p.delay_min = 1; p.delay_max = 20; p.max_steps = 5000;
        break;
    }
    default:
        return fail(SPK_EINVAL, "preset index must be 0..4");
    }
    if (driven && p.neuron_kind == SPK_LIF && p.ext_lambda == 0.0) {
        const double theta = (double)p.v_th - (double)p.v_rest;
        p.ext_lambda = 2.0 * theta * (p.dt_ms / p.tau_m_ms) / (double)p.w_exc;
        p.ext_w = p.w_exc;
    }
    *out = p;
    return SPK_OK;
}

spk_status spk_create(const spk_params *params, void *stream, spk_net **out)
{
    if (!params || !out) return fail(SPK_EINVAL, "null argument");
    *out = nullptr;
    const auto t_begin = std::chrono::steady_clock::now();
    spk_net *net = new (std::nothrow) spk_net();
    if (!net) return fail(SPK_ENOMEM, "host allocation");
    net->P = *params;
    spk_status st = derive(net, false);
    if (st == SPK_OK) st = setup_stream(net, stream);
    if (st == SPK_OK) st = generate(net);
    if (st == SPK_OK) st = alloc_state(net);
    if (st == SPK_OK) st = choose_step_mode(net);
    if (st == SPK_OK) st = sync_flags(net, nullptr);
    if (st != SPK_OK) {
        std::string msg = g_err;
        destroy_net(net);
        g_err = msg;
        return st;
    }
    net->setup_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t_begin).count();
    *out = net;
    return SPK_OK;
}

spk_status spk_create_from_csr(const spk_params *params, uint32_t n, const uint64_t *row_ptr,
                               const uint32_t *col, const float *w, const uint8_t *delay,
                               void *stream, spk_net **out)
{
    if (!params || !out || !row_ptr || (row_ptr[n] && (!col || !w)))
        return fail(SPK_EINVAL, "null argument");
    *out = nullptr;
    const auto t_begin = std::chrono::steady_clock::now();
    spk_net *net = new (std::nothrow) spk_net();
    if (!net) return fail(SPK_ENOMEM, "host allocation");
    net->P = *params;
    net->P.n = n;
    net->P.conn_kind = SPK_CONN_EXPLICIT;
    auto run = [&]() -> spk_status {
        SPK_TRY(derive(net, true));
        if (row_ptr[0] != 0) return fail(SPK_EINVAL, "row_ptr[0] must be 0");
        uint64_t max_row = 0;
        for (uint32_t s = 0; s < n; s++) {
            if (row_ptr[s + 1] < row_ptr[s]) return fail(SPK_EINVAL, "row_ptr not monotone");
            max_row = std::max<uint64_t>(max_row, row_ptr[s + 1] - row_ptr[s]);
        }
        const uint64_t nnz = row_ptr[n];
        std::vector<uint32_t> distinct;  // weight bit patterns, first-seen order, up to 5
        for (uint64_t e = 0; e < nnz && distinct.size() <= kMaxClasses; e++) {
            uint32_t b;
            std::memcpy(&b, &w[e], 4);
            if (std::find(distinct.begin(), distinct.end(), b) == distinct.end()) distinct.push_back(b);
        }
        {
            float cls[kMaxClasses] = {};
            const bool fits = distinct.size() <= kMaxClasses;
            for (size_t k = 0; fits && k < distinct.size(); k++) std::memcpy(&cls[k], &distinct[k], 4);
            if (fits && distinct.empty()) cls[0] = 0.0f;
            SPK_TRY(choose_format(net, fits ? cls : nullptr,
                                  fits ? std::max<uint32_t>(1, (uint32_t)distinct.size()) : 0));
        }
        for (uint64_t e = 0; e < nnz; e++) {
            if (col[e] >= n) return fail(SPK_EINVAL, "target id out of range");
            const uint32_t d = delay ? delay[e] : net->P.delay_min;
            if (d < net->P.delay_min || d > net->P.delay_max)
                return fail(SPK_EINVAL, "delay out of [delay_min, delay_max]");
            if (net->P.acc_mode == SPK_ACC_FIXED) {
                int32_t q;
                if (!quantise(w[e], net->P.fixed_shift, &q))
                    return fail(SPK_EOVERFLOW, "a weight does not fit int32 at this fixed_shift");
            }
        }
        net->nnz = nnz;
        net->max_row = (uint32_t)std::min<uint64_t>(max_row, 0xffffffffull);
        SPK_TRY(setup_stream(net, stream));
        hipStream_t s = net->stream;
        uint32_t *in_col = nullptr;
        float *in_w = nullptr;
        uint8_t *in_d = nullptr;
        void *tmp = nullptr, *syn = nullptr;
        SPK_TRY(dalloc(net, &net->row_ptr, (size_t)n + 1));
        SPK_TRY(alloc_syn(net, &tmp, nnz));
        SPK_TRY(dalloc(net, &in_col, nnz));
        SPK_TRY(dalloc(net, &in_w, nnz));
        SPK_HIP(hipMemcpyAsync(net->row_ptr, row_ptr, ((size_t)n + 1) * 8, hipMemcpyHostToDevice, s));
        if (nnz) {
            SPK_HIP(hipMemcpyAsync(in_col, col, nnz * 4, hipMemcpyHostToDevice, s));
            SPK_HIP(hipMemcpyAsync(in_w, w, nnz * 4, hipMemcpyHostToDevice, s));
        }
        if (delay) {
            SPK_TRY(dalloc(net, &in_d, nnz));
            if (nnz) SPK_HIP(hipMemcpyAsync(in_d, delay, nnz, hipMemcpyHostToDevice, s));
        }
        SPK_HIP(csr_fill(conn_args(net), nnz, in_col, in_w, in_d, tmp, s));
        uint64_t in_max[2] = {nnz, nnz};
        if (net->compact && net->n_cls <= 2 && nnz > 65535) SPK_TRY(in_degrees(net, tmp, nnz, in_max));
        plan_ring(net, nnz, in_max);  // (chooses the tiling)
        RowIndex ix{};
        SPK_TRY(choose_delivery(net, &ix));
        SPK_TRY(alloc_syn(net, &syn, nnz));
        if (net->compact) net->syn32 = (uint32_t *)syn;
        else net->syn = (int2 *)syn;
        SPK_HIP(bucket_rows(conn_args(net), net->row_ptr, tmp, syn, ix, s));
        SPK_HIP(hipStreamSynchronize(s));
        dfree(net, tmp);
        dfree(net, in_col);
        dfree(net, in_w);
        dfree(net, in_d);
        SPK_TRY(finish_rows(net));
        SPK_TRY(alloc_state(net));
        SPK_TRY(choose_step_mode(net));
        return sync_flags(net, nullptr);
    };
    spk_status st = run();
    if (st != SPK_OK) {
        std::string msg = g_err;
        destroy_net(net);
        g_err = msg;
        return st;
    }
    net->setup_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t_begin).count();
    *out = net;
    return SPK_OK;
}

spk_status spk_step(spk_net *net, uint64_t n_steps)
{
    SPK_TRY(check_ready(net));
    if (net->t + n_steps > net->P.max_steps)
        return fail(SPK_EOVERFLOW, "max_steps exceeded");
    hipStream_t s = net->stream;
    if (net->persistent) {  // one cooperative launch per (at most 2^24) steps
        uint64_t left = n_steps;
        while (left) {
            const uint64_t B = std::min<uint64_t>(left, kRunMaxSteps);
            hipEvent_t e0 = nullptr, e1 = nullptr;
            if (net->profiling) {
                SPK_TRY(get_event(net, &e0));
                SPK_TRY(get_event(net, &e1));
            }
            SPK_HIP(reset_control(net, s));
            if (e0) SPK_HIP(hipEventRecord(e0, s));
            SPK_HIP(launch_persistent(net, net->t, B, s));
            if (e1) {
                SPK_HIP(hipEventRecord(e1, s));
                net->ev_run.push_back({e0, e1});
                net->run_launches++;
                net->launches += B;
            }
            left -= B;
            net->t += B;
        }
        return SPK_OK;
    }
    if (net->profiling) {  // plain launches with events around every kernel
        const StepArgs a = step_args(net);
        for (uint64_t k = 0; k < n_steps; k++) {
            const int64_t t = (int64_t)(net->t + k);
            hipEvent_t e0 = nullptr, e1 = nullptr, e2 = nullptr, e3 = nullptr;
            SPK_TRY(get_event(net, &e0));
            SPK_TRY(get_event(net, &e1));
            SPK_HIP(hipEventRecord(e0, s));
            SPK_HIP(launch_tile(a, 0, t, s));
            SPK_HIP(hipEventRecord(e1, s));
            net->ev_tile.push_back({e0, e1});
            if (!net->direct) {
                SPK_TRY(get_event(net, &e2));
                SPK_TRY(get_event(net, &e3));
                SPK_HIP(hipEventRecord(e2, s));
                SPK_HIP(launch_push(a, 0, t, s));
                SPK_HIP(hipEventRecord(e3, s));
                net->ev_push.push_back({e2, e3});
            }
            if (net->P.raster_capacity) SPK_HIP(launch_record(a, 0, t, s));
            net->launches++;
        }
        if (n_steps) SPK_HIP(launch_advance(net->t_base, (uint32_t)n_steps, s));
        net->t += n_steps;
        return SPK_OK;
    }
    uint64_t left = n_steps;
    while (left) {
        const uint32_t B = (uint32_t)std::min<uint64_t>(left, kBatch);
        hipGraphExec_t ge = nullptr;
        SPK_TRY(batch_graph(net, B, &ge));
        SPK_HIP(hipGraphLaunch(ge, s));
        left -= B;
        net->t += B;
    }
    return SPK_OK;
}

spk_status spk_sync(spk_net *net)
{
    SPK_TRY(check_ready(net));
    return sync_flags(net, nullptr);
}

spk_status spk_read_spike_counts(spk_net *net, uint64_t t0, uint64_t n, uint32_t *out)
{
    SPK_TRY(check_ready(net));
    if (t0 + n > net->P.max_steps || (n && !out)) return fail(SPK_EINVAL, "range");
    return read_groups(net, net->counts8, 4, t0, n, out);
}

spk_status spk_read_events(spk_net *net, uint64_t t0, uint64_t n, uint64_t *out)
{
    SPK_TRY(check_ready(net));
    if (t0 + n > net->P.max_steps || (n && !out)) return fail(SPK_EINVAL, "range");
    return read_groups(net, net->events8, 8, t0, n, out);
}

spk_status spk_read_delivered(spk_net *net, uint64_t t0, uint64_t n, uint64_t *out)
{
    SPK_TRY(check_ready(net));
    if (t0 + n > net->P.max_steps || (n && !out)) return fail(SPK_EINVAL, "range");
    if (net->ring && net->lists == 1) {
        // one delay: the events delivered at t are those emitted at t - dmin
        for (uint64_t k = 0; k < n && t0 + k < net->dmin; k++) out[k] = 0;
        const uint64_t skip = t0 < net->dmin ? std::min<uint64_t>(n, net->dmin - t0) : 0;
        const uint64_t last = std::max<uint64_t>(net->t, t0 + skip);  // steps not run yet deliver nothing
        const uint64_t m = std::min<uint64_t>(n - skip, last - (t0 + skip));
        SPK_TRY(read_groups(net, net->events8, 8, m ? t0 + skip - net->dmin : 0, m, out + skip));
        for (uint64_t k = skip + m; k < n; k++) out[k] = 0;
        return SPK_OK;
    }
    return read_groups(net, net->delivered8, 8, t0, n, out);
}

spk_status spk_read_raster(spk_net *net, uint64_t t0, uint64_t n, uint64_t *offs, uint32_t *ids,
                           uint64_t cap)
{
    SPK_TRY(check_ready(net));
    if (!net->P.raster_capacity) return fail(SPK_ESTATE, "raster recording is off");
    if (t0 + n > net->t || !offs) return fail(SPK_EINVAL, "range");
    uint32_t f = 0;
    SPK_TRY(sync_flags(net, &f));
    if (f & 2u) return fail(SPK_EOVERFLOW, "raster capacity exceeded during the run");
    std::vector<uint64_t> o(n + 1);
    SPK_HIP(hipMemcpy(o.data(), net->raster_offs + t0, (n + 1) * 8, hipMemcpyDeviceToHost));
    const uint64_t total = o[n] - o[0];
    if (total > cap || (total && !ids)) return fail(SPK_EOVERFLOW, "ids buffer too small");
    if (total) SPK_HIP(hipMemcpy(ids, net->raster + o[0], total * 4, hipMemcpyDeviceToHost));
    for (uint64_t k = 0; k <= n; k++) offs[k] = o[k] - o[0];
    for (uint64_t k = 0; k < n; k++) std::sort(ids + offs[k], ids + offs[k + 1]);
    return SPK_OK;
}

spk_status spk_read_state(spk_net *net, float *v, uint8_t *ref)
{
    SPK_TRY(check_ready(net));
    if (net->stage && (uint64_t)net->n * 5 + 8 <= kStageBytes - kStageWords * 4) {
        SPK_HIP(read_state(net->V, net->ref, net->n, net->flags, net->stage, net->stream));
        SPK_HIP(hipStreamSynchronize(net->stream));
        SPK_TRY(check_flags(net, net->stage[0], nullptr));
        if (v) std::memcpy(v, net->stage + kStageWords, (size_t)net->n * 4);
        if (ref) std::memcpy(ref, net->stage + kStageWords + net->n, net->n);
        return SPK_OK;
    }
    SPK_TRY(sync_flags(net, nullptr));
    if (v) SPK_HIP(hipMemcpy(v, net->V, (size_t)net->n * 4, hipMemcpyDeviceToHost));
    if (ref) SPK_HIP(hipMemcpy(ref, net->ref, net->n, hipMemcpyDeviceToHost));
    return SPK_OK;
}

spk_status spk_debug_deliver(spk_net *net, const uint32_t *spikes, uint64_t n_spikes, uint32_t delay,
                             float *out_f32, int32_t *out_i32)
{
    SPK_TRY(check_ready(net));
    const bool fixed = net->P.acc_mode == SPK_ACC_FIXED;
    if ((fixed && !out_i32) || (!fixed && !out_f32))
        return fail(SPK_EINVAL, "output buffer for this accumulation mode is required");
    if (n_spikes > 0x3fffffffull || (n_spikes && !spikes)) return fail(SPK_EINVAL, "spikes");
    for (uint64_t k = 0; k < n_spikes; k++)
        if (spikes[k] >= net->n) return fail(SPK_EINVAL, "spike id out of range");
    if (delay && (delay < net->dmin || delay >= net->dmin + net->lists))
        return fail(SPK_EINVAL, "delay not in [delay_min, delay_max]");
    hipStream_t s = net->stream;
    SPK_TRY(sync_flags(net, nullptr));
    const Tiling &tl = net->tl;
    // scratch: the spike list, and for binned delivery pages of one arrival
    // slot with their fill counters and overflow accumulators, so that the
    // network's own pages (events in flight) are left untouched
    std::vector<void *> tmp;
    auto scratch = [&](void **p, size_t bytes) -> spk_status {
        uint8_t *q = nullptr;
        SPK_TRY(dalloc(net, &q, bytes));
        tmp.push_back(q);
        *p = q;
        return SPK_OK;
    };
    spk_status st = SPK_OK;
    do {
        uint32_t *d_sp = nullptr;
        if ((st = scratch((void **)&d_sp, n_spikes * 4 + 4)) != SPK_OK) break;
        StepArgs a = step_args(net);
        a.dbg_spikes = d_sp;
        a.dbg_n = (uint32_t)n_spikes;
        a.dbg_j = delay ? (int32_t)(delay - net->dmin) : -1;
        a.dbg_out = net->dbg_out;
        hipError_t e = hipSuccess;
        if (n_spikes) e = hipMemcpyAsync(d_sp, spikes, n_spikes * 4, hipMemcpyHostToDevice, s);
        if (e == hipSuccess && !net->direct) {
            const uint64_t n_pages = (uint64_t)kGroups * net->pg1 * tl.T8;
            const uint64_t cap = std::min<uint64_t>(kDebugPageCap, std::max<uint64_t>(16, net->page_cap));
            const size_t acc_elems = (size_t)tl.T * tl.W;
            void *pg = nullptr;
            if ((st = scratch(&pg, n_pages * cap * (net->compact ? 2 : 8))) != SPK_OK) break;
            a.pages = net->compact ? nullptr : (int2 *)pg;
            a.pages16 = net->compact ? (uint16_t *)pg : nullptr;
            if ((st = scratch((void **)&a.pfill, n_pages * 4)) != SPK_OK) break;
            if ((st = scratch((void **)&a.ovf_flag, (size_t)tl.T * 4)) != SPK_OK) break;
            if ((st = scratch(&a.acc_ovf, acc_elems * 8)) != SPK_OK) break;
            a.page_cap = (uint32_t)cap;
            a.pslots = 1;
            e = hipMemsetAsync(a.pfill, 0, n_pages * 4, s);
            if (e == hipSuccess) e = hipMemsetAsync(a.ovf_flag, 0, (size_t)tl.T * 4, s);
            if (e == hipSuccess) e = hipMemsetAsync(a.acc_ovf, 0, acc_elems * 8, s);
            if (e == hipSuccess) e = launch_push(a, 0, 0, s);
        }
        if (e == hipSuccess) e = launch_tile(a, 0, 0, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e == hipSuccess)
            e = hipMemcpy(fixed ? (void *)out_i32 : (void *)out_f32, net->dbg_out,
                          (size_t)net->n * 4, hipMemcpyDeviceToHost);
        if (e != hipSuccess) st = fail(SPK_EHIP, hipGetErrorString(e));
    } while (0);
    (void)hipStreamSynchronize(s);
    for (void *p : tmp) dfree(net, p);
    return st;
}

spk_status spk_deliver_noalloc(spk_net *net, const uint32_t *d_spikes, uint64_t n_spikes, uint32_t delay,
                               void *d_out)
{
    SPK_TRY(check_ready(net));
    if (!d_out) return fail(SPK_EINVAL, "output buffer required");
    if (n_spikes > 0x3fffffffull || (n_spikes && !d_spikes)) return fail(SPK_EINVAL, "spikes");
    if (delay && (delay < net->dmin || delay >= net->dmin + net->lists))
        return fail(SPK_EINVAL, "delay not in [delay_min, delay_max]");
    hipStream_t s = net->stream;
    const Tiling &tl = net->tl;
    StepArgs a = step_args(net);
    a.dbg_spikes = n_spikes ? d_spikes : nullptr;
    a.dbg_n = (uint32_t)n_spikes;
    a.dbg_j = delay ? (int32_t)(delay - net->dmin) : -1;
    a.dbg_out = d_out;  // (no spikes: the tile kernel writes zeros)
    hipError_t e = hipSuccess;
    bool capturing = false;
    uint32_t *zero_area = nullptr;  // binned delivery: the scratch's
    bool binned = !net->direct;
    if (binned_pays(net, n_spikes, delay)) {
        binned = true;
        a.direct = 0;
        a.pg1 = push_blocks_per_group();
    }
    if (binned) {
        // Carve the zero area: fill counters, overflow flags and overflow
        // accumulators of one arrival slot; pages of as many records as the
        // bytes they leave of one area's size hold (at most the debug
        // capacity; events beyond it take the overflow accumulators, with the
        // same sums)
        auto up = [](uint64_t b) { return (b + 255) / 256 * 256; };
        const uint64_t n_pages = (uint64_t)kGroups * a.pg1 * tl.T8;
        const uint64_t acc_bytes = (uint64_t)tl.T * tl.W * (net->P.acc_mode == SPK_ACC_FIXED ? 4 : 8);
        const uint64_t o_fill = 0, o_flag = up(n_pages * 4), o_acc = o_flag + up((uint64_t)tl.T * 4);
        const uint64_t used = o_acc + up(acc_bytes);
        const uint64_t rec = net->compact ? 2 : 8;
        const uint64_t room = used < kNoAllocScratchBytes ? kNoAllocScratchBytes - used : 0;
        uint64_t cap = std::min<uint64_t>(room / (n_pages * rec), kDebugPageCap);
        if (!net->direct) cap = std::min<uint64_t>(cap, net->page_cap);
        cap = cap / 16 * 16;
        if (cap < 16)
            return fail(SPK_EOVERFLOW, "network too large for the fixed scratch of spk_deliver_noalloc (" +
                                           std::to_string(kNoAllocScratchBytes >> 20) + " MiB per device)");
        hipStreamCaptureStatus cap_st = hipStreamCaptureStatusNone;
        SPK_HIP(hipStreamIsCapturing(s, &cap_st));
        capturing = cap_st != hipStreamCaptureStatusNone;
        bool clear = false;
        const Scratch x = scratch_take(net->device, capturing, &clear);
        if (!x.pages) return fail(SPK_ESTATE, "no scratch address for the network's device");
        zero_area = (uint32_t *)x.zero;
        a.pfill = (uint32_t *)(x.zero + o_fill);
        a.ovf_flag = (uint32_t *)(x.zero + o_flag);
        a.acc_ovf = x.zero + o_acc;
        a.pages = net->compact ? nullptr : (int2 *)x.pages;
        a.pages16 = net->compact ? (uint16_t *)x.pages : nullptr;
        a.page_cap = (uint32_t)cap;
        a.pslots = 1;
        // (a fill kernel, not a memset: usable under capture)
        if (clear) e = zero_words(zero_area, kNoAllocScratchBytes / 4, s);
        if (e == hipSuccess && n_spikes) e = launch_push(a, 0, 0, s);
    }
    if (e == hipSuccess) e = launch_tile(a, 0, 0, s);
    // after a failed launch the area is cleared at once, so that graphs
    // captured before find it at zero too; where even that cannot be
    // launched, the next call clears
    if (zero_area)
        scratch_done(net->device, capturing,
                     e == hipSuccess || zero_words(zero_area, kNoAllocScratchBytes / 4, s) == hipSuccess);
    if (e != hipSuccess) return fail(SPK_EHIP, hipGetErrorString(e));
    return SPK_OK;
}

spk_status spk_export_rows(spk_net *net, const uint32_t *rows, uint64_t n_rows, uint64_t *offs,
                           uint32_t *col, float *w, int32_t *wq, uint8_t *delay, uint64_t cap)
{
    SPK_TRY(check_ready(net));
    if (!offs || (n_rows && !rows)) return fail(SPK_EINVAL, "null argument");
    for (uint64_t r = 0; r < n_rows; r++)
        if (rows[r] >= net->n) return fail(SPK_EINVAL, "row id out of range");
    SPK_TRY(sync_flags(net, nullptr));
    offs[0] = 0;
    if (!n_rows) return SPK_OK;
    hipStream_t s = net->stream;
    std::vector<uint32_t> deg(net->n);
    SPK_HIP(hipMemcpy(deg.data(), net->outdeg, (size_t)net->n * 4, hipMemcpyDeviceToHost));
    uint64_t tot = 0;
    for (uint64_t r = 0; r < n_rows; r++) {
        tot += deg[rows[r]];
        offs[r + 1] = tot;
    }
    if (tot > cap) return fail(SPK_EOVERFLOW, "export buffers too small");
    uint32_t *d_rows = nullptr, *d_col = nullptr, *d_wb = nullptr;
    uint64_t *d_off = nullptr;
    uint8_t *d_del = nullptr;
    SPK_TRY(dalloc(net, &d_rows, n_rows));
    SPK_TRY(dalloc(net, &d_off, n_rows));
    SPK_TRY(dalloc(net, &d_col, tot));
    SPK_TRY(dalloc(net, &d_wb, tot));
    SPK_TRY(dalloc(net, &d_del, tot));
    SPK_HIP(hipMemcpyAsync(d_rows, rows, n_rows * 4, hipMemcpyHostToDevice, s));
    SPK_HIP(hipMemcpyAsync(d_off, offs, n_rows * 8, hipMemcpyHostToDevice, s));
    if (net->proc)
        SPK_HIP(export_proc(step_args(net), net->ctab, d_rows, n_rows, d_off, d_col, d_wb, d_del, s));
    else
        SPK_HIP(export_gather(net->row_ptr, net->outdeg, syn_ptr(net), net->compact, net->ctab, net->dmin, d_rows, n_rows,
                              d_off, d_col, d_wb, d_del, s));
    std::vector<uint32_t> hc(tot), hw(tot);
    std::vector<uint8_t> hd(tot);
    if (tot) {
        SPK_HIP(hipMemcpyAsync(hc.data(), d_col, tot * 4, hipMemcpyDeviceToHost, s));
        SPK_HIP(hipMemcpyAsync(hw.data(), d_wb, tot * 4, hipMemcpyDeviceToHost, s));
        SPK_HIP(hipMemcpyAsync(hd.data(), d_del, tot, hipMemcpyDeviceToHost, s));
    }
    SPK_HIP(hipStreamSynchronize(s));
    dfree(net, d_rows); dfree(net, d_off);
    dfree(net, d_col); dfree(net, d_wb); dfree(net, d_del);
    // canonical order per row: (target, delay, stored weight bits)
    std::vector<uint64_t> idx;
    for (uint64_t r = 0; r < n_rows; r++) {
        const uint64_t a = offs[r], b = offs[r + 1];
        idx.resize(b - a);
        for (uint64_t e = a; e < b; e++) idx[e - a] = e;
        std::sort(idx.begin(), idx.end(), [&](uint64_t x, uint64_t y) {
            if (hc[x] != hc[y]) return hc[x] < hc[y];
            if (hd[x] != hd[y]) return hd[x] < hd[y];
            return hw[x] < hw[y];
        });
        for (uint64_t e = a; e < b; e++) {
            const uint64_t src = idx[e - a];
            if (col) col[e] = hc[src];
            if (delay) delay[e] = hd[src];
            if (w) std::memcpy(&w[e], &hw[src], 4);
            if (wq) wq[e] = (int32_t)hw[src];
        }
    }
    return SPK_OK;
}

spk_status spk_poisson_table(spk_net *net, uint64_t *thr, uint32_t cap, uint32_t *len)
{
    SPK_TRY(check_ready(net));
    if (!len) return fail(SPK_EINVAL, "null len");
    *len = net->pois_len;
    if (net->pois_len > cap || (net->pois_len && !thr)) return fail(SPK_EOVERFLOW, "cap");
    for (uint32_t k = 0; k < net->pois_len; k++) thr[k] = net->pois[k];
    return SPK_OK;
}

spk_status spk_stats(spk_net *net, spk_stats_t *out)
{
    SPK_TRY(check_ready(net));
    if (!out) return fail(SPK_EINVAL, "null output");
    spk_stats_t st{};
    st.n = net->n;
    st.nnz = net->nnz;
    st.steps = net->t;
    st.device_bytes = net->device_bytes;
    st.n_exc = net->n_exc;
    st.ref_steps = net->ref_steps;
    st.ring_slots = net->spk_slots;
    st.delay_lists = net->lists;
    st.max_row = net->max_row;
    st.pois_len = net->pois_len;
    st.fixed_shift = net->P.acc_mode == SPK_ACC_FIXED ? net->P.fixed_shift : net->shift64;
    st.k = net->k;
    st.bytes_per_synapse = net->proc ? 0.0 : net->compact ? 4.0 : 8.0;
    st.tile_width = net->ring ? net->rtl.W : net->tl.W;
    st.tiles = net->ring ? net->rtl.T : net->tl.T;
    st.delivery = net->direct && !ring_binned(net) ? SPK_DELIVERY_DIRECT : SPK_DELIVERY_BINNED;
    st.page_cap = net->page_cap;
    st.step_mode = net->persistent ? SPK_STEP_PERSISTENT : SPK_STEP_GRAPH;
    st.batch_steps = net->persistent && (!net->direct || net->ring) ? net->run_D : 1u;
    st.setup_ms = net->setup_ms;
    st.gen_ms = net->gen_ms;
    st.range_ms = net->range_ms;
    *out = st;
    return SPK_OK;
}

spk_status spk_set_profiling(spk_net *net, int on)
{
    SPK_TRY(check_ready(net));
    SPK_TRY(collect_profile(net));
    net->profiling = on != 0;
    net->ms_push = net->ms_tile = net->ms_run = 0;
    net->launches = net->run_launches = 0;
    return SPK_OK;
}

spk_status spk_read_kernel_ms(spk_net *net, double *push_ms, double *tile_ms, double *run_ms,
                              uint64_t *steps, uint64_t *run_launches)
{
    SPK_TRY(check_ready(net));
    SPK_TRY(collect_profile(net));
    if (push_ms) *push_ms = net->ms_push;
    if (tile_ms) *tile_ms = net->ms_tile;
    if (run_ms) *run_ms = net->ms_run;
    if (steps) *steps = net->launches;
    if (run_launches) *run_launches = net->run_launches;
    return SPK_OK;
}

spk_status spk_hbm_copy(spk_net *net, uint64_t bytes, int reps, double *ms)
{
    SPK_TRY(check_ready(net));
    if (bytes == 0 || bytes % 16 || reps < 1) return fail(SPK_EINVAL, "bytes multiple of 16, reps >= 1");
    hipStream_t s = net->stream;
    void *a = nullptr, *b = nullptr;
    SPK_TRY(dalloc(net, (uint8_t **)&a, bytes));
    SPK_TRY(dalloc(net, (uint8_t **)&b, bytes));
    hipEvent_t e0 = nullptr, e1 = nullptr;
    spk_status st = SPK_OK;
    do {
        hipError_t e = hipMemsetAsync(a, 1, bytes, s);
        if (e == hipSuccess) e = stream_copy(a, b, bytes, s);  // warm-up
        if (e == hipSuccess) e = hipEventCreate(&e0);
        if (e == hipSuccess) e = hipEventCreate(&e1);
        if (e == hipSuccess) e = hipEventRecord(e0, s);
        for (int r = 0; r < reps && e == hipSuccess; r++) e = stream_copy(a, b, bytes, s);
        if (e == hipSuccess) e = hipEventRecord(e1, s);
        if (e == hipSuccess) e = hipEventSynchronize(e1);
        float t = 0;
        if (e == hipSuccess) e = hipEventElapsedTime(&t, e0, e1);
        if (e != hipSuccess) { st = fail(SPK_EHIP, hipGetErrorString(e)); break; }
        if (ms) *ms = t;
    } while (0);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    dfree(net, a);
    dfree(net, b);
    return st;
}

spk_status spk_hbm_read(spk_net *net, uint64_t bytes, int reps, double *ms)
{
    SPK_TRY(check_ready(net));
    if (bytes == 0 || bytes % 16 || reps < 1) return fail(SPK_EINVAL, "bytes multiple of 16, reps >= 1");
    hipStream_t s = net->stream;
    uint8_t *a = nullptr;
    uint32_t *sink = nullptr;
    SPK_TRY(dalloc(net, &a, bytes));
    SPK_TRY(dalloc(net, &sink, 1));
    hipEvent_t e0 = nullptr, e1 = nullptr;
    spk_status st = SPK_OK;
    do {
        hipError_t e = hipMemsetAsync(a, 1, bytes, s);
        if (e == hipSuccess) e = stream_read(a, bytes, sink, s);  // warm-up
        if (e == hipSuccess) e = hipEventCreate(&e0);
        if (e == hipSuccess) e = hipEventCreate(&e1);
        if (e == hipSuccess) e = hipEventRecord(e0, s);
        for (int r = 0; r < reps && e == hipSuccess; r++) e = stream_read(a, bytes, sink, s);
        if (e == hipSuccess) e = hipEventRecord(e1, s);
        if (e == hipSuccess) e = hipEventSynchronize(e1);
        float t = 0;
        if (e == hipSuccess) e = hipEventElapsedTime(&t, e0, e1);
        if (e != hipSuccess) { st = fail(SPK_EHIP, hipGetErrorString(e)); break; }
        if (ms) *ms = t;
    } while (0);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    dfree(net, a);
    dfree(net, sink);
    return st;
}

void spk_destroy(spk_net *net) { destroy_net(net); }

}  // extern "C"
