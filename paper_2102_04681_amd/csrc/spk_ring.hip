// spk_ring.hip -- the resident step kernel: many simulation steps in one
// launch of one workgroup per target tile, with the inputs of every pending
// arrival step held in LDS.
//
// What it is for: networks whose tile fits in LDS together with its input of
// every step up to the longest delay (delay_max x W accumulators).  The
// events of a spike then need no page in memory: right after a step (or a
// batch of D <= delay_min steps) every tile reads, for each neuron that
// fired anywhere, the run of its row that falls into the tile, and adds each
// event to the accumulator of its arrival step.  One hand-off per batch is
// left (the spike lists), against two for pages, and an event is read once
// and never written; a network of one tile has no hand-off at all.
//
// A batch:
//   1. update: the tile's neurons take the batch's steps, potentials and
//      refractory counters in registers, inputs from the ring slots of the
//      batch (which restart at zero); spikes as (step << 24 | neuron);
//   2. publication: a 16-byte mailbox per tile and batch parity holds the
//      batch's stamp, the spike count and up to three spikes; more go to the
//      tile's segment of the spike list (stored and waited for before the
//      mailbox).  Both 8-byte words carry the stamp, so they need no order
//      between them;
//   3. hand-off: wave w polls the mailboxes of tiles w, w + 16, ... itself
//      (agent-scope loads; the data crosses XCDs), drawing the next batch's
//      external input a unit at a time between looks (draws are private to
//      a thread).  No barrier, list or prefix stands between a mailbox and
//      its gather: lane l of the wave holds the mailbox of tile l / LP and
//      takes its spikes l % LP, l % LP + LP, ... (LP = 64 / tiles per wave;
//      with fewer than 16 tiles several waves share a tile's spikes);
//   4. gather: the lane resolves its spike's run (one unaligned 4-byte load
//      gives the run's two ends, the next spike's in flight meanwhile); the
//      wave's runs are then walked 64 records at a time, the record's run
//      found from a bit mask of run starts by a population count instead of
//      a search.
//
// The gather of a launch's last batch may be left to the next launch (defer,
// pending): the spikes stay in the mailboxes and segments of their parity.  A
// call of one batch then needs no hand-off inside the launch and is an
// ordinary launch; only launches that wait for other tiles are cooperative
// (all workgroups resident at once).
//
// A network of one tile keeps each neuron's row (start and length) in
// registers and puts them into the list beside the spike, so that the gather
// starts with the synapse loads.
//
// Accumulators: networks of at most two weight classes whose in-degrees per
// class stay below 2^16 count events instead of summing weights: two 16-bit
// counts in a 32-bit word, multiplied by the class weights in the update.
// The sum is the same integer (an event adds one to a count; the product and
// the sum are exact), an LDS add takes 4 bytes instead of 8 and needs no
// weight lookup.  Others sum as the page kernels do (Acc<FIXED>).
//
// Every wait is bounded as in the persistent page kernel (10 s of the
// real-time clock, an abort flag that every waiter polls).
#include <hip/hip_runtime.h>

#include "spk_dev.h"

namespace spk {

namespace {

constexpr uint32_t kRT = 1024;                        // threads
constexpr uint32_t kRW = kRT / kWave;                 // waves
constexpr uint32_t kList1 = 1024;                     // one tile: spikes gathered at once
constexpr int kMany = 4;                              // runs per lane walked together, where there are many
constexpr int kWin = 8;                               // 64-record windows in flight per wave
constexpr uint64_t kTicks = 10ull * 100000000ull;     // 10 s of the 100 MHz clock
constexpr uint32_t kStopped = 4u;                     // the network's device flag: a launch stopped early
constexpr uint32_t kInline = 3;                       // spikes carried by a mailbox
constexpr uint32_t kIdBits = 28;                      // step of the batch << 24 | neuron
constexpr uint64_t kIdMask = (1ull << kIdBits) - 1;
constexpr uint64_t kBegMask = (1ull << 48) - 1;
static_assert(kRT == kBlockThreads, "the block-wide helpers assume workgroups of kBlockThreads");
static_assert(kRW == kRingWaves, "ring_share deals the tiles to the waves");
static_assert(kRingMaxT <= kRW * 16, "a wave serves at most 16 tiles, four lanes each");

// Mailbox words.  a: spike 0 << 36 | count << 18 | 18-bit stamp (count <=
// kMaxTileW); b: spike 2 << 36 | spike 1 << 8 | 8-bit stamp.  The same
// parity's stamps differ by 2 from batch to batch.
struct Box {
    uint64_t a, b;
};
__device__ __forceinline__ uint64_t box_a(uint32_t e, uint32_t cnt, uint32_t s0)
{
    return (uint64_t)s0 << 36 | (uint64_t)cnt << 18 | (e & 0x3ffffu);
}
__device__ __forceinline__ uint64_t box_b(uint32_t e, uint32_t s1, uint32_t s2)
{
    return (uint64_t)s2 << 36 | (uint64_t)s1 << 8 | (e & 0xffu);
}
__device__ __forceinline__ uint32_t box_cnt(Box x) { return (uint32_t)(x.a >> 18) & 0x3ffffu; }
// Spike i < kInline of a mailbox.
__device__ __forceinline__ uint32_t box_spike(Box x, uint32_t i)
{
    return i == 0 ? (uint32_t)(x.a >> 36) : i == 1 ? (uint32_t)(x.b >> 8) & (uint32_t)kIdMask : (uint32_t)(x.b >> 36);
}
__device__ __forceinline__ bool box_ready(Box x, uint32_t e)
{
    const uint32_t c = box_cnt(x);  // (a word that carries none of the c spikes need not have arrived)
    return ((uint32_t)x.a & 0x3ffffu) == (e & 0x3ffffu) && (c < 2 || c > kInline || ((uint32_t)x.b & 0xffu) == (e & 0xffu));
}

__device__ __forceinline__ void st_ag64(uint64_t *p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Both words of mailbox k in one 16-byte load at agent scope (sc1; volatile:
// polled in loops).  The two words may be of different stores: each is
// checked on its own.  The halves of one 8-byte word have to be of one store,
// which rests on the hardware and not on the language's memory model: an
// aligned 8-byte store and an aligned 16-byte load of a lane are each one
// access within a 128-byte line.  (A stamp in each 4-byte word, which needs no
// such thing, took 250,000 neurons from 8.8 to 9.9 us per step.)  One request
// per mailbox and look instead of two took 250,000 neurons from 9.5 to 9.3
// us per step, four instead of two had cost 1.7: the looks of every workgroup
// queue.
__device__ __forceinline__ Box box_load(const uint64_t *boxes, uint32_t k)
{
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)boxes, 0, kRingBoxBytes, 0x00027000);
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(k * kRingBoxStride * 8), 0, (int)(0x80000000u | 16u));
    return Box{(uint64_t)v.y << 32 | v.x, (uint64_t)v.w << 32 | v.z};
}

// Accumulators of a variant: packed event counts (CNT), or sums.
template <bool FIXED, bool CNT> struct RingAcc { using T = typename Acc<FIXED>::T; };
template <bool FIXED> struct RingAcc<FIXED, true> { using T = uint32_t; };

template <bool FIXED, bool CNT, bool MULTI>
struct RingLDS {
    using AccT = typename RingAcc<FIXED, CNT>::T;
    static constexpr uint32_t kBytes = MULTI ? kRingBytes : kRingBytes1;
    AccT ring[kBytes / sizeof(AccT)];      // input of (arrival slot, neuron of the tile)
    uint8_t kp[kMaxTileW];                 // Poisson counts of step u of the batch at u * W
    uint64_t pois[256];
    uint16_t guide[256];
    uint64_t list1[MULTI ? 1 : kList1];    // one tile: the batch's spikes, step << 48 | row length << 32 | row start
    uint64_t wst[kRW][MULTI ? kMany * kWave : kWave];  // per wave: run r's (start - records before it) | step << 48
    uint32_t hm[kRW][2 * kWin];            // per wave: bit f set: a run starts at record f of the windows
    uint32_t tw[kRW][16], ti[kRW][64], tm[kRW][2 * kMany];  // per wave: its tiles' spikes as one sequence
    uint32_t cnt[kRingMaxT];               // raster: every tile's spikes in the batch
    uint32_t stop;                         // a wave gave up waiting
    uint32_t own[kInline + 1];             // the tile's first spikes (the last entry: a dummy)
    uint32_t ntot[2];                      // spikes of the batch, by batch parity
    uint32_t nb[kRunMaxD];                 // ... of each step
    unsigned long long ev[kRunMaxD];       // events emitted at each step
    uint32_t dlv[kRunMaxD];                // events delivered at each step (several delays)
    uint32_t rtot[kRunMaxD], rbef[kRunMaxD], rk[kRunMaxD], rokm;
    unsigned long long rb[kRunMaxD];
    long long wtab[kMaxClasses];
};

// One unit of the next batch's draws (unit k: step k / nr, round k % nr):
// thread-private (the neuron's Poisson count in kp, a source's decision in
// bit k of *fire).
template <class L_>
__device__ __forceinline__ void ring_draw(const ModelArgs &m, L_ &L, uint32_t W, uint32_t tile_lo, uint32_t tile_n,
                                          uint64_t t, uint32_t k, uint32_t nr, uint32_t *fire)
{
    const uint32_t u = k / nr, q = (k - u * nr) * kRT + threadIdx.x;
    if (q >= tile_n) return;
    const uint32_t gi = tile_lo + q;
    if (m.pois_len) {  // K = min { k : hi32 < T_k }, searched from the guide entry
        const uint32_t h = hash_hi32(step_hash(m.keys.pois, gi, t + u));
        uint32_t kk = L.guide[h >> 24];
        while ((uint64_t)h >= L.pois[kk]) kk++;
        L.kp[u * W + q] = (uint8_t)kk;
    }
    if (m.kind == SPK_SOURCE) {
        const bool f = (uint64_t)hash_hi32(step_hash(m.keys.bern, gi, t + u)) < m.src_thr;
        *fire = (*fire & ~(1u << k)) | (uint32_t)f << k;
    }
}

// The input of one neuron from its accumulator and Poisson count.
template <bool FIXED, bool CNT, class AccT>
__device__ __forceinline__ float ring_input(const ModelArgs &m, AccT acc, uint32_t K, double w0, double w1, int32_t q0,
                                            int32_t q1)
{
    if constexpr (FIXED) {
        int32_t s;
        if constexpr (CNT) s = (int32_t)(acc & 0xffffu) * q0 + (int32_t)(acc >> 16) * q1;
        else s = (int32_t)acc;
        return ldexpf((float)(s + (int32_t)K * m.ext_wq + m.bias_q), -m.shift);
    } else {
        float isyn;
        if constexpr (CNT) isyn = counts_to_float(acc, w0, w1);
        else isyn = fixed64_to_float(acc, m.shift64);
        return __fadd_rn(__fadd_rn(isyn, __fmul_rn((float)K, m.ext_w)), m.i_bias);
    }
}

// Forward Euler step of the membrane, every operation rounded on its own.
__device__ __forceinline__ float ring_integrate(float V, float I, float k, float v_rest)
{
    return __fadd_rn(__fadd_rn(V, __fmul_rn(k, __fsub_rn(v_rest, V))), I);
}

// One neuron, one step: true if it fires.  Without branches, for both neuron
// kinds and whether the neuron is refractory or not.
__device__ __forceinline__ bool ring_neuron(const ModelArgs &m, float &V, uint32_t &r, float I, bool src_fires)
{
    const float vn = ring_integrate(V, I, m.k, m.v_rest);
    const bool src = m.kind == SPK_SOURCE;  // (uniform)
    const bool refr = r > 0;
    const bool fire = !refr && vn >= m.v_th;
    V = !src && (refr || fire) ? m.v_reset : vn;
    const uint32_t rn = refr ? r - 1u : (fire ? m.ref_steps : 0u);
    r = src ? r : rn;
    return src ? src_fires : fire;
}

// Add the records of N windows (64 records each, from record f0 of the
// wave's runs on) to the ring: every load is issued before the first add.
template <bool FIXED, bool CMP, bool CNT, int N, class L_>
__device__ __forceinline__ void ring_windows(const StepArgs &a, L_ &L, uint32_t w, uint32_t lane,
                                             uint32_t mw, uint32_t f0, uint32_t tot, uint32_t &base, uint32_t slot0)
{
    using Rec = typename SynRec<CMP>::T;
    Rec rec[N];
    uint32_t su[N];
#pragma unroll
    for (int i = 0; i < N; i++) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)mw, 2 * i),
                       hi = (uint32_t)__builtin_amdgcn_readlane((int)mw, 2 * i + 1);
        // run of this lane's record: starts at or before it, minus one
        const uint64_t m = (uint64_t)hi << 32 | lo, m1 = m >> 1;
        const uint32_t r = __builtin_amdgcn_mbcnt_hi((uint32_t)(m1 >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)m1, base + (lo & 1u) - 1u));
        base += (uint32_t)__popcll(m);
        const uint64_t st = L.wst[w][r];
        const uint32_t f = f0 + i * kWave + lane;
        su[i] = (uint32_t)(st >> 48);
        rec[i] = SynRec<CMP>::load(a, f < tot ? (st + f) & kBegMask : 0ull);  // (unconditional, from a clamped index)
    }
#pragma unroll
    for (int i = 0; i < N; i++) {
        const uint32_t key = rec_key(rec[i]);
        uint32_t sl = slot0 + su[i] + rec_delay(key);
        sl = sl >= a.pslots ? sl - a.pslots : sl;
        const uint32_t at = (sl << a.tl.logW) + (key & (a.tl.W - 1u));
        if (f0 + i * kWave + lane < tot) {
            if constexpr (CNT) atomicAdd(&L.ring[at], 1u << ((key >> (kClassShift - 4)) & 0x30u));
            else if constexpr (CMP) Acc<FIXED>::add(&L.ring[at], L.wtab[rec_class(key)]);
            else Acc<FIXED>::add(&L.ring[at], units_of<FIXED>(rec[i].y, a.m.shift64));
        }
    }
}

// Walk a wave's runs (R per lane, len records from synapse beg on each) and
// add their records to the ring.
template <bool FIXED, bool CMP, bool CNT, int R, class L_>
__device__ __forceinline__ void ring_walk(const StepArgs &a, L_ &L, uint32_t w, uint32_t lane, const uint64_t *beg,
                                          const uint32_t *len, const uint32_t *u, uint32_t slot0)
{
    uint32_t pre[R], tot = 0, runs = 0;
#pragma unroll
    for (int r = 0; r < R; r++) {
        const uint32_t inc = wave_scan_incl_u32(len[r]);
        pre[r] = tot + inc - len[r];
        tot += (uint32_t)__builtin_amdgcn_readlane((int)inc, kWave - 1);
        const uint64_t some = __ballot(len[r] != 0);
        if (len[r]) {
            const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(some >> 32),
                                                            __builtin_amdgcn_mbcnt_lo((uint32_t)some, runs));
            L.wst[w][rank] = ((beg[r] - pre[r]) & kBegMask) | (uint64_t)u[r] << 48;
        }
        runs += (uint32_t)__popcll(some);
    }
    uint32_t base = 0;  // runs that start before the windows
    for (uint32_t f0 = 0; f0 < tot; f0 += kWin * kWave) {
        if (lane < 2 * kWin) L.hm[w][lane] = 0;
        lds_wave_sync();
#pragma unroll
        for (int r = 0; r < R; r++) {
            const uint32_t o = pre[r] - f0;
            if (len[r] && o < kWin * kWave) atomicOr(&L.hm[w][o >> 5], 1u << (o & 31u));
        }
        lds_wave_sync();
        const uint32_t mw = L.hm[w][lane & (2 * kWin - 1)];
        const uint32_t nwin = (tot - f0 + kWave - 1) / kWave;
        switch (nwin < (uint32_t)kWin ? nwin : (uint32_t)kWin) {
        case 1: ring_windows<FIXED, CMP, CNT, 1>(a, L, w, lane, mw, f0, tot, base, slot0); break;
        case 2: ring_windows<FIXED, CMP, CNT, 2>(a, L, w, lane, mw, f0, tot, base, slot0); break;
        case 3: ring_windows<FIXED, CMP, CNT, 3>(a, L, w, lane, mw, f0, tot, base, slot0); break;
        case 4: ring_windows<FIXED, CMP, CNT, 4>(a, L, w, lane, mw, f0, tot, base, slot0); break;
        case 5: ring_windows<FIXED, CMP, CNT, 5>(a, L, w, lane, mw, f0, tot, base, slot0); break;
        case 6: ring_windows<FIXED, CMP, CNT, 6>(a, L, w, lane, mw, f0, tot, base, slot0); break;
        case 7: ring_windows<FIXED, CMP, CNT, 7>(a, L, w, lane, mw, f0, tot, base, slot0); break;
        default: ring_windows<FIXED, CMP, CNT, 8>(a, L, w, lane, mw, f0, tot, base, slot0); break;
        }
        lds_wave_sync();
    }
}

// One tile: deliver the K spikes of the list into the ring; each wave takes
// groups of at most 64.
template <bool FIXED, bool CMP, bool CNT, class L_>
__device__ __forceinline__ void ring_gather1(const StepArgs &a, L_ &L, uint32_t K, uint32_t slot0)
{
    const uint32_t lane = lane_id(), w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    uint32_t G = (K + kRW - 1) / kRW;  // spikes per wave and round
    G = G > (uint32_t)kWave ? (uint32_t)kWave : G;
    for (uint32_t p0 = w * G; p0 < K; p0 += kRW * G) {
        const bool live = lane < G && p0 + lane < K;
        const uint64_t en = L.list1[live ? p0 + lane : p0];
        const uint64_t beg = (uint32_t)en;
        const uint32_t len = live ? (uint32_t)(en >> 32) & 0xffffu : 0u, u = (uint32_t)(en >> 48);
        ring_walk<FIXED, CMP, CNT, 1>(a, L, w, lane, &beg, &len, &u, slot0);
    }
}

// Deliver the wave's spikes (the mailboxes of the lanes' tiles have arrived)
// into the ring.  Few spikes: one or two per lane, as the lanes hold them.
// More: the tiles' spikes as one sequence in tile order, up to kMany * 64 at a
// time: neighbouring lanes then read rows and row offsets of one tile's
// neurons, whose pages are few (lanes spread over all of the wave's tiles
// instead took 75 us per step on 1e6 sources at 10 Hz, 41 spikes per tile;
// the sequence takes 50; one tile after the other from a list of all
// spikes, 64 at a time, 60).  Where each tile has a lane per spike, the
// sequence's extra LDS round trips cost more than they save (120,000
// neurons, 1 spike per tile: 6.3 against 5.5 us).
template <bool FIXED, bool CMP, bool CNT, class L_>
__device__ __forceinline__ void ring_gather(const StepArgs &a, L_ &L, uint32_t tile, uint32_t w, uint32_t lane,
                                            const RingShare &h, Box box, const uint32_t *seg0, uint32_t seg_cap,
                                            uint32_t slot0)
{
    const uint32_t c = h.mine ? box_cnt(box) : 0u, i = h.i0;
    if (!__ballot(c != 0)) return;
    const uint32_t row_len = a.row_len;
    // where spike id's run starts (*beg: its row) and ends in the row
    auto resolve = [&](bool in, uint32_t id, uint64_t *beg, uint32_t *ends) {
        const uint32_t s = in ? id & kTargetMask : 0u;
        // (the run's two ends are neighbouring u16: one 4-byte load at 2-byte alignment)
        __builtin_memcpy(ends, a.toff + (uint64_t)s * (a.tl.T + 1) + tile, 4);
        // rows of equal length start at a multiple of it; no load then
        *beg = row_len ? (uint64_t)s * row_len : a.row_ptr[s];
    };
    if (!__ballot(ring_many(h, c))) {
        const bool in = i < c;
        if (!__ballot(in)) return;  // (several waves share the tile)
        uint32_t id = box_spike(box, i);
        if (c > kInline) id = ld_ag(seg0 + (uint64_t)h.tile * seg_cap + (in ? i : 0u));
        const uint32_t u = id >> kTargetBits;
        uint64_t beg;
        uint32_t ends;
        resolve(in, id, &beg, &ends);
        beg += ends & 0xffffu;
        const uint32_t len = in ? (ends >> 16) - (ends & 0xffffu) : 0u;
        ring_walk<FIXED, CMP, CNT, 1>(a, L, w, lane, &beg, &len, &u, slot0);
        return;
    }
    uint32_t id[kMany], at[kMany], base = 0;
    // the first lane of each tile: its spikes are positions pre .. pre + n - 1
    const bool first = h.mine && (h.i0 & (kWave - 1u)) == 0;
    uint32_t n0, n1;
    ring_range(h, c, &n0, &n1);
    const uint32_t n = first ? n1 - n0 : 0u;
    const uint32_t inc = wave_scan_incl_u32(n), pre = inc - n;
    const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)inc, kWave - 1);
    const uint64_t some = __ballot(n != 0);
    if (n) {
        const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(some >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)some, 0u));
        // position p of rank r's spikes: word tw[r] + p of the segments, or of
        // the carried spikes in ti (bit 31)
        L.tw[w][rank] = c > kInline ? h.tile * seg_cap + n0 - pre : 0x80000000u | ((rank * 4 + n0 - pre) & 0x7fffffffu);
#pragma unroll
        for (uint32_t k = 0; k < kInline; k++) L.ti[w][rank * 4 + k] = box_spike(box, k);
    }
    lds_wave_sync();
    // the places of the R * 64 spikes of the sequence from p0 on (base: tiles
    // that start before p0)
    auto locate = [&](uint32_t p0) {
        if (lane < 2 * kMany) L.tm[w][lane] = 0;
        lds_wave_sync();
        const uint32_t o = pre - p0;
        if (n && o < kMany * kWave) atomicOr(&L.tm[w][o >> 5], 1u << (o & 31u));
        lds_wave_sync();
        const uint32_t mw = L.tm[w][lane & (2 * kMany - 1)];
#pragma unroll
        for (int r = 0; r < kMany; r++) {
            const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)mw, 2 * r),
                           hi = (uint32_t)__builtin_amdgcn_readlane((int)mw, 2 * r + 1);
            const uint64_t m = (uint64_t)hi << 32 | lo, m1 = m >> 1;
            const uint32_t k = __builtin_amdgcn_mbcnt_hi((uint32_t)(m1 >> 32),
                                                         __builtin_amdgcn_mbcnt_lo((uint32_t)m1, base + (lo & 1u) - 1u));
            base += (uint32_t)__popcll(m);
            const uint32_t v = L.tw[w][k & 15u], p = p0 + r * kWave + lane;
            at[r] = (v & 0x80000000u) | ((v + p) & 0x7fffffffu);
            if (p < tot && !(at[r] >> 31)) id[r] = ld_ag(seg0 + at[r]);
        }
    };
#pragma unroll
    for (int r = 0; r < kMany; r++) id[r] = 0;
    locate(0);
    for (uint32_t p0 = 0; p0 < tot; p0 += kMany * kWave) {
        uint64_t beg[kMany];
        uint32_t len[kMany], u[kMany], ends[kMany];
#pragma unroll
        for (int r = 0; r < kMany; r++) {
            const bool in = p0 + r * kWave + lane < tot;
            if (in && (at[r] >> 31)) id[r] = L.ti[w][at[r] & 63u];  // (carried by the mailbox)
            u[r] = id[r] >> kTargetBits;
            resolve(in, id[r], &beg[r], &ends[r]);
        }
        if (p0 + kMany * kWave < tot) locate(p0 + kMany * kWave);  // (uniform) the next IDs, in flight during the walk
#pragma unroll
        for (int r = 0; r < kMany; r++) {
            beg[r] += ends[r] & 0xffffu;
            len[r] = p0 + r * kWave + lane < tot ? (ends[r] >> 16) - (ends[r] & 0xffffu) : 0u;
        }
        ring_walk<FIXED, CMP, CNT, kMany>(a, L, w, lane, beg, len, u, slot0);
    }
}

// Mailbox of a tile: the tiles that one wave polls (every 16th) lie together.
__device__ __forceinline__ uint32_t ring_box(uint32_t tile)
{
    return (tile % kRW) * (kRingMaxT / kRW) + tile / kRW;
}

// The kernel's arguments, read again in each phase (scalar loads) instead of
// being held, and spilled, across the whole step: the pointer is opaque to
// the optimiser.
__device__ __forceinline__ const RingArgs &ring_kargs()
{
    auto p = (const __attribute__((address_space(4))) RingArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const RingArgs *)p;
}

// MULTI: several tiles (mailboxes); otherwise the network is one tile.
// NR: neurons per thread (W <= NR * kRT).
template <bool FIXED, bool CMP, bool CNT, bool MULTI, int NR>
__global__ __launch_bounds__(kRT) void k_ring(RingArgs)
{
    using LT = RingLDS<FIXED, CNT, MULTI>;
    using AccT = typename LT::AccT;
    __shared__ LT L;
    const uint32_t tid = threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(tid / kWave);
    const uint32_t T8 = ring_kargs().s.tl.T8, Tn = ring_kargs().Tn;
    // a row's neighbouring tiles on one XCD (workgroups of a cooperative
    // launch go to the XCDs in turn); results do not depend on it
    const uint32_t x = MULTI ? blockIdx.x % kGroups : 0u, tile = MULTI ? x * T8 + blockIdx.x / kGroups : 0u;
    if (tile >= Tn) return;
    const uint32_t W = ring_kargs().s.tl.W, n = ring_kargs().s.n;
    const uint32_t tile_lo = tile * W, tile_n = n - tile_lo < W ? n - tile_lo : W;
    const uint32_t nr = (tile_n + kRT - 1) / kRT;
    const uint32_t pslots = ring_kargs().s.pslots;

    float V[NR];
    uint32_t Rp[(NR + 3) / 4];    // refractory counters, a byte per neuron
    uint32_t rowb[NR], rowl[NR];  // one tile: the neuron's row
    {
        const RingArgs &ra = ring_kargs();
        const StepArgs &a = ra.s;
#pragma unroll
        for (int r = 0; r < NR; r++) {
            const uint32_t q = r * kRT + tid, qc = q < tile_n ? tile_lo + q : tile_lo;
            V[r] = a.V[qc];
            if (r % 4 == 0) Rp[r / 4] = 0;
            Rp[r / 4] |= (uint32_t)a.ref[qc] << (8 * (r % 4));
            if constexpr (!MULTI) {
                rowb[r] = (uint32_t)a.row_ptr[qc];
                rowl[r] = a.outdeg[qc];
            }
        }
        const AccT *ring_g = (const AccT *)ra.ring + (uint64_t)tile * pslots * W;
        for (uint32_t q = tid; q < pslots * W; q += kRT) L.ring[q] = ring_g[q];
        if (a.m.pois_len && tid < 256) {
            L.pois[tid] = a.pois[tid < a.m.pois_len ? tid : 0u];
            L.guide[tid] = a.pois_guide[tid];
        }
        if (tid < kRunMaxD) {
            L.nb[tid] = 0;
            L.ev[tid] = 0;
            L.dlv[tid] = 0;
        }
        if (tid < kMaxClasses) L.wtab[tid] = a.wval[tid];
        if (tid < 2) L.ntot[tid] = 0;
    }
    const uint32_t D = ring_kargs().D;
    uint32_t fire = 0;
    __syncthreads();
    const uint64_t n_steps = ring_kargs().n_steps;
    uint64_t t = ring_kargs().t0;  // the batch's first step
    {
        const RingArgs &ra = ring_kargs();
        const uint32_t n_first = (uint32_t)(n_steps < D ? n_steps : D) * nr;
        for (uint32_t k = 0; k < n_first; k++) ring_draw(ra.s.m, L, W, tile_lo, tile_n, t, k, nr, &fire);
    }
    uint64_t rbase = ring_kargs().s.raster_cap ? ring_kargs().s.raster_offs[t] : 0;
    uint32_t ps = (uint32_t)(t % pslots);  // ring slot of the batch's first step
    uint32_t e = ring_kargs().e0;
    const uint32_t dm = ring_kargs().s.dmin % pslots;

    const RingShare share = ring_share(Tn, w, lane);
    // where the events of a batch whose first step is in slot p are filed from
    auto file_slot = [&](uint32_t p) { return p + dm < pslots ? p + dm : p + dm - pslots; };
    if (tid == 0) L.stop = 0;
    lds_sync();

    // the first round gathers the last launch's last batch, if that was left
    // to this launch, and nothing else
    uint32_t left = MULTI ? ring_kargs().pending : 0u;
    for (uint64_t s = 0; s < n_steps || left;) {
        const bool run = !MULTI || left == 0;
        const uint32_t Db = run ? (uint32_t)(n_steps - s < D ? n_steps - s : D) : left;
        if (run) {
            s += Db;
            e++;
        } else {
            ps = ps >= Db ? ps - Db : ps + pslots - Db;
            t -= Db;
        }
        uint32_t *ntot = &L.ntot[e & 1u];
        const uint32_t lists = ring_kargs().s.lists, row_len = ring_kargs().s.row_len;
        uint32_t od[NR];  // out-degrees of the thread's neurons that fired (one-step batches; loads in flight)
#pragma unroll
        for (int r = 0; r < NR; r++) od[r] = 0;

        // 1. update
        if (run) {
            const RingArgs &ra = ring_kargs();
            const ModelArgs &m = ra.s.m;
            uint32_t *seg = ra.seg + ((uint64_t)(e & 1u) * Tn + tile) * ra.seg_cap;
            double w0 = 0, w1 = 0;
            int32_t q0 = 0, q1 = 0;
            if constexpr (CNT && FIXED) {
                q0 = (int32_t)ra.s.wval[0];
                q1 = (int32_t)ra.s.wval[1];
            } else if constexpr (CNT) {
                w0 = ra.w0;
                w1 = ra.w1;
            }
            const bool drive = m.pois_len != 0;
            // a firing neuron's place in the batch's spike list
            auto put = [&](uint32_t at, uint32_t u, int r) {
                const uint32_t id = u << kTargetBits | (tile_lo + r * kRT + tid);
                if constexpr (MULTI) {
                    L.own[at < kInline ? at : kInline] = id;
                    st_ag(seg + at, id);
                } else {
                    if (at < kList1) L.list1[at] = (uint64_t)u << 48 | (uint64_t)rowl[r] << 32 | rowb[r];
                    if (at >= kList1 || ra.s.raster_cap) st_ag(seg + at, id);
                }
            };
            if (Db == 1) {
                uint64_t bal[NR];
                uint32_t mine = 0, dl = 0;
                const uint32_t at0 = ps * W;
#pragma unroll
                for (int r = 0; r < NR; r++) {
                    bal[r] = 0;
                    if (NR > 1 && r * kRT >= tile_n) continue;  // (uniform)
                    const uint32_t q = r * kRT + tid;
                    const bool live = q < tile_n;
                    const uint32_t qc = live ? q : 0u;
                    const AccT acc = L.ring[at0 + qc];
                    const uint32_t kq = L.kp[qc];
                    if (live) L.ring[at0 + qc] = 0;
                    if constexpr (CNT) dl += live ? (acc & 0xffffu) + (acc >> 16) : 0u;
                    const float I = ring_input<FIXED, CNT>(m, acc, drive ? kq : 0u, w0, w1, q0, q1);
                    uint32_t ref = (Rp[r / 4] >> (8 * (r % 4))) & 0xffu;
                    bal[r] = __ballot(ring_neuron(m, V[r], ref, I, (fire >> r) & 1u) && live);
                    Rp[r / 4] = (Rp[r / 4] & ~(0xffu << (8 * (r % 4)))) | ref << (8 * (r % 4));
                    mine += (uint32_t)__popcll(bal[r]);
                }
                if (mine) {  // (uniform) one position counter update per wave
                    uint32_t wb = 0, el = 0;
                    if (lane == 0) wb = atomicAdd(ntot, mine);
                    wb = (uint32_t)__builtin_amdgcn_readlane((int)wb, 0);
#pragma unroll
                    for (int r = 0; r < NR; r++) {
                        if ((bal[r] >> lane) & 1ull) {
                            put(wb + __builtin_amdgcn_mbcnt_hi((uint32_t)(bal[r] >> 32),
                                                              __builtin_amdgcn_mbcnt_lo((uint32_t)bal[r], 0u)), 0u, r);
                            if constexpr (!MULTI) el += rowl[r];
                            else if (!row_len) od[r] = ra.s.outdeg[tile_lo + r * kRT + tid];
                        }
                        wb += (uint32_t)__popcll(bal[r]);
                    }
                    if constexpr (!MULTI)
                        if (el) atomicAdd(&L.ev[0], (unsigned long long)el);
                }
                if (CNT && lists > 1) {
                    const uint32_t sum = wave_scan_incl_u32(dl);
                    if (lane == kWave - 1 && sum) atomicAdd(&L.dlv[0], sum);
                }
            } else {
#pragma unroll
                for (int r = 0; r < NR; r++) {
                    if (NR > 1 && r * kRT >= tile_n) continue;  // (uniform)
                    const uint32_t q = r * kRT + tid;
                    const bool live = q < tile_n;
                    const uint32_t qc = live ? q : 0u;
                    if (!__ballot(live)) continue;  // (a wave without neurons)
                    uint32_t ref = (Rp[r / 4] >> (8 * (r % 4))) & 0xffu;
                    for (uint32_t u = 0; u < Db; u++) {
                        const uint32_t sl = ps + u < pslots ? ps + u : ps + u - pslots;
                        const AccT acc = L.ring[sl * W + qc];
                        const uint32_t kq = L.kp[u * W + qc];
                        if (live) L.ring[sl * W + qc] = 0;
                        const float I = ring_input<FIXED, CNT>(m, acc, drive ? kq : 0u, w0, w1, q0, q1);
                        const bool f = ring_neuron(m, V[r], ref, I, (fire >> (u * nr + r)) & 1u) && live;
                        const uint64_t bal = __ballot(f);
                        if (bal) {  // (uniform)
                            uint32_t wb = 0;
                            if (lane == 0) {
                                wb = atomicAdd(ntot, (uint32_t)__popcll(bal));
                                atomicAdd(&L.nb[u], (uint32_t)__popcll(bal));
                            }
                            wb = (uint32_t)__builtin_amdgcn_readlane((int)wb, 0);
                            if (f) {
                                put(wb + __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                                  __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u)), u, r);
                                if constexpr (!MULTI) atomicAdd(&L.ev[u], (unsigned long long)rowl[r]);
                            }
                        }
                        if (CNT && lists > 1) {
                            const uint32_t sum = wave_scan_incl_u32(live ? (uint32_t)(acc & 0xffffu) + (uint32_t)(acc >> 16) : 0u);
                            if (lane == kWave - 1 && sum) atomicAdd(&L.dlv[u], sum);
                        }
                    }
                    Rp[r / 4] = (Rp[r / 4] & ~(0xffu << (8 * (r % 4)))) | ref << (8 * (r % 4));
                }
            }
        }
        // 2. publication
        lds_sync();
        const uint32_t cnt = run ? *ntot : 0u;
        if (MULTI ? cnt > kInline : cnt > kList1 || ring_kargs().s.raster_cap) {
            // (spikes in the segment: stored before they are announced or read)
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
        }
        if (MULTI && run && w == kRW - 1) {
            const RingArgs &ra = ring_kargs();
            if (ra.s.raster_cap && Db > 1) {  // each step's count, for the raster positions
                if (lane < Db) st_ag(&ra.cnts[((uint64_t)(e & 1u) * kRunMaxD + lane) * Tn + tile], L.nb[lane]);
                __builtin_amdgcn_s_waitcnt(0);
            }
            if (lane == 0) {
                uint64_t *box = ra.ctl->box[e & 1u] + (uint64_t)ring_box(tile) * kRingBoxStride;
                st_ag64(box, box_a(e, cnt, L.own[0]));
                st_ag64(box + 1, box_b(e, L.own[1], L.own[2]));
            }
        }
        // the tile's i-th spike of the batch
        auto own_spike = [&](uint32_t i) -> uint32_t {
            if (MULTI && cnt <= kInline) return L.own[i];
            const RingArgs &ra = ring_kargs();
            return ld_ag(ra.seg + ((uint64_t)(e & 1u) * Tn + tile) * ra.seg_cap + i);
        };
        // the steps' records: spikes, events emitted, events delivered
        if (run && w == kRW - 2 && lane < Db) {
            const StepArgs &a = ring_kargs().s;
            const uint64_t g = (t + lane) * kGroups + x;
            const uint32_t ns = Db == 1 ? cnt : L.nb[lane];
            const unsigned long long ev = MULTI ? (unsigned long long)ns * row_len : L.ev[lane];
            if (ns) atomicAdd(&a.counts8[g], ns);
            if (ev) atomicAdd((unsigned long long *)&a.events8[g], ev);
            if (CNT && lists > 1 && L.dlv[lane])
                atomicAdd((unsigned long long *)&a.delivered8[g], (unsigned long long)L.dlv[lane]);
            L.dlv[lane] = 0;
            L.ev[lane] = 0;
            if (!a.raster_cap) L.nb[lane] = 0;
        }
        // rows of unequal length: the out-degrees of the tile's spikes, after
        // the gather (their loads are in flight meanwhile)
        auto emitted = [&] {
            if (!MULTI || !run || row_len) return;
            const StepArgs &a = ring_kargs().s;
            if (Db == 1) {
                uint32_t sum = 0;
#pragma unroll
                for (int r = 0; r < NR; r++) sum += od[r];
                if (__ballot(sum != 0)) {
                    const uint64_t ev = wave_sum_u64(sum);
                    if (lane == 0) atomicAdd((unsigned long long *)&a.events8[t * kGroups + x], (unsigned long long)ev);
                }
            } else if (w == kRW - 2) {
                for (uint32_t i = lane; i < cnt; i += kWave) {
                    const uint32_t sp = own_spike(i);
                    atomicAdd((unsigned long long *)&a.events8[(t + (sp >> kTargetBits)) * kGroups + x],
                              (unsigned long long)a.outdeg[sp & kTargetMask]);
                }
            }
        };
        if (MULTI && run && s >= n_steps && ring_kargs().defer) {  // the next launch gathers this batch
            emitted();
            break;
        }

        // 3. the other tiles, the next batch's draws, 4. the gather
        const uint32_t Dn = (uint32_t)(n_steps - s < D ? n_steps - s : D), units = run ? Dn * nr : 0u;
        uint32_t dk = 0, fire_n = 0;
        {
            const RingArgs &ra = ring_kargs();
            const ModelArgs &m = ra.s.m;
            if constexpr (MULTI) {
                const uint64_t *box = ra.ctl->box[e & 1u];
                const uint32_t bk = ring_box(share.tile);
                Box v{(e ^ 1u) & 0x3ffffu, 0};  // (not this batch's)
                bool ok = true;
                uint64_t c0 = 0;
                for (uint32_t k = 0;; k++) {
                    if (share.mine && !box_ready(v, e)) v = box_load(box, bk);
                    const bool draw = dk < units;
                    if (draw) ring_draw(m, L, W, tile_lo, tile_n, t + Db, dk++, nr, &fire_n);
                    if (__all(!share.mine || box_ready(v, e))) break;
                    if (draw) continue;
                    if (!c0) c0 = wall_clock64();
                    if ((k & 31u) == 31u) {
                        if (ld_ag(&ra.ctl->abort_flag)) {
                            ok = false;
                            break;
                        }
                        if (wall_clock64() - c0 > kTicks) {
                            if (lane == 0) atomicOr(&ra.ctl->abort_flag, kRunAbortTimeout);
                            ok = false;
                            break;
                        }
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
                if (ok) {
                    if (ra.s.raster_cap && share.mine && share.i0 == 0) L.cnt[share.tile] = box_cnt(v);
                    ring_gather<FIXED, CMP, CNT>(ra.s, L, tile, w, lane, share, v,
                                                 ra.seg + (uint64_t)(e & 1u) * Tn * ra.seg_cap, ra.seg_cap,
                                                 file_slot(ps));
                } else if (lane == 0) {
                    L.stop = 1;
                    atomicOr(ra.s.flags, kStopped);
                }
            } else {
                for (uint32_t c0 = 0; c0 < cnt; c0 += kList1) {
                    const uint32_t K = cnt - c0 < kList1 ? cnt - c0 : kList1;
                    if (c0) {  // (spikes past the list's room, from the segment)
                        lds_sync();
                        const uint32_t *src = ra.seg + (uint64_t)(e & 1u) * ra.seg_cap + c0;
                        for (uint32_t i = tid; i < K; i += kRT) {
                            const uint32_t sp = ld_ag(src + i), sn = sp & kTargetMask;
                            const uint64_t b = ra.s.row_ptr[sn];
                            L.list1[i] = (uint64_t)(sp >> kTargetBits) << 48 | (uint64_t)ra.s.outdeg[sn] << 32 | b;
                        }
                        lds_sync();
                    }
                    ring_gather1<FIXED, CMP, CNT>(ra.s, L, K, file_slot(ps));
                }
            }
            emitted();
            for (; dk < units; dk++) ring_draw(m, L, W, tile_lo, tile_n, t + Db, dk, nr, &fire_n);
        }
        if (run) fire = fire_n;
        if (tid == 0) L.ntot[(e + 1u) & 1u] = 0;  // (last used before the previous batch's barriers)
        lds_sync();  // every event of the batch is in the ring
        if (MULTI && L.stop) return;
        left = 0;

        // raster: every tile appends its own spikes
        if (run && ring_kargs().s.raster_cap) {
            const RingArgs &ra = ring_kargs();
            const StepArgs &a = ra.s;
            uint32_t before = 0, M = cnt;
            if (MULTI) {  // (each wave for itself)
                uint32_t tot = 0, bef = 0;
                for (uint32_t k = lane; k < Tn; k += kWave) {
                    const uint32_t c = L.cnt[k];
                    tot += c;
                    bef += k < tile ? c : 0u;
                }
                M = (uint32_t)__builtin_amdgcn_readlane((int)wave_scan_incl_u32(tot), kWave - 1);
                before = (uint32_t)__builtin_amdgcn_readlane((int)wave_scan_incl_u32(bef), kWave - 1);
            }
            if (Db == 1) {
                const bool fits = rbase + M <= a.raster_cap;
                if (fits)
                    for (uint32_t i = tid; i < cnt; i += kRT) a.raster[rbase + before + i] = own_spike(i) & kTargetMask;
                if (tile == 0 && tid == 0) {
                    a.raster_offs[t + 1] = fits ? rbase + M : rbase;
                    if (!fits) atomicOr(a.flags, 2u);
                }
                rbase = fits ? rbase + M : rbase;
            } else {
                if (w < Db) {  // wave u: the spikes of step u, of all tiles and of those before this one
                    uint32_t tot = 0, bef = 0;
                    if (MULTI) {
                        for (uint32_t k = lane; k < Tn; k += kWave) {
                            const uint32_t c = ld_ag(&ra.cnts[((uint64_t)(e & 1u) * kRunMaxD + w) * Tn + k]);
                            tot += c;
                            bef += k < tile ? c : 0u;
                        }
                        tot = (uint32_t)__builtin_amdgcn_readlane((int)wave_scan_incl_u32(tot), kWave - 1);
                        bef = (uint32_t)__builtin_amdgcn_readlane((int)wave_scan_incl_u32(bef), kWave - 1);
                    } else {
                        tot = L.nb[w];
                    }
                    if (lane == 0) {
                        L.rtot[w] = tot;
                        L.rbef[w] = bef;
                        L.rk[w] = 0;
                    }
                }
                __syncthreads();
                uint64_t rb = rbase;  // (every thread the same)
                uint32_t okm = 0;
                for (uint32_t u = 0; u < Db; u++) {
                    const bool fits = rb + L.rtot[u] <= a.raster_cap;
                    if (tid == 0) L.rb[u] = rb + L.rbef[u];
                    okm |= (uint32_t)fits << u;
                    rb = fits ? rb + L.rtot[u] : rb;
                    if (tile == 0 && tid == 0) {
                        a.raster_offs[t + u + 1] = rb;
                        if (!fits) atomicOr(a.flags, 2u);
                    }
                }
                rbase = rb;
                __syncthreads();
                for (uint32_t i = tid; i < cnt; i += kRT) {
                    const uint32_t sp = own_spike(i), u = sp >> kTargetBits, rk = atomicAdd(&L.rk[u], 1u);
                    if ((okm >> u) & 1u) a.raster[L.rb[u] + rk] = sp & kTargetMask;
                }
            }
        }
        if (run && ring_kargs().s.raster_cap) {
            __syncthreads();  // (own spikes and counts read before the next batch's)
            if (tid < kRunMaxD) L.nb[tid] = 0;
            __syncthreads();
        }
        t += Db;
        ps = ps + Db < pslots ? ps + Db : ps + Db - pslots;
    }

    const RingArgs &ra = ring_kargs();
    const StepArgs &a = ra.s;
#pragma unroll
    for (int r = 0; r < NR; r++) {
        const uint32_t q = r * kRT + tid;
        if (q < tile_n) {
            a.V[tile_lo + q] = V[r];
            if (a.m.kind != SPK_SOURCE) a.ref[tile_lo + q] = (uint8_t)(Rp[r / 4] >> (8 * (r % 4)));
        }
    }
    AccT *ring_g = (AccT *)ra.ring + (uint64_t)tile * pslots * W;
    for (uint32_t q = tid; q < pslots * W; q += kRT) ring_g[q] = L.ring[q];
    if (tid == 0 && tile == 0) *(uint64_t *)a.t_base = ra.t0 + ra.n_steps;
}

template <bool FIXED, bool CMP, bool CNT, bool MULTI, int NR>
hipError_t launch_ring_k(const RingArgs &ra, hipStream_t s)
{
    if (!MULTI || !ra.waits) {
        hipLaunchKernelGGL((k_ring<FIXED, CMP, CNT, MULTI, NR>), dim3(MULTI ? ra.s.tl.T : 1u), dim3(kRT), 0, s, ra);
        return hipGetLastError();
    }
    RingArgs arg = ra;
    void *args[] = {&arg};
    return hipLaunchCooperativeKernel((const void *)k_ring<FIXED, CMP, CNT, MULTI, NR>, dim3(ra.s.tl.T), dim3(kRT), args, 0,
                                      s);
}

template <bool FIXED, bool CMP, bool CNT>
hipError_t launch_ring_t(const RingArgs &ra, hipStream_t s)
{
    const uint32_t nr = (ra.s.tl.W + kRT - 1) / kRT;
    if (ra.Tn == 1) {
        static_assert(kRingW1 == 2 * kRT, "the kernel for one tile holds two neurons per thread");
        if (nr <= 1) return launch_ring_k<FIXED, CMP, CNT, false, 1>(ra, s);
        if (nr <= 2) return launch_ring_k<FIXED, CMP, CNT, false, 2>(ra, s);
    }
    if (nr <= 1) return launch_ring_k<FIXED, CMP, CNT, true, 1>(ra, s);
    if (nr <= 2) return launch_ring_k<FIXED, CMP, CNT, true, 2>(ra, s);
    if (nr <= 4) return launch_ring_k<FIXED, CMP, CNT, true, 4>(ra, s);
    return launch_ring_k<FIXED, CMP, CNT, true, 8>(ra, s);
}

}  // namespace

// Bytes of one accumulator of the ring.
uint32_t ring_acc_bytes(bool fixed, bool counts) { return fixed || counts ? 4u : 8u; }

bool ring_supported(const RingArgs &ra)
{
    const StepArgs &a = ra.s;
    const Tiling &tl = a.tl;
    if (!a.direct || a.proc || !a.toff || a.m.pois_len > 256 || a.pslots == 0 || a.dmin == 0) return false;
    if (ra.Tn == 0 || ra.Tn > kRingMaxT || (uint64_t)ra.Tn * tl.W < a.n || tl.T > kRingMaxT || tl.W > kMaxTileW) return false;
    if (ra.D == 0 || ra.D > kRunMaxD || ra.D > a.dmin || ra.D * tl.W > kMaxTileW || ra.seg_cap < ra.D * tl.W) return false;
    if (a.pslots != a.dmin + a.lists - 1) return false;
    if (ra.counts && !a.compact) return false;
    if (!ra.counts && a.lists > 1) return false;  // (deliveries per step are counted from the event counts)
    if (a.compact ? !a.syn32 : !a.syn) return false;
    return (uint64_t)a.pslots * tl.W * ring_acc_bytes(a.m.fixed, ra.counts) <= (ra.Tn == 1 && tl.W <= kRingW1 ? kRingBytes1 : kRingBytes);
}

hipError_t launch_ring(const RingArgs &ra, hipStream_t s)
{
    if (!ring_supported(ra)) return hipErrorInvalidValue;
    const bool F = ra.s.m.fixed, C = ra.s.compact;
    if (ra.counts) return F ? launch_ring_t<true, true, true>(ra, s) : launch_ring_t<false, true, true>(ra, s);
    if (C) return F ? launch_ring_t<true, true, false>(ra, s) : launch_ring_t<false, true, false>(ra, s);
    return F ? launch_ring_t<true, false, false>(ra, s) : launch_ring_t<false, false, false>(ra, s);
}

}  // namespace spk
