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
//      mailbox).  Both 8-byte halves carry the stamp, so neither needs an
//      order between them;
//   3. hand-off: four waves poll the mailboxes (agent-scope loads; the data
//      crosses XCDs) while all threads draw the next batch's external input
//      a unit at a time between looks;
//   4. gather: the spikes as one list in LDS, shared among the 16 waves.
//      Lane l of a wave resolves spike l (one unaligned 4-byte load gives
//      the run's two ends); the wave's runs are then walked 64 records at a
//      time, the record's run found from a bit mask of run starts by a
//      population count instead of a search.
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
constexpr uint32_t kList = 2048;                      // spikes gathered at once
constexpr uint32_t kList1 = kList / 2;                // ... of a network of one tile (8-byte entries)
constexpr int kWin = 8;                               // 64-record windows in flight per wave
constexpr uint64_t kTicks = 10ull * 100000000ull;     // 10 s of the 100 MHz clock
constexpr uint32_t kStopped = 4u;                     // the network's device flag: a launch stopped early
constexpr uint32_t kInline = 3;                       // spikes carried by a mailbox
constexpr uint32_t kIdBits = 28;                      // step of the batch << 24 | neuron
constexpr uint64_t kIdMask = (1ull << kIdBits) - 1;
constexpr uint64_t kBegMask = (1ull << 48) - 1;
static_assert(kRT == kBlockThreads, "the block-wide helpers assume workgroups of kBlockThreads");
static_assert(kRingMaxT <= 4 * kWave, "four polling waves");

// Mailbox halves.  a: spike 0 << 36 | count << 18 | 18-bit stamp (count <=
// kMaxTileW < 2^14 ... 2^18); b: spike 2 << 36 | spike 1 << 8 | 8-bit stamp.
// The same parity's stamps differ by 2 from batch to batch.
__device__ __forceinline__ uint64_t box_a(uint32_t e, uint32_t cnt, uint32_t s0)
{
    return (uint64_t)s0 << 36 | (uint64_t)cnt << 18 | (e & 0x3ffffu);
}
__device__ __forceinline__ uint64_t box_b(uint32_t e, uint32_t s1, uint32_t s2)
{
    return (uint64_t)s2 << 36 | (uint64_t)s1 << 8 | (e & 0xffu);
}
__device__ __forceinline__ uint32_t box_cnt(uint64_t a) { return (uint32_t)(a >> 18) & 0x3ffffu; }
__device__ __forceinline__ bool box_ready(uint64_t a, uint64_t b, uint32_t e)
{
    if (((uint32_t)a & 0x3ffffu) != (e & 0x3ffffu)) return false;
    const uint32_t c = box_cnt(a);
    return c < 2 || c > kInline || ((uint32_t)b & 0xffu) == (e & 0xffu);
}

__device__ __forceinline__ uint64_t ld_ag64(const uint64_t *p)
{
    return __hip_atomic_load(const_cast<uint64_t *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_ag64(uint64_t *p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Accumulators of a variant: packed event counts (CNT), or sums.
template <bool FIXED, bool CNT> struct RingAcc { using T = typename Acc<FIXED>::T; };
template <bool FIXED> struct RingAcc<FIXED, true> { using T = uint32_t; };

template <bool FIXED, bool CNT>
struct RingLDS {
    using AccT = typename RingAcc<FIXED, CNT>::T;
    AccT ring[kRingBytes / sizeof(AccT)];  // input of (arrival slot, neuron of the tile)
    uint8_t kp[kMaxTileW];                 // Poisson counts of step u of the batch at u * W
    uint64_t pois[256];
    uint16_t guide[256];
    union {
        uint32_t list[kList];              // spikes being gathered: step of the batch << 24 | neuron
        uint64_t list1[kList1];            // one tile: step << 48 | row length << 32 | row start
    };
    uint64_t wst[kRW][kWave];              // per wave: run r's (start - records before it) | step << 48
    uint32_t hm[kRW][2 * kWin];            // per wave: bit f set: a run starts at record f of the windows
    uint32_t cnt[kRingMaxT], pre[kRingMaxT];
    uint32_t inl[kRingMaxT][kInline];
    uint32_t ptot[4], pq[2][4], pstop[4];
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
        // (w0, w1: the classes' units scaled by 2^-shift64; the products and
        // their sum are integers below 2^53 times that, so exact)
        if constexpr (CNT) isyn = (float)__fma_rn((double)(acc & 0xffffu), w0, __dmul_rn((double)(acc >> 16), w1));
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
template <bool FIXED, bool CMP, bool CNT, int N>
__device__ __forceinline__ void ring_windows(const StepArgs &a, RingLDS<FIXED, CNT> &L, uint32_t w, uint32_t lane,
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

// Where a spike's run in this tile starts, and how long it is: loads issued
// here, used later (the next group's are in flight while a group is walked).
struct RunAt {
    uint64_t row;    // the row's first synapse
    uint32_t ends;   // the run's two ends in the row
    uint32_t u;
};
__device__ __forceinline__ RunAt run_at(const StepArgs &a, uint32_t tile, uint32_t spike)
{
    const uint32_t s = spike & kTargetMask;
    RunAt r;
    // (the two ends are neighbouring u16: one 4-byte load at 2-byte alignment)
    __builtin_memcpy(&r.ends, a.toff + (uint64_t)s * (a.tl.T + 1) + tile, 4);
    // rows of equal length start at a multiple of it; no load then
    r.row = a.row_ptr[a.row_len ? 0u : s];
    if (a.row_len) r.row = (uint64_t)s * a.row_len;
    r.u = spike >> kTargetBits;
    return r;
}

// Walk a wave's runs (one per lane, len records from synapse beg on) and add
// their records to the ring.
template <bool FIXED, bool CMP, bool CNT>
__device__ __forceinline__ void ring_walk(const StepArgs &a, RingLDS<FIXED, CNT> &L, uint32_t w, uint32_t lane,
                                          uint64_t beg, uint32_t len, uint32_t u, uint32_t slot0)
{
    const uint32_t inc = wave_scan_incl_u32(len), pre = inc - len;
    const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)inc, kWave - 1);
    const uint64_t some = __ballot(len != 0);
    if (len) {
        const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(some >> 32),
                                                        __builtin_amdgcn_mbcnt_lo((uint32_t)some, 0u));
        L.wst[w][rank] = ((beg - pre) & kBegMask) | (uint64_t)u << 48;
    }
    uint32_t base = 0;  // runs that start before the windows
    for (uint32_t f0 = 0; f0 < tot; f0 += kWin * kWave) {
        if (lane < 2 * kWin) L.hm[w][lane] = 0;
        lds_wave_sync();
        const uint32_t o = pre - f0;
        if (len && o < kWin * kWave) atomicOr(&L.hm[w][o >> 5], 1u << (o & 31u));
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

// Deliver the K spikes of the list into the ring: each wave takes groups of
// at most 64.
template <bool FIXED, bool CMP, bool CNT, bool MULTI>
__device__ __forceinline__ void ring_gather(const StepArgs &a, RingLDS<FIXED, CNT> &L, uint32_t tile, uint32_t K,
                                            uint32_t slot0)
{
    const uint32_t lane = lane_id(), w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    uint32_t G = (K + kRW - 1) / kRW;  // spikes per wave and round
    G = G > (uint32_t)kWave ? (uint32_t)kWave : G;
    uint32_t p0 = w * G;
    if (p0 >= K) return;
    if constexpr (!MULTI) {
        for (; p0 < K; p0 += kRW * G) {
            const bool live = lane < G && p0 + lane < K;
            const uint64_t en = L.list1[live ? p0 + lane : p0];
            ring_walk<FIXED, CMP, CNT>(a, L, w, lane, (uint32_t)en, live ? (uint32_t)(en >> 32) & 0xffffu : 0u,
                                       (uint32_t)(en >> 48), slot0);
        }
    } else {
        RunAt nx = run_at(a, tile, L.list[lane < G && p0 + lane < K ? p0 + lane : p0]);
        for (; p0 < K; p0 += kRW * G) {
            const RunAt r = nx;
            const bool live = lane < G && p0 + lane < K;
            const uint32_t n0 = p0 + kRW * G;
            nx = run_at(a, tile, L.list[lane < G && n0 + lane < K ? n0 + lane : p0]);
            const uint32_t b = r.ends & 0xffffu;
            ring_walk<FIXED, CMP, CNT>(a, L, w, lane, r.row + b, live ? (r.ends >> 16) - b : 0u, r.u, slot0);
        }
    }
}

// What a polling lane has seen of its tile's mailbox.
struct Seen {
    uint64_t a, b;
};

// A wave's mailboxes are complete: their counts, the exclusive prefix of the
// counts within the wave, their sum and the carried spikes go to LDS.
template <class L_>
__device__ __forceinline__ void ring_take(L_ &L, uint32_t w, uint32_t lane, bool mine, const Seen &v)
{
    uint32_t c = mine ? box_cnt(v.a) : 0u;
    c = c < kMaxTileW ? c : kMaxTileW;
    const uint32_t inc = wave_scan_incl_u32(c), tile = w * kWave + lane;
    if (mine) {
        L.cnt[tile] = c;
        L.pre[tile] = inc - c;
        L.inl[tile][0] = (uint32_t)(v.a >> 36);
        L.inl[tile][1] = (uint32_t)((v.b >> 8) & kIdMask);
        L.inl[tile][2] = (uint32_t)(v.b >> 36);
    }
    if (lane == kWave - 1) L.ptot[w] = inc;
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
    using LT = RingLDS<FIXED, CNT>;
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
    uint32_t R[NR];
    uint32_t rowb[NR], rowl[NR];  // one tile: the neuron's row
    {
        const RingArgs &ra = ring_kargs();
        const StepArgs &a = ra.s;
#pragma unroll
        for (int r = 0; r < NR; r++) {
            const uint32_t q = r * kRT + tid, qc = q < tile_n ? tile_lo + q : tile_lo;
            V[r] = a.V[qc];
            R[r] = a.ref[qc];
            if constexpr (!MULTI) {
                rowb[r] = (uint32_t)a.row_ptr[qc];
                rowl[r] = (uint32_t)a.row_ptr[qc + 1] - rowb[r];
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
    uint32_t e = ring_kargs().e0, look = 0;
    const uint32_t dm = ring_kargs().s.dmin % pslots;

    // Gather the spikes of batch e (first step in slot p): M of them, their
    // counts and carried spikes in LDS (MULTI), or in the list (one tile).
    auto gather = [&](uint32_t M, uint32_t p) {
        const RingArgs &ra = ring_kargs();
        const uint32_t sl0 = p + dm, slot0 = sl0 < pslots ? sl0 : sl0 - pslots;
        constexpr uint32_t kChunk = MULTI ? kList : kList1;
        for (uint32_t c0 = 0; c0 < M; c0 += kChunk) {
            const uint32_t K = M - c0 < kChunk ? M - c0 : kChunk;
            if constexpr (MULTI) {  // four threads per tile copy its spikes into the list
                const uint32_t ti = tid >> 2, sub = tid & 3u;
                static_assert(kRingMaxT * 4 <= kRT, "four threads per tile");
                if (ti < Tn) {
                    const uint32_t c = L.cnt[ti];
                    uint32_t off = L.pre[ti];
                    for (uint32_t k = 0; k < ti / kWave; k++) off += L.ptot[k];
                    if (c <= kInline) {
                        if (sub < c && off + sub - c0 < K) L.list[off + sub - c0] = L.inl[ti][sub];
                    } else if (off < c0 + K && off + c > c0) {
                        const uint32_t *src = ra.seg + ((uint64_t)(e & 1u) * Tn + ti) * ra.seg_cap;
                        const uint32_t i0 = off < c0 ? c0 - off : 0u, i1 = off + c > c0 + K ? c0 + K - off : c;
                        for (uint32_t i = i0 + sub; i < i1; i += 16) {
                            uint32_t id[4];
#pragma unroll
                            for (int k = 0; k < 4; k++) id[k] = ld_ag(src + (i + 4 * k < i1 ? i + 4 * k : i));
#pragma unroll
                            for (int k = 0; k < 4; k++)
                                if (i + 4 * k < i1) L.list[off + i + 4 * k - c0] = id[k];
                        }
                    }
                }
                lds_sync();
            } else if (c0) {  // (spikes past the list's room, from the segment)
                const uint32_t *src = ra.seg + (uint64_t)(e & 1u) * ra.seg_cap + c0;
                for (uint32_t i = tid; i < K; i += kRT) {
                    const uint32_t sp = ld_ag(src + i), s = sp & kTargetMask;
                    const uint64_t b = ra.s.row_ptr[s];
                    L.list1[i] = (uint64_t)(sp >> kTargetBits) << 48 | (ra.s.row_ptr[s + 1] - b) << 32 | b;
                }
                lds_sync();
            }
            ring_gather<FIXED, CMP, CNT, MULTI>(ra.s, L, tile, K, slot0);
            if (c0 + K < M) lds_sync();  // the list is rebuilt
        }
    };

    if constexpr (MULTI) {
        if (const uint32_t Dp = ring_kargs().pending) {  // the last launch's last batch
            if (w * kWave < Tn) {
                const uint32_t pt = w * kWave + lane;
                const uint64_t *box = ring_kargs().ctl->box[e & 1u] + (uint64_t)(pt < Tn ? pt : 0u) * kRingBoxStride;
                Seen v;
                v.a = ld_ag64(box);
                v.b = ld_ag64(box + 1);
                ring_take(L, w, lane, pt < Tn, v);
            }
            lds_sync();
            uint32_t M = 0;
            for (uint32_t k = 0; k * kWave < Tn; k++) M += L.ptot[k];
            gather(M, ps >= Dp ? ps - Dp : ps + pslots - Dp);
            lds_sync();
        }
    }

    for (uint64_t s = 0; s < n_steps;) {
        const uint32_t Db = (uint32_t)(n_steps - s < D ? n_steps - s : D);
        s += Db;
        e++;
        uint32_t *ntot = &L.ntot[e & 1u];
        const uint32_t lists = ring_kargs().s.lists;

        // 1. update
        {
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
                    bal[r] = __ballot(ring_neuron(m, V[r], R[r], I, (fire >> r) & 1u) && live);
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
                    for (uint32_t u = 0; u < Db; u++) {
                        const uint32_t sl = ps + u < pslots ? ps + u : ps + u - pslots;
                        const AccT acc = L.ring[sl * W + qc];
                        const uint32_t kq = L.kp[u * W + qc];
                        if (live) L.ring[sl * W + qc] = 0;
                        const float I = ring_input<FIXED, CNT>(m, acc, drive ? kq : 0u, w0, w1, q0, q1);
                        const bool f = ring_neuron(m, V[r], R[r], I, (fire >> (u * nr + r)) & 1u) && live;
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
                }
            }
        }
        // 2. publication (the waves that poll are not those that store)
        if (MULTI || ring_kargs().s.raster_cap) __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        const uint32_t cnt = *ntot;
        if (!MULTI && cnt > kList1) {  // (spikes in the segment: stored before they are read)
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
        }
        if (MULTI && w == kRW - 1) {
            const RingArgs &ra = ring_kargs();
            if (ra.s.raster_cap && Db > 1) {  // each step's count, for the raster positions
                if (lane < Db) st_ag(&ra.cnts[((uint64_t)(e & 1u) * kRunMaxD + lane) * Tn + tile], L.nb[lane]);
                __builtin_amdgcn_s_waitcnt(0);
            }
            if (lane == 0) {
                uint64_t *box = ra.ctl->box[e & 1u] + (uint64_t)tile * kRingBoxStride;
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
        if (MULTI && !ring_kargs().s.row_len) {  // events emitted: the out-degrees of the tile's spikes
            for (uint32_t i = tid; i < cnt; i += kRT) {
                const uint32_t sp = own_spike(i);
                atomicAdd(&L.ev[sp >> kTargetBits], (unsigned long long)ring_kargs().s.outdeg[sp & kTargetMask]);
            }
            __syncthreads();
        }
        if (w == kRW - 2 && lane < Db) {  // the steps' records
            const StepArgs &a = ring_kargs().s;
            const uint64_t g = (t + lane) * kGroups + x;
            const uint32_t ns = Db == 1 ? cnt : L.nb[lane];
            const unsigned long long ev = MULTI && a.row_len ? (unsigned long long)ns * a.row_len : L.ev[lane];
            if (ns) atomicAdd(&a.counts8[g], ns);
            if (ev) atomicAdd((unsigned long long *)&a.events8[g], ev);
            if (CNT && lists > 1 && L.dlv[lane]) atomicAdd((unsigned long long *)&a.delivered8[g], (unsigned long long)L.dlv[lane]);
            L.dlv[lane] = 0;
            L.ev[lane] = 0;
        }
        if (MULTI && s >= n_steps && ring_kargs().defer) {  // the next launch gathers this batch
            t += Db;
            break;
        }

        // 3. the other tiles, and the next batch's draws
        const uint32_t Dn = (uint32_t)(n_steps - s < D ? n_steps - s : D), units = Dn * nr;
        uint32_t dk = 0, M = cnt, fire_n = 0;
        if constexpr (MULTI) {
            const RingArgs &ra = ring_kargs();
            const ModelArgs &m = ra.s.m;
            const bool poller = w * kWave < Tn;
            const uint32_t ptile = w * kWave + lane;
            const bool mine = poller && ptile < Tn;
            const uint64_t *box = ra.ctl->box[e & 1u] + (uint64_t)(mine ? ptile : 0u) * kRingBoxStride;
            Seen v{(uint64_t)((e ^ 1u) & 0x3ffffu), 0};  // (not this batch's)
            bool ready = false;
            while (!ready && dk < units) {
                if (mine && !box_ready(v.a, v.b, e)) {
                    v.a = ld_ag64(box);
                    v.b = ld_ag64(box + 1);
                }
                ring_draw(m, L, W, tile_lo, tile_n, t + Db, dk++, nr, &fire_n);
                if (poller) {
                    const bool ok = __all(!mine || box_ready(v.a, v.b, e));
                    if (ok) ring_take(L, w, lane, mine, v);
                    if (lane == 0) L.pq[look & 1u][w] = ok ? 1u : 0u;
                }
                __syncthreads();
                ready = true;
                for (uint32_t k = 0; k * kWave < Tn; k++) ready = ready && L.pq[look & 1u][k] != 0;
                look++;  // (pq of this parity is written again two looks later, after a barrier)
            }
            if (!ready) {
                if (poller) {
                    const uint64_t c0 = wall_clock64();
                    bool ok = true;
                    for (uint32_t k = 0;; k++) {
                        if (mine && !box_ready(v.a, v.b, e)) {
                            v.a = ld_ag64(box);
                            v.b = ld_ag64(box + 1);
                        }
                        if (__all(!mine || box_ready(v.a, v.b, e))) break;
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
                    if (ok) ring_take(L, w, lane, mine, v);
                    if (lane == 0) {
                        L.pstop[w] = ok ? 0u : 1u;
                        if (!ok) atomicOr(ra.s.flags, kStopped);
                    }
                }
                __syncthreads();
                uint32_t stop = 0;
                for (uint32_t k = 0; k * kWave < Tn; k++) stop |= L.pstop[k];
                if (stop) return;
            }
            M = 0;
            for (uint32_t k = 0; k * kWave < Tn; k++) M += L.ptot[k];
        }
        if (tid == 0) L.ntot[(e + 1u) & 1u] = 0;  // (last used before the previous batch's barriers)

        // raster: every tile appends its own spikes
        if (ring_kargs().s.raster_cap) {
            const RingArgs &ra = ring_kargs();
            const StepArgs &a = ra.s;
            uint32_t before = 0;
            if (MULTI) {
                before = L.pre[tile];
                for (uint32_t k = 0; k < tile / kWave; k++) before += L.ptot[k];
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
        if (Db > 1 && w == kRW - 2 && lane < Db) L.nb[lane] = 0;  // (read by this wave, and above before a barrier)

        // 4. gather, and the draws that are left
        gather(M, ps);
        {
            const ModelArgs &m = ring_kargs().s.m;
            for (; dk < units; dk++) ring_draw(m, L, W, tile_lo, tile_n, t + Db, dk, nr, &fire_n);
        }
        fire = fire_n;
        t += Db;
        ps = ps + Db < pslots ? ps + Db : ps + Db - pslots;
        lds_sync();  // every event of the batch is in the ring
    }

    const RingArgs &ra = ring_kargs();
    const StepArgs &a = ra.s;
#pragma unroll
    for (int r = 0; r < NR; r++) {
        const uint32_t q = r * kRT + tid;
        if (q < tile_n) {
            a.V[tile_lo + q] = V[r];
            if (a.m.kind != SPK_SOURCE) a.ref[tile_lo + q] = (uint8_t)R[r];
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
    return (uint64_t)a.pslots * tl.W * ring_acc_bytes(a.m.fixed, ra.counts) <= kRingBytes;
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
