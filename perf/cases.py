"""Performance cases of libspk: what a program that simulates spiking networks
has the library do, through the Python binding's public entry points.

A case is a dict of plain values.  ``what`` names the use:

  step     a closed loop: a call of one or a few steps, after which the program
           reads the step's spike counts and the neurons' state
  run      a simulation: many steps in one call on a network that has settled
           into its steady activity, then the per-step records and the state
  build    a network created from its parameters (or an adjacency list), its
           first steps, and what they gave
  deliver  spike transmission alone: a list of spikes in device memory delivered
           through a network's synapses into the caller's buffer

The networks are this repository's workloads and sizes between and around
them: leaky integrate-and-fire neurons with an external Poisson drive that
keeps them active, or Bernoulli sources with a weight per synapse; Bernoulli,
fixed out-degree and fixed in-degree connectivity; one delay or several; fp32
or fixed-point accumulation; stored or procedural synapses.  How steps are
run, how events are delivered and how synapses are stored is left to the
library, as programs do (procedural synapses are asked for).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2102_04681_amd import Net

BERNOULLI, FIXED_OUT, FIXED_IN, EXPLICIT = 0, 1, 2, 3
CONN = {"bernoulli": BERNOULLI, "out": FIXED_OUT, "in": FIXED_IN, "csr": EXPLICIT}
LARGEST_N = 2_000_000
MAX_STEPS = 1 << 20  # per network: many calls on one state


def _case(what, n, conn, deg, steps, delays=(1, 1), rate=0.0, acc="f32", proc=False, raster=False, spikes=0,
          delay=0, **name):
    """n neurons; deg synapses per neuron on average; rate > 0: Bernoulli
    sources of that many Hz, each synapse with its own weight."""
    return dict(name, what=what, n=n, conn=conn, deg=deg, steps=steps, dmin=delays[0], dmax=delays[1], rate=rate,
                acc=acc, proc=proc, raster=raster, spikes=spikes, delay=delay)


def listed():
    return [
        # The smallest call: a program in a loop with its network (an agent, a
        # clamp experiment) steps once and looks at what happened.
        _case("step", 1000, "bernoulli", 20, 1, name="step_1k"),
        # The small network (1,000 neurons, p = 0.02, weights 0.27 / -4.5 mV) over 100 ms with its raster.
        _case("run", 1000, "bernoulli", 20, 1000, raster=True, name="run_1k"),
        # An ordinary model of odd size: 30,011 neurons, fan-out 333, delays 0.1 to 1 ms.
        _case("run", 30_011, "out", 333, 500, (1, 10), name="run_30k_delays"),
        # 250,000 neurons, p = 0.02 (1.25e9 synapses), one delay.
        _case("run", 250_000, "bernoulli", 5000, 500, name="run_250k"),
        # Brunel's shape: 100,000 neurons, in-degree 8,000 + 2,000, delay 1.5 ms.
        _case("run", 100_000, "in", 10_000, 1000, (15, 15), name="run_brunel"),
        # 1e6 Bernoulli sources at 10 Hz, fan-out 1,000, a weight per synapse, dt = 1 ms.
        _case("run", 1_000_000, "out", 1000, 100, rate=10.0, name="run_sources"),
        # A mid-size network of odd size in fixed-point arithmetic with delays of 0.3 to 1.2 ms.
        _case("run", 500_009, "out", 1201, 300, (3, 12), acc="fixed", name="run_500k_fixed"),
        # The largest: 2e6 neurons, fan-out 1,500 (3e9 synapses), delays 0.1 to 2 ms.
        _case("run", 2_000_000, "out", 1500, 400, (1, 20), name="run_3e9"),
        # The same with its synapses generated when they are needed instead of stored.
        _case("run", 2_000_000, "out", 1500, 100, (1, 20), proc=True, name="run_3e9_procedural"),
        # The setup study's network: density 5 %, delay 1 (1.8e8 synapses).
        _case("build", 60_000, "bernoulli", 3000, 10, name="build_synth"),
        # A network of fixed out-degree from its parameters to its first steps (2e8 synapses).
        _case("build", 400_000, "out", 500, 10, (1, 20), name="build_out"),
        # Spike transmission alone: one step's spikes of a 1e6-neuron network through all delays.
        _case("deliver", 1_000_000, "out", 1500, 1, (1, 20), spikes=1000, name="deliver_1m"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["step", "run", "run", "run", "run", "run", "build", "deliver"])
    acc = rng.choice(["f32", "f32", "f32", "fixed"])
    delays = rng.choice([(1, 1), (1, 1), None, None, (15, 15)])
    if delays is None:
        lo = rng.choice([1, 1, 2, 3, 5])
        delays = (lo, lo + rng.randint(1, 19))
    conn = rng.choice(["bernoulli", "out", "out", "in"])
    rate, proc = 0.0, False
    if what == "step":
        n = _log(rng, 300, 20_000)
        deg = min(n // 2, _log(rng, 20, 300))
        return _case("step", n, conn, deg, rng.randint(1, 3), delays, acc=acc)
    top = {"bernoulli": 250_000, "in": 100_000, "out": LARGEST_N}[conn]
    if what == "deliver":
        n = _log(rng, 20_000, min(top, 1_000_000))
        deg = min(n // 4, _log(rng, 100, 1500))
        delay = rng.choice([0, 0, rng.randint(*delays)])
        return _case("deliver", n, conn, deg, 1, delays, acc=acc, spikes=_log(rng, 30, min(n // 4, 4000)), delay=delay)
    if what == "build":
        conn = rng.choice(["bernoulli", "out", "in", "csr"])
        if conn == "csr":
            n = _log(rng, 2000, 50_000)
            return _case("build", n, conn, _log(rng, 20, 200), 10, delays, acc=acc)
        n = _log(rng, 5000, {"bernoulli": 60_000, "in": 60_000, "out": 400_000}[conn])
        deg = max(50, min(n // 20, 500 if conn == "out" else 3000, _log(rng, 100, 3000)))
        return _case("build", n, conn, deg, 10, delays, acc=acc)
    n = _log(rng, 500, top)
    deg = max(20, min(n // 10, 1500 if conn == "out" else 10_000, _log(rng, 50, 10_000)))
    if conn == "out" and rng.random() < 0.35:
        rate = float(rng.choice([1, 5, 10, 20, 50]))
        delays = rng.choice([(1, 1), delays])
        deg = min(deg, 1000)
    elif conn == "out" and rng.random() < 0.25:
        proc = True
    steps = max(20, min(1000, _log(rng, 100, 1000), int(1e-2 / (1.2e-5 + _events(n, deg, rate) / 1e11))))
    return _case("run", n, conn, deg, steps, delays, rate=rate, acc=acc, proc=proc, raster=n <= 3000 and rng.random() < 0.5)


def _events(n, deg, rate):
    """Synaptic events per step: the source rate at dt = 1 ms, or about 10 Hz at 0.1 ms."""
    return n * deg * (rate * 1e-3 if rate else 1e-3)


def _f32(x):
    return float(np.float32(x))


def _params(case, seed):
    n, deg = case["n"], case["deg"]
    sc = min(1.0, 80.0 / deg)
    c = dict(neuron_kind=0, frac_exc=0.8, dt_ms=0.1, tau_m_ms=20.0, t_ref_ms=5.0, v_rest=-60.0, v_th=-50.0,
             v_reset=-60.0, v0_lo=-60.0, v0_hi=-50.0, i_bias=0.0, p=0.0, k_out=0, k_in_exc=0, k_in_inh=0, w_uniform=0,
             w_lo=0.0, w_hi=0.0, w_exc=_f32(0.27 * sc), w_inh=_f32(-4.5 * sc), delay_min=case["dmin"],
             delay_max=case["dmax"], src_rate_hz=0.0, acc_mode=1 if case["acc"] == "fixed" else 0, fixed_shift=20,
             n=n, seed=int(seed), conn_kind=CONN[case["conn"]])
    if case["conn"] == "bernoulli":
        c["p"] = deg / n
    elif case["conn"] == "out":
        c["k_out"] = deg
    elif case["conn"] == "in":
        c.update(k_in_exc=deg - deg // 5, k_in_inh=deg // 5, w_exc=_f32(0.1), w_inh=_f32(-0.5))
    if case["rate"]:
        c.update(neuron_kind=1, frac_exc=1.0, dt_ms=1.0, w_uniform=1, w_lo=0.0, w_hi=_f32(1e-3), w_exc=0.0, w_inh=0.0,
                 src_rate_hz=case["rate"])
    else:  # the external drive, at twice the rate that would hold V at threshold
        c["ext_lambda"] = 2.0 * 10.0 * (0.1 / 20.0) / c["w_exc"]
        c["ext_w"] = c["w_exc"]
    if case["proc"]:
        c["syn_format"] = 3
    return c


def _csr(case, seed):
    """An adjacency list as a program holds it: Poisson out-degrees, targets in
    no order, two weights by population."""
    rng = np.random.default_rng(seed)
    n, c = case["n"], _params(case, seed)
    deg = rng.poisson(case["deg"], n)
    ptr = np.zeros(n + 1, np.uint64)
    ptr[1:] = np.cumsum(deg)
    m = int(ptr[-1])
    w = np.repeat(np.where(np.arange(n) < round(0.8 * n), c["w_exc"], c["w_inh"]).astype(np.float32), deg)
    return ptr, rng.integers(0, n, m, dtype=np.uint32), w, rng.integers(case["dmin"], case["dmax"] + 1, m).astype(np.uint8)


_stream = None


def _the_stream():
    """One stream for every network: calls of spk_deliver_noalloc on one device are ordered by their caller."""
    global _stream
    if _stream is None:
        _stream = torch.cuda.Stream()
    return _stream


def _settle(case):
    """Steps to the steady state: 30 ms and twice the longest delay."""
    return max(2 * case["dmax"], 30 if case["rate"] else 300)


def prepare(case, seed):
    cfg, stream = _params(case, seed), _the_stream()
    st = {"case": case, "cfg": cfg, "stream": stream}
    if case["what"] == "build":
        if case["conn"] == "csr":
            st["csr"] = _csr(case, seed)
        return st
    steps = 1 if case["what"] == "deliver" else MAX_STEPS
    net = st["net"] = Net(cfg, stream=stream, max_steps=steps, raster_capacity=(1 << 25) if case["raster"] else 0)
    if case["what"] == "deliver":
        st["spikes"] = _spikes(case, seed).to(torch.int32).cuda()
        st["out"] = torch.zeros(case["n"], dtype=torch.int32 if case["acc"] == "fixed" else torch.float32, device="cuda")
        torch.cuda.synchronize()
    else:
        net.step(_settle(case))
        net.sync()
        st["t"] = _settle(case)
    return st


def _spikes(case, seed):
    g = torch.Generator().manual_seed(int(seed))
    return torch.randperm(case["n"], generator=g)[:case["spikes"]]


def _records(net, t0, steps):
    v, ref = net.state()
    return {"counts": net.spike_counts(t0, steps).astype(np.int64), "events": net.events(t0, steps).astype(np.int64),
            "delivered": net.delivered(t0, steps).astype(np.int64), "v": v, "ref": ref}


def run(state):
    case = state["case"]
    what, steps = case["what"], case["steps"]
    if what == "deliver":
        state["net"].deliver_noalloc(state["spikes"].data_ptr(), case["spikes"], state["out"].data_ptr(), case["delay"])
        return state["out"]
    if what == "build":
        net = Net(state["cfg"], stream=state["stream"], max_steps=steps, csr=state.get("csr"))
        net.step(steps)
        out = _records(net, 0, steps)
        out["synapses"] = net.stats()["nnz"]
        net.close()
        return out
    net, t0 = state["net"], state["t"]
    net.step(steps)
    state["t"] = t0 + steps
    if what == "step":
        v, ref = net.state()
        return {"counts": net.spike_counts(t0, steps).astype(np.int64), "v": v, "ref": ref}
    out = _records(net, t0, steps)
    if case["raster"]:
        offsets, ids = net.raster(t0, steps)
        out["offsets"], out["ids"] = offsets.astype(np.int64), np.zeros(steps * (case["n"] // 32 + 8), np.int32)
        m = min(len(ids), len(out["ids"]))
        out["ids"][:m] = ids[:m]
    return out


def work(case):
    """Bytes: every fired row read once (4 bytes per synapse with one weight
    per population, 8 with a weight per synapse, none where synapses are
    generated), the neurons' state read and written once per call, and spike
    IDs.  Operations: one addition per event, six per neuron update; a build
    draws each synapse, or each ordered pair of neurons, once (about ten
    integer operations per draw) and writes the synapses."""
    n, deg, steps = case["n"], case["deg"], case["steps"]
    rec = 0 if case["proc"] else 8 if case["rate"] else 4
    ev = case["spikes"] * deg if case["what"] == "deliver" else _events(n, deg, case["rate"]) * steps
    b, f = ev * rec + 10.0 * n + 4.0 * ev / deg, ev + 6.0 * n * steps
    if case["what"] == "deliver":
        b, f = ev * rec + 4.0 * n + 4.0 * case["spikes"], float(ev)
    if case["what"] == "build":
        nnz = float(n) * deg
        b += nnz * rec + (13.0 * nnz if case["conn"] == "csr" else 0.0)
        f += 10.0 * (float(n) * n if case["conn"] == "bernoulli" else nnz)
    if case["proc"]:
        f += 20.0 * ev
    return {"bytes": b, "flops": f}


def tolerance(case):
    """Sums are exact integers rounded once and every fp32 operation of the
    neuron update is rounded on its own, in one stated order: spike trains,
    records and state are the same bits whatever the implementation."""
    return "exact"


# ------------------------------------------------------------- 64-bit values
# The network's definition in plain torch: SplitMix64-based counter hash, rows
# drawn again for the neurons that fire, float64 state and sums.

_TAG = dict(conn=1, tgt=2, src_e=3, src_i=4, w=5, delay=6, v0=7, pois=8, bern=9)


def _s64(x):
    x &= (1 << 64) - 1
    return x - (1 << 64) if x >> 63 else x


def _shr(z, k):
    return (z >> k) & ((1 << (64 - k)) - 1)


def _mix(z):
    z = z + _s64(0x9E3779B97F4A7C15)
    z = (z ^ _shr(z, 30)) * _s64(0xBF58476D1CE4E5B9)
    z = (z ^ _shr(z, 27)) * _s64(0x94D049BB133111EB)
    return z ^ _shr(z, 31)


class _Network:
    def __init__(self, case, seed):
        self.case, self.c = case, _params(case, seed)
        self.dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
        s = torch.tensor(_s64(int(seed)), dtype=torch.int64)
        self.key = {k: int(_mix(_mix(s) ^ t)) for k, t in _TAG.items()}
        self.n, self.n_exc = case["n"], int(math.floor(self.c["frac_exc"] * case["n"] + 0.5))
        self.lists = case["dmax"] - case["dmin"] + 1

    def prefix(self, tag, a):
        return _mix(a ^ self.key[tag])

    def _range(self, h, m):
        return (_shr(h, 32) * m) >> 32

    def rows(self, src):
        """Every synapse of the given neurons, in parts: (target, delay, weight)."""
        c, n, dev = self.c, self.n, self.dev
        conn = c["conn_kind"]

        def finish(s, tgt, a, b):
            j = self._range(_mix(self.prefix("delay", a) ^ b), self.lists) if self.lists > 1 else torch.zeros_like(tgt)
            if c["w_uniform"]:
                u = _shr(_mix(self.prefix("w", a) ^ b), 40).to(torch.float32) * (1.0 / 16777216.0)
                w = (u * np.float32(c["w_hi"] - c["w_lo"]).item() + c["w_lo"])
            else:
                w = torch.where(s < self.n_exc, c["w_exc"], c["w_inh"]).to(torch.float32)
            if c["acc_mode"] == 1:
                w = torch.round(w * 2.0 ** c["fixed_shift"]).double() * 2.0 ** -c["fixed_shift"]
            return tgt, j + c["delay_min"], w.double()

        if conn == FIXED_OUT:
            part = max(1, 20_000_000 // c["k_out"])
            for k in range(0, len(src), part):
                s = src[k:k + part].repeat_interleave(c["k_out"])
                j = torch.arange(c["k_out"], device=dev).repeat(len(src[k:k + part]))
                yield finish(s, self._range(_mix(self.prefix("tgt", s) ^ j), n), s, j)
        elif conn == BERNOULLI:
            thr, part, t = int(math.floor(c["p"] * 4294967296.0)), max(1, 20_000_000 // n), torch.arange(n, device=dev)
            for k in range(0, len(src), part):
                s0 = src[k:k + part]
                hit = (_shr(_mix(self.prefix("conn", s0)[:, None] ^ t[None, :]), 32) < thr).nonzero()
                s, tgt = s0[hit[:, 0]], hit[:, 1]
                yield finish(s, tgt, s, tgt)
        else:
            ke, ki = c["k_in_exc"], c["k_in_inh"]
            fired = torch.zeros(n, dtype=torch.bool, device=dev)
            fired[src] = True
            part = max(1, 20_000_000 // (ke + ki))
            for t0 in range(0, n, part):
                t = torch.arange(t0, min(n, t0 + part), device=dev)
                e = self._range(_mix(self.prefix("src_e", t)[:, None] ^ torch.arange(ke, device=dev)[None, :]), self.n_exc)
                i = self._range(_mix(self.prefix("src_i", t)[:, None] ^ torch.arange(ki, device=dev)[None, :]), n - self.n_exc)
                s = torch.cat([e, i + self.n_exc], 1)
                hit = fired[s].nonzero()
                yield finish(s[hit[:, 0], hit[:, 1]], hit[:, 0] + t0, hit[:, 0] + t0, hit[:, 1])

    def simulate(self, steps):
        """V after the given steps from t = 0, and how close a neuron that
        could fire came to its threshold."""
        c, n, dev, dmax = self.c, self.n, self.dev, self.case["dmax"]
        ids = torch.arange(n, device=dev)
        V = c["v0_lo"] + (c["v0_hi"] - c["v0_lo"]) * (_shr(_mix(self.prefix("v0", ids)), 40).double() / 16777216.0)
        ref = torch.zeros(n, dtype=torch.int64, device=dev)
        k = _f32(c["dt_ms"] / c["tau_m_ms"])
        ext_w = c.get("ext_w", 0.0)
        if c["acc_mode"] == 1:
            ext_w = float(np.rint(ext_w * 2.0 ** c["fixed_shift"])) * 2.0 ** -c["fixed_shift"]
        thr = []
        if c.get("ext_lambda"):
            pk = cdf = math.exp(-c["ext_lambda"])
            while math.floor(cdf * 4294967296.0) < 4294967295.0:
                thr.append(math.floor(cdf * 4294967296.0))
                pk = pk * c["ext_lambda"] / len(thr)
                cdf += pk
        thr = torch.tensor(thr, dtype=torch.int64, device=dev)
        src_thr = math.floor(c["src_rate_hz"] * c["dt_ms"] * 1e-3 * 4294967296.0)
        ring = torch.zeros(dmax + 1, n, dtype=torch.float64, device=dev)
        ref_steps = int(round(c["t_ref_ms"] / c["dt_ms"]))
        near = math.inf
        for t in range(steps):
            slot = t % (dmax + 1)
            I = ring[slot].clone()
            ring[slot] = 0
            ctr = ids | (t << 32)
            if len(thr):
                I = I + torch.searchsorted(thr, _shr(_mix(ctr ^ self.key["pois"]), 32), right=True) * ext_w
            vn = V + k * (c["v_rest"] - V) + I
            if c["neuron_kind"] == 1:
                V = vn
                fire = _shr(_mix(ctr ^ self.key["bern"]), 32) < src_thr
            else:
                held = ref > 0
                fire = ~held & (vn >= c["v_th"])
                near = min(near, float(torch.where(held, math.inf, (vn - c["v_th"]).abs()).min()))
                V = torch.where(held | fire, c["v_reset"], vn)
                ref = torch.where(held, ref - 1, torch.where(fire, ref_steps, 0))
            for tgt, d, w in self.rows(fire.nonzero()[:, 0]):
                ring.view(-1).index_add_(0, ((t + d) % (dmax + 1)) * n + tgt, w)
        return V, near


def exact(case, seed):
    """Delivered sums, and the state of networks whose V has a value in 64
    bits: sources (no threshold) at any length, and the first steps of a
    build where no neuron came so near its threshold that fp32 rounding
    decides (10 steps of up to two roundings of 4e-6 at 50 mV, which partly
    cancel).  The V of a network of firing neurons after hundreds of steps
    has none: one rounding moves a spike, and the spike trains part."""
    if case["conn"] == "csr":
        return None
    net = _Network(case, seed)
    if case["what"] == "deliver":
        out = torch.zeros(case["n"], dtype=torch.float64, device=net.dev)
        for tgt, d, w in net.rows(_spikes(case, seed).to(net.dev)):
            keep = (d == case["delay"]) if case["delay"] else torch.ones_like(d, dtype=torch.bool)
            out.index_add_(0, tgt[keep], w[keep])
        return out if case["acc"] == "f32" else None
    if case["what"] == "build":
        steps = case["steps"]
    elif case["what"] == "run" and case["rate"]:
        steps = _settle(case) + case["steps"]
    else:
        return None
    ev = _events(case["n"], case["deg"], case["rate"]) * steps
    if case["conn"] == "in":
        ev = float(case["n"]) * case["deg"] * steps
    elif case["conn"] == "bernoulli":
        ev = ev / case["deg"] * case["n"] * 10  # (a start fires about ten times the steady rate)
    if ev > 2e10:
        return None
    V, near = net.simulate(steps)
    if near < 2e-5:
        return None
    return {"counts": None, "events": None, "delivered": None, "v": V.cpu().numpy(), "ref": None, "synapses": None}
