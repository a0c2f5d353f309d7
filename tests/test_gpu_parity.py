"""GPU parity: libspk (HIP, through the C ABI) against the CPU oracle.

Bar (per the method's two accumulation modes):
  - connectivity: every row identical (targets, delays, weight bits);
  - delivery of a given spike set: exact in fixed-point mode; in fp32 mode
    |I_gpu - I_ref| <= 1e-5 * max(|I_ref|, sum |w|) per target, I_ref summed
    in double (the bar for any fp32 summation order), and in addition
    within one fp32 ulp of I_ref, since the library sums exactly and rounds
    once;
  - whole simulation in fixed-point mode: bit-identical rasters, counts,
    events, delivered events and final state, for both delivery strategies
    and for every way of running the steps (graph replay, plain launches,
    the persistent kernel);
  - the persistent kernel and the graph path: bit-identical in fp32 mode
    too (both sum exactly and round once);
  - fp32 mode: mean firing rate within 1 % (the oracle adds fp32 inputs one
    by one in push order, the library rounds the exact sum once, so spike
    trains diverge chaotically after the first difference).
Both synapse formats (8-byte full records, 4-byte compact records with a
weight class) are held to the same bar.
Sizes span several tiles, many delay lists, ragged row lengths and the bin
overflow path.
"""
import sys

import numpy as np
import pytest

import inputs as I
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def spk():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2102_04681_amd import spk as mod
    mod.lib()
    return mod


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


_ORACLE_NETS = {}
_ORACLE_RUNS = {}


def _key(cfg):
    return tuple(sorted((k, v) for k, v in cfg.items() if k not in ("delivery", "syn_format", "step_mode")))


def _oracle_net(cfg):
    """Oracle network for cfg (delivery strategy and synapse format do not change it)."""
    k = _key(cfg)
    if k not in _ORACLE_NETS:
        _ORACLE_NETS.clear()
        _ORACLE_NETS[k] = oracle.Net(cfg)
    return _ORACLE_NETS[k]


def _oracle_run(cfg, T):
    """(run record, final V, final ref, csr) of a fresh oracle network."""
    k = (_key(cfg), T)
    if k not in _ORACLE_RUNS:
        _ORACLE_RUNS.clear()
        o = oracle.Net(cfg)
        r = o.run(T)
        v, ref = o.state()
        _ORACLE_RUNS[k] = (r, v, ref, o.csr())
    return _ORACLE_RUNS[k]


def _canon(col, d, wbits):
    """Row-local canonical order key (target, delay, weight bits)."""
    return np.lexsort((wbits, d, col))


def _compare_rows(g_offs, g_col, g_w, g_d, o_rp, o_col, o_w, o_d, rows, fixed, shift=20):
    for k, s in enumerate(rows):
        a, b = int(g_offs[k]), int(g_offs[k + 1])
        oa, ob = int(o_rp[s]), int(o_rp[s + 1])
        assert b - a == ob - oa, f"row {s}: length {b - a} vs oracle {ob - oa}"
        gc, gd = g_col[a:b], g_d[a:b]
        oc, od = o_col[oa:ob], o_d[oa:ob]
        if fixed:
            ow = np.rint(o_w[oa:ob].astype(np.float64) * 2.0**shift).astype(np.int32).view(np.uint32)
            gw = g_w[a:b].view(np.uint32)
        else:
            ow = o_w[oa:ob].view(np.uint32)
            gw = g_w[a:b].view(np.uint32)
        gi, oi = _canon(gc, gd, gw), _canon(oc, od, ow)
        assert np.array_equal(gc[gi], oc[oi]), f"row {s}: targets differ"
        assert np.array_equal(gd[gi], od[oi]), f"row {s}: delays differ"
        assert np.array_equal(gw[gi], ow[oi]), f"row {s}: weights differ"


GEN_CASES = [
    ("C0", lambda: I.config(0, seed=1)),
    ("C0s2", lambda: I.config(0, seed=2, driven=True)),
    ("C1-3000", lambda: I.scaled(1, 3000)),
    ("C2-4000", lambda: I.scaled(2, 4000, k_in_exc=300, k_in_inh=75)),
    ("C3-5000", lambda: I.scaled(3, 5000, k_out=300)),
    ("C4-6000", lambda: I.scaled(4, 6000, k_out=400)),
    ("bern-delays", lambda: I.config(0, n=1500, p=0.05, delay_min=2, delay_max=9, seed=4)),
    ("C4-fixed", lambda: I.scaled(4, 4000, k_out=300, acc_mode=I.ACC_FIXED)),
]


FORMATS = [(1, "full"), (0, "auto")]


def _two_pass_rows(spk, cfg):
    """Bernoulli rows of a network that is not drawn in one pass (graph path
    or binned delivery), against the oracle's."""
    for over in (dict(step_mode=1), dict(delivery=2)):
        g = spk.Net(dict(cfg, **over), max_steps=1)
        st = g.stats()
        assert st["step_mode"] == 1 or st["page_cap"] > 0
        o = oracle.Net(cfg)
        o_rp, o_col, o_w, o_d = o.csr()
        assert st["nnz"] == len(o_col)
        offs, col, w, d = g.csr()
        _compare_rows(offs, col, w, d, o_rp, o_col, o_w, o_d, range(cfg["n"]), cfg["acc_mode"] == I.ACC_FIXED)


@pytest.mark.parametrize("keys", ["0", "1"], ids=["drawn-again", "kept"])
@pytest.mark.parametrize("name", ["C0", "C1-3000", "bern-delays"])
def test_generator_two_draws_equals_oracle(spk, name, keys, monkeypatch):
    """Bernoulli rows placed by drawing every row a second time (the path
    taken in small networks and where a row is longer than the first pass can
    keep), and from the synapses that the first pass kept, equal the
    oracle's rows."""
    monkeypatch.setenv("SPK_GEN_KEYS", keys)
    cfg = dict(GEN_CASES)[name]()
    _say(f"[gen two draws] {name} n={cfg['n']}")
    _two_pass_rows(spk, cfg)


def test_generator_without_count_keeping_equals_oracle(spk, monkeypatch):
    """Bernoulli rows placed without the count pass's per-row bucket counts
    (the path taken where they cannot be allocated: SPK_GEN_HIST=0) equal the
    oracle's rows."""
    monkeypatch.setenv("SPK_GEN_HIST", "0")
    _two_pass_rows(spk, I.config(0, n=1500, p=0.05, delay_min=2, delay_max=9, seed=4))


@pytest.mark.parametrize("atomics", ["0", "1"], ids=["lds", "per-synapse"])
def test_fixed_in_generator_several_source_ranges(spk, atomics, monkeypatch):
    """Fixed in-degree rows of a network larger than one LDS source range
    (70,000 neurons: three ranges of 32,768 sources), counted per block in LDS
    or (SPK_GEN_IN_ATOMICS=1) with one global atomic per synapse, equal the
    oracle's rows."""
    monkeypatch.setenv("SPK_GEN_IN_ATOMICS", atomics)
    cfg = I.config(2, n=70_000, k_in_exc=40, k_in_inh=10, seed=5)
    g = spk.Net(cfg, max_steps=1)
    o = oracle.Net(cfg)
    o_rp, o_col, o_w, o_d = o.csr()
    assert g.stats()["nnz"] == len(o_col)
    offs, col, w, d = g.csr()
    _compare_rows(offs, col, w, d, o_rp, o_col, o_w, o_d, range(cfg["n"]), False)


@pytest.mark.parametrize("name,mk", GEN_CASES, ids=[c[0] for c in GEN_CASES])
@pytest.mark.parametrize("fmt", [f for f, _ in FORMATS], ids=[n for _, n in FORMATS])
def test_generator_equals_oracle(spk, name, mk, fmt):
    cfg = mk()
    cfg["syn_format"] = fmt
    _say(f"[gen] {name} n={cfg['n']} format={fmt}")
    g = spk.Net(cfg, max_steps=1)
    o = oracle.Net(cfg)
    o_rp, o_col, o_w, o_d = o.csr()
    st = g.stats()
    # population weights are stored compactly unless the full format is asked for
    assert st["bytes_per_synapse"] == (4.0 if fmt == 0 and not cfg["w_uniform"] else 8.0)
    assert st["nnz"] == len(o_col)
    offs, col, w, d = g.csr()
    fixed = cfg["acc_mode"] == I.ACC_FIXED
    _compare_rows(offs, col, w, d, o_rp, o_col, o_w, o_d, range(cfg["n"]), fixed)
    # out-degree bookkeeping and the maximum run length
    assert st["max_row"] >= 1


def test_fig_adj_delivery(spk):
    fx = I.fig_adj()
    for acc in (I.ACC_F32, I.ACC_FIXED):
      for fmt in (1, 2):
        cfg = I.explicit_params(fx["n"], acc_mode=acc, syn_format=fmt)
        _say(f"[fig_adj] acc={acc} format={fmt}")
        g = spk.Net(cfg, max_steps=1, csr=(fx["row_ptr"], fx["col"], fx["w"], fx["delay"]))
        assert g.stats()["bytes_per_synapse"] == (8.0 if fmt == 1 else 4.0)
        out = g.debug_deliver(fx["spikes"])
        want = np.array(fx["expect_input"], dtype=np.float64)
        if acc == I.ACC_FIXED:
            assert np.array_equal(out.astype(np.int64), (want * 2**20).astype(np.int64))
        else:
            assert np.array_equal(out.astype(np.float64), want)
        offs, col, _, _ = g.export_rows([9])
        assert col.tolist() == fx["expect_row9"]


def _abs_sum(o, spikes, delay):
    """Per target: sum of |w| over contributing synapses, and their number."""
    rp, col, w, d = o.csr()
    s = np.asarray(spikes, dtype=np.int64)
    a, b = rp[s].astype(np.int64), rp[s + 1].astype(np.int64)
    lens = b - a
    # the synapse positions of every spike's row, spikes repeated as given
    idx = np.repeat(a - (np.cumsum(lens) - lens), lens) + np.arange(int(lens.sum()), dtype=np.int64)
    if delay:
        idx = idx[d[idx] == delay]
    out = np.bincount(col[idx], weights=np.abs(w[idx].astype(np.float64)), minlength=o.n)
    cnt = np.bincount(col[idx], minlength=o.n).astype(np.float64)
    return out, cnt


def _fp32_tolerance(want, abs_sum, terms):
    """Tolerance for an fp32 sum of `terms` values added in an arbitrary
    order (atomics): 1e-5 relative to max(|I|, sum|w|), widened to the
    worst-case recursive-summation bound gamma_{m-1} * sum|w|,
    gamma_k = k u / (1 - k u), u = 2^-24, for targets receiving so many
    terms that 1e-5 is below what fp32 guarantees (m > 168)."""
    u = 2.0**-24
    k = np.maximum(terms - 1.0, 0.0)
    gamma = k * u / (1.0 - k * u)
    return np.maximum(1e-5, gamma) * np.maximum(np.abs(want), abs_sum)


def _check_deliver(o, got, spikes, delay, acc):
    """The inputs one delivery of `spikes` leaves (synapses of `delay`, 0 =
    all) against the oracle's: equal in fixed point; in fp32 within 1e-5
    relative (widened where fp32 summation cannot promise it) and within one
    ulp of the double-precision sum, since the library sums exactly and
    rounds once."""
    if acc == I.ACC_FIXED:
        _, want = o.deliver(spikes, delay=delay, fixed=True)
        assert np.array_equal(got.astype(np.int64), want), "fixed-point inputs differ"
        return
    want = o.deliver(spikes, delay=delay)
    abs_sum, terms = _abs_sum(o, spikes, delay)
    tol = _fp32_tolerance(want, abs_sum, terms)
    err = np.abs(got.astype(np.float64) - want)
    scale = np.maximum(np.abs(want), abs_sum) + 1e-30
    assert np.all(err <= tol), f"max rel err {np.max(err / scale)}"
    if terms.max() <= 168:  # the plain 1e-5 relative bar applies
        assert np.all(err <= 1e-5 * scale)
    ulp = np.spacing(np.abs(want).astype(np.float32)).astype(np.float64)
    assert np.all(err <= ulp), f"not the rounded exact sum: {np.max(err / ulp)} ulp"


DELIVER_CASES = [
    ("C0", lambda acc: I.config(0, acc_mode=acc), [0]),
    ("C1-4000", lambda acc: I.scaled(1, 4000, acc_mode=acc), [0]),
    ("C4-8000", lambda acc: I.scaled(4, 8000, k_out=700, acc_mode=acc), [0, 1, 7, 20]),
    ("C3-8000", lambda acc: I.scaled(3, 8000, k_out=1000, acc_mode=acc), [0]),
    ("C2-5000", lambda acc: I.scaled(2, 5000, k_in_exc=400, k_in_inh=100, acc_mode=acc), [0, 15]),
]


DELIVERY = [(0, "auto"), (1, "direct"), (2, "binned")]


@pytest.mark.parametrize("name,mk,delays", DELIVER_CASES, ids=[c[0] for c in DELIVER_CASES])
@pytest.mark.parametrize("acc", [I.ACC_F32, I.ACC_FIXED], ids=["f32", "fixed"])
@pytest.mark.parametrize("delivery", [1, 2], ids=["direct", "binned"])
@pytest.mark.parametrize("fmt", [f for f, _ in FORMATS], ids=[n for _, n in FORMATS])
def test_debug_deliver_matches_oracle(spk, name, mk, delays, acc, delivery, fmt):
    cfg = mk(acc)
    cfg["delivery"] = delivery
    cfg["syn_format"] = fmt
    n = cfg["n"]
    g = spk.Net(cfg, max_steps=1)
    assert g.stats()["delivery"] == delivery
    o = _oracle_net(cfg)
    # spike-set sizes: empty, single, a typical step at ~10-50 Hz (n*r*dt with
    # r*dt ~ 0.005), a third of the network, every neuron, every neuron 3x
    for k, (count, uniq) in enumerate([(0, True), (1, True), (37, True), (max(1, n // 200), True),
                                       (n // 3, True), (n, False), (3 * n, False)]):
        spikes = I.spike_set(n, count, seed=10 + k, unique=uniq)
        for delay in delays:
            _say(f"[deliver] {name} acc={acc} spikes={len(spikes)} delay={delay}")
            _check_deliver(o, g.debug_deliver(spikes, delay=delay), spikes, delay, acc)


def test_debug_deliver_rejects_bad_input(spk):
    g = spk.Net(I.config(0), max_steps=1)
    with pytest.raises(spk.SpkError) as e:
        g.debug_deliver(np.array([5, 1000], dtype=np.uint32))
    assert e.value.code == spk.SPK_EINVAL
    with pytest.raises(spk.SpkError):
        g.debug_deliver(np.array([5], dtype=np.uint32), delay=2)


RUN_CASES = [
    ("C0-driven", lambda: I.config(0, driven=True, seed=1), 1000),
    ("C0-driven-s3", lambda: I.config(0, driven=True, seed=3), 400),
    ("C1-6000", lambda: I.scaled(1, 6000), 300),
    ("C2-6000", lambda: I.scaled(2, 6000, k_in_exc=480, k_in_inh=120), 300),
    ("C3-20000", lambda: I.scaled(3, 20000, k_out=1000), 100),
    ("C3-d4-6", lambda: I.scaled(3, 20000, k_out=1000, delay_min=4, delay_max=6), 100),
    ("C4-12000", lambda: I.scaled(4, 12000, k_out=1500), 400),
    ("C4-d3-9", lambda: I.scaled(4, 12000, k_out=1500, delay_min=3, delay_max=9), 300),
    ("C0-literal", lambda: I.config(0, seed=1), 200),
]


# how the steps run: graph replay, plain launches with events (profiling),
# the persistent kernel as chosen (binned delivery with a smallest delay >= 2:
# batches of up to 8 steps), the same with events around it, and the
# persistent kernel with batches capped at 1, 4 and 16 steps (SPK_BATCH_STEPS)
MODES = [("graph", 1, False, None), ("launch", 1, True, None), ("persist", 2, False, None),
         ("persist-prof", 2, True, None), ("persist-batch1", 2, False, "1"),
         ("persist-batch4", 2, False, "4"), ("persist-batch16", 2, False, "16"),
         # direct delivery in the persistent kernel that reads the due rows,
         # which the resident kernel else stands in for (SPK_RING=0)
         ("persist-rows", 2, False, None)]


def _expected_batch(cfg, batch):
    return min(cfg["delay_min"], int(batch) if batch else 8)


def _general_tile_width(n):
    """Neurons per tile outside the resident kernel (up to 256 tiles, at least 64 neurons)."""
    w = 64
    while -(-n // (8 * w)) > 32:
        w *= 2
    return w


def _persistent_applies(cfg, delivery):
    """Shapes the persistent kernel takes: direct delivery with one delay,
    or binned delivery (the test shapes are all small enough)."""
    return delivery == 2 or cfg["delay_min"] == cfg["delay_max"]


@pytest.mark.parametrize("name,mk,T", RUN_CASES, ids=[c[0] for c in RUN_CASES])
@pytest.mark.parametrize("delivery", [1, 2], ids=["direct", "binned"])
@pytest.mark.parametrize("mode,step_mode,profiled,batch", MODES, ids=[m[0] for m in MODES])
@pytest.mark.parametrize("fmt", [f for f, _ in FORMATS], ids=[n for _, n in FORMATS])
def test_fixed_point_simulation_bit_identical(spk, name, mk, T, delivery, mode, step_mode, profiled, batch,
                                              fmt, monkeypatch):
    cfg = mk()
    cfg["acc_mode"] = I.ACC_FIXED
    cfg["delivery"] = delivery
    cfg["syn_format"] = fmt
    cfg["step_mode"] = step_mode
    if profiled and name not in ("C0-driven", "C4-12000"):
        pytest.skip("profiled paths checked on two shapes")
    if step_mode == 2 and not _persistent_applies(cfg, delivery):
        pytest.skip("the persistent kernel takes direct delivery with one delay only")
    if batch and (delivery == 1 or cfg["delay_min"] < 2):
        pytest.skip("steps are batched only with binned delivery and a smallest delay >= 2")
    if batch:
        monkeypatch.setenv("SPK_BATCH_STEPS", batch)
    if mode == "persist-rows":
        if delivery == 2:
            pytest.skip("binned delivery does not take the resident kernel")
        monkeypatch.setenv("SPK_RING", "0")
    _say(f"[run] {name} n={cfg['n']} T={T} delivery={delivery} mode={mode} format={fmt}")
    g = spk.Net(cfg, max_steps=T, raster_capacity=cfg["n"] * T)
    st = g.stats()
    assert st["step_mode"] == step_mode
    if mode == "persist-rows":
        assert st["tile_width"] == _general_tile_width(cfg["n"])
    persist_binned = step_mode == 2 and delivery == 2
    assert st["batch_steps"] == (_expected_batch(cfg, batch) if persist_binned else 1)
    g.set_profiling(profiled)
    g.step(T)
    offs, ids = g.raster()
    r, ov, orf, (rp, col, w, d) = _oracle_run(cfg, T)
    assert np.array_equal(g.spike_counts(), r["counts"]), "spike counts differ"
    assert np.array_equal(offs, r["offs"])
    assert np.array_equal(ids, r["raster"]), "rasters differ"
    assert np.array_equal(g.events(), r["events"]), "event counts differ"
    gv, gr = g.state()
    assert np.array_equal(gv.view(np.uint32), ov.view(np.uint32)), "membrane potentials differ"
    assert np.array_equal(gr, orf)
    if name != "C0-literal":
        assert r["counts"].sum() > 0
    else:
        assert r["counts"].sum() == 0
    # delivered events: every spike emitted at t arrives at t + d
    dl = g.delivered()
    want = np.zeros(T, np.uint64)
    for t in range(T):
        for s in r["raster"][int(r["offs"][t]):int(r["offs"][t + 1])]:
            dd = d[int(rp[s]):int(rp[s + 1])].astype(np.int64) + t
            np.add.at(want, dd[dd < T], 1)
    assert np.array_equal(dl, want), "delivered-event counts differ"
    if profiled:
        km = g.kernel_ms()
        assert km["steps"] == T
        if step_mode == 2:
            assert km["run_launches"] == 1 and km["run_ms"] > 0 and km["tile_ms"] == 0
        else:
            assert km["tile_ms"] > 0 and km["run_launches"] == 0


# long pages in the persistent kernel's one-step drain, which loads the
# first part of every page before the fill counts are known and the rest
# through its chunk tables: 16,384 Bernoulli sources firing with
# probability 0.5 per step (256 tiles), fan-out 800, delays 1-4, one weight
# (compact records) or full records: ~800 records per page and step, within
# the page capacity, and two sorting windows per push block; fixed point,
# bit-identical to the oracle
@pytest.mark.parametrize("fmt", [f for f, _ in FORMATS], ids=[n for _, n in FORMATS])
def test_long_pages_one_step_drain_bit_identical(spk, fmt):
    cfg = I.scaled(3, 16384, rate_hz=500.0, k_out=800, delay_min=1, delay_max=4, w_uniform=0, w_exc=1e-3)
    cfg["acc_mode"] = I.ACC_FIXED
    cfg["delivery"] = 2
    cfg["syn_format"] = fmt
    cfg["step_mode"] = 2
    T = 40
    _say(f"[long pages] n={cfg['n']} T={T} format={fmt}")
    g = spk.Net(cfg, max_steps=T, raster_capacity=cfg["n"] * T)
    st = g.stats()
    assert st["step_mode"] == 2 and st["batch_steps"] == 1 and st["delivery"] == 2
    if fmt == 0:
        assert st["bytes_per_synapse"] == 4.0  # compact records
    g.step(T)
    offs, ids = g.raster()
    r, ov, orf, _ = _oracle_run(cfg, T)
    # records per page and step once every delay contributes: a step's events
    # over the tiles and the push blocks of each group (32 on MI355X)
    per_page = float(np.mean(r["events"][8:])) / (st["tiles"] * 32)
    assert 600 < per_page and 1.2 * per_page < st["page_cap"], (per_page, st["page_cap"])
    assert np.array_equal(g.spike_counts(), r["counts"]), "spike counts differ"
    assert np.array_equal(offs, r["offs"]) and np.array_equal(ids, r["raster"]), "rasters differ"
    assert np.array_equal(g.events(), r["events"]), "event counts differ"
    assert np.array_equal(g.delivered(), r["delivered"]), "delivered-event counts differ"
    gv, gr = g.state()
    assert np.array_equal(gv.view(np.uint32), ov.view(np.uint32)), "membrane potentials differ"
    assert np.array_equal(gr, orf)


# degenerate shapes: a single neuron with its autapse, two neurons fully
# connected, a network with no synapse at all (nnz = 0), one partial tile
# (n = 37 < the smallest tile), every pair connected, in-degree 1, and 64
# delay lists (pages for 64 arrival slots)
DEGENERATE = [
    ("one-neuron", lambda: I.config(0, n=1, p=1.0, driven=True, v0_lo=-50.5, v0_hi=-50.1), 300),
    ("two-neurons", lambda: I.config(0, n=2, p=1.0, driven=True, v0_lo=-50.5, v0_hi=-50.1), 300),
    ("no-synapses", lambda: I.config(0, n=500, p=0.0, driven=True), 100),
    ("partial-tile", lambda: I.scaled(4, 37, k_out=5), 100),
    ("all-pairs", lambda: I.config(0, n=200, p=1.0, driven=True, w_exc=0.05, w_inh=-0.2), 100),
    ("in-degree-1", lambda: I.scaled(2, 300, k_in_exc=1, k_in_inh=0), 100),
    ("64-delays", lambda: I.scaled(4, 3000, k_out=300, delay_min=1, delay_max=64), 100),
]


@pytest.mark.parametrize("name,mk,T", DEGENERATE, ids=[c[0] for c in DEGENERATE])
@pytest.mark.parametrize("delivery", [1, 2], ids=["direct", "binned"])
@pytest.mark.parametrize("step_mode,ring", [(1, None), (2, None), (2, "0")], ids=["graph", "persist", "persist-rows"])
def test_degenerate_networks_bit_identical(spk, name, mk, T, delivery, step_mode, ring, monkeypatch):
    cfg = mk()
    if ring:
        if delivery == 2:
            pytest.skip("binned delivery does not take the resident kernel")
        monkeypatch.setenv("SPK_RING", ring)
    cfg["acc_mode"] = I.ACC_FIXED
    cfg["delivery"] = delivery
    cfg["step_mode"] = step_mode
    if step_mode == 2 and not _persistent_applies(cfg, delivery):
        pytest.skip("the persistent kernel takes direct delivery with one delay only")
    _say(f"[degenerate] {name} n={cfg['n']} T={T} delivery={delivery} step_mode={step_mode}")
    g = spk.Net(cfg, max_steps=T, raster_capacity=max(1, cfg["n"] * T))
    assert g.stats()["step_mode"] == step_mode
    g.step(T)
    offs, ids = g.raster()
    r, ov, orf, (rp, col, w, d) = _oracle_run(cfg, T)
    assert int(g.stats()["nnz"]) == int(rp[-1])
    assert r["counts"].sum() > 0
    assert np.array_equal(g.spike_counts(), r["counts"]), "spike counts differ"
    assert np.array_equal(offs, r["offs"]) and np.array_equal(ids, r["raster"]), "rasters differ"
    assert np.array_equal(g.events(), r["events"]), "event counts differ"
    assert np.array_equal(g.delivered(), r["delivered"]), "delivered-event counts differ"
    gv, gr = g.state()
    assert np.array_equal(gv.view(np.uint32), ov.view(np.uint32)), "membrane potentials differ"
    assert np.array_equal(gr, orf)


# a sweep over seeded random shapes (tests/inputs.random_shape): sizes,
# connectivity kinds, delays and formats the fixed cases do not hit
RANDOM_SEEDS = list(range(1, 25))


@pytest.mark.parametrize("seed", RANDOM_SEEDS)
def test_random_shapes_bit_identical(spk, seed, monkeypatch):
    base = I.random_shape(seed)
    base["acc_mode"] = I.ACC_FIXED
    base["syn_format"] = FORMATS[seed % len(FORMATS)][0]
    T = 150
    r, ov, orf, _ = _oracle_run(base, T)
    assert r["counts"].sum() > 0
    # (delivery, step mode, SPK_RING): pages, the due rows, and AUTO (the resident kernel)
    runs = [(2, 1, None), (2, 2, None), (0, 2, None)]
    if base["delay_min"] == base["delay_max"]:
        runs += [(1, 1, None), (1, 2, None), (1, 2, "0")]
    for delivery, step_mode, ring in runs:
        if ring:
            monkeypatch.setenv("SPK_RING", ring)
        cfg = dict(base, delivery=delivery, step_mode=step_mode)
        _say(f"[random] seed={seed} n={cfg['n']} kind={cfg['conn_kind']} delays={cfg['delay_min']}-"
             f"{cfg['delay_max']} format={cfg['syn_format']} delivery={delivery} step_mode={step_mode}")
        g = spk.Net(cfg, max_steps=T, raster_capacity=cfg["n"] * T)
        assert g.stats()["step_mode"] == step_mode
        g.step(T // 3)
        g.step(T - T // 3)  # (across two calls)
        offs, ids = g.raster()
        assert np.array_equal(g.spike_counts(), r["counts"]), "spike counts differ"
        assert np.array_equal(offs, r["offs"]) and np.array_equal(ids, r["raster"]), "rasters differ"
        assert np.array_equal(g.events(), r["events"]) and np.array_equal(g.delivered(), r["delivered"])
        gv, gr = g.state()
        assert np.array_equal(gv.view(np.uint32), ov.view(np.uint32)) and np.array_equal(gr, orf)
        g.close()


@pytest.mark.parametrize("seed", RANDOM_SEEDS)
@pytest.mark.parametrize("acc", [I.ACC_F32, I.ACC_FIXED], ids=["f32", "fixed"])
def test_random_shapes_deliver_matches_oracle(spk, seed, acc):
    # one delivery of a given spike set on random shapes (both deliveries,
    # the shape's format, the smallest, largest and a middle delay and all
    # delays at once): the inputs equal the oracle's to the bar above
    base = dict(I.random_shape(seed), acc_mode=acc)
    base["syn_format"] = FORMATS[seed % len(FORMATS)][0]
    n, d0, d1 = base["n"], base["delay_min"], base["delay_max"]
    o = _oracle_net(base)
    delays = sorted({0, d0, (d0 + d1) // 2, d1})
    for delivery in (1, 2):
        g = spk.Net(dict(base, delivery=delivery), max_steps=1)
        for k, count in enumerate([1, max(1, n // 100), n // 3]):
            spikes = I.spike_set(n, count, seed=100 * seed + k)
            for delay in delays:
                _say(f"[random deliver] seed={seed} n={n} kind={base['conn_kind']} delays={d0}-{d1} "
                     f"format={base['syn_format']} delivery={delivery} spikes={len(spikes)} delay={delay}")
                _check_deliver(o, g.debug_deliver(spikes, delay=delay), spikes, delay, acc)
        g.close()


@pytest.mark.parametrize("seed", RANDOM_SEEDS[:12])
def test_random_procedural_shapes_bit_identical(spk, seed, monkeypatch):
    # procedural synapses on random fixed out-degree shapes (both push
    # kernels): fixed-point runs bit-identical to the oracle
    base = I.random_shape(seed)
    base.update(conn_kind=I.FIXED_OUT, k_out=int(min(base["n"], 50 + 37 * seed)), p=0.0, k_in_exc=0,
                k_in_inh=0, acc_mode=I.ACC_FIXED, syn_format=3)
    sc = min(1.0, 80.0 / base["k_out"])
    base["w_exc"], base["w_inh"] = I._f32(0.27 * sc), I._f32(-4.5 * sc)
    base["ext_w"] = base["w_exc"]
    base["ext_lambda"] = I.drive_lambda(base)
    T = 120
    r, ov, orf, _ = _oracle_run(base, T)
    assert r["counts"].sum() > 0
    for once in ("1", "0"):
        monkeypatch.setenv("SPK_PROC_ONCE", once)
        _say(f"[random proc] seed={seed} n={base['n']} k_out={base['k_out']} delays={base['delay_min']}-"
             f"{base['delay_max']} once={once}")
        g = spk.Net(base, max_steps=T, raster_capacity=base["n"] * T)
        g.step(T // 2)
        g.step(T - T // 2)
        offs, ids = g.raster()
        assert np.array_equal(g.spike_counts(), r["counts"]) and np.array_equal(ids, r["raster"]), once
        assert np.array_equal(g.events(), r["events"]) and np.array_equal(g.delivered(), r["delivered"])
        gv, gr = g.state()
        assert np.array_equal(gv.view(np.uint32), ov.view(np.uint32)) and np.array_equal(gr, orf)
        g.close()


@pytest.mark.parametrize("seed", RANDOM_SEEDS[:12])
def test_random_shapes_fp32_persistent_equals_graph(spk, seed):
    # fp32 mode: exact sums, so the two step modes agree bit for bit
    base = I.random_shape(seed)
    base["syn_format"] = FORMATS[seed % len(FORMATS)][0]
    T = 150
    out = []
    for step_mode in (1, 2):
        g = spk.Net(dict(base, delivery=2, step_mode=step_mode), max_steps=T)
        g.step(T)
        v, ref = g.state()
        out.append((g.spike_counts(), g.events(), v.view(np.uint32), ref))
        g.close()
    assert out[0][0].sum() > 0
    for a_, b_ in zip(out[0], out[1]):
        assert np.array_equal(a_, b_)


@pytest.mark.parametrize("acc", [I.ACC_F32, I.ACC_FIXED], ids=["f32", "fixed"])
@pytest.mark.parametrize("fmt", [f for f, _ in FORMATS], ids=[n for _, n in FORMATS])
@pytest.mark.parametrize("step_mode", [1, 2], ids=["graph", "persist"])
@pytest.mark.parametrize("delays", [(1, 1), (2, 4)], ids=["d1", "d2-4"])
def test_bin_overflow_fallback(spk, acc, fmt, step_mode, delays, monkeypatch):
    # 64 neurons, 200 synapses each (multapses), all above threshold at t=0:
    # the one tile receives 12 800 events (delay 1; with delays 2-4, spread
    # over three arrival steps of batches of 2), ~400 per push block, while
    # every page is capped at 64 records, so the global-atomic fallback must
    # deliver the rest (in the simulation and in debug_deliver).
    monkeypatch.setenv("SPK_PAGE_CAP", "64")
    cfg = I.config(4, n=64, k_out=200, delay_min=delays[0], delay_max=delays[1], v0_lo=-49.0, v0_hi=-49.0,
                   t_ref_ms=0.0, acc_mode=acc, delivery=2, syn_format=fmt, step_mode=step_mode)
    T = 9
    g = spk.Net(cfg, max_steps=T, raster_capacity=64 * T)
    st = g.stats()
    assert st["page_cap"] == 64
    if step_mode == 2:
        assert st["batch_steps"] == delays[0]
    spikes = np.arange(64, dtype=np.uint32)
    got = g.debug_deliver(spikes)
    o = oracle.Net(cfg)
    if acc == I.ACC_FIXED:
        assert np.array_equal(got.astype(np.int64), o.deliver(spikes, fixed=True)[1])
        g.step(T)
        r = o.run(T)
        assert np.array_equal(g.raster()[1], r["raster"])
        assert np.array_equal(g.state()[0].view(np.uint32), o.state()[0].view(np.uint32))
    else:
        want = o.deliver(spikes)
        ulp = np.spacing(np.abs(want).astype(np.float32)).astype(np.float64)
        assert np.all(np.abs(got - want) <= ulp)
        # fp32 sums are exact: the simulation equals the graph path's bit for bit
        g.step(T)
        ref = spk.Net(dict(cfg, step_mode=1), max_steps=T, raster_capacity=64 * T)
        ref.step(T)
        assert np.array_equal(g.raster()[1], ref.raster()[1])
        assert np.array_equal(g.state()[0].view(np.uint32), ref.state()[0].view(np.uint32))


@pytest.mark.parametrize("delays", [(1, 20), (3, 9), (15, 15)], ids=["d1-20", "d3-9", "d15"])
@pytest.mark.parametrize("step_mode,ring", [(1, None), (2, None), (2, "0")], ids=["graph", "resident", "pages"])
def test_resume_matches_single_run(spk, step_mode, ring, delays, monkeypatch):
    # calls of 50 and 70 steps, and of one step each: batches of several steps
    # (smallest delay 3 or 15) end early at the end of a call
    cfg = I.scaled(4, 5000, k_out=500, acc_mode=I.ACC_FIXED, step_mode=step_mode,
                   delay_min=delays[0], delay_max=delays[1])
    if ring:
        monkeypatch.setenv("SPK_RING", ring)
    a = spk.Net(cfg, max_steps=120, raster_capacity=5000 * 120)
    assert (a.stats()["page_cap"] == 0) == (delays[0] == delays[1] if step_mode == 1 else not ring)
    b = spk.Net(cfg, max_steps=120, raster_capacity=5000 * 120)
    a.step(50)
    a.step(70)
    for _ in range(120):
        b.step(1)
    # events filed near a launch boundary arrive up to 20 steps later: both
    # must equal the oracle's single run, raster and state
    r, ov, orf, _ = _oracle_run(cfg, 120)
    assert r["counts"].sum() > 0
    for g in (a, b):
        assert np.array_equal(g.raster()[1], r["raster"]), "raster differs from the oracle"
        assert np.array_equal(g.state()[0].view(np.uint32), ov.view(np.uint32))
        assert np.array_equal(g.state()[1], orf)
    assert np.array_equal(a.delivered(), b.delivered())


@pytest.mark.parametrize("step_mode,ring", [(1, None), (2, None), (2, "0")], ids=["graph", "resident", "pages"])
def test_delay_chain_spike_timing(spk, step_mode, ring, monkeypatch):
    if ring:
        monkeypatch.setenv("SPK_RING", ring)
    delays = [1, 3, 2, 5]
    n = 5
    row_ptr = np.array([0, 1, 2, 3, 4, 4], dtype=np.uint64)
    col = np.array([1, 2, 3, 4], dtype=np.uint32)
    w = np.full(4, 15.0, dtype=np.float32)
    cfg = I.explicit_params(n, v0_lo=-49.0, v0_hi=-49.0, t_ref_ms=0.0, delay_min=1, delay_max=5,
                            step_mode=step_mode)
    g = spk.Net(cfg, max_steps=20, raster_capacity=100,
                csr=(row_ptr, col, w, np.array(delays, dtype=np.uint8)))
    g.step(20)
    offs, ids = g.raster()
    fire = [{0}]
    for j in range(1, n):
        fire.append({0} | {t + delays[j - 1] for t in fire[j - 1]})
    for t in range(20):
        got = set(ids[int(offs[t]):int(offs[t + 1])].tolist())
        assert got == {j for j in range(n) if t in fire[j]}, t


def test_poisson_table_equals_oracle(spk):
    for lam in (0.37, 1.0, 6.94, 23.15):
        cfg = I.config(0, ext_lambda=lam, ext_w=0.1)
        g = spk.Net(cfg, max_steps=1)
        assert np.array_equal(g.poisson_table(), oracle.poisson_table(lam))


def test_torch_stream_and_overflow_errors(spk):
    import torch
    s = torch.cuda.Stream()
    cfg = I.config(0, driven=True)
    g = spk.Net(cfg, stream=s, max_steps=10, raster_capacity=5)
    g.step(10)
    s.synchronize()
    with pytest.raises(spk.SpkError) as e:
        g.step(1)  # beyond max_steps
    assert e.value.code == spk.SPK_EOVERFLOW
    if int(g.spike_counts().sum()) > 5:
        with pytest.raises(spk.SpkError) as e:
            g.raster()
        assert e.value.code == spk.SPK_EOVERFLOW


def test_fixed_point_guard_matches_oracle(spk):
    cfg = I.config(0, n=60, p=1.0, w_exc=2000.0, w_inh=-2000.0, acc_mode=I.ACC_FIXED, fixed_shift=20)
    with pytest.raises(spk.SpkError) as e:
        spk.Net(cfg, max_steps=1)
    assert e.value.code == spk.SPK_EOVERFLOW
    cfg["fixed_shift"] = 8
    spk.Net(cfg, max_steps=1)


def test_fixed_point_guard_fixed_in_degree(spk):
    # fixed in-degree with population weights: the range is known without a
    # pass over the synapses; the library refuses exactly the networks the
    # oracle refuses (largest per-neuron sum of |quantised weights| beyond
    # int32: 50 x 42,949,672 fits, 50 x 42,960,159 does not)
    for w, fits in ((40.95, True), (40.97, False)):
        cfg = I.config(2, n=400, k_in_exc=40, k_in_inh=10, w_exc=w, w_inh=-w, ext_lambda=0.0,
                       ext_w=0.0, acc_mode=I.ACC_FIXED, fixed_shift=20)
        if fits:
            assert int(oracle.Net(cfg).in_abs_sum_q().max()) <= 2**31 - 1
            spk.Net(cfg, max_steps=1)
        else:
            with pytest.raises(oracle.OracleError) as eo:
                oracle.Net(cfg)
            assert eo.value.code == -4  # the oracle's overflow status
            with pytest.raises(spk.SpkError) as e:
                spk.Net(cfg, max_steps=1)
            assert e.value.code == spk.SPK_EOVERFLOW


@pytest.mark.parametrize("w_uniform", [0, 1], ids=["population", "per-synapse"])
def test_range_pass_per_target_matches_oracle(spk, w_uniform, monkeypatch):
    # Bernoulli networks: the largest per-neuron sum of |quantised weights|
    # is found per target from the pair predicate (no atomics) or with one
    # atomic per synapse; both must refuse exactly the networks the oracle
    # refuses.  Weights are scaled so that the oracle's largest sum lands
    # just inside and just outside int32.
    base = dict(n=800, p=0.05, acc_mode=I.ACC_FIXED, fixed_shift=20, ext_lambda=0.0, ext_w=0.0)
    if w_uniform:
        base.update(w_uniform=1, w_lo=-1.0, w_hi=1.0)
    probe = oracle.Net(I.config(0, **base))
    m1 = int(probe.in_abs_sum_q().max())  # at unit scale
    assert m1 > 0
    for scale, fits in ((0.999, True), (1.001, False)):
        f = scale * (2**31 - 1) / m1
        over = dict(base, w_lo=-f, w_hi=f) if w_uniform else dict(base, w_exc=0.27 * f, w_inh=-4.5 * f)
        cfg = I.config(0, **over)
        try:
            ok = int(oracle.Net(cfg).in_abs_sum_q().max()) <= 2**31 - 1
        except oracle.OracleError as e:
            assert e.code == -4
            ok = False
        assert ok == fits
        for mode in ("targets", "atomics"):
            monkeypatch.setenv("SPK_RANGE_PASS", mode)
            if fits:
                spk.Net(cfg, max_steps=1)
            else:
                with pytest.raises(spk.SpkError) as e:
                    spk.Net(cfg, max_steps=1)
                assert e.value.code == spk.SPK_EOVERFLOW


@pytest.mark.parametrize("mode", ["tiles", "atomics"])
def test_range_pass_fixed_out_matches_oracle(spk, mode, monkeypatch):
    # fixed out-degree networks with population weights: the largest
    # per-neuron sum of |quantised weights| from the synapses filed by target
    # tile (default) or one atomic per synapse; both must refuse exactly the
    # networks the oracle refuses, weights scaled to land just inside and
    # just outside int32
    monkeypatch.setenv("SPK_RANGE_PASS", mode)
    base = dict(n=3000, k_out=300, acc_mode=I.ACC_FIXED, fixed_shift=20, ext_lambda=0.0, ext_w=0.0)
    unit = I.config(4, **base)
    m1 = int(oracle.Net(unit).in_abs_sum_q().max())
    assert m1 > 0
    for scale, fits in ((0.999, True), (1.001, False)):
        f = scale * (2**31 - 1) / m1
        cfg = I.config(4, **dict(base, w_exc=unit["w_exc"] * f, w_inh=unit["w_inh"] * f))
        try:
            ok = int(oracle.Net(cfg).in_abs_sum_q().max()) <= 2**31 - 1
        except oracle.OracleError as e:
            assert e.code == -4
            ok = False
        assert ok == fits
        if fits:
            st = spk.Net(cfg, max_steps=1).stats()
            assert st["range_ms"] > 0
        else:
            with pytest.raises(spk.SpkError) as e:
                spk.Net(cfg, max_steps=1)
            assert e.value.code == spk.SPK_EOVERFLOW


@pytest.mark.parametrize("seed", [1, 2])
def test_fp32_mode_mean_rate_within_one_percent(spk, seed):
    # fp32 atomics: spike trains diverge after the first rounding
    # difference; the network's mean rate must still agree.  Pooled over
    # enough spikes that finite-sample noise stays well below 1 %.
    cfg = I.scaled(4, 20000, k_out=1500, seed=seed)
    T = 8000
    g = spk.Net(cfg, max_steps=T)
    g.step(T)
    gc = g.spike_counts().astype(np.float64)
    r = oracle.Net(cfg).run(T)
    oc = r["counts"].astype(np.float64)
    warm = 1000
    rg, ro = gc[warm:].sum(), oc[warm:].sum()
    _say(f"[rate] seed={seed} gpu={rg} oracle={ro}")
    assert ro > 1e5
    assert abs(rg - ro) / ro < 0.01


def _random_csr(n, n_w, seed):
    """Ragged random adjacency (0..250 synapses per row, multapses allowed),
    delays 1..12, weights drawn from n_w distinct values (n_w = 0: every
    synapse its own weight)."""
    rng = np.random.default_rng(seed)
    deg = rng.integers(0, 251, n)
    deg[rng.choice(n, n // 10, replace=False)] = 0
    row_ptr = np.zeros(n + 1, np.uint64)
    row_ptr[1:] = np.cumsum(deg)
    nnz = int(row_ptr[-1])
    col = rng.integers(0, n, nnz).astype(np.uint32)
    delay = rng.integers(1, 13, nnz).astype(np.uint8)
    if n_w:
        vals = np.array([0.37, -1.25, 0.05, 2.0, -0.61][:n_w], np.float32)
        w = vals[rng.integers(0, n_w, nnz)]
    else:
        w = rng.uniform(-1.0, 1.0, nnz).astype(np.float32)
    return row_ptr, col, w, delay


@pytest.mark.parametrize("n_w", [1, 2, 3, 4, 5, 0], ids=["1w", "2w", "3w", "4w", "5w", "perw"])
@pytest.mark.parametrize("fmt", [0, 1, 2], ids=["auto", "full", "compact"])
def test_explicit_adjacency_formats(spk, n_w, fmt):
    n = 3000
    row_ptr, col, w, delay = _random_csr(n, n_w, seed=40 + n_w)
    fits = 1 <= n_w <= 4
    for acc in (I.ACC_FIXED, I.ACC_F32):
        cfg = I.explicit_params(n, acc_mode=acc, delay_min=1, delay_max=12, syn_format=fmt,
                                i_bias=1.2, v0_lo=-65.0, v0_hi=-50.0)
        _say(f"[explicit] n_w={n_w} format={fmt} acc={acc}")
        if fmt == 2 and not fits:
            with pytest.raises(spk.SpkError) as e:
                spk.Net(cfg, max_steps=1, csr=(row_ptr, col, w, delay))
            assert e.value.code == spk.SPK_EINVAL
            return
        T = 60
        g = spk.Net(cfg, max_steps=T, raster_capacity=n * T, csr=(row_ptr, col, w, delay))
        compact = fmt == 2 or (fmt == 0 and fits)
        assert g.stats()["bytes_per_synapse"] == (4.0 if compact else 8.0)
        o = oracle.Net(cfg, csr=(row_ptr, col, w, delay))
        rows = np.arange(0, n, 7, dtype=np.uint32)
        offs, gc, gw, gd = g.export_rows(rows)
        o_rp, o_col, o_w, o_d = o.csr()
        _compare_rows(offs, gc, gw, gd, o_rp, o_col, o_w, o_d, rows, acc == I.ACC_FIXED)
        spikes = I.spike_set(n, n // 3, seed=5, unique=True)
        for dl in (0, 1, 12):
            got = g.debug_deliver(spikes, delay=dl)
            if acc == I.ACC_FIXED:
                assert np.array_equal(got.astype(np.int64), o.deliver(spikes, delay=dl, fixed=True)[1])
            else:
                want = o.deliver(spikes, delay=dl)
                ulp = np.spacing(np.abs(want).astype(np.float32)).astype(np.float64)
                assert np.all(np.abs(got.astype(np.float64) - want) <= ulp)
        if acc == I.ACC_FIXED:
            g.step(T)
            r = o.run(T)
            assert r["counts"].sum() > 0
            assert np.array_equal(g.raster()[1], r["raster"]), "rasters differ"
            assert np.array_equal(g.state()[0].view(np.uint32), o.state()[0].view(np.uint32))


@pytest.mark.parametrize("name,mk,T", [
    ("C4-20000", lambda: I.scaled(4, 20000, k_out=1500), 1500),
    ("C1-8000", lambda: I.scaled(1, 8000), 800),
    ("C3-30000", lambda: I.scaled(3, 30000, k_out=1000), 200),
    ("C2-8000", lambda: I.scaled(2, 8000, k_in_exc=640, k_in_inh=160), 800),
], ids=["C4-20000", "C1-8000", "C3-30000", "C2-8000"])
@pytest.mark.parametrize("fmt", [f for f, _ in FORMATS], ids=[n for _, n in FORMATS])
@pytest.mark.parametrize("delivery", [0, 2], ids=["auto", "binned"])
def test_persistent_equals_graph_fp32(spk, name, mk, T, fmt, delivery, monkeypatch):
    # fp32 mode is deterministic (exact sums, one rounding): every way of
    # running the steps must agree bit for bit over a long active run
    cfg = mk()
    cfg["syn_format"] = fmt
    cfg["delivery"] = delivery
    runs = []
    for step_mode, batch, ring in ((1, None, None), (2, None, None), (2, "1", None), (2, None, "0")):
        if batch:
            monkeypatch.setenv("SPK_BATCH_STEPS", batch)
        if ring:  # AUTO: pages or the due rows instead of the resident kernel
            if delivery == 2:
                continue
            monkeypatch.delenv("SPK_BATCH_STEPS")
            monkeypatch.setenv("SPK_RING", ring)
        c = dict(cfg, step_mode=step_mode)
        g = spk.Net(c, max_steps=T, raster_capacity=cfg["n"] * T)
        st = g.stats()
        assert st["step_mode"] == step_mode
        _say(f"[persist=graph] {name} T={T} mode={step_mode} batch={st['batch_steps']} format={fmt}")
        g.step(T // 3)
        g.step(T - T // 3)
        runs.append((g.spike_counts(), g.raster()[1], g.delivered(), g.events(), g.state()))
    c1, r1, d1, e1, (v1, f1) = runs[0]
    assert c1.sum() > 0
    for c2, r2, d2, e2, (v2, f2) in runs[1:]:
        assert np.array_equal(c1, c2) and np.array_equal(r1, r2), "rasters differ"
        assert np.array_equal(d1, d2) and np.array_equal(e1, e2)
        assert np.array_equal(v1.view(np.uint32), v2.view(np.uint32)) and np.array_equal(f1, f2)


def test_setup_timing_stats(spk):
    # creation reports its wall time and the GPU time of the generation
    # kernels and of the accumulator-range pass (Sec. IV-C); uploaded rows are
    # not generated
    for cfg in (I.synth(4000, 0.05), I.scaled(2, 8000, k_in_exc=640, k_in_inh=160),
                I.scaled(4, 8000, k_out=300)):
        _say(f"[setup] n={cfg['n']} conn={cfg['conn_kind']}")
        st = spk.Net(cfg, max_steps=1).stats()
        assert st["gen_ms"] > 0
        # fixed in-degree with population weights: the range needs no pass
        assert (st["range_ms"] == 0) == (cfg["conn_kind"] == I.FIXED_IN)
        assert st["setup_ms"] >= st["gen_ms"] + st["range_ms"]
    n = 2000
    row_ptr, col, w, delay = _random_csr(n, 2, seed=3)
    cfg = I.explicit_params(n, delay_min=1, delay_max=12)
    st = spk.Net(cfg, max_steps=1, csr=(row_ptr, col, w, delay)).stats()
    assert st["gen_ms"] == 0 and st["range_ms"] > 0 and st["setup_ms"] > 0


def test_step_mode_selection(spk, monkeypatch):
    # AUTO takes the persistent kernel where it applies; asking for it where
    # it does not (direct delivery with several delays) is an error
    # delay-1 events: one step per batch
    st = spk.Net(I.scaled(4, 8000, k_out=300), max_steps=1).stats()
    assert st["step_mode"] == spk.SPK_STEP_PERSISTENT and st["batch_steps"] == 1
    # smallest delay 15: binned delivery in batches of 8 steps (15 when
    # asked for, 1 when batches are capped at 1)
    c2 = I.scaled(2, 8000, k_in_exc=640, k_in_inh=160)
    st = spk.Net(c2, max_steps=1).stats()
    assert st["step_mode"] == spk.SPK_STEP_PERSISTENT
    assert st["delivery"] == spk.SPK_DELIVERY_BINNED and st["batch_steps"] == 8
    monkeypatch.setenv("SPK_BATCH_STEPS", "16")
    assert spk.Net(c2, max_steps=1).stats()["batch_steps"] == 15
    monkeypatch.setenv("SPK_BATCH_STEPS", "1")
    st = spk.Net(c2, max_steps=1).stats()
    assert st["step_mode"] == spk.SPK_STEP_PERSISTENT and st["batch_steps"] == 1
    monkeypatch.delenv("SPK_BATCH_STEPS")
    # delays 3..9: batches of 3 steps
    st = spk.Net(I.scaled(4, 8000, k_out=300, delay_min=3, delay_max=9), max_steps=1).stats()
    assert st["batch_steps"] == 3
    # ... but direct delivery when steps run as graphs
    st = spk.Net(I.scaled(2, 8000, k_in_exc=640, k_in_inh=160, step_mode=1), max_steps=1).stats()
    assert st["delivery"] == spk.SPK_DELIVERY_DIRECT
    # fp32 sums with 8-byte synapses: persistent too
    st = spk.Net(I.scaled(4, 8000, k_out=300, syn_format=1), max_steps=1).stats()
    assert st["step_mode"] == spk.SPK_STEP_PERSISTENT
    g = spk.Net(I.scaled(4, 8000, k_out=300, step_mode=1), max_steps=1)
    assert g.stats()["step_mode"] == spk.SPK_STEP_GRAPH
    cfg = I.scaled(4, 8000, k_out=300, delivery=1)
    assert spk.Net(cfg, max_steps=1).stats()["step_mode"] == spk.SPK_STEP_GRAPH
    with pytest.raises(spk.SpkError) as e:
        spk.Net(dict(cfg, step_mode=2), max_steps=1)
    assert e.value.code == spk.SPK_EINVAL


# ------------------------------------------------ procedural connectivity

PROC_CASES = [
    ("C4-8000", lambda acc: I.scaled(4, 8000, k_out=700, acc_mode=acc)),
    ("C4-d3-9", lambda acc: I.scaled(4, 6000, k_out=500, delay_min=3, delay_max=9, acc_mode=acc)),
    ("C3-8000", lambda acc: I.scaled(3, 8000, k_out=1000, acc_mode=acc)),
]


@pytest.mark.parametrize("name,mk", PROC_CASES, ids=[c[0] for c in PROC_CASES])
@pytest.mark.parametrize("acc", [I.ACC_F32, I.ACC_FIXED], ids=["f32", "fixed"])
@pytest.mark.parametrize("once", ["1", "0"], ids=["rows-once", "per-group"])
def test_procedural_rows_and_delivery_equal_oracle(spk, name, mk, acc, once, monkeypatch):
    # procedural synapses are never stored: the rows the library generates
    # (exported) equal the oracle's, and delivering a spike set through them
    # equals the oracle's sums (exact in fixed mode, the rounded exact sum in
    # fp32 mode) and the stored compact/full format's bit for bit
    monkeypatch.setenv("SPK_PROC_ONCE", once)
    cfg = dict(mk(acc), syn_format=3)
    g = spk.Net(cfg, max_steps=1)
    st = g.stats()
    assert st["bytes_per_synapse"] == 0.0 and st["delivery"] == spk.SPK_DELIVERY_BINNED
    assert st["step_mode"] == spk.SPK_STEP_GRAPH and st["nnz"] == cfg["n"] * cfg["k_out"]
    o = _oracle_net(cfg)
    o_rp, o_col, o_w, o_d = o.csr()
    rows = np.arange(0, cfg["n"], 13, dtype=np.uint32)
    offs, col, w, d = g.export_rows(rows)
    _compare_rows(offs, col, w, d, o_rp, o_col, o_w, o_d, rows, acc == I.ACC_FIXED)
    stored = spk.Net(dict(cfg, syn_format=0, step_mode=1), max_steps=1)
    n = cfg["n"]
    for k, count in enumerate([0, 1, 37, n // 200, n // 3, 3 * n]):
        spikes = I.spike_set(n, count, seed=30 + k, unique=count <= n)
        for delay in sorted({0, cfg["delay_min"], cfg["delay_max"]}):
            _say(f"[proc deliver] {name} acc={acc} spikes={len(spikes)} delay={delay}")
            got = g.debug_deliver(spikes, delay=delay)
            if acc == I.ACC_FIXED:
                _, want = o.deliver(spikes, delay=delay, fixed=True)
                assert np.array_equal(got.astype(np.int64), want), "fixed-point inputs differ"
            else:
                want = o.deliver(spikes, delay=delay)
                ulp = np.spacing(np.abs(want).astype(np.float32)).astype(np.float64)
                assert np.all(np.abs(got.astype(np.float64) - want) <= ulp)
            assert np.array_equal(got.view(np.uint32), stored.debug_deliver(spikes, delay=delay).view(np.uint32))


PROC_RUNS = [
    ("C4-12000", lambda: I.scaled(4, 12000, k_out=1500), 400),
    ("C4-d3-9", lambda: I.scaled(4, 12000, k_out=1500, delay_min=3, delay_max=9), 300),
    ("C3-20000", lambda: I.scaled(3, 20000, k_out=1000), 100),
]


@pytest.mark.parametrize("name,mk,T", PROC_RUNS, ids=[c[0] for c in PROC_RUNS])
@pytest.mark.parametrize("once", ["1", "0"], ids=["rows-once", "per-group"])
def test_procedural_simulation_bit_identical(spk, name, mk, T, once, monkeypatch):
    # fixed point: rasters, counts, events, delivered events and final state
    # equal the oracle's; also with the pages shrunk into the overflow path.
    # Both push kernels: each fired row generated once (the default where its
    # buckets fit) and generated by every XCD group (SPK_PROC_ONCE=0)
    monkeypatch.setenv("SPK_PROC_ONCE", once)
    cfg = dict(mk(), acc_mode=I.ACC_FIXED, syn_format=3)
    r, ov, orf, (rp, col, w, d) = _oracle_run(cfg, T)
    assert r["counts"].sum() > 0
    for cap in (None, "64"):
        if cap:
            monkeypatch.setenv("SPK_PAGE_CAP", cap)
        _say(f"[proc run] {name} T={T} page_cap={cap or 'budget'}")
        g = spk.Net(cfg, max_steps=T, raster_capacity=cfg["n"] * T)
        g.step(T // 3)
        g.step(T - T // 3)
        offs, ids = g.raster()
        assert np.array_equal(g.spike_counts(), r["counts"]), "spike counts differ"
        assert np.array_equal(ids, r["raster"]), "rasters differ"
        assert np.array_equal(g.events(), r["events"])
        assert np.array_equal(g.delivered(), r["delivered"])
        gv, gr = g.state()
        assert np.array_equal(gv.view(np.uint32), ov.view(np.uint32)), "membrane potentials differ"
        assert np.array_equal(gr, orf)


def test_procedural_fp32_equals_stored(spk):
    # fp32 mode sums exactly: the procedural network and the stored one step
    # bit for bit alike (graph path both)
    cfg = dict(I.scaled(4, 20000, k_out=1500), step_mode=1)
    T = 600
    out = []
    for fmt in (3, 0):
        g = spk.Net(dict(cfg, syn_format=fmt), max_steps=T, raster_capacity=cfg["n"] * T)
        g.step(T)
        out.append((g.raster()[1], g.state()[0], g.delivered()))
    assert len(out[0][0]) > 0
    assert np.array_equal(out[0][0], out[1][0])
    assert np.array_equal(out[0][1].view(np.uint32), out[1][1].view(np.uint32))
    assert np.array_equal(out[0][2], out[1][2])


def test_procedural_rejects_what_it_does_not_take(spk):
    for cfg in (dict(I.scaled(2, 4000, k_in_exc=300, k_in_inh=75), syn_format=3),
                dict(I.config(0), syn_format=3),
                dict(I.scaled(4, 4000, k_out=300), syn_format=3, delivery=1),
                dict(I.scaled(4, 4000, k_out=300), syn_format=3, step_mode=2)):
        with pytest.raises(spk.SpkError) as e:
            spk.Net(cfg, max_steps=1)
        assert e.value.code == spk.SPK_EINVAL
