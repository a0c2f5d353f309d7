"""The resident step kernel (one workgroup per tile, every pending input in
LDS) against the oracle and the other step paths, where it can go wrong: one
tile and several, the edges of tiles and of the spike list, the mailbox's
carried spikes, batches, calls whose last batch is gathered by the next one,
and in-degrees beyond the packed event counts.  Fixed-point sums and fp32
sums (exact integers rounded once) are compared bit for bit."""
import os

import numpy as np
import pytest

import inputs as I
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def spk():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2102_04681_amd import spk as mod
    mod.lib()
    return mod


def _records(g, raster=True):
    v, r = g.state()
    out = [g.spike_counts(), g.events(), g.delivered(), v.view(np.uint32), r]
    return out + list(g.raster()) if raster else out


def _same(a, b, what):
    for x, y, name in zip(a, b, ("counts", "events", "delivered", "v", "ref", "offsets", "ids")):
        assert np.array_equal(x, y), f"{what}: {name}"


def _burst(n, k_out, **over):
    """Every neuron starts above threshold: all fire at the first step."""
    return I.config(4, n=n, k_out=k_out, v0_lo=-49.0, v0_hi=-49.0, t_ref_ms=0.3, **over)


CASES = [  # name, parameters, steps, tiles of the resident kernel
    ("one", lambda: I.scaled(4, 1, k_out=1, delay_max=1), 20, 1),
    ("1024", lambda: I.config(0, driven=True, n=1024), 120, 1),
    ("1025", lambda: I.config(0, driven=True, n=1025), 120, 1),
    ("2048", lambda: I.scaled(4, 2048, k_out=100, delay_max=7), 120, 1),
    ("2049", lambda: I.scaled(4, 2049, k_out=100, delay_max=7), 120, 5),
    ("one-tile-list", lambda: _burst(2047, 40, delay_max=5), 12, 1),         # 2,047 spikes in a list of 1,024
    ("list", lambda: _burst(5000, 60, delay_max=5), 12, 10),                 # 5,000 in a list of 2,048
    ("batches-burst", lambda: _burst(3000, 60, delay_min=4, delay_max=9), 21, 6),
    ("batches-one-tile", lambda: I.scaled(4, 900, k_out=90, delay_min=3, delay_max=9), 100, 1),
    ("in-degree", lambda: I.scaled(2, 6000, k_in_exc=480, k_in_inh=120), 120, 12),
    ("sources", lambda: I.scaled(3, 9000, k_out=300), 60, 18),
    ("bernoulli", lambda: I.scaled(1, 6000), 120, 12),
    ("fanout-1", lambda: I.scaled(4, 3000, k_out=1, delay_max=3), 80, 6),
]


@pytest.mark.parametrize("name,mk,T,tiles", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("acc", [I.ACC_FIXED, I.ACC_F32], ids=["fixed", "f32"])
def test_resident_kernel_bit_identical(spk, name, mk, T, tiles, acc, monkeypatch):
    cfg = dict(mk(), acc_mode=acc)
    monkeypatch.setenv("SPK_RING", "512" if tiles > 1 else "1024" if cfg["n"] <= 1024 else "2048")
    cap = cfg["n"] * T
    g = spk.Net(cfg, max_steps=T, raster_capacity=cap)
    st = g.stats()
    assert st["step_mode"] == spk.SPK_STEP_PERSISTENT and st["page_cap"] == 0
    assert -(-cfg["n"] // st["tile_width"]) == tiles
    g.step(T // 3)
    g.step(1)
    g.step(T - T // 3 - 1)
    got = _records(g)
    if acc == I.ACC_FIXED:
        o = oracle.Net(cfg)
        r = o.run(T)
        v, ref = o.state()
        want = [r["counts"], r["events"], r["delivered"], v.view(np.uint32), ref, r["offs"], r["raster"]]
    else:
        h = spk.Net(dict(cfg, step_mode=1), max_steps=T, raster_capacity=cap)
        h.step(T)
        want = _records(h)
    assert got[0].sum() > 0 or name == "one"
    _same(got, want, name)
    # without a raster a call leaves its last batch to the next one: calls of
    # one step, of a few, of several batches
    g = spk.Net(cfg, max_steps=T)
    left = T
    for k in (1, 1, 2, 7, 3, 1, 20, 5, 1, T):
        k = min(k, left)
        g.step(k)
        left -= k
    _same(_records(g, raster=False), want[:5], f"{name}, many calls")


WIDTHS = [  # parameters, neurons per tile of the resident kernel
    (lambda: I.config(0, n=1024), 1024), (lambda: I.config(0, n=1025), 2048),
    (lambda: I.scaled(4, 1000, k_out=300, delay_max=4), 1024),
    (lambda: I.scaled(4, 1000, k_out=300, delay_max=4, t_ref_ms=0.0), 64),   # (may fire every step)
    (lambda: I.scaled(4, 2000, k_out=500, delay_max=4), 2048),
    (lambda: I.scaled(4, 1000, k_out=100, delay_min=2, delay_max=4), 64),    # (batches)
    (lambda: I.scaled(3, 1000, k_out=300, rate_hz=10.0), 1024), (lambda: I.scaled(3, 1000, k_out=300, rate_hz=50.0), 64),
    (lambda: I.scaled(3, 2000, k_out=300, rate_hz=3.0), 2048), (lambda: I.scaled(3, 2000, k_out=300, rate_hz=10.0), 64),
    (lambda: I.scaled(4, 3072, k_out=700, delay_max=4), 64), (lambda: I.scaled(4, 3073, k_out=700, delay_max=4), 128),
    (lambda: I.scaled(4, 12288, k_out=700, delay_max=4), 256), (lambda: I.scaled(4, 12289, k_out=700, delay_max=4), 512),
    (lambda: I.scaled(4, 4852, k_out=68, delay_max=4), 512),  # (few events)
    (lambda: I.scaled(4, 4852, k_out=68, delay_min=2, delay_max=4), 128),
    (lambda: I.scaled(3, 2500, k_out=400, rate_hz=2.0), 256),
    (lambda: I.scaled(4, 12289, k_out=1000, delay_max=4, t_ref_ms=0.0), 256),
    (lambda: I.scaled(4, 65536, k_out=50, delay_max=4), 512), (lambda: I.scaled(4, 65537, k_out=50, delay_max=4), 1024),
    # rows grouped by narrower tiles, and by the same where the narrower ones' offsets take more than 64 MB
    (lambda: I.scaled(4, 120_000, k_out=20, delay_max=4), 1024), (lambda: I.scaled(4, 131_072, k_out=20, delay_max=4), 1024),
    (lambda: I.scaled(3, 20480, k_out=1000, rate_hz=10.0), 512), (lambda: I.scaled(3, 20480, k_out=1000, rate_hz=50.0), 128),
    (lambda: I.scaled(4, 20480, k_out=50, delay_max=253, delay_min=190), 0),  # (its inputs do not fit)
    (lambda: I.scaled(4, 8192, k_out=50, delay_max=253, delay_min=190), 64),  # (only in narrow tiles)
]


@pytest.mark.parametrize("mk,width", WIDTHS, ids=[str(k) for k in range(len(WIDTHS))])
def test_resident_kernel_tile_width(spk, mk, width):
    # the width that the rule takes, and the same steps and deliveries as the
    # graph path's
    cfg, T = mk(), 30
    a, b = spk.Net(cfg, max_steps=T), spk.Net(dict(cfg, step_mode=1), max_steps=T)
    st = a.stats()
    if width:
        assert st["page_cap"] == 0 and st["tile_width"] == width
    else:
        assert st["page_cap"] > 0
    for g in (a, b):
        g.step(11)
        g.step(T - 11)
    _same(_records(a, raster=False), _records(b, raster=False), "width")
    spikes = I.spike_set(cfg["n"], 300, seed=1)
    assert np.array_equal(a.debug_deliver(spikes).view(np.uint32), b.debug_deliver(spikes).view(np.uint32))


@pytest.mark.parametrize("width,n,dmax,resident", [(4096, 3000, 6, True), (4096, 3000, 7, False), (8192, 7000, 3, True),
                                                   (8192, 7000, 4, False), (2048, 2000, 15, True), (2048, 2000, 16, False),
                                                   (64, 16_384, 5, True), (64, 16_385, 5, False)])
def test_resident_kernel_widths_asked_for(spk, width, n, dmax, resident, monkeypatch):
    # one tile wider than 2,048 neurons has the room of several, a narrower one
    # more; at most 256 tiles
    cfg, T = I.scaled(4, n, k_out=60, delay_max=dmax), 40
    monkeypatch.setenv("SPK_RING", str(width))
    a, b = spk.Net(cfg, max_steps=T), spk.Net(dict(cfg, step_mode=1), max_steps=T)
    assert (a.stats()["page_cap"] == 0 and a.stats()["tile_width"] == width) == resident
    for g in (a, b):
        g.step(11)
        g.step(T - 11)
    assert a.spike_counts().sum() > 0
    _same(_records(a, raster=False), _records(b, raster=False), "width")


def test_resident_kernel_serves_one_delay_of_weights_per_synapse(spk):
    cfg = I.scaled(3, 9000, k_out=300, delay_min=2, delay_max=2)
    a, b = spk.Net(cfg, max_steps=50), spk.Net(dict(cfg, step_mode=1), max_steps=50)
    for g in (a, b):
        g.step(17)
        g.step(33)
    assert a.stats()["page_cap"] == 0 and a.stats()["step_mode"] == 2
    _same(_records(a, raster=False), _records(b, raster=False), "d2")
    # deliveries of steps not run yet read as 0
    c = spk.Net(cfg, max_steps=50)
    c.step(20)
    assert not c.delivered(20, 30).any() and np.array_equal(c.delivered(0, 20), a.delivered(0, 20))


@pytest.mark.parametrize("delays", [(1, 1), (1, 2)], ids=["one-delay", "two"])
def test_in_degree_beyond_the_packed_counts(spk, delays):
    # 80,000 synapses of one weight from two sources that fire together into
    # neuron 5: more events in one step than a 16-bit count holds
    n, m = 300, 40_000
    row_ptr = np.zeros(n + 1, dtype=np.uint64)
    row_ptr[1:] = np.minimum(np.arange(1, n + 1), 2) * m
    col = np.full(2 * m, 5, dtype=np.uint32)
    w = np.full(2 * m, 2.0 ** -14, dtype=np.float32)
    d = np.full(2 * m, delays[0], dtype=np.uint8)
    d[: m // 2] = delays[1]
    cfg = I.explicit_params(n, v0_lo=-49.0, v0_hi=-49.0, t_ref_ms=5.0, delay_min=delays[0], delay_max=delays[1],
                            acc_mode=I.ACC_FIXED)
    g = spk.Net(cfg, max_steps=8, csr=(row_ptr, col, w, d))
    o = oracle.Net(cfg, csr=(row_ptr, col, w, d))
    g.step(8)
    r = o.run(8)
    v, ref = o.state()
    _same(_records(g, raster=False), [r["counts"], r["events"], r["delivered"], v.view(np.uint32), ref], "hub")


@pytest.mark.parametrize("first,second", [(40_000, 40_000), (65_535, 300), (300, 65_535), (300, 65_536), (65_536, 0)])
@pytest.mark.parametrize("acc", [I.ACC_FIXED, I.ACC_F32], ids=["fixed", "f32"])
def test_in_degrees_of_two_weights_about_the_packed_counts(spk, acc, first, second):
    # that many synapses of each of two weights into neuron 5, all delivered at
    # the same step: counts up to 2^16 - 1 of each class fit, whatever their sum
    n = 300
    sizes = [first // 2, first - first // 2, second // 2, second - second // 2]  # rows 0 .. 3
    row_ptr = np.zeros(n + 1, dtype=np.uint64)
    row_ptr[1:] = np.cumsum(sizes + [0] * (n - 4))
    m = first + second
    col = np.full(m, 5, dtype=np.uint32)
    w = np.full(m, 2.0 ** -13, dtype=np.float32)
    w[first:] = -(2.0 ** -14)
    cfg = I.explicit_params(n, v0_lo=-49.0, v0_hi=-49.0, t_ref_ms=0.0, acc_mode=acc, delay_max=2)
    csr = (row_ptr, col, w, np.full(m, 1, dtype=np.uint8))
    g = spk.Net(cfg, max_steps=8, csr=csr)
    # (several delays: no sums in the resident kernel, so it takes counts or nothing)
    assert (g.stats()["page_cap"] == 0) == (max(first, second) <= 65_535)
    g.step(8)
    h = spk.Net(dict(cfg, step_mode=1), max_steps=8, csr=csr)
    h.step(8)
    want = _records(h, raster=False)
    assert want[2][1] == m
    _same(_records(g, raster=False), want, f"{first} + {second}")


@pytest.mark.parametrize("mk", [lambda: I.scaled(4, 8000, k_out=300), lambda: I.scaled(1, 6000),
                                lambda: I.scaled(4, 20000, k_out=50, delay_min=2, delay_max=8)],
                         ids=["delays", "one-delay", "short-rows"])
def test_resident_network_deliveries_match_oracle(spk, mk):
    cfg = dict(mk(), acc_mode=I.ACC_FIXED)
    g, o = spk.Net(cfg, max_steps=1), oracle.Net(cfg)
    for count in (0, 1, 37, cfg["n"] // 3):
        spikes = I.spike_set(cfg["n"], count, seed=count)
        for delay in (0, cfg["delay_max"]):
            want = o.deliver(spikes, delay=delay, fixed=True)[1]
            assert np.array_equal(g.debug_deliver(spikes, delay=delay).astype(np.int64), want)


def _hub_csr(n, tiles, c, delays, w_hub, w_rest, fan):
    """Neuron 0 drives c spikes out of every tile's neurons, the first 512 of
    them delays[0] steps after its first spike, the rest at delays[1]; every
    neuron has fan weak synapses to random targets."""
    rng = np.random.default_rng(c)
    width = n // tiles
    first, rest = min(c, width), c - min(c, width)
    base = np.arange(tiles)[:, None] * width
    hub_a, hub_b = (base + np.arange(first)).ravel(), (base + np.arange(rest)).ravel()
    col = np.concatenate([hub_a, hub_b, rng.integers(0, n, n * fan)]).astype(np.uint32)
    d = np.concatenate([np.full(len(hub_a), delays[0]), np.full(len(hub_b), delays[1]),
                        rng.integers(delays[0], delays[1] + 1, n * fan)]).astype(np.uint8)
    w = np.full(len(col), w_rest, np.float32) if w_rest else \
        rng.uniform(1e-4, 4e-4, len(col)).astype(np.float32)
    w[: c * tiles] = w_hub
    row_ptr = np.zeros(n + 1, np.uint64)
    row_ptr[1:] = c * tiles + np.arange(1, n + 1, dtype=np.uint64) * fan
    return row_ptr, col, w, d


# tiles of 512 neurons, q = 16 // tiles waves share one: batch counts per tile
# at the edges of 64 q .. 64 (2 q - 1)
SHARED = [(t, c) for t in range(2, 9) for q in [16 // t]
          for c in (64 * q, 64 * q + 1, 64 * q + 22, 96 * q, 64 * (2 * q - 1), 64 * (2 * q - 1) + 1)]


@pytest.mark.parametrize("tiles,c", sorted(set(SHARED)))
@pytest.mark.parametrize("kind", ["fixed", "f32", "sums"])
def test_spikes_of_tiles_shared_by_waves(spk, tiles, c, kind, monkeypatch):
    # every spike's row is delivered once: V against the oracle (fixed point)
    # and the graph path (fp32: packed counts or, with one delay, sums)
    if kind == "sums" and c > 512:
        pytest.skip("two delays are counted, not summed")
    monkeypatch.setenv("SPK_RING", "512")
    n, T, fan = 512 * tiles, 16, 200
    delays = (5, 5) if kind == "sums" else (5, 6)
    csr = _hub_csr(n, tiles, c, delays, 12.0, 0.0 if kind == "sums" else 2.0 ** -12, fan)
    cfg = I.explicit_params(n, v0_lo=-49.0, v0_hi=-49.0, t_ref_ms=0.0, delay_min=delays[0], delay_max=delays[1],
                            acc_mode=I.ACC_FIXED if kind == "fixed" else I.ACC_F32)
    g = spk.Net(cfg, max_steps=T, csr=csr)
    st = g.stats()
    assert st["step_mode"] == 2 and st["page_cap"] == 0 and st["tile_width"] == 512 and st["batch_steps"] == 5
    g.step(T)
    if kind == "fixed":
        o = oracle.Net(cfg, csr=csr)
        r = o.run(T)
        v, ref = o.state()
        want = [r["counts"], r["events"], r["delivered"], v.view(np.uint32), ref]
    else:
        h = spk.Net(dict(cfg, step_mode=1), max_steps=T, csr=csr)
        h.step(T)
        want = _records(h, raster=False)
    assert want[0][5:10].sum() == c * tiles  # the second batch's spikes
    _same(_records(g, raster=False), want, f"{tiles} tiles, {c} spikes each")


@pytest.mark.parametrize("n,rate", [(2500, 50.0), (4000, 40.0), (1100, 110.0)])
def test_sources_in_batches_on_few_tiles(spk, n, rate, monkeypatch):
    # (per tile and batch about 205, 164 and, on 3 tiles, 450 spikes)
    monkeypatch.setenv("SPK_RING", "512")
    cfg = I.scaled(3, n, k_out=300, rate_hz=rate, delay_min=15, delay_max=15)
    out = []
    for mode in (0, 1):
        g = spk.Net(dict(cfg, step_mode=mode), max_steps=64)
        g.step(64)
        out.append(_records(g, raster=False))
        if mode == 0:
            assert g.stats()["page_cap"] == 0 and g.stats()["batch_steps"] == 8
    _same(*out, f"{n} sources")
