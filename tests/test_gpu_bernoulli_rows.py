"""Bernoulli rows drawn block-wise (the first product of the pair hash split
into a block's scalar and a thread's part) equal the oracle's pair by pair: at
the edges of the 1,024-target blocks, with p = 1, and in rows where a carry
crosses bit 30 inside a block (found by a search over seeds).  The largest
input sum from rows grouped by tile equals the other passes' (the same fp32
accumulator unit, the same refusals)."""
import numpy as np
import pytest

import inputs as I
import oracle

pytestmark = pytest.mark.gpu

GAMMA, M1, M2 = np.uint64(0x9E3779B97F4A7C15), np.uint64(0xBF58476D1CE4E5B9), np.uint64(0x94D049BB133111EB)


def _mix(z):
    z = z + GAMMA
    z = (z ^ (z >> np.uint64(30))) * M1
    z = (z ^ (z >> np.uint64(27))) * M2
    return z ^ (z >> np.uint64(31))


def _crossing_rows(seed, n):
    """Rows (and block) whose z without and with the carry differ above bit 30."""
    with np.errstate(over="ignore"):
        key = _mix(_mix(np.array([seed], np.uint64)) ^ np.uint64(1))
        rk = _mix(key ^ np.arange(n, dtype=np.uint64))
        low = np.uint64(1023)
        for t0 in range(0, n, 1024):
            za = ((rk ^ np.uint64(t0)) & ~low) + (GAMMA & ~low)
            bad = np.nonzero(((za >> np.uint64(30)) ^ ((za + np.uint64(1024)) >> np.uint64(30))) & low)[0]
            if len(bad):
                return [int(s) for s in bad]
    return []


@pytest.fixture(scope="module")
def spk():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2102_04681_amd import spk as mod
    return mod


def _check_rows(spk, cfg, rows):
    g, o = spk.Net(cfg, max_steps=1), oracle.Net(cfg, build_csr=False)
    for s in rows:
        col, d, w = (x for x in _row(g, s))
        t, ow, od = o.row(s)
        k = np.lexsort((ow, od, t))
        assert np.array_equal(col, t[k]) and np.array_equal(d, od[k]) and np.array_equal(w, ow[k]), s


def _row(g, s):
    _, col, w, d = g.export_rows(np.array([s], np.uint32))
    return col, d, w


@pytest.mark.parametrize("n,p", [(1, 0.5), (255, 0.3), (1023, 0.1), (1024, 0.1), (1025, 0.1), (3073, 0.02), (600, 1.0), (900, 0.0)])
def test_rows_at_block_edges(spk, n, p):
    cfg = I.config(0, n=n, p=p, delay_max=4, seed=5)
    _check_rows(spk, cfg, sorted({0, n // 2, n - 1}))


def test_rows_with_a_carry_through_bit_30(spk):
    n = 4096
    seed, rows = next((s, r) for s, r in ((s, _crossing_rows(s, n)) for s in range(1, 5000)) if r)
    _check_rows(spk, I.config(0, n=n, p=0.05, seed=seed), rows[:4])


@pytest.mark.parametrize("over", [dict(), dict(delay_max=5), dict(w_uniform=1, w_lo=-0.5, w_hi=1.0), dict(acc_mode=1),
                                  dict(n=2500, p=0.3)], ids=["pop", "delays", "uniform", "fixed", "wide"])
def test_range_from_tile_rows(spk, over, monkeypatch):
    cfg = I.config(0, driven=True, **over)
    units = []
    for mode in (None, "targets", "atomics"):
        if mode:
            monkeypatch.setenv("SPK_RANGE_PASS", mode)
        units.append(spk.Net(cfg, max_steps=1).stats()["fixed_shift"])
    assert len(set(units)) == 1


@pytest.mark.parametrize("w_uniform", [0, 1], ids=["population", "per-synapse"])
def test_range_from_tile_rows_at_the_int32_boundary(spk, w_uniform):
    base = dict(n=800, p=0.05, acc_mode=I.ACC_FIXED, fixed_shift=20, ext_lambda=0.0, ext_w=0.0)
    if w_uniform:
        base.update(w_uniform=1, w_lo=-1.0, w_hi=1.0)
    m1 = int(oracle.Net(I.config(0, **base)).in_abs_sum_q().max())
    for scale, fits in ((0.999, True), (1.001, False)):
        f = scale * (2**31 - 1) / m1
        over = dict(base, w_lo=-f, w_hi=f) if w_uniform else dict(base, w_exc=0.27 * f, w_inh=-4.5 * f)
        cfg = I.config(0, **over)
        if fits:
            spk.Net(cfg, max_steps=1)
        else:
            with pytest.raises(spk.SpkError) as e:
                spk.Net(cfg, max_steps=1)
            assert e.value.code == spk.SPK_EOVERFLOW


@pytest.mark.parametrize("n,p,ring", [(5000, 0.03, True), (8000, 0.9, True), (9500, 0.9, True), (700, 1.0, False)],
                         ids=["once", "near-stage", "past-stage", "graph"])
def test_whole_networks_drawn_once_and_twice(spk, n, p, ring):
    # expected rows below the stage are drawn once (their order in memory is
    # free), longer ones and networks of the graph path in two passes: the
    # same rows, and the same first steps as the oracle's
    cfg = I.config(0, n=n, p=p, seed=3, w_exc=0.27 * 20 / (n * p), w_inh=-4.5 * 20 / (n * p), driven=True,
                   acc_mode=I.ACC_FIXED, step_mode=0 if ring else 1)
    cfg["ext_lambda"], cfg["ext_w"] = 5.0, 0.1
    rows = [0, 1, n // 3, n - 1]
    g, o = spk.Net(cfg, max_steps=12), oracle.Net(cfg, build_csr=False)
    for s in rows:
        col, d, w = _row(g, s)
        t, ow, od = o.row(s)
        k = np.lexsort((ow, od, t))
        assert np.array_equal(col, t[k]) and np.array_equal(d, od[k])
    r = o.run(12)
    g.step(12)
    assert r["counts"].sum() > 0
    assert np.array_equal(g.spike_counts(), r["counts"]) and np.array_equal(g.events(), r["events"])
    assert np.array_equal(g.state()[0].view(np.uint32), o.state()[0].view(np.uint32))
