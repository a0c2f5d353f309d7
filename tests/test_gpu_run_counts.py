"""The persistent page kernel's packed event counts (fp32 mode, at most two
weight classes) against the graph path's 64-bit sums, bit for bit: one-step
and batched kernels, in-degrees on both sides of the 16-bit bound, counts of
the upper class beyond 2^15, full pages, equal weights and one class."""
import numpy as np
import pytest

import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def spk():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2102_04681_amd import spk as mod
    mod.lib()
    return mod


def _burst(n, k_out, **over):
    """Every neuron starts above threshold and fires at the first step; again
    at most every second one."""
    return I.config(4, n=n, k_out=k_out, v0_lo=-49.0, v0_hi=-49.0, t_ref_ms=0.1, **over)


CASES = [  # parameters, page capacity
    ("plain", lambda: I.scaled(4, 6007, k_out=300, delay_min=1, delay_max=7), None),
    ("batches", lambda: I.scaled(4, 3001, k_out=200, delay_min=4, delay_max=9), None),
    ("full-pages", lambda: _burst(700, 90, delay_min=1, delay_max=3), "64"),
    ("full-pages-batches", lambda: _burst(700, 90, delay_min=3, delay_max=5), "64"),
    # 64 neurons; equal |weights|: the bound is the in-degree itself
    ("upper-class", lambda: _burst(64, 50_000, delay_max=1, frac_exc=0.2, w_exc=1e-3, w_inh=-1e-3), None),
    ("beyond", lambda: _burst(64, 65_500, delay_max=1, frac_exc=0.5, w_exc=1e-3, w_inh=-1e-3), None),
    ("equal", lambda: I.scaled(4, 2000, k_out=100, delay_max=4, w_exc=0.3, w_inh=0.3), None),
    ("all-excitatory", lambda: I.scaled(4, 2000, k_out=100, delay_max=4, frac_exc=1.0), None),
]


@pytest.mark.parametrize("name,mk,cap", CASES, ids=[c[0] for c in CASES])
def test_packed_counts_bit_identical(spk, name, mk, cap, monkeypatch):
    if cap:
        monkeypatch.setenv("SPK_PAGE_CAP", cap)
    T = 40
    cfg = dict(mk(), acc_mode=I.ACC_F32, delivery=2, syn_format=2)
    out = []
    for mode in (1, 2):
        g = spk.Net(dict(cfg, step_mode=mode), max_steps=T, raster_capacity=cfg["n"] * T)
        assert g.stats()["step_mode"] == mode
        g.step(17)
        g.step(T - 17)
        v, r = g.state()
        out.append([g.spike_counts(), g.events(), g.delivered(), v.view(np.uint32), r, *g.raster()])
        g.close()
    assert out[0][0].sum() > 0
    for a, b, what in zip(*out, ("counts", "events", "delivered", "v", "ref", "offsets", "ids")):
        assert np.array_equal(a, b), what


@pytest.mark.parametrize("n_w", [1, 2])
@pytest.mark.parametrize("delays", [(1, 3), (3, 5)], ids=["steps", "batches"])
@pytest.mark.parametrize("cap", [None, "16"], ids=["pages", "full-pages"])
def test_packed_counts_of_an_explicit_adjacency(spk, n_w, delays, cap, monkeypatch):
    # the classes of an explicit adjacency's weights are 0 and 1 in order of
    # first appearance, whichever comes first in a row, in the pages and past
    # them
    if cap:
        monkeypatch.setenv("SPK_PAGE_CAP", cap)
    n, k, T = 900, 120, 40
    rng = np.random.default_rng(n_w)
    row_ptr = np.arange(n + 1, dtype=np.uint64) * k
    col = rng.integers(0, n, n * k, dtype=np.uint32)
    w = np.array([0.02, -0.05][:n_w], np.float32)[rng.integers(0, n_w, n * k)]
    d = rng.integers(delays[0], delays[1] + 1, n * k).astype(np.uint8)
    cfg = I.explicit_params(n, v0_lo=-49.0, v0_hi=-49.0, t_ref_ms=0.0, i_bias=0.06, delay_min=delays[0],
                            delay_max=delays[1], delivery=2, syn_format=2)
    out = []
    for mode in (1, 2):
        g = spk.Net(dict(cfg, step_mode=mode), max_steps=T, csr=(row_ptr, col, w, d))
        assert g.stats()["step_mode"] == mode and g.stats()["page_cap"] > 0
        g.step(17)
        g.step(T - 17)
        v, r = g.state()
        out.append([g.spike_counts(), g.events(), g.delivered(), v.view(np.uint32), r])
        g.close()
    assert out[0][0].sum() > 0
    for a, b, what in zip(*out, ("counts", "events", "delivered", "v", "ref")):
        assert np.array_equal(a, b), what
