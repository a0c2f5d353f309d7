"""Procedural synapses generated once, shares that cut rows: against the
stored synapses of the same network, bit for bit, where a share is empty, one
synapse, part of a row, more spikes than a chunk, and more synapses than one
or several windows."""
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


SHAPES = [  # neurons (all fire at the first step), fan-out, delays
    (1, 1, 1), (40, 3, 2), (257, 97, 5), (3001, 1, 1), (100_003, 1, 3),
    (255, 14_336, 1), (2447, 1500, 20), (5003, 1500, 2), (31, 65_535, 1),
]


@pytest.mark.parametrize("n,k_out,dmax", SHAPES)
@pytest.mark.parametrize("acc,full", [(I.ACC_FIXED, False), (I.ACC_F32, False), (I.ACC_F32, True)],
                         ids=["fixed", "f32", "f32-full"])
def test_shares_that_cut_rows(spk, n, k_out, dmax, acc, full):
    T = 12
    cfg = I.config(4, n=n, k_out=k_out, delay_max=dmax, v0_lo=-49.0, v0_hi=-49.0, t_ref_ms=0.3, acc_mode=acc,
                   fixed_shift=12, delivery=2, step_mode=1)
    if full:
        cfg.update(w_uniform=1, w_lo=0.0, w_hi=1e-3)
    out = []
    for fmt in (3, 0):
        g = spk.Net(dict(cfg, syn_format=fmt), max_steps=T, raster_capacity=n * T)
        g.step(T)
        v, r = g.state()
        out.append([g.spike_counts(), g.events(), g.delivered(), v.view(np.uint32), r, *g.raster()])
        g.close()
    assert out[0][0][0] == n
    for a, b, what in zip(*out, ("counts", "events", "delivered", "v", "ref", "offsets", "ids")):
        assert np.array_equal(a, b), what
