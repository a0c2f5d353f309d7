"""spk_deliver_noalloc's scratch is shared by every network of a device and
kept at zero between calls: networks of different layouts in turn, in their
overflow paths, deliver what spk_debug_deliver (its own scratch) does."""
import numpy as np
import pytest

import inputs as I

pytestmark = pytest.mark.gpu


def test_networks_in_turn_leave_the_scratch_clean(monkeypatch):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2102_04681_amd import spk
    stream = torch.cuda.Stream()
    monkeypatch.setenv("SPK_PAGE_CAP", "16")  # most events overflow their page
    cfgs = [I.scaled(4, 30000, k_out=300, delivery=2), I.scaled(4, 7000, k_out=200, delivery=2, acc_mode=I.ACC_FIXED),
            I.scaled(4, 9000, k_out=250, syn_format=3), I.scaled(4, 12000, k_out=200, delivery=2, syn_format=1)]
    nets = [spk.Net(c, stream=stream, max_steps=1) for c in cfgs]
    for turn in range(3):
        for k, (cfg, g) in enumerate(zip(cfgs, nets)):
            n = cfg["n"]
            spikes = I.spike_set(n, n // (2 + turn), seed=10 * turn + k)
            d = torch.from_numpy(spikes.astype(np.int32)).cuda()
            out = torch.full((n,), 7, dtype=torch.int32 if cfg["acc_mode"] else torch.float32, device="cuda")
            torch.cuda.synchronize()
            g.deliver_noalloc(d.data_ptr(), len(spikes), out.data_ptr(), delay=(0, 3, 20)[turn])
            g.sync()
            want = g.debug_deliver(spikes, delay=(0, 3, 20)[turn])
            assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32)), (turn, k)


@pytest.mark.parametrize("over", [dict(delivery=2), dict(syn_format=3), dict(delivery=1)],
                         ids=["binned", "procedural", "direct"])
def test_captured_deliveries_replayed_among_eager_ones(over, monkeypatch):
    # the call recorded in a graph: every replay delivers what the spike list
    # then holds, with eager calls of the same and of another network between
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2102_04681_amd import spk
    monkeypatch.setenv("SPK_PAGE_CAP", "64")
    stream = torch.cuda.Stream()
    cfg = I.scaled(4, 9000, k_out=250, **over)
    n, k = cfg["n"], 400
    g = spk.Net(cfg, stream=stream, max_steps=1)
    other = spk.Net(I.scaled(4, 7000, k_out=200, delivery=2), stream=stream, max_steps=1)
    d = torch.zeros(k, dtype=torch.int32, device="cuda")
    out = torch.zeros(n, dtype=torch.float32, device="cuda")
    other_spikes = I.spike_set(7000, 100, seed=9)
    other_d = torch.from_numpy(other_spikes.astype(np.int32)).cuda()
    other_out = torch.zeros(7000, dtype=torch.float32, device="cuda")
    other_want = other.debug_deliver(other_spikes)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        g.deliver_noalloc(d.data_ptr(), k, out.data_ptr())
    for r in range(4):
        spikes = I.spike_set(n, k, seed=r)
        d.copy_(torch.from_numpy(spikes.astype(np.int32)))
        out.fill_(7)
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            graph.replay()
        torch.cuda.synchronize()
        want = g.debug_deliver(spikes)
        assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32)), r
        if r % 2:
            g.deliver_noalloc(d.data_ptr(), k, out.data_ptr())
            g.sync()
            assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32)), r
        other.deliver_noalloc(other_d.data_ptr(), 100, other_out.data_ptr())
        other.sync()
        assert np.array_equal(other_out.cpu().numpy().view(np.uint32), other_want.view(np.uint32)), r
