"""Two-layer prediction in launches of many rows against the layers' own forward and readout calls,
batch by batch: at the edges of the launch sizes, and where the rows go batch by batch."""
import numpy as np
import pytest

from paper_2106_05373_amd import bcpnn

pytestmark = pytest.mark.gpu


def _network(in_hcu, in_mcu, max_batch):
    from paper_2106_05373_amd.pipeline import Network
    rng = np.random.default_rng(5)
    net = Network(bcpnn.default_config(in_hcu, in_mcu, 12, 50, max_batch, seed=3), None, 7)
    for layer in (net.hidden, net.readout):
        st = layer.get_state()
        for k in ("w", "b"):
            st[k] = (st[k] + 0.3 * rng.standard_normal(st[k].shape)).astype(np.float32)
        layer.set_state(st)
    return net


def _by_batches(net, x):
    """Classes and the gap of the two largest supports, max_batch rows at a time."""
    import torch
    n = net.max_batch
    best, gap = [], []
    for k in range(0, len(x), n):
        xk = x[k:k + n].clone()
        y = torch.empty(len(xk), net.hidden.n_out, device="cuda")
        p = torch.empty(len(xk), net.n_classes, device="cuda")
        s = torch.empty_like(p)
        net.hidden.forward(xk, y)
        net.readout.forward(y, p, s)
        top = s.topk(2, 1)
        best.append(top.indices[:, 0])
        gap.append(top.values[:, 0] - top.values[:, 1])
    return torch.cat(best), torch.cat(gap)


def _agree(got, best, gap):
    # supports of a few units, sums of 600 activities: an fp32 ulp of y and s is below 1e-6
    assert bool(((got.long() == best) | (gap < 1e-5)).all())


@pytest.mark.parametrize("in_hcu,in_mcu,max_batch,B", [
    (90, 2, 1, 1), (90, 2, 24, 23), (90, 2, 24, 25), (90, 2, 24, 1024), (90, 2, 24, 1025),
    (90, 2, 24, 2500), (37, 3, 4, 1031), (37, 3, 5, 5), (40, 1, 1100, 1101)])
def test_rows_of_any_number(in_hcu, in_mcu, max_batch, B):
    import torch
    net = _network(in_hcu, in_mcu, max_batch)
    x = torch.rand(B, in_hcu * in_mcu, device="cuda")
    best, gap = _by_batches(net, x)
    out = torch.full((B + 1,), -1, device="cuda", dtype=torch.int32)
    assert net.predict(x, out[1:]).data_ptr() == out[1:].data_ptr()
    _agree(out[1:], best, gap)
    assert int(out[0]) == -1
    _agree(net.predict(x), best, gap)
    wide = torch.zeros(B, 2, device="cuda", dtype=torch.int64)        # another type and stride
    _agree(net.predict(x, wide[:, 1]), best, gap)
    net.close()


def test_what_batches_refuse_stays_refused():
    import torch
    net = _network(37, 3, 5)                       # the second batch would start off 16 bytes
    with pytest.raises(RuntimeError, match="aligned"):
        net.predict(torch.rand(6, 111, device="cuda"))
    with pytest.raises(TypeError):
        net.predict(torch.rand(3, 111, device="cuda", dtype=torch.float64))
    assert net.predict(torch.rand(0, 111, device="cuda")).shape == (0,)
    net.close()
