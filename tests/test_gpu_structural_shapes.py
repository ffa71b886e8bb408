"""GPU: the mutual-information scores and the weight pass at the edges of their lane patterns (full
and single columns of a lane, one to many rows per block, unaligned rows, hidden HCUs with unequal
numbers of active inputs) on an arbitrary state, against the oracle."""
import sys

import numpy as np
import pytest

import oracle
from pairs import Pair, TOL_MI_REL, assert_weights_close, gpu_config, oracle_params

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _announce(request):
    print(f"\n[gpu] {request.node.nodeid}", file=sys.stderr, flush=True)
    yield


@pytest.mark.parametrize("in_hcu,in_mcu,out_hcu,out_mcu", [
    (9, 2, 3, 1), (10, 1, 5, 3), (7, 3, 2, 8), (33, 2, 7, 9), (20, 2, 3, 16), (12, 10, 3, 17),
    (40, 2, 9, 24), (30, 3, 4, 33), (64, 2, 11, 100), (25, 2, 3, 257), (49152, 2, 8, 4),
    (30, 5, 3, 10), (30, 5, 3, 15), (17, 2, 2, 25), (40, 2, 300, 5), (1535, 1, 3, 2), (1536, 1, 255, 1), (1536, 1, 256, 1),
])
def test_scores_and_weights_on_any_state(in_hcu, in_mcu, out_hcu, out_mcu):
    rng = np.random.default_rng(in_hcu * 31 + out_mcu)
    cfg = gpu_config(in_hcu, in_mcu, out_hcu, out_mcu, 16, n_swaps=2)
    mask = (rng.random((in_hcu, out_hcu)) < min(0.4, 2000 / in_hcu)).astype(np.uint8)
    mask[0, :] = 1
    mask[:, 1] = 0                                               # a hidden HCU of one input
    mask[in_hcu - 1, 1] = 1
    pair = Pair(cfg, mask)
    st = pair.ora.get_state()
    n_in, n_out = pair.n_in, pair.n_out
    st["pi"] = rng.uniform(1e-9, 1.0, n_in).astype(np.float32)
    st["pj"] = rng.uniform(1e-9, 0.5, n_out).astype(np.float32)
    pij = rng.uniform(0.0, 0.3, (n_in, n_out)).astype(np.float32)
    pij[rng.random((n_in, n_out)) < 0.05] = 0.0
    st["pij"] = pij
    pair.gpu.set_state(st)
    pair.ora.set_state(st)
    pair.gpu.recompute_weights()
    pair.ora.recompute_weights()
    sg = pair.gpu.get_state()
    assert_weights_close(sg["w"], pair.ora.w)
    assert_weights_close(sg["b"], pair.ora.b)
    assert pair.gpu.structural_update() == pair.ora.structural_update()[0]
    want = oracle.mutual_information(oracle_params(cfg), st["pi"], st["pj"], pij)
    # fp64 terms on both sides: the tolerance is relative to the block's sum of |terms|
    e = float(cfg.eps)
    P = np.maximum(pij.astype(np.float64), e)
    ratio = P / np.maximum(st["pi"].astype(np.float64), e)[:, None]
    ratio /= np.maximum(st["pj"].astype(np.float64), e)[None, :]
    size = np.abs(pij * np.log(ratio)).reshape(in_hcu, in_mcu, out_hcu, out_mcu).sum((1, 3))
    assert np.all(np.abs(pair.gpu.get_mi() - want) <= TOL_MI_REL * size)
    np.testing.assert_array_equal(pair.gpu.get_state()["mask"], pair.ora.mask)
    pair.close()


# The weight pass over the whole matrix (dense masks, narrow blocks; 16-byte and scalar rows, rows past
# one pass of a workgroup, full masks) and, with the sparser mask of the same layer, over the active
# blocks.  Silent weights are exactly 0 either way.
@pytest.mark.parametrize("in_hcu,in_mcu,out_hcu,out_mcu,share", [
    (300, 2, 400, 3, 1.0), (300, 2, 400, 3, 0.5), (300, 2, 400, 3, 0.02), (512, 1, 333, 7, 0.9),
    (2100, 1, 97, 33, 1.0), (2100, 1, 97, 33, 0.2), (600, 1, 1025, 1, 0.7), (530, 2, 2051, 4, 0.6),
    (3000, 1, 2, 1024, 1.0), (1024, 3, 450, 50, 0.95),
])
def test_weights_under_masks_of_any_share(in_hcu, in_mcu, out_hcu, out_mcu, share):
    rng = np.random.default_rng(in_hcu + out_mcu)
    cfg = gpu_config(in_hcu, in_mcu, out_hcu, out_mcu, 16)
    mask = (rng.random((in_hcu, out_hcu)) < share).astype(np.uint8)
    mask[rng.integers(in_hcu), :] = 1
    pair = Pair(cfg, mask)
    st = pair.ora.get_state()
    st["pi"] = rng.uniform(1e-9, 1.0, pair.n_in).astype(np.float32)
    st["pj"] = rng.uniform(1e-9, 0.5, pair.n_out).astype(np.float32)
    st["pij"] = rng.uniform(0.0, 0.3, (pair.n_in, pair.n_out)).astype(np.float32)
    pair.gpu.set_state(st)
    pair.ora.set_state(st)
    pair.gpu.recompute_weights()
    pair.ora.recompute_weights()
    sg = pair.gpu.get_state()
    assert_weights_close(sg["w"], pair.ora.w)
    assert_weights_close(sg["b"], pair.ora.b)
    silent = np.repeat(np.repeat(mask == 0, in_mcu, 0), out_mcu, 1)
    assert not np.any(sg["w"].reshape(pair.n_in, pair.n_out)[silent])
    pair.close()
