"""GPU: the support's launch shapes (one chunk, chunks, many rows, a single row, row by row) at the
edges of their column tiles, unit chunks and input vectors, against the oracle's forward pass on a
given state; and a supervised batch without activities, whose support is not computed."""
import sys

import numpy as np
import pytest

from paper_2106_05373_amd import synth
from pairs import TOL_ACT, Pair, assert_state_close, assert_support_close, gpu_config, max_abs

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _announce(request):
    print(f"\n[gpu] {request.node.nodeid}", file=sys.stderr, flush=True)
    yield


def given_state(rng, hin, min_, hout, mout, mask):
    n_in, n_out = hin * min_, hout * mout
    w = rng.normal(0, 0.7, (n_in, n_out)).astype(np.float32)
    w *= np.repeat(np.repeat(mask, min_, 0), mout, 1)
    pj = rng.random(n_out).astype(np.float32) + 0.1
    return dict(pi=np.full(n_in, 1 / min_, np.float32), pj=pj,
                pij=np.full((n_in, n_out), 1e-3, np.float32), w=w,
                b=np.log(pj).astype(np.float32), mask=mask)


# (in_hcu, in_mcu, out_hcu, out_mcu, active input HCUs, batch)
SHAPES = [
    # one chunk: column tiles 1, 5 (16-byte rows and not), 7, 8; odd and even MCUs per input HCU
    (20, 2, 3, 16, 9, 33), (20, 1, 2, 17, 13, 16), (31, 3, 3, 70, 11, 20), (40, 2, 2, 80, 31, 17),
    (40, 4, 2, 81, 20, 5), (90, 2, 3, 100, 78, 129), (60, 2, 2, 128, 50, 31),
    # a single row: one chunk, chunks
    (90, 2, 3, 100, 78, 1), (300, 3, 2, 70, 201, 1), (400, 2, 2, 12, 400, 1),
    # chunks: a partial last one, unit counts one past a chunk, every panel stride
    (300, 3, 2, 70, 201, 40), (700, 1, 3, 6, 613, 18), (600, 2, 2, 100, 599, 20),
    (200, 2, 2, 129, 151, 17), (150, 3, 2, 257, 99, 16), (100, 2, 2, 513, 61, 18),
    # wide hidden HCUs: whole and partial k-steps at the end, shares that leave no room for their sums
    (160, 3, 2, 200, 133, 20), (90, 2, 2, 256, 78, 33), (200, 2, 1, 300, 190, 19), (120, 2, 3, 400, 99, 2),
    (100, 1, 2, 512, 77, 17), (60, 3, 1, 700, 47, 18), (40, 2, 2, 1024, 30, 16), (50, 1, 1, 1000, 45, 1),
    # two workgroups per CU: partial chunks and k-steps, a unit table in parts
    (200, 2, 90, 100, 120, 48), (500, 1, 300, 113, 389, 2), (200, 3, 64, 160, 133, 80),
    (900, 2, 60, 150, 850, 70), (820, 2, 29, 97, 811, 144),
    # many hidden HCUs with one, two and five row tiles, a group's last ones absent; a handful of units
    (30, 1, 1100, 10, 25, 16), (30, 1, 1100, 10, 25, 17), (60, 2, 210, 100, 50, 80), (40, 2, 520, 20, 30, 33),
    (200, 3, 110, 30, 133, 72), (450, 1, 260, 12, 401, 40), (12, 1, 3000, 2, 3, 2), (700, 2, 70, 100, 350, 71),
    # many rows: groups of four row tiles, the last one with 17 rows (weight rows of 4, 8 and 16 bytes)
    (200, 3, 60, 10, 133, 337), (200, 3, 60, 21, 133, 337), (200, 3, 40, 81, 133, 337),
    (160, 2, 80, 100, 150, 337), (90, 2, 60, 128, 78, 465),
    # ... of few units: several one-chunk workgroups per CU instead
    (60, 2, 40, 20, 15, 450), (90, 2, 30, 100, 39, 600), (64, 3, 130, 10, 21, 140),
    # a readout, row by row: weight rows of 16, 8 and 4 bytes, ragged batches
    (30, 100, 1, 16, 30, 40), (30, 100, 1, 10, 30, 128), (50, 13, 1, 7, 49, 19), (600, 1, 1, 2, 513, 1),
    # ... every input unit active: weights past the last 16 bytes, 2 to 96 passes, widths 3 (not 4) to 16
    (105, 5, 1, 13, 105, 3), (513, 1, 1, 7, 513, 2), (6000, 2, 1, 4, 6000, 3), (256, 2, 1, 6, 256, 5),
    (12288, 1, 1, 16, 12288, 3), (40, 100, 1, 15, 40, 2), (171, 3, 1, 3, 171, 9),
    # more active units than the larger stages leave room for in the unit table
    # (the table then holds a part of them at a time)
    (6000, 2, 1, 40, 5900, 18), (12288, 1, 2, 20, 12288, 3), (5000, 1, 2, 11, 4801, 1),
    (1200, 3, 2, 93, 1195, 15), (360, 10, 1, 27, 359, 40), (3500, 1, 2, 100, 3454, 17),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_forward_and_readout_match_oracle(shape):
    hin, min_, hout, mout, k, B = shape
    rng = np.random.default_rng(hin * 7 + mout)
    mask = np.stack([synth.random_mask(hin, 1, k, 50 + c)[:, 0] for c in range(hout)], 1)
    if hout > 1 and k > 2:                       # hidden HCUs of unequal counts
        mask[np.flatnonzero(mask[:, -1])[1], -1] = 0
    pair = Pair(gpu_config(hin, min_, hout, mout, B, gain=2.0), mask)
    pair.ora.set_state(given_state(rng, hin, min_, hout, mout, mask))
    pair.sync_gpu_to_oracle()
    a = rng.random((B, hin, min_)) + 0.05
    x = (a / a.sum(-1, keepdims=True)).reshape(B, -1).astype(np.float32)
    y, s, y_o, s_o = pair.forward(x)
    # supports near zero: fp64 sums in another order differ by 2^-53 of their terms, not of s
    far = np.abs(s_o) > 1e-6
    assert_support_close(s[far], s_o[far])
    assert max_abs(s[~far], s_o[~far]) <= 1e-11
    assert max_abs(y, y_o) <= TOL_ACT
    t = pair.torch
    win = t.empty((B, hout), device="cuda", dtype=t.int32)
    pair.gpu.readout(pair.dev(x), win)
    best = s.reshape(B, hout, mout).argmax(2)    # the argmax of the GPU's own support: exact
    assert np.array_equal(win.cpu().numpy(), best)
    pair.close()


def test_training_batch_of_more_units_than_the_table_holds():
    rng = np.random.default_rng(8)
    hin, hout, mout, k, B = 4100, 2, 21, 4011, 19
    mask = np.stack([synth.random_mask(hin, 1, k, 60 + c)[:, 0] for c in range(hout)], 1)
    pair = Pair(gpu_config(hin, 1, hout, mout, B, alpha=0.05), mask)
    pair.ora.set_state(given_state(rng, hin, 1, hout, mout, mask))
    pair.sync_gpu_to_oracle()
    y, y_o, _ = pair.train(rng.random((B, hin)).astype(np.float32))
    assert max_abs(y, y_o) <= TOL_ACT
    got, want = pair.gpu.get_state(), pair.ora.get_state()
    for key in ("pi", "pj", "pij"):
        assert max_abs(got[key], want[key]) <= TOL_ACT, key
    pair.close()


# (in_hcu, in_mcu, out_hcu, out_mcu, active input HCUs, batch, pairs)
TRAINED = [
    # four row tiles per workgroup, the last group one full row tile and a row of the next: shares of the
    # k-steps and none, weight rows of 4, 8 and 16 bytes
    (200, 3, 60, 10, 133, 337, 0), (300, 2, 70, 10, 200, 337, 1), (200, 3, 60, 21, 133, 337, 0),
    (200, 3, 40, 81, 133, 337, 0), (160, 2, 80, 100, 150, 337, 1), (200, 3, 48, 40, 133, 320, 0),
    # two workgroups per CU; wide hidden HCUs
    (200, 3, 30, 100, 133, 150, 0), (200, 3, 26, 160, 133, 150, 0), (150, 2, 17, 300, 90, 260, 1),
    # one row tile of many hidden HCUs
    (200, 2, 1100, 10, 150, 3, 1),
]


@pytest.mark.parametrize("target", [False, True], ids=["unsupervised", "target"])
@pytest.mark.parametrize("shape", TRAINED, ids=lambda s: "x".join(map(str, s)))
def test_training_batches_match_oracle(shape, target):
    """Two batches in the forms of many row tiles: the activities and the state, with the activity and
    with a target in the traces."""
    hin, min_, hout, mout, k, B, pairs = shape
    rng = np.random.default_rng(hout * 3 + mout)
    mask = np.stack([synth.random_mask(hin, 1, k, 70 + c)[:, 0] for c in range(hout)], 1)
    pair = Pair(gpu_config(hin, min_, hout, mout, B, alpha=0.05, complement_pairs=pairs), mask)
    pair.ora.set_state(given_state(rng, hin, min_, hout, mout, mask))
    pair.sync_gpu_to_oracle()
    for _ in range(2):
        if pairs:
            x = synth.encode_pixels(rng.random((B, hin)).astype(np.float32))
        else:
            p = rng.random((B, hin, min_)) + 0.05
            x = (p / p.sum(-1, keepdims=True)).reshape(B, -1).astype(np.float32)
        t = None
        if target:
            t = np.concatenate([synth.one_hot(rng.integers(0, mout, B), mout) for _ in range(hout)], 1)
        y, y_o, _ = pair.train(x, t)
        assert max_abs(y, y_o) <= TOL_ACT
        assert_state_close(pair.gpu.get_state(), pair.ora.get_state())
        pair.sync_gpu_to_oracle()
    pair.close()


@pytest.mark.parametrize("in_mcu,pairs,out_hcu,B", [(100, 0, 1, 37), (2, 1, 3, 130), (3, 0, 5, 16)])
def test_supervised_batches_without_activities_leave_the_same_state(in_mcu, pairs, out_hcu, B):
    """The traces take the target either way: the same bits."""
    rng = np.random.default_rng(B)
    hin, mout = 40, 10
    p = rng.random((B, hin, in_mcu)) + 0.05
    x = (p / p.sum(-1, keepdims=True)).reshape(B, -1).astype(np.float32)
    if pairs:
        x = synth.encode_pixels(rng.random((B, hin)).astype(np.float32))
    target = np.tile(synth.one_hot(rng.integers(0, mout, B), mout), (1, out_hcu))
    mask = np.stack([synth.random_mask(hin, 1, 25, c)[:, 0] for c in range(out_hcu)], 1)
    states = []
    for ask in (False, True):
        pair = Pair(gpu_config(hin, in_mcu, out_hcu, mout, B, alpha=0.05, complement_pairs=pairs), mask)
        t = pair.torch
        y = t.empty((B, out_hcu * mout), device="cuda") if ask else None
        for _ in range(3):
            pair.gpu.train_batch(pair.dev(x), pair.dev(target), y)
        states.append(pair.gpu.get_state())
        pair.close()
    for k, v in states[0].items():
        assert np.array_equal(v, states[1][k]), k


@pytest.mark.parametrize("k", [30, 29, 5])       # row by row: all units, some; by row tiles
def test_readout_passes_over_columns_that_are_nan(k):
    """An infinite input unit makes the support +inf, -inf or (weight 0) NaN by the sign of its
    weight: the winner is the first +inf column, whatever NaN columns stand before it."""
    hin, min_, mout, B = 30, 100, 10, 5
    rng = np.random.default_rng(k)
    mask = np.zeros((hin, 1), np.uint8)
    mask[:k] = 1
    pair = Pair(gpu_config(hin, min_, 1, mout, B), mask)
    st = given_state(rng, hin, min_, 1, mout, mask)
    st["w"][7] = [0, -1, 0, 2, -1, 0, 2, 1, -1, 0]
    pair.ora.set_state(st)
    pair.sync_gpu_to_oracle()
    x = rng.random((B, hin * min_)).astype(np.float32)
    x[:, 7] = np.inf
    win = pair.torch.empty((B, 1), device="cuda", dtype=pair.torch.int32)
    pair.gpu.readout(pair.dev(x), win)
    assert (win.cpu().numpy() == 3).all()
    pair.close()
