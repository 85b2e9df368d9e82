"""The feature sort in its three forms (inside the output layer's launches, two launches per
pass, three from 49,152 (chunk, digit) counts on) and the step on one stream and on two: the touched
rows bit for bit, and the whole step's W1 update against the oracle."""
import numpy as np
import pytest

import paper_2110_07029_amd as asgd
from oracle import model as om
from paper_2110_07029_amd import synth

from gpu_util import RTOL_FP32, Setup, assert_update_close, flush, step_magnitudes

pytestmark = pytest.mark.gpu


def dataset(F, L, B, nnz, seed):
    """B rows holding exactly nnz entries in all, some rows long, one feature in every row that
    has room."""
    r = np.random.default_rng(seed)
    w = r.lognormal(0.0, 0.7, B)
    counts = np.minimum(np.maximum((w / w.sum() * nnz).astype(np.int64), 0), F)
    while counts.sum() < nnz:
        i = r.integers(0, B)
        counts[i] += int(counts[i] < F)
    while counts.sum() > nnz:
        i = r.integers(0, B)
        counts[i] -= int(counts[i] > 0)
    rows = []
    for c in counts:
        ids = r.choice(F, c, replace=False)
        if c and F - 1 not in ids:
            ids[0] = F - 1
        rows.append(np.sort(ids))
    x = synth.CSR(np.concatenate([[0], np.cumsum(counts)]), np.concatenate(rows).astype(np.int32),
                  r.uniform(0.1, 1.0, nnz).astype(np.float32), F)
    y = synth.CSR(np.arange(B + 1, dtype=np.int64), r.integers(0, L, B).astype(np.int32), None, L)
    wl = synth.Workload("sort", F, L, B, B, 0.5, True, "", 0, 0, 0, 1.05, "", "", 0, None, 7)
    return wl, synth.Dataset(wl, x, y)


# F 2,000: one pass; 3,000 / 100,000 / 600,000 / 2^21: two passes of 6 / 9 / 10 / 11 bits.  Entries:
# around a chunk of 512 or 1,024, where pass 0 starts to leave pass 1's counts (16,384), where the
# offsets get their own launch (47 | 48 chunks of 10 bits, 95 | 96 of 9, 23 | 24 of 11), and at the
# 16-bit counters' limit, where the step goes from one stream to two
@pytest.mark.parametrize("F,nnz", [(2_000, 511), (3_000, 512), (100_000, 513), (100_000, 1_025), (100_000, 16_383), (2_500, 16_384), (1 << 21, 18_600),
                                   (600_000, 48_128), (600_000, 48_129), (100_000, 97_280), (100_000, 97_281), (1 << 21, 23_552),
                                   (1 << 21, 23_553), (3_000, 131_073), (100_000, 49_152), (100_000, 49_153), (100_000, 65_535), (3_000, 65_536),
                                   (100_000, 65_537), (2_000, 131_072),
                                   (100_000, 131_073)])
def test_touched_rows_and_w1_update(F, nnz):
    import torch
    flush(f"sort F={F} nnz={nnz}")
    L, B = 300, 160
    wl, ds = dataset(F, L, B, nnz, 11)
    s = Setup(wl, B, B, bf16=False, ds=ds)
    try:
        ids = torch.empty(nnz, dtype=torch.int32, device="cuda")
        n = asgd.asgd_debug_touched_rows(s.m, s.xb(0, B), ids)
        touched = np.unique(ds.x.indices)
        assert n == len(touched) and np.array_equal(ids[:n].cpu().numpy(), touched)
        p = s.params()
        for _ in range(2):  # the second step on the same buffers
            asgd.asgd_train_step(s.m, s.xb(0, B), s.yb(0, B), wl.lr)
            after = s.params()
            ref, _, g, fw = om.train_step(p, ds.x, ds.y, wl.lr, "fp32")
            mag = step_magnitudes(p, ds.x, ds.y, g, fw, wl.lr)
            assert_update_close("W1", p["W1"][touched], after["W1"][touched], ref["W1"][touched], RTOL_FP32, mag["W1"])
            rest = np.setdiff1d(np.arange(F), touched)
            assert np.array_equal(after["W1"][rest].view(np.uint32), p["W1"][rest].view(np.uint32))
            p = after
    finally:
        s.free()
