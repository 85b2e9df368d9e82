"""Top-k prediction at the edges of its launch shapes, bit for bit against a stable sort of
the library's own logits (``asgd_debug_forward``'s z_dev takes the same products in the same
order), with exact ties planted and with NaN and infinite biases."""
import numpy as np
import pytest

import paper_2110_07029_amd as asgd
from paper_2110_07029_amd import synth

from gpu_util import Setup, flush, write_params
from test_gpu_trained_scale import trained_scale

pytestmark = pytest.mark.gpu


def workload(L):
    return synth.Workload("predict", 4_000, L, 1_100, 256, 0.01, True, "lognormal", 3.0, 0.8, 300, 1.05, "uniform",
                          "poisson", 2.0, 1.2, 2)


def check(s, rows, k, nan=False):
    import torch
    z = torch.empty((rows, s.L), dtype=torch.float32, device="cuda")
    ids = torch.empty((rows, k), dtype=torch.int32, device="cuda")
    sc = torch.empty((rows, k), dtype=torch.float32, device="cuda")
    asgd.asgd_debug_forward(s.m, s.xb(0, rows), None, z_dev=z)
    asgd.asgd_predict_topk(s.m, s.xb(0, rows), k, ids, sc)
    z, ids, sc = z.cpu().numpy(), ids.cpu().numpy(), sc.cpu().numpy()
    key = np.where(np.isnan(z), -np.inf, z)
    order = np.argsort(-key, axis=1, kind="stable")[:, :k]  # ties: the smaller id first
    assert np.array_equal(ids, order)
    assert np.array_equal(sc, np.take_along_axis(key, order, 1))


# rows: one, a wave's edge, the change from 32 to 64 rows per wave (256 / 257), its row
# block (512 / 513); k: one entry, lists of up to 8, lists of up to 32
@pytest.mark.parametrize("rows,k", [(1, 1), (1, 32), (31, 5), (33, 8), (33, 9), (256, 1), (257, 8), (257, 9), (512, 1),
                                    (513, 3), (1025, 8), (1025, 32)])
@pytest.mark.parametrize("bf16", [True, False])
def test_topk_equals_a_stable_sort_of_the_logits(rows, k, bf16):
    flush(f"predict rows={rows} k={k} bf16={bf16}")
    s = Setup(workload(2_987), 1_100, 1_100, bf16=bf16)
    try:
        p = trained_scale(s.F, s.L, 3)
        for a, b in ((4, 7), (0, 40), (33, 2_980), (2_986, 17)):  # equal labels: exact ties
            p["W2"][b], p["b2"][b] = p["W2"][a], p["b2"][a]
            p["b2"][[a, b]] += 2.0
        write_params(s.m, p)
        check(s, rows, k)
    finally:
        s.free()


@pytest.mark.parametrize("L", [1, 31, 32, 33, 97, 8_193])
def test_few_labels_and_extreme_biases(L):
    flush(f"predict L={L}")
    s = Setup(workload(L), 300, 300)
    try:
        p = trained_scale(s.F, s.L, 4)
        if L > 40:
            p["b2"][5], p["b2"][36], p["b2"][37], p["b2"][38] = np.inf, np.nan, -np.inf, -np.finfo(np.float32).max
        write_params(s.m, p)
        check(s, 300, min(L, 4))
    finally:
        s.free()


@pytest.mark.parametrize("rows,k", [(40, 1), (40, 5), (300, 8), (300, 12)])
def test_rows_with_fewer_ranked_labels_than_k(rows, k):
    """NaN logits are never ranked: the places of a row without a ranked label hold id 2^31 - 1 and
    score -inf."""
    import torch
    flush(f"predict few ranked labels: rows={rows} k={k}")
    s = Setup(workload(2_987), 300, 300)
    try:
        p = trained_scale(s.F, s.L, 4)
        p["b2"][:] = np.nan
        ranked = [7, 1_000, 2_986][:k - 1]
        p["b2"][ranked] = 0.0
        write_params(s.m, p)
        ids = torch.empty((rows, k), dtype=torch.int32, device="cuda")
        sc = torch.empty((rows, k), dtype=torch.float32, device="cuda")
        asgd.asgd_predict_topk(s.m, s.xb(0, rows), k, ids, sc)
        ids, sc = ids.cpu().numpy(), sc.cpu().numpy()
        n = len(ranked)
        assert np.array_equal(np.sort(ids[:, :n], axis=1), np.tile(np.array(ranked, np.int32), (rows, 1)))
        assert np.all(np.isfinite(sc[:, :n])) and np.all(np.isneginf(sc[:, n:]))
        assert np.all(ids[:, n:] == 2 ** 31 - 1)
    finally:
        s.free()
