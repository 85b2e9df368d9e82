"""GPU parity with weights of a trained model's scale (logits that differ by units).

At the first step's weights every logit is about zero, so a wrong operand of the
recomputed logits hardly shows in the update; here it shows in the bias update of every
label, which is the sum of the label's probabilities."""
import numpy as np
import pytest

import paper_2110_07029_amd as asgd
from oracle import model as om
from paper_2110_07029_amd import synth

from gpu_util import RTOL_BF16, RTOL_FP32, Setup, assert_update_close, flush, step_magnitudes, write_params

pytestmark = pytest.mark.gpu

H = asgd.HIDDEN
LABELS = synth.Workload("labels-3000", 5_000, 2_999, 700, 256, 0.01, True, "lognormal", 3.5, 0.8, 500, 1.05,
                        "uniform", "poisson", 4.0, 1.2, 2)


def trained_scale(F, L, seed):
    r = np.random.default_rng(seed)
    f = lambda scale, *shape: (r.standard_normal(shape) * scale).astype(np.float32)  # noqa: E731
    return {"W1": f(0.5, F, H), "b1": f(0.1, H), "W2": f(0.15, L, H), "b2": f(0.3, L)}


@pytest.mark.parametrize("bf16", [True, False])
@pytest.mark.parametrize("B", [31, 96, 128, 129, 256, 257, 300, 512, 611])
def test_bias_update_of_labels_without_targets(B, bf16):
    """Labels with no entry in the batch: their bias changes by -lr * mean_i softmax(Z_i)_j.

    Against the oracle that rounds the same operands: the kernel's fp32 A1 may flip the bf16
    rounding of an H1 entry (2^-8 of it), a logit moves by at most 2^-8 |h||w| for that one of
    128 terms, here below 0.005, and the sum over rows by less; the stored bias rounds to
    2 ulp."""
    flush(f"trained scale: B={B} bf16={bf16}")
    s = Setup(LABELS, 700, B, bf16=bf16)
    try:
        p = trained_scale(s.F, s.L, 5)
        write_params(s.m, p)
        lr = 0.5
        asgd.asgd_train_step(s.m, s.xb(0, B), s.yb(0, B), lr)
        x, y = s.host_batch(0, B)
        ref = om.train_step(p, x, y, lr, "bf16" if bf16 else "fp32")[0]["b2"].astype(np.float64) - p["b2"]
        got = asgd.asgd_model_get_params(s.m, asgd.ASGD_PARAM_B2, (s.L,)).astype(np.float64) - p["b2"]
        free = np.setdiff1d(np.arange(s.L), y.indices)
        want = ref[free]
        bound = (5e-3 if bf16 else 1e-4) * np.abs(want) + 2.0 * np.spacing(np.abs(p["b2"][free]))
        err = np.abs(got[free] - want)
        assert np.all(err <= bound), (err / bound).max()
    finally:
        s.free()


@pytest.mark.parametrize("bf16", [True, False])
@pytest.mark.parametrize("label", [0, 5, 34, 39])
def test_one_label_far_above_the_rest(label, bf16):
    """A bias 200 above the others, at labels that either half of a wavefront owns: the online
    softmax has to raise its reference to it, or 2^(200 log2 e) overflows."""
    flush(f"far label {label} bf16={bf16}")
    B = 64
    s = Setup(LABELS, 256, B, bf16=bf16)
    try:
        p = trained_scale(s.F, s.L, 6)
        p["b2"][label] = 200.0
        write_params(s.m, p)
        x, y = s.host_batch(0, B)
        loss = asgd.asgd_train_step(s.m, s.xb(0, B), s.yb(0, B), 0.5, want_loss=True)
        ref, ref_loss, g, _ = om.train_step(p, x, y, 0.5, "bf16" if bf16 else "fp32")
        assert np.isfinite(loss) and abs(loss - ref_loss) <= 1e-3 * abs(ref_loss), (loss, ref_loss)
        got = asgd.asgd_model_get_params(s.m, asgd.ASGD_PARAM_B1, (H,)).astype(np.float64)
        d, dr = got - p["b1"], ref["b1"].astype(np.float64) - p["b1"]
        assert np.linalg.norm(d - dr) <= 2e-2 * np.linalg.norm(dr)
    finally:
        s.free()


# forwards: waves on tiles of their own (one tile each; several), workgroups on shared tiles (one
# stream; two, by the batch's entries)
@pytest.mark.parametrize("B,L,nnz,bf16", [(64, 2_999, 20, True), (33, 2_999, 20, False), (256, 30_000, 20, True),
                                          (40, 33_000, 20, False), (1_000, 33_600, 20, True), (1_000, 33_600, 50, True),
                                          (1_000, 33_600, 20, False)])
def test_labels_masked_by_infinite_biases(B, L, nnz, bf16):
    """Labels of bias -inf (a label space with ids out of use) have probability zero: whole tiles of
    them, at any place of a wavefront's or a split's tiles, whole splits, and single ones.  They stay
    as they are, and the others step as if the masked ones were not there."""
    flush(f"masked labels: B={B} L={L} nnz={nnz} bf16={bf16}")
    r = np.random.default_rng(21)
    tiles = np.arange((L + 31) // 32)
    masked = np.isin(tiles % 11, (0, 4)) | ((tiles >= 40) & (tiles < 75)) | (tiles == tiles[-1])
    mask = np.repeat(masked, 32)[:L] | (r.random(L) < 0.1)
    F = 4_000
    ind = np.sort(np.argsort(r.random((B, F)), axis=1)[:, :nnz], axis=1).astype(np.int32)
    x = synth.CSR(np.arange(B + 1, dtype=np.int64) * nnz, ind.ravel(),
                  r.uniform(0.1, 0.5, B * nnz).astype(np.float32), F)
    y = synth.CSR(np.arange(B + 1, dtype=np.int64), r.choice(np.flatnonzero(~mask), B).astype(np.int32), None, L)
    wl = synth.Workload("masked", F, L, B, B, 0.5, True, "", 0, 0, 0, 1.05, "", "", 0, None, 7)
    s = Setup(wl, B, B, bf16=bf16, ds=synth.Dataset(wl, x, y))
    try:
        p = trained_scale(F, L, 9)
        p["b2"][mask] = -np.inf
        write_params(s.m, p)
        loss = asgd.asgd_train_step(s.m, s.xb(0, B), s.yb(0, B), 0.5, want_loss=True)
        ref, ref_loss, g, fw = om.train_step(p, x, y, 0.5, "fp32")
        assert abs(loss - ref_loss) <= 2e-3 * max(1.0, abs(ref_loss)), (loss, ref_loss)
        got = s.params()
        assert np.all(np.isneginf(got["b2"][mask]))
        assert np.array_equal(got["W2"][mask].view(np.uint32), p["W2"][mask].view(np.uint32))
        mag = step_magnitudes(p, x, y, g, fw, 0.5)
        rtol = RTOL_BF16 if bf16 else RTOL_FP32
        for k in ("W2", "b2"):
            assert_update_close(k, p[k][~mask], got[k][~mask], ref[k][~mask], rtol, mag[k][~mask])
        assert_update_close("b1", p["b1"], got["b1"], ref["b1"], rtol, mag["b1"])
        t = g["touched"]
        assert_update_close("W1", p["W1"][t], got["W1"][t], ref["W1"][t], rtol, mag["W1"])
    finally:
        s.free()


# The same two checks for the kernels of long label spaces, which 2,999 labels do not reach: the
# forward with shared tiles, the bf16 backward with a label block per wave, the chunked one, and the
# fp32 one that reads H1 from global memory.
@pytest.mark.parametrize("B,L,bf16", [(256, 131_105, True), (96, 16_500, True), (300, 65_700, True), (513, 65_700, True),
                                      (256, 131_105, False), (33, 20_640, False)])
def test_bias_update_of_labels_without_targets_in_long_label_spaces(B, L, bf16):
    """Bounds as above; here the probabilities are 1/L on average, so the update of one bias is
    near the rounding of the bias itself: the rate is 0.1 L, and the updates' bound is the same
    share of them."""
    flush(f"trained scale, long label space: B={B} L={L} bf16={bf16}")
    wl = synth.Workload("labels-long", 5_000, L, 700, B, 0.01, True, "lognormal", 3.5, 0.8, 500, 1.05, "uniform",
                        "poisson", 4.0, 1.2, 2)
    s = Setup(wl, 700, B, bf16=bf16)
    try:
        p = trained_scale(s.F, s.L, 5)
        write_params(s.m, p)
        lr = 0.1 * L
        asgd.asgd_train_step(s.m, s.xb(0, B), s.yb(0, B), lr)
        x, y = s.host_batch(0, B)
        ref = om.train_step(p, x, y, lr, "bf16" if bf16 else "fp32")[0]["b2"].astype(np.float64) - p["b2"]
        got = asgd.asgd_model_get_params(s.m, asgd.ASGD_PARAM_B2, (s.L,)).astype(np.float64) - p["b2"]
        free = np.setdiff1d(np.arange(s.L), y.indices)
        want = ref[free]
        assert np.median(np.abs(want)) > 1e-2  # far above the bias' rounding
        bound = (5e-3 if bf16 else 1e-4) * np.abs(want) + 2.0 * np.spacing(np.abs(p["b2"][free]) + np.abs(want)).astype(float)
        err = np.abs(got[free] - want)
        assert np.all(err <= bound), (err / bound).max()
    finally:
        s.free()


@pytest.mark.parametrize("bf16", [True, False])
@pytest.mark.parametrize("label", [5, 39, 70_001])
def test_one_label_far_above_the_rest_in_a_long_label_space(label, bf16):
    flush(f"far label {label} of 131,105 bf16={bf16}")
    B = 256
    wl = synth.Workload("labels-long", 5_000, 131_105, 256, B, 0.01, True, "lognormal", 3.5, 0.8, 500, 1.05, "uniform",
                        "poisson", 4.0, 1.2, 2)
    s = Setup(wl, 256, B, bf16=bf16)
    try:
        p = trained_scale(s.F, s.L, 6)
        p["b2"][label] = 200.0
        write_params(s.m, p)
        x, y = s.host_batch(0, B)
        loss = asgd.asgd_train_step(s.m, s.xb(0, B), s.yb(0, B), 0.5, want_loss=True)
        ref, ref_loss, g, _ = om.train_step(p, x, y, 0.5, "bf16" if bf16 else "fp32")
        assert np.isfinite(loss) and abs(loss - ref_loss) <= 1e-3 * abs(ref_loss), (loss, ref_loss)
        got = asgd.asgd_model_get_params(s.m, asgd.ASGD_PARAM_B1, (H,)).astype(np.float64)
        d, dr = got - p["b1"], ref["b1"].astype(np.float64) - p["b1"]
        assert np.linalg.norm(d - dr) <= 2e-2 * np.linalg.norm(dr)
    finally:
        s.free()
