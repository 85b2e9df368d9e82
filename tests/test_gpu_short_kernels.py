"""The whole step at trained-scale weights where the output layer changes kernels: the forward
with waves on tiles of their own and the backward with waves on row blocks of their own, and the
kernels past the lines of their rules, with remainders in rows, labels and waves."""
import numpy as np
import pytest

import paper_2110_07029_amd as asgd
from oracle import model as om
from paper_2110_07029_amd import synth

from gpu_util import RTOL_BF16, RTOL_FP32, Setup, assert_update_close, flush, step_magnitudes, write_params
from test_gpu_trained_scale import trained_scale

pytestmark = pytest.mark.gpu


# All of these run the forward for short label splits; L = 7, 32, 33: less than a tile, a tile and
# one more.  Its splits have one tile each up to 1,024 labels and eight from 8,192 on; 65 and 129
# splits at 16,640 and 33,000 (the per-row pass takes 64 at a time).  Backward with bf16 operands:
# a workgroup per label block up to 512 blocks at 256 rows or less (16,384 | 16,385 labels), else
# up to 2,048 (65,536 | 65,537); the lines with fp32 operands and the forward's are below.
@pytest.mark.parametrize("B,L", [(1, 7), (1, 33), (33, 32), (64, 257), (65, 1_000), (256, 16_384), (255, 16_385),
                                 (257, 1_000), (300, 65_536), (257, 65_537), (1_000, 2_001),
                                 (128, 1_024), (128, 1_025), (40, 8_192), (40, 8_193),
                                 (16, 16_640), (20, 33_000)])
@pytest.mark.parametrize("bf16", [True, False])
def test_step_parity(B, L, bf16):
    if not bf16 and B * L > 5_000_000:
        pytest.skip("the oracle's time")
    flush(f"short kernels: B={B} L={L} bf16={bf16}")
    step_parity(B, L, bf16)


def step_parity(B, L, bf16):
    w = synth.Workload("short", 3_000, L, B, B, 0.5, True, "lognormal", 2.5, 0.6, 100, 1.05, "uniform", "poisson",
                       2.0, 1.1, 2)
    s = Setup(w, B, B, bf16=bf16)
    try:
        p = trained_scale(s.F, s.L, 8)
        write_params(s.m, p)
        x, y = s.host_batch(0, B)
        loss = asgd.asgd_train_step(s.m, s.xb(0, B), s.yb(0, B), 0.5, want_loss=True)
        ref, ref_loss, g, fw = om.train_step(p, x, y, 0.5, "fp32")
        assert abs(loss - ref_loss) <= 2e-3 * max(1.0, abs(ref_loss))
        got = s.params()
        mag = step_magnitudes(p, x, y, g, fw, 0.5)
        rtol = RTOL_BF16 if bf16 else RTOL_FP32
        for k in ("W2", "b2", "b1"):
            assert_update_close(k, p[k], got[k], ref[k], rtol, mag[k])
        t = g["touched"]
        assert_update_close("W1", p["W1"][t], got["W1"][t], ref["W1"][t], rtol, mag["W1"])
    finally:
        s.free()


def bwd_line(B):
    """Label blocks up to which the fp32 backward gives every block a workgroup."""
    return 2_048 if B > 512 else min(1_536, 512 + 4 * B)


@pytest.mark.parametrize("past", [0, 1])
@pytest.mark.parametrize("B", [1, 40, 128, 300, 513])
def test_step_parity_at_the_line_of_the_fp32_backward(B, past):
    """The last label count of the backward with a workgroup per label block, and one label more:
    the backward whose wavefronts own blocks and read H1 from global memory."""
    L = 32 * bwd_line(B) + past
    flush(f"fp32 backward's line: B={B} L={L}")
    step_parity(B, L, False)


# The forward's line: 32,768 (tile, 32-row block) products, where B is above 64.  The last on one
# side and the first on the other, by labels and by rows, up to the largest batch; the bf16 backward
# is the one with a block per wave (256 rows), the chunked one (520 rows at 65,568 labels) or that
# of few blocks, the fp32 one reads H1 from global memory at 256 rows.
@pytest.mark.parametrize("B,L", [(256, 131_072), (256, 131_073), (2_048, 16_384), (2_048, 16_385), (1_024, 32_768),
                                 (1_025, 32_768), (520, 65_568)])
@pytest.mark.parametrize("bf16", [True, False])
def test_step_parity_at_the_line_of_the_forward(B, L, bf16):
    flush(f"forward's line: B={B} L={L} bf16={bf16}")
    step_parity(B, L, bf16)
