"""Graph replay that runs several blocks at once (uniform partitions tiled in
time, 16 to 256 bins): bit for bit what one rta_process_device call per
block gives, for runs of whole and partial batches, replayed and mixed with
single blocks and resets, and with input and output in the same buffer."""
import numpy as np
import pytest

import oracle
from paper_2509_04390_amd import workloads

from test_graph_gpu import blocks_of, direct, to_signal
from test_parity_gpu import FP32_DB, check_db, make_filters, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rta():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    from paper_2509_04390_amd import rta as mod
    return mod


@pytest.mark.parametrize("M", [1, 5, 8, 16, 21, 64])
@pytest.mark.parametrize("B,lens,spectra", [(64, [[64 * 18, 64 * 30, 0], [64 * 33 + 5, 700, 64 * 19]], "fp32"),
                                            (16, [[16 * 20, 16 * 300 + 7]], "fp32"), (32, [[32 * 25], [32 * 18]], "bf16"),
                                            (128, [[128 * 45 + 1, 128 * 20]], "fp16"),
                                            (256, [[256 * 40]], "fp32")])
def test_runs_of_blocks_equal_single_blocks(rta, B, lens, spectra, M):
    import torch
    Q, L = len(lens), len(lens[0])
    filt = make_filters(840 + B, lens)
    total = 4 * M + 3 + max(0, 60 - 4 * M)
    x = workloads.white_noise(841, Q, total * B)
    xb = blocks_of(x, B)
    say(f"B={B} {spectra} M={M} blocks={total}")
    with rta.Convolver(filt, B, spectra=spectra) as cv:
        ref = direct(cv, xb)
        cv.reset()
        gin = torch.empty((M, Q, B), device="cuda")
        gout = torch.empty((M, L, B), device="cuda")
        yb = torch.empty_like(ref)
        with cv.graph(gin, gout, M) as g:
            for turn in range(2):  # the same graph again after a reset
                yb.zero_()
                pos = 0
                for step in ("g", "g", "d", "g", "d", "d", "g", "rest"):
                    n = M if step == "g" else 1 if step == "d" else total - pos
                    if step == "g":
                        gin.copy_(xb[pos:pos + M])
                        g.launch()
                        yb[pos:pos + M].copy_(gout)
                    else:
                        for b in range(pos, pos + n):
                            cv.process_device(xb[b], yb[b])
                    pos += n
                torch.cuda.synchronize()
                assert torch.equal(yb, ref), f"turn {turn}"
                cv.reset()
    if spectra == "fp32":
        check_db(to_signal(yb), oracle.direct(x, filt, 0, x.shape[1]), FP32_DB, f"graph runs M={M}")


def test_input_and_output_in_one_buffer(rta):
    import torch
    B, M = 128, 20
    filt = make_filters(850, [[B * 25]])
    x = workloads.white_noise(851, 1, 2 * M * B)
    xb = blocks_of(x, B)
    with rta.Convolver(filt, B) as cv:
        ref = direct(cv, xb)
        cv.reset()
        buf = torch.empty((M, 1, B), device="cuda")
        with cv.graph(buf, buf, M) as g:
            for k in range(2):
                buf.copy_(xb[k * M:(k + 1) * M])
                g.launch()
                torch.cuda.synchronize()
                assert torch.equal(buf, ref[k * M:(k + 1) * M])
