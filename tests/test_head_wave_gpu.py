"""Heads that run by wavefronts (first tiers of 16 to 256 bins): inputs
beyond one round of the four wavefronts, partial slots beyond what is
prefetched, later tiers' rings, the separate and the fused feedback
convolution, and unaligned device buffers, against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2509_04390_amd import workloads

from test_parity_gpu import FP32_DB, check_db, make_filters, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rta():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    from paper_2509_04390_amd import rta as mod
    return mod


@pytest.mark.parametrize("B", [16, 32, 64, 128, 256])
@pytest.mark.parametrize("Q,rows", [(1, 1), (1, 70), (4, 30), (5, 9), (9, 4)])
def test_inputs_and_slots(rta, B, Q, rows):
    """rows partitions read one to an item: up to 68 slots per input."""
    L = 3
    lens = [[max(1, B * rows - 7 * q - 3 * l) for l in range(L)] for q in range(Q)]
    filt = make_filters(800 + B + Q, lens)
    n = B * (rows + 6)
    x = workloads.white_noise(801, Q, n)
    say(f"B={B} Q={Q} rows={rows}")
    with rta.Convolver(filt, B, tuning=rta.make_tuning(tail_rows=1)) as cv:
        y = cv.run(x)
        cv.reset()
        assert np.array_equal(cv.run_device(x), y)
    check_db(y, oracle.direct(x, filt, 0, n), FP32_DB, f"B={B} Q={Q} rows={rows}")


@pytest.mark.parametrize("B,scheme", [(16, [(16, 8), (64, 3), (256, 0)]), (32, [(32, 12), (256, 0)]), (64, [(64, 12), (512, 0)]), (128, [(128, 15), (1024, 14), (8192, 0)]),
                                      (256, [(256, 15), (2048, 0)]),
                                      (64, [(64, 12), (256, 8), (512, 8), (1024, 0)])])
def test_rings_and_feedback(rta, B, scheme):
    Q, L = 2, 5
    lens = [[9000 + 100 * l for l in range(L)] for _ in range(Q)]
    filt = make_filters(820, lens)
    # (loop gain about 0.1: the room's gain is about 32 per path)
    fb = [[(5e-5 * f).astype(np.float32) for f in row] for row in make_filters(821, [[3 * B + 5] * L] * Q)]
    n = -(-12000 // B) * B
    x = workloads.white_noise(822, Q, n)
    with rta.Convolver(filt, B, scheme=scheme) as cv:
        check_db(cv.run_device(x), oracle.direct(x, filt, 0, n), FP32_DB, f"B={B} {scheme}")
        ref = oracle.feedback_loop(x, filt, fb, B)[0]
        for spectra, fused in (("fp32", 1), ("fp16", 0)):
            cv.set_feedback(fb, spectra=spectra)
            assert cv.info()["feedback_fused"] == fused
            y = cv.run_device(x)
            # (16-bit paths: their rounding, 60 dB down, on a feedback signal
            # that is itself below the output)
            check_db(y, ref, FP32_DB if fused else -60.0, f"feedback {spectra}")


@pytest.mark.parametrize("B", [16, 32, 64, 128, 256])
def test_unaligned_device_buffers(rta, B):
    import torch
    filt = make_filters(830, [[B * 20, B * 3], [B * 7, B]])
    n = B * 30
    x = workloads.white_noise(831, 2, n)
    with rta.Convolver(filt, B) as cv:
        want = cv.run_device(x)
        cv.reset()
        buf = torch.empty(2 * B + 3, device="cuda")
        out = torch.empty(2 * B + 3, device="cuda")
        got = np.empty_like(want)
        for b in range(n // B):
            buf[1:1 + 2 * B] = torch.from_numpy(np.ascontiguousarray(x[:, b * B:(b + 1) * B])).reshape(-1)
            cv.process_device(buf[1:1 + 2 * B], out[3:3 + 2 * B])
            got[:, b * B:(b + 1) * B] = out[3:3 + 2 * B].reshape(2, B).cpu().numpy()
    assert np.array_equal(got, want)


from test_parity_gpu import BF16_DB, FP16_DB  # noqa: E402


@pytest.mark.parametrize("B,spectra,flags", [(256, "fp16", 0), (256, "bf16", 0), (512, "fp32", 0), (1024, "fp16", 0),
                                             (16, "fp32", 2), (32, "fp16", 2), (128, "fp32", 2), (512, "fp32", 2)])
@pytest.mark.parametrize("Q,rows", [(1, 40), (4, 17), (5, 9), (9, 4)])
def test_workgroup_heads(rta, B, spectra, flags, Q, rows):
    """Heads that run by workgroups: inputs and partial slots that are whole and
    broken multiples of those a thread has in flight (rows partitions read one
    to an item), plain and as feedback heads of Q outputs."""
    L = 3
    lens = [[max(1, B * rows - 7 * q - 3 * l) for l in range(L)] for q in range(Q)]
    filt = [[(f / 64).astype(np.float32) for f in row] for row in make_filters(870 + Q, lens)]
    n = B * (rows + 6)
    x = workloads.white_noise(871, Q, n)
    limit = {"fp32": FP32_DB, "fp16": FP16_DB, "bf16": BF16_DB}[spectra]
    say(f"B={B} Q={Q} rows={rows} {spectra} flags={flags}")
    with rta.Convolver(filt, B, spectra=spectra, flags=flags, tuning=rta.make_tuning(tail_rows=1)) as cv:
        y = cv.run(x)
        cv.reset()
        assert np.array_equal(cv.run_device(x), y)
    check_db(y, oracle.direct(x, filt, 0, n), limit, f"B={B} Q={Q} rows={rows}")
    # outputs of this room fed back into L microphones (loop gain about 0.1)
    fb = [[(0.004 * f).astype(np.float32) for f in row] for row in make_filters(872, [[B * 3 + q for q in range(Q)]] * L)]
    room = [[filt[q][l] for q in range(Q)] for l in range(L)]
    m = workloads.white_noise(873, L, n)
    with rta.Convolver(room, B, spectra=spectra, flags=flags) as cv:
        cv.set_feedback(fb, spectra=spectra)
        assert cv.info()["feedback_fused"] == 1
        y = cv.run_device(m)
    check_db(y, oracle.feedback_loop(m, room, fb, B)[0], limit, f"feedback B={B} Q={Q}")
