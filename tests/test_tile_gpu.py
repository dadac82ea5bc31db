"""Far partitions tiled in time (one reading of a far partition row serves
eight blocks): the shapes at the edges of that tiling against the FP64 oracle,
sample by sample past the filters' ends, and the window of spectra it reads
(Sec. IV step 2: block n needs spectra n - p only)."""
import numpy as np
import pytest

import oracle
from paper_2509_04390_amd import workloads

from test_parity_gpu import BF16_DB, FP16_DB, FP32_DB, check_db, make_filters, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rta():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    from paper_2509_04390_amd import rta as mod
    return mod


# (B, lens[q][l], flags): 18 partitions are the first to be tiled (9 far
# ones); runs of 8 rows, 16 runs of a 16-bin slice make 128-row chunks
SHAPES = [
    (16, [[16 * 17]], 0), (16, [[16 * 18]], 0), (16, [[16 * 18 + 1]], 0),
    (16, [[16 * 1100, 16 * 500 + 3]], 0),
    (64, [[64 * 25, 64 * 26 + 1, 64 * 18 + 5], [64 * 200 - 3, 0, 700]], 0),
    (128, [[128 * 137]], 0), (128, [[128 * 138, 128 * 10, 128 * 9 + 1]], 0),
    (128, [[128 * (20 + 3 * l) - l for l in range(17)]], 0),      # two outputs per item, one left
    (128, [[128 * 40 - 5] * 3 for _ in range(5)], 0),             # more inputs than a head prefetches
    (64, [[64 * 20 - q, 64 * 18 + q, 0 if q % 3 else 64 * 40] for q in range(40)], 0),  # several inputs per slot
    (256, [[256 * 70 + 100, 256 * 30]], 0),
    (512, [[512 * 40, 512 * 33 + 7]], 0),
    (4096, [[4096 * 19, 5]], 0),
    (16, [[16 * 60, 16 * 21]], 2), (128, [[128 * 45 + 7], [128 * 19]], 2),   # n_f = 3B
]


@pytest.mark.parametrize("spectra,limit", [("fp32", FP32_DB), ("fp16", FP16_DB), ("bf16", BF16_DB)])
@pytest.mark.parametrize("shape", range(len(SHAPES)))
def test_tiled_shapes_match_oracle(rta, shape, spectra, limit):
    B, lens, flags = SHAPES[shape]
    filt = make_filters(700 + shape, lens)
    n = max(max(r) for r in lens) // B * B + 20 * B
    x = workloads.white_noise(701 + shape, len(lens), n)
    say(f"B={B} lens={lens} flags={flags} {spectra}")
    with rta.Convolver(filt, B, spectra=spectra, flags=flags) as cv:
        y = cv.run_device(x)
        cv.reset()
        assert np.array_equal(cv.run(x[:, :40 * B]), y[:, :40 * B])
    rng = np.random.default_rng(shape)
    idx = np.unique(np.r_[0, B - 1, B, n - 1, rng.integers(0, n, 300)])
    check_db(y[:, idx], oracle.direct_at(x, filt, idx), limit, f"tiled B={B}")


@pytest.mark.parametrize("G", [1, 2, 4])
def test_tiled_outputs_per_group(rta, G):
    B, L = 64, 9
    lens = [[64 * (30 + 2 * l) + l for l in range(L)], [64 * 50] * L]
    filt = make_filters(740, lens)
    n = 90 * B
    x = workloads.white_noise(741, 2, n)
    with rta.Convolver(filt, B, tuning=rta.make_tuning(outputs_per_group=G)) as cv:
        y = cv.run_device(x)
    check_db(y, oracle.direct(x, filt, 0, n), FP32_DB, f"tiled G={G}")


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_a_bad_block_is_heard_for_its_partitions_only(rta, bad):
    """Blocks before a NaN or infinite one are untouched bit for bit, and the
    outputs recover as soon as the last partition has passed it."""
    B, K, at = 64, 40, 60
    filt = make_filters(750, [[B * K, B * K]])
    x = workloads.white_noise(751, 1, (at + K + 40) * B)
    xb = x.copy()
    xb[0, at * B + 5] = bad
    with rta.Convolver(filt, B) as cv:
        y = cv.run_device(x)
        cv.reset()
        yb = cv.run_device(xb)
    assert np.array_equal(y[:, :at * B], yb[:, :at * B])
    assert not np.isfinite(yb[:, at * B:(at + K) * B]).any()
    # block at + K's window still begins with the bad block; partition K - 1
    # pairs block at + K with the spectrum of [x(at), x(at + 1)]
    assert np.array_equal(y[:, (at + K + 1) * B:], yb[:, (at + K + 1) * B:])


@pytest.mark.parametrize("B,rows", [(32, 18), (64, 17), (64, 18), (64, 41), (128, 19), (128, 130), (256, 30), (512, 20)])
@pytest.mark.parametrize("Q,L,spectra,limit", [(1, 6, "fp32", FP32_DB), (3, 2, "fp32", FP32_DB), (1, 3, "fp16", FP16_DB)])
def test_tiled_feedback_paths(rta, B, rows, Q, L, spectra, limit):
    """Feedback paths around and beyond the first tiled length, of unequal
    lengths, in a loop of small gain (rooms of about 30 per path)."""
    filt = make_filters(760 + B, [[3 * B + 7 * l + q for l in range(L)] for q in range(Q)])
    fb = make_filters(761 + rows, [[B * rows - 11 * l - q for l in range(L)] for q in range(Q)])
    fb = [[(5e-5 * f).astype(np.float32) for f in row] for row in fb]
    if spectra == "fp16":  # normal numbers in 16 bits, the same loop gain
        fb = [[64 * f for f in row] for row in fb]
        filt = [[f / 64 for f in row] for row in filt]
    n = (rows + 24) * B
    x = workloads.white_noise(762, Q, n)
    say(f"B={B} rows={rows} Q={Q} L={L} {spectra}")
    with rta.Convolver(filt, B, spectra=spectra) as cv:
        cv.set_feedback(fb, spectra=spectra)
        assert cv.info()["feedback_fused"] == 1
        y = cv.run_device(x)
    check_db(y, oracle.feedback_loop(x, filt, fb, B)[0], limit, f"feedback rows={rows}")


def block_us(cv, blocks=64):
    import torch
    x = torch.zeros((cv.n_in, cv.block), device="cuda")
    y = torch.empty((cv.n_out, cv.block), device="cuda")
    best = 1e9
    for _ in range(6):
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0.record()
        for _ in range(blocks):
            cv.process_device(x, y)
        t1.record()
        t1.synchronize()
        best = min(best, t0.elapsed_time(t1) * 1e3 / blocks)
    return best


def test_near_rows_of_many_outputs_take_the_whole_chip(rta):
    """8 inputs to 64 outputs, 18 partitions: most rows are near ones.  All on
    one XCD they took 13.9 us per block where reading every row every block
    takes 6.9."""
    B = 128
    filt = make_filters(790, [[B * 18] * 64] * 8)
    with rta.Convolver(filt, B) as cv:
        tiled = block_us(cv)
    with rta.Convolver(filt, B, tuning=rta.make_tuning(tail_rows=8)) as cv:
        plain = block_us(cv)
    say(f"  tiled {tiled:.1f} us, every row every block {plain:.1f} us")
    assert tiled < 1.4 * plain


def one_filter(B, parts, Q, L, seed):
    """Q x L paths through the same few filters (host memory for one)."""
    f = (make_filters(seed, [[B * parts - 3]])[0][0] * 0.1).astype(np.float32)
    return [[f] * L for _ in range(Q)]


def test_tiled_where_only_graphs_lack_room(rta):
    """64 inputs of 18 partitions: the partial sums of 32 blocks (a graph's 16
    at once) take more than the spectra, those of 16 do not.  The far rows are
    then still read once for eight blocks, and a graph runs one block after
    another."""
    import torch
    B, parts, Q, L = 128, 18, 64, 128
    filt = one_filter(B, parts, Q, L, 770)
    x = workloads.white_noise(771, Q, 40 * B)
    xb = torch.from_numpy(np.ascontiguousarray(x.reshape(Q, 40, B).transpose(1, 0, 2))).cuda()
    with rta.Convolver(filt, B, spectra="fp16") as cv:
        info = cv.info()
        # (9 near rows and an eighth of 9 far ones, of 18)
        assert info["h_bytes_per_block"] == pytest.approx(info["spectra_bytes"] * (9 + 9 / 8) / 18)
        y = cv.run_device(x)
        cv.reset()
        out = torch.empty((20, L, B), device="cuda")
        with cv.graph(xb[:20].contiguous(), out, 20) as g:
            g.launch()
            torch.cuda.synchronize()
    assert np.array_equal(out.permute(1, 0, 2).reshape(L, -1).cpu().numpy(), y[:, :20 * B])
    ref = oracle.direct(np.sum(x, axis=0, dtype=np.float64)[None].astype(np.float32), [[filt[0][0]]], 0, x.shape[1])
    check_db(y[:1], ref, FP16_DB, "64 x 128 of 18 partitions")
    assert (y == y[0]).all()


def test_little_memory_left(rta):
    """Where the device has no room for the partial sums of 32 blocks, a context
    is made with fewer: same output, less memory."""
    import torch
    B, parts, Q, L = 128, 40, 128, 128
    filt = one_filter(B, parts, Q, L, 780)
    x = workloads.white_noise(781, Q, 50 * B)
    with rta.Convolver(filt, B, spectra="fp16") as cv:
        full = cv.info()["device_bytes"]
        y = cv.run_device(x)
    # room for all but 40 MB of it and of the 64 MB that stage the taps
    left = full + (64 << 20) - (40 << 20)
    torch.cuda.empty_cache()
    hold = []
    try:
        for size in (8 << 30, 1 << 30, 64 << 20, 2 << 20):
            while torch.cuda.mem_get_info()[0] - size >= left:
                hold.append(torch.empty(size, dtype=torch.uint8, device="cuda"))
        say(f"free {torch.cuda.mem_get_info()[0] >> 20} MB of {left >> 20}, full context {full >> 20} MB")
        with rta.Convolver(filt, B, spectra="fp16") as cv:
            assert cv.info()["device_bytes"] < full
            del hold[:]
            torch.cuda.empty_cache()
            assert np.array_equal(cv.run_device(x), y)
    finally:
        del hold[:]
        torch.cuda.empty_cache()
