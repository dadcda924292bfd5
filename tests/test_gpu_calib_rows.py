"""Calibration's two min/max kernels (whole 16-byte chunks and general) against
the oracle, bit for bit, at the edges of their tiles; zeros of both signs,
the extremes, and non-finite values anywhere in a row block."""
import numpy as np
import pytest
import torch

from oracle import ot_oracle as O
from paper_2406_18832_amd import ot

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _same(got, ref):
    torch.cuda.synchronize()
    for g, r, name in zip(got, ref, ["minmax", "z", "s", "inv_s"]):
        assert np.array_equal(g.cpu().numpy().view(np.uint32), r.view(np.uint32)), name


# K: one chunk, ragged against a wave's 512 channels, general widths, and past
# the one-launch finalize (65536); rows: one, ragged against the 8 rows a wave
# takes and the 32 of a workgroup, more than the grid takes at once
@pytest.mark.parametrize("rows,K", [(1, 8), (7, 520), (33, 512), (131, 1032), (64, 4096), (9, 37),
                                    (3, 1004), (300, 16), (5000, 24), (3, 65536), (2, 65544)])
def test_calibrate_widths(rows, K):
    print(f"[case] calibrate rows={rows} K={K}", flush=True)
    r = np.random.default_rng(rows + K)
    a = r.normal(0, 3, size=(rows, K)).astype(np.float16)
    a[:, 0] = -0.0
    a[:, K // 2] = 2.0
    a[rows // 2, K - 1] = np.float16(65504)
    a[rows - 1, K - 1] = np.float16(-65504)
    a[:, K // 3] = -np.abs(a[:, K // 3])
    b = r.normal(1, 1, size=(5, K)).astype(np.float16)
    b[:, 0] = -0.0
    _same(ot.calibrate([a, b], 8), O.calibrate([a, b], 8))


@pytest.mark.parametrize("K", [512, 37, 65544])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_calibrate_non_finite_leaves_outputs(K, bad):
    print(f"[case] calibrate non-finite {bad} K={K}", flush=True)
    for row, col in [(0, 0), (40, K - 1), (8, K // 2)]:
        x = np.ones((41, K), np.float16)
        x[row, col] = bad
        minmax = torch.empty(2 * K, dtype=torch.float32, device="cuda")
        z, s, inv_s = (torch.full((K,), 7.0, device="cuda") for _ in range(3))
        with pytest.raises(ot.OTError) as e:
            ot.ot_calibrate(dev(x), 8, True, minmax, z, s, inv_s)
        assert e.value.code == ot.OT_ENONFINITE
        good = dev(np.ones((3, K), np.float16))
        with pytest.raises(ot.OTError):  # the state stays poisoned
            ot.ot_calibrate(good, 8, False, minmax, z, s, inv_s)
        assert torch.all(z == 7.0) and torch.all(s == 7.0) and torch.all(inv_s == 7.0)
        ot.ot_calibrate(good, 8, True, minmax, z, s, inv_s)
        assert torch.all(z == 1.0) and torch.all(s == 1.0)


def test_calibrate_misaligned_rows():
    print("[case] calibrate misaligned", flush=True)
    a = np.random.default_rng(2).normal(0, 3, size=(50, 256)).astype(np.float16)
    flat = torch.empty(a.size + 1, dtype=torch.float16, device="cuda")
    view = flat[1:].view(a.shape)
    view.copy_(dev(a))
    _same(ot.calibrate([view], 6), O.calibrate([a], 6))


def test_synchronous_calls_from_threads():
    """Folds and calibrations on several threads and streams at once, some
    with non-finite input: each reports its own."""
    import threading
    print("[case] synchronous calls from threads", flush=True)
    K, N = 256, 8
    good, poor = np.ones((16, K), np.float16), np.ones((16, K), np.float16)
    poor[5, 9] = np.nan
    W, V = np.ones((N, K), np.float16), np.ones((N, K), np.float16)
    V[3, 3] = np.inf
    data = [[dev(a) for a in (good, W)], [dev(a) for a in (poor, V)]]
    z, s = torch.zeros(K, device="cuda"), torch.ones(K, device="cuda")
    torch.cuda.synchronize()
    wrong = []

    def work(i):
        st = torch.cuda.Stream()
        x, w = data[i % 2]
        with torch.cuda.stream(st):
            for _ in range(20):
                for call in (lambda: ot.calibrate([x], 8), lambda: ot.fold_weights(w, None, 8, z, s)):
                    try:
                        call()
                        code = ot.OT_OK
                    except ot.OTError as e:
                        code = e.code
                    if code != (ot.OT_ENONFINITE if i % 2 else ot.OT_OK):
                        wrong.append((i, code))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not wrong
