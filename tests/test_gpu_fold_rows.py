"""The weight fold's two kernels (whole 16-byte chunks held in registers, and
the general one) against the oracle: codes, scales and zero points bit for
bit, bias within one fp32 unit, in every mode, at the edges of their ranges."""
import numpy as np
import pytest
import torch

from oracle import ot_oracle as O
from paper_2406_18832_amd import ot
from tests._tol import assert_fp32_within_ulps

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _check(mode, W, b, z, s, bits, Wdev=None):
    Wd = dev(W) if Wdev is None else Wdev
    bd = None if b is None else dev(b)
    if mode == "channel":
        got = ot.fold_weights(Wd, bd, bits, dev(z), dev(s))
        ref = O.fold_weights(W, b, z, s, bits)
    elif mode == "token":
        got = ot.fold_weights_per_token(Wd, bd, None, bits)
        ref = O.fold_weights_per_token(W, b, None, bits)
    else:
        got = ot.fold_weights_asym(Wd, bd, bits, dev(z), dev(s))
        ref = O.fold_weights_asym(W, b, z, s, bits)
    torch.cuda.synchronize()
    got = [t.cpu().numpy() for t in got]
    for g, r in zip(got[:-1], ref[:-1]):
        assert np.array_equal(g, r), mode
    assert_fp32_within_ulps(got[-1], ref[-1], 1)


# K: one chunk; ragged against the 64-lane waves; both sides of the register
# kernel's configurations (6144, 8192, 16384, 20480, 32768, 65536); not whole chunks (general
# kernel).  N: not a multiple of its 4 rows per workgroup.
@pytest.mark.parametrize("N,K", [(1, 8), (5, 40), (7, 520), (6, 6144), (6, 6152), (3, 8192), (9, 8200),
                                 (5, 16384), (3, 16392), (2, 20480), (2, 20488), (5, 32768), (3, 32776), (2, 65536), (2, 65544),
                                 (6, 37), (4, 1004)])
@pytest.mark.parametrize("mode", ["channel", "token", "asym"])
def test_fold_widths(mode, N, K):
    print(f"[case] fold {mode} N={N} K={K}", flush=True)
    r = np.random.default_rng(N + 3 * K)
    W = (r.standard_normal((N, K)) * 0.02).astype(np.float16)
    b = r.normal(0, 0.02, N).astype(np.float16) if K % 16 else None
    z = r.normal(0, 3, K).astype(np.float32)
    s = r.uniform(0.01, 0.8, K).astype(np.float32)
    _check(mode, W, b, z, s, 8 if N % 2 else 6)


@pytest.mark.parametrize("bits", [8, 6, 2])
@pytest.mark.parametrize("mode", ["channel", "token", "asym"])
def test_fold_ties_and_extremes(mode, bits):
    """Quotients exactly on and one fp16 unit beside half-integers (where the
    fp32 estimate cannot decide), one-sided and zero rows, scales at fp32's ends."""
    print(f"[case] fold ties {mode} bits={bits}", flush=True)
    K = 512
    r = np.random.default_rng(bits)
    top = 2 ** bits - 1 if mode == "asym" else 2 ** (bits - 1) - 1
    halves = r.integers(-2 * top, 2 * top + 1, size=K) / 2.0   # integers and halves
    halves[0], halves[1] = top, -top if mode != "asym" else 0.0
    if mode == "asym":
        halves = np.abs(halves) / 2.0
        halves[0] = top
    rows = [halves, np.nextafter(halves.astype(np.float16), np.float16(0)).astype(np.float64),
            np.abs(halves), -np.abs(halves), np.zeros(K), halves * 0.125,
            r.standard_normal(K) * 100, np.where(np.arange(K) == 3, 65504.0, 2.0 ** -24)]
    W = np.stack(rows).astype(np.float16)
    b = r.normal(0, 1, len(rows)).astype(np.float16)
    z = r.normal(0, 2, K).astype(np.float32)
    for scale in (1.0, 0.1, 1e-37, 1e33):
        s = np.full(K, scale, dtype=np.float32)
        _check(mode, W, b, z, s, bits)


def test_fold_misaligned_weights_take_the_general_kernel():
    print("[case] fold misaligned", flush=True)
    r = np.random.default_rng(1)
    N, K = 5, 256
    W = (r.standard_normal((N, K)) * 0.02).astype(np.float16)
    flat = torch.empty(N * K + 1, dtype=torch.float16, device="cuda")
    view = flat[1:].view(N, K)
    view.copy_(dev(W))
    z = r.normal(0, 3, K).astype(np.float32)
    s = r.uniform(0.01, 0.8, K).astype(np.float32)
    for mode in ("channel", "token", "asym"):
        _check(mode, W, None, z, s, 8, view)


@pytest.mark.parametrize("K", [512, 37])
@pytest.mark.parametrize("mode", ["channel", "token", "asym"])
def test_fold_reports_non_finite_and_recovers(mode, K):
    print(f"[case] fold non-finite {mode} K={K}", flush=True)
    z, s = np.zeros(K, np.float32), np.ones(K, np.float32)
    for where, bad in [((2, K - 1), np.inf), ((0, 0), np.nan), ((6, 9), -np.inf)]:
        W = np.ones((7, K), np.float16)
        W[where] = bad
        with pytest.raises(ot.OTError) as e:
            _check(mode, W, None, z, s, 8)
        assert e.value.code == ot.OT_ENONFINITE
        _check(mode, np.ones((7, K), np.float16), None, z, s, 8)
    b = np.array([0, 1, np.inf, 0, 0, 0, 0], np.float16)
    with pytest.raises(ot.OTError):
        _check(mode, np.ones((7, K), np.float16), b, z, s, 8)
