"""Dispatch lines of the calls with few rows, each side against the oracle bit
for bit: the decode GEMM's 16-row tiles (up to 16 tokens), the static
quantizer's rows per wave, the per-token quantizer's and the fused LayerNorm's
chunks per thread."""
import numpy as np
import pytest
import torch

from oracle import ot_oracle as O
from paper_2406_18832_amd import ot
from tests._tol import assert_fp16_close

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


# channels up to 16 a CU (8 K groups), between 32-row tile lines on 256 CUs
# (9221, 12288: 16-row tiles even the CUs out), and past them (12289, 16384);
# K shorter than one stage, ragged, and several stages
@pytest.mark.parametrize("M,N,K", [(16, 4090, 272), (5, 2048, 4112), (1, 33, 48), (7, 9221, 528),
                                   (16, 12288, 272), (3, 12289, 144), (9, 16384, 272)])
@pytest.mark.parametrize("flavour", ["channel", "token", "asym"])
def test_decode_tiles_up_to_16_tokens(M, N, K, flavour):
    print(f"[case] decode {flavour} M={M} N={N} K={K} plan={ot.ot_qlinear_plan(M, N, K)}", flush=True)
    r = np.random.default_rng(M + N + K)
    Xq = r.integers(-127, 128, size=(M, K)).astype(np.int8)
    Wq = r.integers(-127, 128, size=(N, K)).astype(np.int8)
    sW = (r.uniform(0.5, 2.0, size=N) * 1e-4).astype(np.float32)
    bp = r.normal(0, 1, size=N).astype(np.float32)
    acc = O.int_gemm(Xq, Wq)
    if flavour == "channel":
        ref = O.epilogue(acc, sW, bp)
        Y, got = ot.qlinear(dev(Xq), dev(Wq), dev(sW), dev(bp), 8, 8, want_acc=True)
    elif flavour == "token":
        sX = r.uniform(0.01, 0.2, size=M).astype(np.float32)
        ref = O.epilogue_per_token(acc, sX, sW, bp)
        Y, got = ot.qlinear_per_token(dev(Xq), dev(Wq), dev(sX), dev(sW), dev(bp), 8, 8,
                                      want_acc=True)
    else:
        zW = r.integers(-128, 128, size=N).astype(np.int32)
        acc = O.int_gemm_asym(Xq, Wq, zW)
        ref = O.epilogue(acc, sW, bp)
        Y, got = ot.qlinear_asym(dev(Xq), dev(Wq), dev(sW), dev(zW), dev(bp), 8, 8, want_acc=True)
    assert np.array_equal(host(got), acc)
    assert_fp16_close(host(Y), ref)


# 256 CUs: one row per wave below 2048 row-waves (512 channels each), two
# below 8192, eight from there
@pytest.mark.parametrize("M,K", [(1, 16), (9, 528), (1023, 1024), (1025, 1024), (2047, 1040),
                                 (4097, 1024)])
def test_quantize_rows_per_wave(M, K):
    print(f"[case] quantize M={M} K={K}", flush=True)
    r = np.random.default_rng(M + K)
    x = (r.standard_normal((M, K)) * 3 + r.uniform(-5, 5, K)).astype(np.float16)
    z = r.uniform(-5, 5, K).astype(np.float32)
    inv_s = r.uniform(5, 30, K).astype(np.float32)
    assert np.array_equal(host(ot.quantize_act(dev(x), 8, dev(z), dev(inv_s))),
                          O.quantize_act(x, z, inv_s, 8))


@pytest.mark.parametrize("M,K", [(3, 16), (5, 1552), (2, 24576), (2, 24592), (1030, 784)])
def test_per_token_chunks_per_thread(M, K):
    print(f"[case] per-token M={M} K={K}", flush=True)
    r = np.random.default_rng(M + K)
    x = (r.standard_normal((M, K)) * 3).astype(np.float16)
    x[1] = 0
    Xq, sX = ot.quantize_act_per_token(dev(x), 8)
    rq, rs = O.quantize_act_per_token(x, 8)
    assert np.array_equal(host(Xq), rq) and np.array_equal(host(sX), rs)


# 4 chunks per thread (2048, 3088, 4096), 8 in 2, 3 and 4 waves, and beside them
@pytest.mark.parametrize("M,K", [(3, 2048), (2, 3088), (3, 4096), (1024, 7696), (1023, 10240),
                                 (1024, 10240), (2, 12288), (3, 12304), (2, 16384), (2, 16400),
                                 (1792, 16400)])
def test_per_token_fewer_threads(M, K):
    test_per_token_chunks_per_thread(M, K)


@pytest.mark.parametrize("M,K", [(1024, 784), (1025, 784), (2, 16384), (2, 16400)])
def test_layernorm_chunks_per_thread(M, K):
    print(f"[case] ln M={M} K={K}", flush=True)
    r = np.random.default_rng(M + K)
    h = (r.standard_normal((M, K)) * 2 + r.normal(0, 2, K)).astype(np.float16)
    h[1] -= h[1].mean(dtype=np.float64).astype(np.float16)
    gamma, beta = r.uniform(0.5, 1.5, K).astype(np.float16), r.normal(0, 1, K).astype(np.float16)
    z, inv_s = r.normal(0, 1, K).astype(np.float32), r.uniform(10, 40, K).astype(np.float32)
    got = host(ot.ln_quantize_act(dev(h), dev(gamma), dev(beta), 1e-5, 8, dev(z), dev(inv_s)))
    assert np.array_equal(got, O.ln_quantize_act(h, gamma, beta, 1e-5, z, inv_s, 8))
