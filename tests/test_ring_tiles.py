"""The deep-ring prefill tiles (launches that leave the large tiles' CUs idle):
every tile and epilogue against the oracle at the edges of its tiles, and the
register budget of their kernels."""
import os
import re

import numpy as np
import pytest
import torch

from oracle import ot_oracle as O
from paper_2406_18832_amd import ot
from tests._tol import assert_fp16_close
from tests.test_kernel_resources import CSRC, kernel_resources

# (tokens, channels, K) -> the tile that runs on 256 CUs.  Ragged tokens,
# channels and K (K = 16: less than one K step of most waves; 144, 272: a K
# tail; 48 .. 528: fewer K tiles than ring stages), whole 16-byte output rows
# and odd ones, exact multiples of the tile.
TILES = {(65, 33, 16): "32x32", (97, 515, 48): "32x32", (131, 104, 2064): "32x32",
         (97, 2050, 272): "32x64", (128, 4096, 528): "32x64",
         (67, 4102, 528): "64x64", (127, 4104, 1040): "64x64",
         (65, 8197, 272): "64x128", (128, 10240, 768): "64x128",
         (161, 8250, 8208): "128x96", (131, 8197, 272): "128x128", (256, 8200, 1040): "128x128",
         (129, 16390, 272): "192x128", (300, 1000, 272): "32x64", (383, 16390, 272): "256x128"}

# The same over a K that fills every stage of the ring more than twice, with a
# tail: K tiles loaded into stages that hold older ones, where a wrong count of
# loads in flight, a stage handed over early or a missing barrier would show.
REUSED = {(131, 107, 4368): "32x32", (97, 2050, 2832): "32x64", (67, 4102, 2320): "64x64",
          (97, 8197, 2064): "64x128", (191, 10250, 2064): "128x96", (131, 8197, 1296): "128x128",
          (129, 16390, 1040): "192x128", (383, 16390, 1040): "256x128"}
RING = {"32x32": (256, 8), "32x64": (256, 5), "64x64": (256, 4), "64x128": (256, 3),
        "128x96": (128, 5), "128x128": (128, 4), "192x128": (128, 3), "256x128": (128, 3)}  # BK, stages


def test_rings_and_their_reuse():
    """RING is what the library compiles, and REUSED goes round each ring twice."""
    with open(os.path.join(CSRC, "ot_ring.hip")) as f:
        made = re.findall(r"^  OT_RING\((\d+), (\d+), (\d+), \d+, \d+, \d+, (\d+)\);", f.read(), re.M)
    assert {f"{bn}x{bm}": (int(bk), int(stages)) for bn, bm, bk, stages in made} == RING
    assert sorted(REUSED.values()) == sorted(RING)
    for (M, N, K), tile in REUSED.items():
        bk, stages = RING[tile]
        assert -(-K // bk) >= 2 * stages + 1 and K % bk and N % 8, (M, N, K)


def test_every_ring_tile_is_picked():
    if torch.cuda.is_available() and torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the tile choice depends on the CU count")
    for shape, tile in [*TILES.items(), *REUSED.items()]:
        assert ot.ot_qlinear_plan(*shape) == "prefill " + tile, shape


@pytest.mark.timeout(900)
def test_ring_kernels_do_not_spill(tmp_path):
    res = kernel_resources(os.path.join(CSRC, "ot_ring.hip"), tmp_path)
    ring = {k: v for k, v in res.items() if "qgemm_ring" in k}
    assert len(ring) == 24  # 8 tiles, 3 epilogues
    assert not {k: v for k, v in ring.items() if v["spill"] != 0}


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [*TILES, *REUSED])
@pytest.mark.parametrize("flavour", ["channel", "token", "asym"])
def test_ring_tiles_match_the_oracle(M, N, K, flavour):
    print(f"[case] ring {flavour} M={M} N={N} K={K} plan={ot.ot_qlinear_plan(M, N, K)}", flush=True)
    r = np.random.default_rng(M + 3 * N + 7 * K)
    Xq = r.integers(-127, 128, size=(M, K)).astype(np.int8)
    Wq = r.integers(-127, 128, size=(N, K)).astype(np.int8)
    sW = (r.uniform(0.5, 2.0, size=N) * 1e-4).astype(np.float32)
    bp = r.normal(0, 1, size=N).astype(np.float32)
    args, acc = [dev(Xq), dev(Wq)], O.int_gemm(Xq, Wq)
    if flavour == "channel":
        ref = O.epilogue(acc, sW, bp)
        run = lambda **k: ot.qlinear(*args, dev(sW), dev(bp), 8, 8, **k)
    elif flavour == "token":
        sX = r.uniform(0.01, 0.2, size=M).astype(np.float32)
        ref = O.epilogue_per_token(acc, sX, sW, bp)
        run = lambda **k: ot.qlinear_per_token(*args, dev(sX), dev(sW), dev(bp), 8, 8, **k)
    else:
        zW = r.integers(-128, 128, size=N).astype(np.int32)
        acc = O.int_gemm_asym(Xq, Wq, zW)
        ref = O.epilogue(acc, sW, bp)
        run = lambda **k: ot.qlinear_asym(*args, dev(sW), dev(zW), dev(bp), 8, 8, **k)
    Y = run()
    Y2, got = run(want_acc=True)
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), acc)
    assert_fp16_close(Y.cpu().numpy(), ref)
    assert torch.equal(Y, Y2)
