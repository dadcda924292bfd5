"""Grids and workgroups that the entry points launch, without a GPU: the launch
configurations that the library hands to the HIP runtime are recorded and the
launches left out (a preloaded library), in a process of its own.  256 CUs, as
on MI355X, without a device."""
import os
import shutil
import subprocess
import sys

import pytest

from paper_2406_18832_amd import ot

RECORDER = r"""
#include <stddef.h>
#include <stdint.h>
struct dim3 { uint32_t x, y, z; };
extern "C" {
uint64_t ot_test_grid[3], ot_test_block[3], ot_test_launches;
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t, void *) {
  ot_test_grid[0] = g.x; ot_test_grid[1] = g.y; ot_test_grid[2] = g.z;
  ot_test_block[0] = b.x; ot_test_block[1] = b.y; ot_test_block[2] = b.z;
  ++ot_test_launches;
  return 1;  // nonzero: the launch is left out
}
}
"""

CALLER = r"""
import ctypes, sys
R, L = ctypes.CDLL(sys.argv[1]), ctypes.CDLL(sys.argv[2])
grid, block = ((ctypes.c_uint64 * 3).in_dll(R, n) for n in ("ot_test_grid", "ot_test_block"))
launches = ctypes.c_uint64.in_dll(R, "ot_test_launches")
vp, i64, ci, P = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int, 4096   # P: aligned, never read
for line in sys.stdin:
    name, M, N, K = line.split()
    M, N, K = int(M), int(N), int(K)
    launches.value = 0
    if name == "qlinear":
        L.ot_qlinear(vp(P), vp(P), vp(P), vp(P), i64(M), i64(N), i64(K), ci(8), ci(8), vp(P), None, None, None)
    else:
        L.ot_quantize_act_per_token(vp(P), i64(M), i64(K), ci(8), vp(P), vp(P), None)
    print(launches.value, *grid, *block, flush=True)
"""


@pytest.fixture(scope="module")
def launch(tmp_path_factory):
    """launch([(call, M, N, K), ...]) -> (grid, block) of each call's one launch."""
    d = tmp_path_factory.mktemp("launches")
    src, so = d / "recorder.cpp", d / "recorder.so"
    src.write_text(RECORDER)
    subprocess.run([os.environ.get("CXX") or shutil.which("g++") or "c++", "-shared", "-fPIC", "-O1",
                    str(src), "-o", str(so)], check=True)

    def run(calls):
        env = dict(os.environ, LD_PRELOAD=str(so))
        out = subprocess.run([sys.executable, "-c", CALLER, str(so), ot.LIB_PATH], env=env,
                             input="".join("%s %d %d %d\n" % c for c in calls), text=True,
                             capture_output=True, timeout=300)
        assert out.returncode == 0, out.stderr[-2000:]
        rows = [[int(v) for v in line.split()] for line in out.stdout.splitlines()]
        assert len(rows) == len(calls) and all(r[0] == 1 for r in rows), rows
        return [(r[1:4], r[4:7]) for r in rows]
    return run


# A launch takes fewer than 2^32 work-items per dimension.  Tall calls (tokens
# in the hundreds of millions by few channels, within 288 GB) on which the tile
# of the least estimated time has more, and the largest of the 256-token tiles'.
TALL = [(1 << 30, 1, 16), (1 << 30, 16, 16), (1 << 30, 33, 32), (1300000000, 64, 16),
        (1073741825, 8, 64), (2147483391, 1, 16), (1 << 29, 16, 16), (65, 1 << 30, 16)]


def test_prefill_grids_stay_within_the_launch_limit(launch):
    for (M, N, K), (grid, block) in zip(TALL, launch([("qlinear", *s) for s in TALL])):
        bn, bm = (int(v) for v in ot.ot_qlinear_plan(M, N, K).split()[1].split("x"))
        assert grid == [-(-M // bm) * -(-N // bn), 1, 1]
        assert grid[0] * block[0] < 1 << 32, (M, N, K, grid, block)


def test_per_token_quantizer_grids_stay_within_the_launch_limit(launch):
    """One workgroup per row: tens of millions of rows, within 288 GB."""
    sizes = [(33554432, 1552), (67108863, 2048), (22369622, 3104), (33554431, 4096), (22369622, 4112)]
    for (M, K), (grid, block) in zip(sizes, launch([("per_token", M, 0, K) for M, K in sizes])):
        assert grid == [M, 1, 1]
        assert grid[0] * block[0] < 1 << 32, (M, K, grid, block)


# (rows, K) -> threads of a row: 3 chunks each, except where 4 need a wave fewer
# up to K = 4096, and 8 beyond at the widths, rows and elements where their 2 to 4
# waves measured faster (either side of each line)
@pytest.mark.parametrize("M,K,threads", [
    (512, 1536, 64), (512, 1552, 64), (14544, 1696, 64), (4096, 2048, 64), (4096, 2064, 128),
    (9089, 3072, 128), (4096, 3088, 128), (8192, 4096, 128), (4096, 4112, 192), (4096, 5120, 256),
    (4096, 7680, 320), (1023, 7696, 384), (1024, 7696, 128), (4096, 8192, 128), (5197, 7696, 128),
    (5198, 7696, 384), (2048, 8416, 192), (1024, 10240, 192), (4000, 10256, 448),
    (4000, 12288, 512), (4000, 12304, 256), (100, 14768, 256), (4448, 14768, 256),
    (5468, 16384, 256), (5469, 16384, 704), (8496, 16304, 704), (1791, 16400, 704),
    (1792, 16400, 320), (3988, 17120, 320), (4374, 20480, 320), (4375, 20480, 896),
    (3000, 20496, 896),
    (3000, 24576, 1024), (4, 24592, 448)])
def test_per_token_quantizer_threads(launch, M, K, threads):
    (grid, block), = launch([("per_token", M, 0, K)])
    assert grid == [M, 1, 1] and block == [threads, 1, 1]
