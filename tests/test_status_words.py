"""How the synchronous calls (calibration, fold) learn of non-finite values:
from a status word in pinned host memory, or from their outputs read back where
there is no word.  The host code of ot_api.hip against a stand-in runtime and
stand-in launchers, on the CPU, each scene in a process of its own."""
import subprocess

import pytest

from paper_2406_18832_amd import build_lib

DRIVER = r"""
#include <math.h>
#include <stdlib.h>
#include <string.h>
#include <thread>
#include <vector>
#include "ot_common.h"

// ---- the runtime and the launchers -------------------------------------------
static bool g_capturing = false, g_pinned = true, g_bad = false;
static hipError_t g_launch = hipSuccess;
static int g_copies = 0, g_finalized = 0;
extern "C" {
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
  *s = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  return g_capturing ? hipErrorStreamCaptureUnsupported : hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
  if (!g_pinned) return hipErrorOutOfMemory;
  *p = calloc(1, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
  if (!g_capturing) memcpy(d, s, n);
  ++g_copies;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *) { return hipSuccess; }
}
namespace ot {
static hipError_t fold(int64_t N, float *sW, float *bp, int *status) {
  for (int64_t n = 0; n < N; ++n) sW[n] = 1.f, bp[n] = 0.f;
  if (g_bad && g_launch == hipSuccess && !g_capturing) {
    sW[N - 1] = NAN;
    if (status) *status = 1;
  }
  return g_launch;
}
hipError_t launch_fold(const uint16_t *, const uint16_t *, int64_t N, int64_t, int, const float *,
                       const float *, int8_t *, float *sW, float *bp, int *st, hipStream_t) {
  return fold(N, sW, bp, st);
}
hipError_t launch_fold_per_token(const uint16_t *, const uint16_t *, const float *, int64_t N, int64_t,
                                 int, int8_t *, float *sW, float *bp, int *st, hipStream_t) {
  return fold(N, sW, bp, st);
}
hipError_t launch_fold_asym(const uint16_t *, const uint16_t *, int64_t N, int64_t, int, const float *,
                            const float *, int8_t *, float *sW, int32_t *, float *bp, int *st,
                            hipStream_t) {
  return fold(N, sW, bp, st);
}
hipError_t launch_calib_reset(float *, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_calib_minmax(const uint16_t *, int64_t, int64_t K, float *mm, hipStream_t) {
  for (int64_t k = 0; k < 2 * K; ++k) mm[k] = k < K ? -1.f : 1.f;
  if (g_bad) mm[K] = NAN;
  return hipSuccess;
}
bool calib_finish_ok(int64_t K) { return K <= 65536; }
hipError_t launch_calib_finish(const float *, int64_t K, int, float *z, float *, float *, int *status,
                               hipStream_t) {
  if (g_launch != hipSuccess || g_capturing) return g_launch;
  if (g_bad) *status = 1;
  else z[0] = 1.f;
  return hipSuccess;
}
hipError_t launch_calib_finalize(const float *, int64_t, int, int, float *z, float *, float *,
                                 hipStream_t) {
  ++g_finalized;
  z[0] = 1.f;
  return hipSuccess;
}
}  // namespace ot

// ---- the four calls ------------------------------------------------------------
constexpr int64_t N = 8, K = 16;
static uint16_t W[N * K];
static int8_t Wq[N * K];
static ot_status call(int which, float *first = nullptr) {
  float z[K] = {}, s[K] = {}, inv[K] = {}, mm[2 * K], sW[N], bp[N];
  int32_t zW[N];
  ot_status rc;
  if (which == 0) rc = ot_fold_weights(W, nullptr, N, K, 8, z, s, Wq, sW, bp, nullptr);
  else if (which == 1) rc = ot_fold_weights_per_token(W, nullptr, nullptr, N, K, 8, Wq, sW, bp, nullptr);
  else if (which == 2) rc = ot_fold_weights_asym(W, nullptr, N, K, 8, z, s, Wq, sW, zW, bp, nullptr);
  else rc = ot_calibrate(W, N, K, 8, 1, mm, z, s, inv, nullptr);
  if (first) *first = z[0];
  return rc;
}
#define CHECK(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); exit(1); } } while (0)
static void both_outcomes() {  // and that bad calibration data leave the outputs
  for (int round = 0; round < 3; ++round)
    for (int w = 0; w < 4; ++w) {
      float z0;
      g_bad = false;
      CHECK(call(w, &z0) == OT_OK);
      if (w == 3) CHECK(z0 == 1.f);
      g_bad = true;
      CHECK(call(w, &z0) == OT_ENONFINITE);
      if (w == 3) CHECK(z0 == 0.f);
      g_bad = false;
    }
}
int main(int, char **argv) {
  const char *scene = argv[1];
  if (!strcmp(scene, "words")) {
    both_outcomes();
    CHECK(g_copies == 0 && g_finalized == 0);
  } else if (!strcmp(scene, "no pinned memory")) {
    g_pinned = false;
    both_outcomes();
    CHECK(g_copies == 3 * (3 * 2 * 2 + 2) && g_finalized == 3);
  } else if (!strcmp(scene, "capture")) {  // calls that fail under capture take no word with them
    both_outcomes();
    g_capturing = true;
    for (int i = 0; i < 200; ++i) CHECK(call(i & 3) == OT_EHIP);
    g_capturing = false;
    g_copies = 0;
    both_outcomes();
    CHECK(g_copies == 0);
  } else if (!strcmp(scene, "launch errors")) {
    g_launch = hipErrorInvalidConfiguration;
    for (int i = 0; i < 200; ++i) CHECK(call(i & 3) == OT_EHIP);
    g_launch = hipSuccess;
    both_outcomes();
    CHECK(g_copies == 0);
  } else {
    return 2;
  }
  printf("passed\n");
  return 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("status_words")
    (d / "driver.hip").write_text(DRIVER)
    objs = []
    for src in (build_lib.CSRC + "/ot_api.hip", str(d / "driver.hip")):
        objs.append(str(d / (src.rsplit("/", 1)[1] + ".o")))
        run = subprocess.run([build_lib.hipcc(), "-O1", "-std=c++17", "--cuda-host-only", "-I" + build_lib.CSRC,
                              "-x", "hip", "-c", src, "-o", objs[-1]], capture_output=True, text=True,
                             timeout=300)
        assert run.returncode == 0, run.stderr[-3000:]
    # the runtime's calls are the driver's; the launchers of the other entry
    # points stay unresolved and are never reached
    run = subprocess.run(["g++", "-no-pie", *objs, "-Wl,--unresolved-symbols=ignore-in-object-files",
                          "-lpthread", "-o", str(d / "driver")], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stderr[-3000:]
    return str(d / "driver")


@pytest.mark.parametrize("scene", ["words", "no pinned memory", "capture", "launch errors"])
def test_non_finite_values_are_reported(driver, scene):
    run = subprocess.run([driver, scene], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and "passed" in run.stdout, (run.returncode, run.stdout, run.stderr)
