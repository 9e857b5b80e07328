"""Which kernel a MatMul call is sent to, on the CPU: the host side of the
library compiled into small programs of its own, no kernel launched."""

import os
import subprocess

import pytest

from paper_1603_04467_amd import build as B

pytestmark = pytest.mark.timeout(600)

# api.cpp against stand-ins of what its fused calls launch. The route answers
# with the other kernel each time it is asked, as it may when a tuning knob is
# set on another thread during a call.
STAND_INS = r"""
#include <cstdio>
#include <cstdlib>
#include "include/tfdense.h"
#include "paper_1603_04467_amd/csrc/kernels.h"
namespace tfd {
static int asked, start;
static int64_t launched_rows, launched_tiles, summed_rows, summed_tiles;
GemmRoute gemm_fused_route(const GemmDesc&) {
  return (start + asked++) % 2 ? GemmRoute::kBf16Tiles128 : GemmRoute::kBf16Whole256;
}
static int64_t up(int64_t a, int64_t b) { return (a + b - 1) / b; }
int64_t gemm_bf16_128_tile_rows(const GemmDesc& d) { return up(d.m, 128); }
int64_t gemm_bf16_128_tiles(const GemmDesc& d) { return up(d.m, 128) * up(d.n, 128); }
hipError_t launch_gemm_bf16_256(const GemmDesc& d, hipStream_t) {
  launched_rows = d.m / 256, launched_tiles = launched_rows * (d.n / 256);
  return hipSuccess;
}
hipError_t launch_gemm_bf16_128(const GemmDesc& d, hipStream_t) {
  launched_rows = up(d.m, 128), launched_tiles = launched_rows * up(d.n, 128);
  return hipSuccess;
}
hipError_t launch_colsum_final(const float*, float*, int64_t chunks, int64_t, hipStream_t) {
  summed_rows = chunks;
  return hipSuccess;
}
hipError_t launch_loss_final(const double*, int n, double*, hipStream_t) {
  summed_tiles = n;
  return hipSuccess;
}
size_t reduction_ws_bytes(int64_t, int64_t, bool) { return 1 << 20; }
size_t loss_ws_bytes(int64_t, bool) { return 1 << 20; }
}  // namespace tfd
using namespace tfd;
int main() {
  static char mem[16][1 << 20] __attribute__((aligned(256)));
  void *a = mem[0], *b = mem[1], *c = mem[2], *f = mem[3], *g = mem[4], *ws = mem[5];
  uint32_t* mask = reinterpret_cast<uint32_t*>(mem[6]);
  float *bias = reinterpret_cast<float*>(mem[7]), *db = reinterpret_cast<float*>(mem[8]);
  double* loss = reinterpret_cast<double*>(mem[9]);
  const int64_t m = 512, n = 512, k = 64;
  for (start = 0; start < 2; ++start)
    for (int call = 0; call < 4; ++call) {
      asked = 0, launched_rows = launched_tiles = summed_rows = summed_tiles = -1;
      tfd_status st = TFD_EHIP;
      if (call == 0)
        st = tfd_matmul_relu_mask(0, 0, m, n, k, a, k, b, n, bias, c, n, mask, TFD_BF16, TFD_ROUND_NEAREST_EVEN, 0);
      if (call == 1)
        st = tfd_matmul_relu_grad_bias_add_grad(0, 0, m, n, k, a, k, b, n, f, c, db, TFD_BF16,
                                                TFD_ROUND_NEAREST_EVEN, ws, sizeof mem[5], 0);
      if (call == 2)
        st = tfd_matmul_relu_mask_grad_bias_add_grad(0, 0, m, n, k, a, k, b, n, mask, c, db, TFD_BF16,
                                                     TFD_ROUND_NEAREST_EVEN, ws, sizeof mem[5], 0);
      if (call == 3)
        st = tfd_matmul_l2_loss_grad(0, 0, m, n, k, a, k, b, n, bias, c, f, g, loss, db, TFD_BF16,
                                     TFD_ROUND_NEAREST_EVEN, ws, sizeof mem[5], 0);
      if (call == 0) summed_rows = launched_rows;
      if (call != 3) summed_tiles = launched_tiles;
      printf("call %d start %d status %d asked %d rows %lld %lld tiles %lld %lld\n", call, start, (int)st, asked,
             (long long)launched_rows, (long long)summed_rows, (long long)launched_tiles, (long long)summed_tiles);
    }
}
"""


def _build(tmp, source, objects):
    """A program of `source` and compiled objects; what it never calls stays unresolved."""
    src, obj, exe = (os.path.join(tmp, "main" + e) for e in (".cpp", ".o", ""))
    with open(src, "w") as f:
        f.write(source)
    for cmd in ([B._hipcc(), "-O1", "-std=c++17", "-I", B.ROOT, "-c", src, "-o", obj],
                [B._hipcc(), obj, *objects, "-Wl,--unresolved-symbols=ignore-all", "-o", exe]):
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
    return exe


def _object(name):
    path = os.path.join(B.OBJ, name)
    if not os.path.exists(path):
        B.build()
    return path


def test_fused_calls_decide_their_kernel_once(tmp_path):
    exe = _build(tmp_path, STAND_INS, [_object("api.o")])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stderr
    lines = out.stdout.splitlines()
    assert len(lines) == 8
    for line in lines:
        w = line.split()
        assert w[5] == "0" and int(w[9]) > 0, line              # launched, through a fused kernel
        assert w[9] == w[10] and w[12] == w[13], line           # sums and partials of the kernel that ran
        assert w[7] == "1", line


# gemm.hip as it is built, with a stand-in for the small-problem kernel; the
# launch of any other fails without a GPU
SMALL_STAND_IN = r"""
#include <cstdio>
#include <cstdlib>
#include "paper_1603_04467_amd/csrc/kernels.h"
namespace tfd {
static bool small;
hipError_t launch_gemm_small_f32(const GemmDesc&, hipStream_t) {
  small = true;
  return hipSuccess;
}
int tuning(TuneKnob) { return 0; }
}  // namespace tfd
int main(int argc, char** argv) {
  for (int i = 1; i + 5 < argc; i += 6) {
    tfd::GemmDesc d = {};
    d.ta = argv[i][0] == 'T', d.tb = argv[i][1] == 'T';
    d.m = atoll(argv[i + 1]), d.n = atoll(argv[i + 2]), d.k = atoll(argv[i + 3]);
    d.lda = (d.ta ? d.m : d.k) + atoll(argv[i + 4]), d.ldb = (d.tb ? d.k : d.n) + atoll(argv[i + 4]), d.ldc = d.n;
    const uintptr_t at = 4096 + 4 * (uintptr_t)atoll(argv[i + 5]);
    d.a = reinterpret_cast<const void*>(at), d.b = reinterpret_cast<const void*>(at), d.c = reinterpret_cast<void*>(4096);
    tfd::small = false;
    (void)tfd::launch_gemm(d, nullptr);
    puts(tfd::small ? "small" : "tiles");
  }
}
"""

# Far from the break-even. The small kernel's: single tiles, few columns, rows
# shorter than a unit, rows that start anywhere; the tile kernels': enough tiles
# of any size, k over 64 x 64 tiles' wave groups.
SMALL = ["NN 1 49 100 0 0", "NN 143 2 1267 0 0", "NT 57 6 6231 1 1", "NT 2426 1 1702 0 0", "TN 1 262 144 1 0",
         "NN 8 160 104 0 0", "TN 6992 24 56 0 0", "NT 200 25 2 1 0", "NN 8 8 3216 1 0", "TN 128 2048 3456 0 1",
         "NN 100 100 784 0 0"]
TILES = ["NN 1000 1000 1000 0 0", "NT 8192 4096 4096 0 0", "TN 1024 784 1000 0 0", "NN 300 1024 784 1 1",
         "NT 2368 4096 64 0 0", "TN 4096 4096 33 0 0"]


def test_small_fp32_problems_take_the_small_kernel(tmp_path):
    exe = _build(tmp_path, SMALL_STAND_IN, [_object("gemm.o")])
    out = subprocess.run([exe, *" ".join(SMALL + TILES).split()], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stderr
    assert dict(zip(SMALL + TILES, out.stdout.split())) == {**{s: "small" for s in SMALL}, **{t: "tiles" for t in TILES}}


# the routes of gemm.hip as they are built
ROUTES = r"""
#include <cstdio>
#include <cstdlib>
#include "paper_1603_04467_amd/csrc/kernels.h"
namespace tfd {
int tuning(TuneKnob) { return 0; }
}  // namespace tfd
int main(int argc, char** argv) {
  for (int i = argc % 4 == 2 ? 2 : 1; i + 3 < argc; i += 4) {  // (a word more: fused calls)
    tfd::GemmDesc d = {};
    d.in_bf16 = d.out_bf16 = true;
    d.ta = argv[i][0] == 'T', d.tb = argv[i][1] == 'T';
    d.m = atoll(argv[i + 1]), d.n = atoll(argv[i + 2]), d.k = atoll(argv[i + 3]);
    d.lda = d.ta ? d.m : d.k, d.ldb = d.tb ? d.k : d.n, d.ldc = d.n;
    d.a = d.b = reinterpret_cast<const void*>(4096), d.c = reinterpret_cast<void*>(4096);
    const tfd::GemmRoute r = argc % 4 == 2 ? tfd::gemm_fused_route(d) : tfd::gemm_route(d);
    if (r != tfd::GemmRoute::kBf16Tiles128)
      puts(r == tfd::GemmRoute::kBf16Whole256 ? "whole" : "other");
    else if (tfd::gemm_bf16_128_tile_rows(d) == (d.m + 255) / 256 && d.m > 128)
      puts("tall");
    else
      puts(tfd::gemm_bf16_128_tiles(d) <= 256 ? "four" : "two");
  }
}
"""


def test_16_bit_routes(tmp_path):
    """Which kernel, and which of its forms (128 x 128 tiles in four or two stages, 256 x 128 tiles), the sizes of
    the GPU tests of the fused epilogues take, and sizes far to either side of the rules."""
    exe = _build(tmp_path, ROUTES, [_object(o) for o in ("gemm.o", "gemm_bf16.o", "gemm_bf16_tn.o", "gemm_bf16_128.o")])
    want = {(1800, 2040, 1000): "four", (3000, 2504, 328): "two", (2176, 2056, 1288): "tall", (2048, 4096, 576): "tall",
            (16384, 4096, 4096): "whole", (4096, 8192, 512): "whole", (2048, 4096, 4096): "tall",
            (2048, 2048, 4096): "four", (16000, 1000, 1000): "tall", (256, 1024, 1024): "other", (100, 100, 784): "other",
            (1000, 1001, 1000): "other"}
    # fused calls: as the plain ones, but for problems on 64 x 64 tiles and whole k-tiles without wave groups
    fused = {**want, (2048, 1792, 128): "four", (8448, 768, 128): "two", (1792, 3584, 128): "two",
             (1000, 1024, 200): "other"}
    plain = {**want, (2048, 1792, 128): "other", (8448, 768, 128): "other", (1792, 3584, 128): "other",
             (1000, 1024, 200): "other"}
    for words, table in (([], plain), (["fused"], fused)):
        keys = [(lay, *size) for lay in ("NN", "NT", "TN") for size in table]
        out = subprocess.run([exe, *words, *[str(v) for k in keys for v in k]], capture_output=True, text=True, timeout=60)
        assert out.returncode == 0, out.stderr
        assert dict(zip(keys, out.stdout.split())) == {k: table[k[1:]] for k in keys}
