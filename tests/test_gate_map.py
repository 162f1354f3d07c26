"""The raw gate map (csrc/gate_map.h) within its stated bound.

CPU: the header's host side, which has the device's IEEE operations and so its
results bit for bit, against numpy in 80-bit over every binade of fp32 and both
tails.  The bound of 0.8 ulp is half an ulp of the one rounding to fp32, the two
polynomials' relative errors (2^-28.5 + 2^-30.1 of the result: 0.06 ulp) and the
roundings of their fp32 tails, at most 0.16 times the result (a quarter ulp).

GPU: a decode step with write strength 0 multiplies the state by e^g, which
shows g in units of |g|: the gate's own error (|g| 0.8 2^-23), then the library's
expf and one product (within 2 x 2^-23)."""

import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

MAIN = r"""
#include <stdio.h>
#include <vector>
#include "gate_map.h"
int main(int, char **argv) {
  FILE *f = fopen(argv[1], "rb"), *g = fopen(argv[2], "wb");
  if (!f || !g) return 1;
  std::vector<float> x(1 << 16);
  for (size_t n; (n = fread(x.data(), 4, x.size(), f)) > 0;) {
    for (size_t i = 0; i < n; ++i) x[i] = hagdn::neg_softplus(x[i]);
    if (fwrite(x.data(), 4, n, g) != n) return 1;
  }
  return fclose(f) | fclose(g);
}
"""


def _points():
    rng = np.random.default_rng(3)
    every = rng.integers(0, 1 << 32, 1 << 20, dtype=np.uint64).astype(np.uint32).view(np.float32)
    spans = [rng.uniform(a, b, 1 << 18) for a, b in
             ((-110, -103), (-104, -87), (-88, -20), (-20, -1), (-1, 1), (1, 20), (20, 120))]
    edges = [0.0, -0.0, np.inf, -np.inf, np.nan, 1e-45, -1e-45, 3.4e38, -3.4e38, -110.0, -87.336548, -103.97208]
    return np.concatenate([every, np.asarray(edges, np.float32)] + [s.astype(np.float32) for s in spans])


def _softplus(x):
    with np.errstate(over="ignore", under="ignore", invalid="ignore"):
        x = x.astype(np.longdouble)
        return np.where(x < 0, 0, x) + np.log1p(np.exp(-np.abs(x)))


def test_gate_map_within_its_bound(tmp_path):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("hipcc not available")
    src = tmp_path / "main.cpp"
    src.write_text(MAIN)
    cmd = [HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O2", "-std=c++17",
           "-I", os.path.join(ROOT, "paper_2609_32114_amd", "csrc"), str(src), "-o", str(tmp_path / "m")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    x = _points()
    x.tofile(tmp_path / "x")
    r = subprocess.run([str(tmp_path / "m"), str(tmp_path / "x"), str(tmp_path / "y")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    y, ref = np.fromfile(tmp_path / "y", np.float32), -_softplus(x)
    assert np.array_equal(np.isnan(y), np.isnan(x))
    fin = np.isfinite(x)
    assert np.array_equal(y[np.isinf(x)], ref[np.isinf(x)].astype(np.float32))
    ulp = np.spacing(np.abs(ref[fin]).astype(np.float32)).astype(np.longdouble)
    err = np.abs(y[fin] - ref[fin]) / ulp
    assert np.max(err) <= 0.8, (float(np.max(err)), x[fin][np.argmax(err)])


@pytest.mark.gpu
def test_gate_map_through_decode():
    import torch
    import paper_2609_32114_amd as P
    rng = np.random.default_rng(4)
    N, D = 64, 128
    x = rng.uniform(-110, 60, (N, 1, D)).astype(np.float32)
    x[0] = rng.uniform(-1, 1, D)
    x[1], x[2], x[3] = np.inf, -np.inf, np.nan
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    zero = np.zeros((N, 1, D), np.float32)
    state = torch.ones((N, 1, D, D), device="cuda")
    P.kda_decode(t(zero), t(zero), t(zero), t(x), t(zero[:, :, 0]), state, preprocess=P.PRE_GATE_SOFTPLUS)
    torch.cuda.synchronize()
    s = state.cpu().numpy().astype(np.float64)[:, 0]
    assert np.all(s[1] == 0) and np.all(s[2] == 1) and np.all(np.isnan(s[3]))
    g = -_softplus(x[:, 0]).astype(np.float64)
    ok = np.arange(N) != 3
    with np.errstate(invalid="ignore"):
        tol = np.where(np.isinf(g), 0, np.abs(g) * 0.8 * 2**-23 + 2 * 2**-23)
        err = np.abs(s / np.where(np.isinf(g), 1, np.exp(g))[..., None] - np.where(np.isinf(g), 0, 1)[..., None])
    assert np.all(err[ok] <= tol[ok][..., None]), float(np.max((err / np.maximum(tol, 1e-30)[..., None])[ok]))
