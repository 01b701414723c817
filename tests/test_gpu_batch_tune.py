"""The batch autotuner's choice and who follows it: automatic calls run the way it
found faster, calls that name the persistent kernel its best shape there, entries of
the cache file that were made without timing the windows leave automatic calls to
the rule.  Each case in a process of its own (the table belongs to the process)."""
import json
import os
import subprocess
import sys

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2607_01735_amd as rb  # noqa: E402

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SIZES = [63, 127, 255]
SWEEPS = 20  # windows: 4 passes; persistent: 5 passes of 4 in a launch, or 3 of 6 and one of 2

CHILD = f"""
import json, sys
import torch
import paper_2607_01735_amd as rb
us = [torch.zeros((n + 2, n + 2), dtype=torch.float32, device="cuda:0") for n in {SIZES}]
fs = [torch.ones_like(u) for u in us]
out = {{k: rb.rbgs_sweep_batched(us, fs, {SWEEPS}, timing=True, kernel=k)["sweep_launches"]
       for k in ("auto", "blocked")}}
with rb.BatchPlan(us, fs, {SWEEPS}) as plan:
    plan.launch()
    plan.check()
want = [torch.zeros_like(u) for u in us]
for u, f in zip(want, fs):
    rb.rbgs_sweep(u, f, 3 * {SWEEPS}, kernel="plain")
out["equal"] = all(torch.equal(a, b) for a, b in zip(us, want))
print(json.dumps(out))
"""


def key(version):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    return f"{version}/f32/cu{cus}" + "".join(f"/{n}x1" for n in SIZES)


@pytest.mark.parametrize("lines,auto,blocked", [
    ([], 4, 1),
    (["{v3} 6 64 -1 0.01 0"], 2, 2),                          # persistent was faster
    (["{v3} 6 64 -1 0.01 1"], 4, 2),                          # windows were
    (["{v2} 6 64 -1 0.01"], 4, 2),                            # windows were not timed
    (["{v3} 6 64 -1 0.01 0", "{v2} 4 64 -1 0.01"], 2, 2),     # which replaces no timed entry
    (["{v2} 4 64 -1 0.01", "{v3} 6 64 -1 0.01 0"], 2, 2),
    (["{v3} 6 64 -1 0.01", "{v3} 6 64 -1 0.01 2", "{v3} 0 64 -1 0.01 0", "junk"], 4, 1),
])
def test_cache_file(tmp_path, lines, auto, blocked):
    print(f"tune cache {lines}", flush=True)
    path = tmp_path / "tune.txt"
    path.write_text("".join(s.format(v3=key("v3"), v2=key("v2")) + "\n" for s in lines))
    res = subprocess.run([sys.executable, "-c", CHILD], cwd=ROOT, capture_output=True, text=True,
                         timeout=100, env={**os.environ, "RBGS_TUNE_CACHE": str(path)})
    assert res.returncode == 0, res.stderr
    assert json.loads(res.stdout.splitlines()[-1]) == {"auto": auto, "blocked": blocked,
                                                       "equal": True}


def inputs(sizes, dtype):
    us = [W.random_ring(n, seed=g).astype(dtype) for g, n in enumerate(sizes)]
    fs = [W.normal_rhs(n, seed=50 + g).astype(dtype) for g, n in enumerate(sizes)]
    return us, fs, [torch.from_numpy(f).to("cuda:0") for f in fs]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_tuned_calls_equal_oracle(oracle, dtype):
    """After tuning: automatic calls on the way that was faster, and the persistent
    kernel at its tuned shape."""
    sizes = [255, 300, 127, 63, 31]
    print(f"tuned calls {dtype.__name__}", flush=True)
    us, fs, ft = inputs(sizes, dtype)
    start = [torch.from_numpy(u).to("cuda:0") for u in us]
    best = rb.rbgs_autotune_batched(start, ft)
    assert best["kernel"] in ("auto", "blocked") and best["ms_per_sweep"] > 0
    for u, t in zip(us, start):
        assert np.array_equal(t.cpu().numpy(), u)
    sweeps = 3 * best["fuse"] + 1
    for n, u, f in zip(sizes, us, fs):
        oracle.sweep(u, f, W.spacing(n), sweeps)
    for kernel in ("auto", "blocked"):
        got = [t.clone() for t in start]
        rb.rbgs_sweep_batched(got, ft, sweeps, kernel=kernel)
        for u, t in zip(us, got):
            assert np.array_equal(t.cpu().numpy(), u), kernel


@pytest.mark.parametrize("check", [300, 301])
def test_persistent_solve_equals_oracle(oracle, check):
    """kernel "blocked": 300 sweeps at depth 4 are 75 passes, so that the iterate
    changes buffers from round to round; 301 are 76."""
    sizes = [63, 31, 127, 7]
    print(f"persistent batched solve check_every={check}", flush=True)
    fs = [W.fourier_rhs(n, seed=g + 1, count=8, kmax=8) for g, n in enumerate(sizes)]
    us = [W.random_ring(n, seed=50 + g) for g, n in enumerate(sizes)]
    ut, ft = [[torch.from_numpy(x).to("cuda:0") for x in xs] for xs in (us, fs)]
    infos = rb.rbgs_solve_batched(ut, ft, 200_000, 1e-8, check, precision="f64", kernel="blocked",
                                  fuse=4)
    for n, u, f, t, info in zip(sizes, us, fs, ut, infos):
        ref = u.copy()
        rc, done, _ = oracle.solve(ref, f, W.spacing(n), 200_000, 1e-8, check)
        assert rc == 0 and info["status"] == 0 and info["sweeps"] == done
        assert np.array_equal(t.cpu().numpy(), ref), n
