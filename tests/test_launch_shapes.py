"""The launch shapes the host planner picks (CPU), and list calls against flat ones in each of them (GPU)."""

import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

import oracle
import paper_2609_38095_amd as zo
import streaming

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_38095_amd", "csrc")


def test_launch_shapes(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no g++")
    exe = str(tmp_path / "launch_shapes")
    subprocess.run([cxx, "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-Wall",
                    "-Werror", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "helpers", "launch_shapes_check.cpp"),
                    os.path.join(CSRC, "zo_plan.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stderr[:4000]


def _sizes(tensors, weights):
    """Ragged tensors of about `weights` in all, among them ones of no, one and a few row groups."""
    part = np.random.default_rng(tensors).uniform(0.5, 1.5, tensors)
    sizes = (weights * part / part.sum()).astype(int)
    sizes[:6] = [1, 7, 1023, 1024, 1025, 16_385]
    sizes[-1] += weights - sizes.sum()
    return [int(s) for s in sizes]


@pytest.fixture(scope="module", params=[(dt, t) for dt in ("bf16", "f32") for t in (40, 150)],
                ids=lambda p: f"{p[0]}-{p[1]}tensors")
def lists(request):
    """A call of 300 MiB: 40 tensors make one launch of 300 MiB, 150 make launches of 128 MiB."""
    dtype, tensors = request.param
    bf16 = dtype == "bf16"
    sizes = _sizes(tensors, (300 << 20) // (2 if bf16 else 4))
    g = torch.Generator(device="cuda").manual_seed(3)
    flat = torch.empty(sum(sizes), device="cuda", dtype=torch.bfloat16 if bf16 else torch.float32)
    flat.normal_(0.0, 0.02, generator=g)
    return flat, sizes


def _check(lists, flat_call, list_call):
    flat, sizes = lists
    base, starts = 777, np.concatenate([[0], np.cumsum(sizes)[:-1]])
    whole = flat.clone()
    flat_call(whole, base)
    ts = [flat[a:a + s].clone() for a, s in zip(starts, sizes)]
    list_call(ts, [base + int(a) for a in starts])
    bits = torch.int16 if flat.dtype == torch.bfloat16 else torch.int32
    differ = [i for i, (t, a, s) in enumerate(zip(ts, starts, sizes))
              if not torch.equal(t.view(bits), whole[a:a + s].view(bits))]
    assert differ == []
    return whole, base


def _check_windows(base, whole, offset, c, k_restore, eps, k_base=0):
    """The update's values on windows of a flat result against the oracle, within the update's bar."""
    dtype = "bf16" if base.dtype == torch.bfloat16 else "f32"
    for a, ln in streaming.windows(base.numel()):
        th = streaming.host(base[a:a + ln], dtype)
        want = oracle.update_restore(th, dtype, offset + a, 5, 7, c, 1e-3, k_restore, eps, k_base=k_base)
        w64, g64 = (x.astype(np.float64) if dtype == "f32" else oracle.bf16_to_f64(x)
                    for x in (want, streaming.host(whole[a:a + ln], dtype)))
        # 1e-6 of max(|theta|, lr sum |c| and the restore), and for bf16 one neighbouring value
        allow = 1e-6 * np.maximum(np.abs(w64), 1e-3 * np.abs(c.astype(np.float64)).sum() + abs(eps))
        if dtype == "bf16":
            allow = allow + np.maximum(np.abs(w64), 2.0 ** -126) * 2.0 ** -7
        assert np.all(np.abs(g64 - w64) <= allow)


@pytest.mark.gpu
@pytest.mark.parametrize("groups", list(range(1, 18)))
def test_list_updates_equal_flat_ones(lists, groups):
    """Bit for bit, with k_base inside a group and a restore in the first group (even counts) or none; the flat
    one within the update's bar of the oracle."""
    K, k_base = 8 * groups - 5, 3
    c = np.random.default_rng(groups).normal(0, 0.5, K).astype(np.float32)
    eps = 1e-3 if groups % 2 == 0 else 0.0
    whole, offset = _check(lists, lambda t, o: zo.zo_update_restore(t, c, 1e-3, 5, 7, 4, eps, o, k_base),
                           lambda ts, os_: zo.zo_update_segments(ts, os_, c, 1e-3, 5, 7, 4, eps, k_base))
    _check_windows(lists[0], whole, offset, c, 4, eps, k_base)


@pytest.mark.gpu
@pytest.mark.parametrize("k_b,eps_b", [(0, 0.0), (6, -1e-3), (12, -1e-3)])
def test_list_perturbs_equal_flat_ones(lists, k_b, eps_b):
    _check(lists, lambda t, o: zo.zo_perturb2(t, 3, 1e-3, k_b, eps_b, 5, 7, o),
           lambda ts, os_: zo.zo_perturb_segments(ts, os_, 3, 1e-3, k_b, eps_b, 5, 7))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,mib,K", [("bf16", 1000, 48), ("bf16", 1000, 96), ("bf16", 1100, 128), ("f32", 1000, 64)])
@pytest.mark.parametrize("restore", [False, True])
def test_four_chunks_per_stream(dtype, mib, K, restore):
    """Buffers whose flat update walks four chunks per stream: the bits that a list of their parts gives (one
    chunk per stream), and on windows the oracle's values within the update's bar."""
    n = (mib << 20) // (2 if dtype == "bf16" else 4) - 77
    base = streaming.weights(dtype, n)
    c = np.random.default_rng(K).normal(0, 0.5, K).astype(np.float32)
    eps, offset = (1e-3, 5) if restore else (0.0, 5)
    whole, parts = base.clone(), base.clone()
    zo.zo_update_restore(whole, c, 1e-3, 5, 7, K - 1, eps, offset)
    at = [0, n // 3, n // 3 + 1025, n]
    zo.zo_update_segments([parts[a:b] for a, b in zip(at, at[1:])], [offset + a for a in at[:-1]], c, 1e-3, 5, 7, K - 1, eps)
    bits = torch.int16 if dtype == "bf16" else torch.int32
    same = torch.equal(whole.view(bits), parts.view(bits))
    assert same
    _check_windows(base, whole, offset, c, K - 1, eps)
