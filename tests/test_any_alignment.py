"""Tensors stored at any weight's address (a shard that starts at an odd global index, a view
in the middle of a buffer): small launches sweep them element by element, in larger ones the full row
groups take the vector path wherever they lie."""

import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

import oracle
import paper_2609_38095_amd as zo
import workloads

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_38095_amd", "csrc")
GUARD = 64


def test_planner_at_any_alignment(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no g++")
    exe = str(tmp_path / "any_alignment")
    subprocess.run([cxx, "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-Wall",
                    "-Werror", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "helpers", "any_alignment_check.cpp"),
                    os.path.join(CSRC, "zo_plan.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stderr


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,shift", [("bf16", s) for s in range(1, 8)] + [("f32", s) for s in (1, 2, 3)])
@pytest.mark.parametrize("n,offset", [(1023, 0), (1024, 0), (1025, 1023), (2 * 1024 + 5, 2 ** 35 + 7), (70_001, 3)])
def test_any_alignment_matches_oracle(dtype, shift, n, offset):
    """Perturb bit for bit and the K = 9 update within its bar; the weights around the view stay."""
    f32 = dtype == "f32"
    total = n + 2 * GUARD
    host = workloads.normal_f32(total, n + shift) if f32 else workloads.normal_bf16_bits(total, n + shift)
    buf = torch.from_numpy(host.copy() if f32 else host.view(np.int16).copy()).to("cuda:0")
    buf = buf if f32 else buf.view(torch.bfloat16)
    view = buf[GUARD + shift:GUARD + shift + n]
    th = host[GUARD + shift:GUARD + shift + n]

    def get(t):
        return t.cpu().numpy() if f32 else t.view(torch.int16).cpu().numpy().view(np.uint16)

    zo.zo_perturb(view, 11, 1e-3, 77, 5, offset=offset)
    want = oracle.perturb(th, dtype, offset, 77, 5, 11, 1e-3)
    np.testing.assert_array_equal(get(view), want)
    c = np.linspace(-0.4, 0.5, 9).astype(np.float32)
    zo.zo_update_ex(view, c, 1e-3, 77, 5, offset=offset)
    up = oracle.update(want, dtype, offset, 77, 5, c, 1e-3)
    # the bar of the update: 1e-6 of max(|theta|, lr sum |c|), and for bf16 one neighbouring value
    w64 = up.astype(np.float64) if f32 else oracle.bf16_to_f64(up)
    g64 = get(view).astype(np.float64) if f32 else oracle.bf16_to_f64(get(view))
    allow = 1e-6 * np.maximum(np.abs(w64), 1e-3 * np.abs(c.astype(np.float64)).sum())
    if not f32:
        allow = allow + np.maximum(np.abs(w64), 2.0 ** -126) * 2.0 ** -7
    assert np.all(np.abs(g64 - w64) <= allow)
    whole = get(buf)
    np.testing.assert_array_equal(whole[:GUARD + shift], host[:GUARD + shift])
    np.testing.assert_array_equal(whole[GUARD + shift + n:], host[GUARD + shift + n:])


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,shift", [("bf16", s) for s in range(1, 8)] + [("f32", s) for s in (1, 2, 3)])
@pytest.mark.parametrize("n,offset,K", [(2 ** 20 + 2 ** 19 + 5, 1023, 9), (5_300_021, 2 ** 35 + 7, 133)])
def test_row_groups_at_any_alignment(dtype, shift, n, offset, K):
    """Launches large enough for row groups: the perturb and the update equal those of the same weights in aligned
    storage bit for bit, the weights around the view stay, and the ends and middle match the oracle."""
    f32 = dtype == "f32"
    g = torch.Generator(device="cuda").manual_seed(shift)
    buf = torch.empty(n + 2 * GUARD, device="cuda", dtype=torch.float32 if f32 else torch.bfloat16)
    buf.normal_(0.0, 0.02, generator=g)
    bits = torch.int32 if f32 else torch.int16
    before = buf.clone()
    view = buf[GUARD + shift:GUARD + shift + n]
    room = torch.empty(n + 16, device="cuda", dtype=buf.dtype)
    at = -(room.data_ptr() // room.element_size() - offset) % 8  # element `offset` where an aligned vector has it
    aligned = room[at:at + n].copy_(view)
    c = np.linspace(-0.4, 0.5, K).astype(np.float32)

    def host(t):
        return t.cpu().numpy() if f32 else t.view(torch.int16).cpu().numpy().view(np.uint16)

    for t in (view, aligned):
        zo.zo_perturb(t, 11, 1e-3, 77, 5, offset=offset)
    same = torch.equal(view.view(bits), aligned.view(bits))
    assert same
    for a in (0, n // 2, n - 3000):
        want = oracle.perturb(host(before[GUARD + shift + a:GUARD + shift + a + 3000]), dtype, offset + a, 77, 5, 11, 1e-3)
        np.testing.assert_array_equal(host(view[a:a + 3000]), want)
    for t in (view, aligned):
        zo.zo_update_ex(t, c, 1e-3, 77, 5, offset=offset)
    same = torch.equal(view.view(bits), aligned.view(bits))
    assert same
    for part in (slice(0, GUARD + shift), slice(GUARD + shift + n, None)):
        assert torch.equal(buf[part].view(bits), before[part].view(bits))
