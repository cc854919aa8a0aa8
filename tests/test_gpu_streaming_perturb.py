"""Perturbs of streaming buffers (256 MiB and more)."""

import numpy as np
import pytest
import torch

import oracle
import paper_2609_38095_amd as zo

SEED, STEP, OFFSET = 0x1234_5678_9ABC, 7, 3
EPS = 1e-3
# 256 MiB and a ragged tail: the whole call streams, each half of it does not
N = {"bf16": 2 ** 27 + 4099, "f32": 2 ** 26 + 4099}
TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}


@pytest.fixture(scope="module", params=["bf16", "f32"])
def theta(request):
    g = torch.Generator(device="cuda").manual_seed(1)
    return request.param, torch.empty(N[request.param], device="cuda", dtype=TORCH[request.param]).normal_(
        0.0, 0.02, generator=g)


def _host(t, dtype):
    return t.cpu().numpy() if dtype == "f32" else t.view(torch.int16).cpu().numpy().view(np.uint16)


def _windows(n):
    return [(0, 1500), (n // 2 - 700, 1400), (n - 1500, 1500)]


@pytest.mark.gpu
@pytest.mark.parametrize("two", [False, True])
def test_streaming_perturb(theta, two):
    """Bit for bit the oracle's on windows, and the same in two cache-sized calls over the whole buffer."""
    dtype, base = theta
    n, m = base.numel(), base.numel() // 2

    def call(t, offset):
        if two:
            zo.zo_perturb2(t, 7, EPS, 8, -2 * EPS, SEED, STEP, offset)
        else:
            zo.zo_perturb(t, 5, EPS, SEED, STEP, offset)

    whole, halves = base.clone(), base.clone()
    call(whole, OFFSET)
    call(halves[:m], OFFSET)
    call(halves[m:], OFFSET + m)
    bits = torch.int16 if dtype == "bf16" else torch.int32
    assert torch.equal(whole.view(bits), halves.view(bits))
    if two:
        return
    for at, ln in _windows(n):
        want = oracle.perturb(_host(base[at:at + ln], dtype), dtype, OFFSET + at, SEED, STEP, 5, EPS)
        np.testing.assert_array_equal(_host(whole[at:at + ln], dtype), want)
