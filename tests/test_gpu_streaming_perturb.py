"""Perturbs of streaming buffers (256 MiB and more)."""

import numpy as np
import pytest
import torch

import oracle
import paper_2609_38095_amd as zo
import streaming

SEED, STEP, OFFSET = 0x1234_5678_9ABC, 7, 3
EPS = 1e-3


@pytest.fixture(scope="module", params=["bf16", "f32"])
def theta(request):
    return request.param, streaming.weights(request.param)


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
    same = torch.equal(whole.view(bits), halves.view(bits))
    assert same
    for at, ln in streaming.windows(n):
        th = streaming.host(base[at:at + ln], dtype)
        if two:
            want = oracle.perturb2(th, dtype, OFFSET + at, SEED, STEP, 7, EPS, 8, -2 * EPS)
        else:
            want = oracle.perturb(th, dtype, OFFSET + at, SEED, STEP, 5, EPS)
        np.testing.assert_array_equal(streaming.host(whole[at:at + ln], dtype), want)
