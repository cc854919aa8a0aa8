"""Updates of every probe-group count from 1 to 17, each with the kernels of streaming buffers (256 MiB
and more) and of cache-sized ones."""

import numpy as np
import pytest
import torch

import oracle
import paper_2609_38095_amd as zo
import streaming

SEED, STEP, OFFSET = 0x1234_5678_9ABC, 7, 3
LR, EPS = 1e-3, 1e-3


@pytest.fixture(scope="module", params=["bf16", "f32"])
def theta(request):
    return request.param, streaming.weights(request.param)


@pytest.mark.gpu
@pytest.mark.parametrize("restore", [False, True])
@pytest.mark.parametrize("groups", list(range(1, 18)))
def test_update_of_every_group_count(theta, groups, restore):
    """Bit for bit the same in one streaming call and in two cache-sized ones (both sum the tables in the
    same order), and within the update's bar of the oracle on windows at the start, middle and end."""
    dtype, base = theta
    n, K = base.numel(), 8 * groups - (3 if groups % 2 else 0)
    c = np.random.default_rng(groups).normal(0, 0.5, K).astype(np.float32)

    def call(t, offset):
        if restore:
            zo.zo_update_restore(t, c, LR, SEED, STEP, K - 1, EPS, offset)
        else:
            zo.zo_update_ex(t, c, LR, SEED, STEP, offset)

    whole, halves = base.clone(), base.clone()
    call(whole, OFFSET)
    m = n // 2
    call(halves[:m], OFFSET)
    call(halves[m:], OFFSET + m)
    bits = torch.int16 if dtype == "bf16" else torch.int32
    assert torch.equal(whole.view(bits), halves.view(bits))
    for at, ln in streaming.windows(n):
        th = streaming.host(base[at:at + ln], dtype)
        if restore:
            want = oracle.update_restore(th, dtype, OFFSET + at, SEED, STEP, c, LR, K - 1, EPS)
        else:
            want = oracle.update(th, dtype, OFFSET + at, SEED, STEP, c, LR)
        w64, g64 = (x.astype(np.float64) if dtype == "f32" else oracle.bf16_to_f64(x)
                    for x in (want, streaming.host(whole[at:at + ln], dtype)))
        # 1e-6 of max(|theta|, lr sum |c| and the restore), and for bf16 one neighbouring value
        scale = LR * np.abs(c.astype(np.float64)).sum() + (EPS if restore else 0.0)
        allow = 1e-6 * np.maximum(np.abs(w64), scale)
        if dtype == "bf16":
            allow = allow + np.maximum(np.abs(w64), 2.0 ** -126) * 2.0 ** -7
        assert np.all(np.abs(g64 - w64) <= allow)
