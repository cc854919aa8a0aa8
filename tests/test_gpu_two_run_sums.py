"""Updates of 9 to 16 probe groups (two runs of up to eight) at the ends of fp32: every weight's sum is
compensated across the runs (NaN where it overflows, +0 where it is zero), on full row groups and on
head and tail tiles alike, so that a weight's result does not depend on where a call is cut."""

import numpy as np
import pytest
import torch

import oracle
import paper_2609_38095_amd as zo

SEED, STEP, OFFSET = 0x1234_5678_9ABC, 7, 3
SIZES = {"bf16": (70_001, 2 ** 27 + 4099), "f32": (70_001,)}  # bf16 streams from 2^27 weights on
TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}
CASES = [(dt, n) for dt in ("bf16", "f32") for n in SIZES[dt]]


def _bits(t):
    return t.view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32)


@pytest.mark.gpu
@pytest.mark.parametrize("groups", list(range(9, 17)))
@pytest.mark.parametrize("dtype,n", CASES)
def test_zero_step_keeps_every_bit(dtype, n, groups):
    """lr = 0 makes every term of the sum a zero of either sign: weights of -0 stay -0."""
    c = np.random.default_rng(groups).normal(0, 0.5, 8 * groups - 2).astype(np.float32)
    t = torch.full((n,), -0.0, device="cuda", dtype=TORCH[dtype])
    want = _bits(t)[0].item()
    zo.zo_update_ex(t, c, 0.0, SEED, STEP, OFFSET)
    changed = int((_bits(t) != want).sum())
    assert changed == 0


@pytest.mark.gpu
@pytest.mark.parametrize("groups", list(range(9, 17)))
@pytest.mark.parametrize("dtype,n", CASES)
def test_overflow_across_runs(dtype, n, groups):
    """One term of 3e38 in the first run and one in the second: where they agree in sign the sum
    overflows and the weight becomes NaN, elsewhere they cancel and the weight keeps its value."""
    K = 8 * groups
    c = np.zeros(K, np.float32)
    c[3] = c[K - 2] = 3e38
    g = torch.Generator(device="cuda").manual_seed(groups)
    base = torch.empty(n, device="cuda", dtype=TORCH[dtype]).normal_(0.0, 0.02, generator=g)
    t = base.clone()
    zo.zo_update_ex(t, c, 1.0, SEED, STEP, OFFSET)
    for at, ln in ((0, 4000), (n // 2 - 700, 1400), (n - 2500, 2500)):
        over = oracle.signs(OFFSET + at, ln, SEED, STEP, 3) == oracle.signs(OFFSET + at, ln, SEED, STEP, K - 2)
        got = t[at:at + ln].float().cpu().numpy()
        np.testing.assert_array_equal(np.isnan(got), over)
        np.testing.assert_array_equal(got[~over], base[at:at + ln].float().cpu().numpy()[~over])
        # the same weights cut into pieces too short for a row group
        cut = base[at:at + ln].clone()
        for a in range(0, ln, 500):
            zo.zo_update_ex(cut[a:a + 500], c, 1.0, SEED, STEP, OFFSET + at + a)
        same = torch.equal(torch.isnan(cut), torch.isnan(t[at:at + ln]))
        assert same
