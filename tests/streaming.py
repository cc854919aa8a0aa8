"""Streaming buffers of the GPU tests: 256 MiB and a ragged tail, so that a call over the whole buffer
streams and a call over either half of it does not."""

import numpy as np
import torch

N = {"bf16": 2 ** 27 + 4099, "f32": 2 ** 26 + 4099}
TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}


def weights(dtype, n=0, seed=1):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.empty(n or N[dtype], device="cuda", dtype=TORCH[dtype]).normal_(0.0, 0.02, generator=g)


def host(t, dtype):
    return t.cpu().numpy() if dtype == "f32" else t.view(torch.int16).cpu().numpy().view(np.uint16)


def windows(n):
    """(start, weights) at the start, in the middle and at the end."""
    return [(0, 1500), (n // 2 - 700, 1400), (n - 1500, 1500)]
