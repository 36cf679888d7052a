"""Second moments stored through sqrt(v) at block scales whose square is subnormal in fp32.

With zero inputs the step only decays: v' = beta2 (s q)^2, a normal number here although s^2 is
not (s down to 1.2e-21, 3e-22 for fp8).  The stored scale (int8: the largest sqrt(v') / 127; fp8:
the ring's amax) is sqrt(beta2) s q up to the rounding of s q, its square, beta2 v, the
hardware's square root (1 ulp) and the division: below 6 2^-24 = 3.6e-7.
"""
import math

import pytest
import torch

from gpu_util import HP
from paper_2606_22932_amd import forge

pytestmark = pytest.mark.gpu
TOL = 3.6e-7
STEP = 100                                     # slot 0 of an amax ring is written, 2 and 3 are read


def _zeros(T, d_in, d_out):
    z = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device="cuda")
    return z(T, d_in), z(T, d_out), z(d_out, d_in)


# the pipelined kernel, the long-loop kernel, and the stand-alone optimizer
@pytest.mark.parametrize("T,d_in,d_out,alone", [(32, 136, 264, False), (32, 4104, 8264, False), (0, 136, 264, True)])
def test_int8_columns_keep_small_scales(T, d_in, d_out, alone):
    print("case", T, d_in, d_out, alone, flush=True)
    X, dY, W = _zeros(T, d_in, d_out)
    m = torch.zeros((d_out, d_in), dtype=torch.int8, device="cuda")
    v = torch.full((d_out, d_in), 127, dtype=torch.int8, device="cuda")
    ms = torch.zeros(((d_out + 255) // 256, d_in), device="cuda")
    vs = torch.empty_like(ms).copy_(torch.linspace(1.2e-21, 3e-21, ms.numel()).view(ms.shape))
    want = vs.double() * math.sqrt(torch.tensor(HP["beta2"]).item())
    if alone:
        forge.forge_adamw(torch.zeros((d_out, d_in), device="cuda"), W, m, v, ms, vs, step=STEP, **HP)
    else:
        forge.forge_linear_step(X, dY, W, m, v, ms, vs, step=STEP, **HP)
    torch.cuda.synchronize()
    assert bool((v == 127).all())
    assert float(((vs.double() - want) / want).abs().max()) < TOL


# 128 x 128 tiles and the long-loop kernel, with bf16 and with fp8 weights
@pytest.mark.parametrize("wfp8", [False, True])
@pytest.mark.parametrize("T,d_in,d_out", [(32, 136, 264), (512, 4104, 8264)])
@pytest.mark.parametrize("amax", [3.1e-19, 2.3e-19, 1.7e-19])
def test_fp8_moments_keep_small_scales(T, d_in, d_out, amax, wfp8):
    print("case", T, d_in, d_out, amax, wfp8, flush=True)
    X, dY, W = _zeros(T, d_in, d_out)
    code = lambda c: torch.full((d_out, d_in), c, dtype=torch.uint8, device="cuda").view(torch.float8_e4m3fn)
    ring = lambda a: torch.tensor([0.0, 0.0, a, a], device="cuda")
    m, v, ms, vs = code(0), code(0x7E), ring(0.0), ring(amax)
    want = float(vs[2]) * math.sqrt(torch.tensor(HP["beta2"]).item())
    if wfp8:
        forge.forge_linear_step_wfp8(X, dY, code(0), ring(0.0), m, v, ms, vs, step=STEP, **HP)
    else:
        forge.forge_linear_step(X, dY, W, m, v, ms, vs, step=STEP, **HP)
    torch.cuda.synchronize()
    assert bool((v.view(torch.uint8) == 0x7E).all())
    assert abs(float(vs[0]) - want) < TOL * want
