"""The input gradient on every tile shape, against the oracle: sizes at which the tile choice (by
rounds of tiles over the chip) falls on 64 x 128, 128 x 128 and 256 x 256 tiles, with remainders
on both axes and in the last K chunk, around the point where a larger tile takes over.

On a 256-CU device, by token rows: (520, 4104) 128 (the 64-row grid just passes one round),
(505, 4096) 64, (1000, 14344) 256 (four rounds of 128-row tiles against one), (265, 14344) 128,
(4090, 4088) 256 (a full round), (4100, 3976) 256 with d_out = 40 and 128 with 1032 (256-row tiles
pass a full round by a few), (805, 4688) 128 (two short rounds of 64-row tiles against one).
"""
import pytest
import torch

from gpu_util import bits
from paper_2606_22932_amd import forge
from test_gpu_backward import _rand, check_dx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(520, 4104, 72), (505, 4096, 136), (1000, 14344, 40), (265, 14344, 72),
                                   (4090, 4088, 40), (4100, 3976, 40), (4100, 3976, 1032), (805, 4688, 288)],
                         ids=lambda s: "x".join(map(str, s)))
def test_input_grad_tile_choice(shape):
    T, d_in, d_out = shape
    print("input_grad", shape, flush=True)
    dY, W = _rand((T, d_out), 1e-3, 9300 + T), _rand((d_out, d_in), 0.02, 9400 + d_in)
    dX = torch.full((T, d_in), float("nan"), dtype=torch.bfloat16, device="cuda")
    forge.forge_input_grad(dY.cuda(), W.cuda(), dX)
    torch.cuda.synchronize()
    check_dx(bits(dX), [(bits(dY), bits(W))])
