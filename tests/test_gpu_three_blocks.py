"""Three 64-row blocks in one patch of weight slices (129 to 192 rows): the same sums as in patches of two and one, bit for bit,
and the oracle's within the tolerance."""
import pytest
import torch

from paper_2512_12949_amd import binding as ff
from paper_2512_12949_amd import inputs
from paper_2512_12949_amd.inputs import ACT_GELU_TANH, ACT_SILU

import gpu_util as gu

# one row in the third block, a full one; fewer items than workgroups, about as many, and more in one phase or both
SHAPES = [(129, 72, 328, 264), (150, 136, 5448, 136), (192, 40, 8392, 1032), (192, 264, 72, 8)]


@pytest.mark.gpu
@pytest.mark.parametrize("bh,gated", [(64, False), (64, True), (128, False), (128, True)])
def test_one_patch_is_two(bh, gated):
    for M, K, N1, N2 in SHAPES:
        w = inputs.custom("three", M, K, N1, N2, dtype="bf16", act=ACT_SILU if gated else ACT_GELU_TANH, gated=gated, cfg_id=1400)
        host = inputs.make(w)
        dev = {k: gu.to_device(v, "bf16") for k, v in host.items()}
        ref = gu.oracle_rows(w, host)
        for splits in (2, 8):
            what = f"gated={gated} {(M, K, N1, N2)} bh={bh} splits={splits}"
            print(what, flush=True)
            Y = [gu.run(w, dev, plan=ff.make_plan(ff.FAMILY_TWOPHASE, bm=64, bh=bh, bn2=256, bk=32, splits=splits, raster=r)) for r in (3, 2)]
            gu.check(Y[0], ref, "bf16", what=what)
            assert torch.equal(Y[0], Y[1]), what
