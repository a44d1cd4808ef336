"""The two-phase family's LDS-direct kernels that run with eight waves: parity where the loads' split over the waves, the
rings and the tiles end, with the load hint and with the gated branches as separate items."""
import pytest
import torch

from paper_2512_12949_amd import binding as ff
from paper_2512_12949_amd import inputs
from paper_2512_12949_amd.inputs import ACT_GELU_TANH, ACT_SILU

import gpu_util as gu

# K (and ranges) below, on and past one step of 32, one super-stage of 64, the fill of a ring of 4 and of 8 steps; odd and even
# numbers of steps; ragged rows and columns; fewer and more items than workgroups.
SHAPES = [(1, 8, 8, 8), (65, 32, 72, 264), (128, 40, 136, 8), (130, 72, 328, 520), (200, 96, 264, 256), (129, 136, 640, 264),
          (256, 232, 520, 136), (70, 264, 1096, 72), (254, 296, 8328, 1032)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("bm,bh,gated", [(64, 128, False), (64, 128, True), (128, 64, False), (128, 64, True), (128, 128, False),
                                         (128, 128, True), (128, 256, False)])
def test_parity_at_the_edges(bm, bh, gated, dtype, monkeypatch):
    for M, K, N1, N2 in SHAPES:
        w = inputs.custom("eight", M, K, N1, N2, dtype=dtype, act=ACT_SILU if gated else ACT_GELU_TANH, gated=gated, cfg_id=1300)
        host = inputs.make(w)
        dev = {k: gu.to_device(v, dtype) for k, v in host.items()}
        ref = gu.oracle_rows(w, host)
        for splits in (1, 3):
            plan = ff.make_plan(ff.FAMILY_TWOPHASE, bm=bm, bh=bh, bn2=256, bk=32, splits=splits, raster=2)
            what = f"{dtype} gated={gated} {(M, K, N1, N2)} bm={bm} bh={bh} splits={splits}"
            print(what, flush=True)
            Y = gu.run(w, dev, plan=plan)
            gu.check(Y, ref, dtype, what=what)
            monkeypatch.setenv("FFUSE_NT", "1")
            assert torch.equal(Y, gu.run(w, dev, plan=plan)), what + " with the load hint"
            monkeypatch.delenv("FFUSE_NT")
            if gated and N1 % 64 == 0:
                plan.gate_split = 1
                gu.check(gu.run(w, dev, plan=plan), ref, dtype, what=what + " branches apart")
