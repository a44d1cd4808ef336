"""The small row blocks' kernel on more workgroups than compute units, where they share one: ranges of one slice and of
several, the last range shorter than the others, with K inside the short form (256) and past it."""
import pytest

from paper_2512_12949_amd import binding as ff
from paper_2512_12949_amd import inputs
from paper_2512_12949_amd.inputs import ACT_GELU_TANH, ACT_SILU

import gpu_util as gu

# (M, K, N1, N2, ranges), row blocks x ranges just below, on and past 256 workgroups on 16 and on 32 rows; K below, on and
# past a wave's step of 32, a turn of four and of eight waves (128, 256) and the short form
SHAPES = [(4080, 8, 40, 16, 1), (4097, 64, 64, 64, 1), (1100, 72, 248, 256, 4), (2210, 136, 256, 128, 4), (1090, 256, 256, 192, 4),
          (8210, 40, 64, 72, 1), (1100, 128, 496, 136, 4), (2100, 256, 328, 256, 3), (1100, 264, 456, 264, 4), (700, 256, 720, 512, 6)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("gated", [False, True])
@pytest.mark.parametrize("bm", [16, 32])
def test_parity_on_more_workgroups_than_units(bm, gated, dtype):
    for M, K, N1, N2, splits in SHAPES:
        w = inputs.custom("slices", M, K, N1, N2, dtype=dtype, act=ACT_SILU if gated else ACT_GELU_TANH, gated=gated, cfg_id=1400)
        host = inputs.make(w)
        dev = {k: gu.to_device(v, dtype) for k, v in host.items()}
        plan = ff.make_plan(ff.FAMILY_REDUCE, bm=bm, bh=64, bk=32, splits=splits)
        what = f"{dtype} gated={gated} {(M, K, N1, N2)} bm={bm} splits={splits}"
        print(what, flush=True)
        gu.check(gu.run(w, dev, plan=plan), gu.oracle_rows(w, host), dtype, what=what)
