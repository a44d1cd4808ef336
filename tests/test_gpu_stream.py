"""The two-phase family's streaming kernel (plan.bk = 128): up to 32 rows, weights straight to registers.  Parity at the
edges of its steps and tiles, both load hints, one phase per launch, and its barrier's failure path."""
import ctypes
import random

import pytest
import torch

from paper_2512_12949_amd import binding as ff
from paper_2512_12949_amd import inputs
from paper_2512_12949_amd.inputs import ACT_GELU_TANH, ACT_RELU, ACT_SILU

import gpu_util as gu


def _plan(bm, splits):
    return ff.make_plan(ff.FAMILY_TWOPHASE, bm=bm, bh=64, bn2=64, bk=128, splits=splits, raster=1)


def _case(M, K, N1, N2, dtype, gated, act=None, cfg_id=1200):
    w = inputs.custom("stream", M, K, N1, N2, dtype=dtype, act=act if act is not None else (ACT_SILU if gated else ACT_GELU_TANH),
                      gated=gated, cfg_id=cfg_id)
    host = inputs.make(w)
    return w, host, {k: gu.to_device(v, dtype) for k, v in host.items()}


# One unit of everything; K and ranges on and beside the lane octets (8), a wave's halves (32, 64) and a step (512), past
# one and two; one to 32 rows; whole and ragged 64-column slices; more slices than workgroups; more output items than workgroups.
SHAPES = [(1, 8, 8, 8), (16, 64, 64, 64), (3, 40, 72, 136), (17, 136, 200, 264), (32, 512, 328, 72), (5, 520, 1096, 200),
          (31, 1096, 640, 328), (2, 24, 16456, 40), (20, 16, 576, 4104)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("gated", [False, True])
def test_parity_at_the_edges(dtype, gated, monkeypatch):
    for M, K, N1, N2 in SHAPES:
        w, host, dev = _case(M, K, N1, N2, dtype, gated)
        ref = gu.oracle_rows(w, host)
        for bm in (16, 32):
            if M > bm:
                with pytest.raises(ff.FfuseError):
                    ff.ffuse_traffic_model(_plan(bm, 1), ff.DTYPE_CODE[dtype], gated, M, K, N1, N2)
                continue
            for splits in (1, 2, 5):
                what = f"{dtype} gated={gated} {(M, K, N1, N2)} bm={bm} splits={splits}"
                print(what, flush=True)
                Y = gu.run(w, dev, plan=_plan(bm, splits))
                gu.check(Y, ref, dtype, what=what)
                monkeypatch.setenv("FFUSE_NT", "1")
                assert torch.equal(Y, gu.run(w, dev, plan=_plan(bm, splits))), what + " with the load hint"
                monkeypatch.delenv("FFUSE_NT")
                monkeypatch.setenv("FFUSE_GROUP_BARRIER", "0")
                assert torch.equal(Y, gu.run(w, dev, plan=_plan(bm, splits))), what + " behind the device-wide barrier"
                monkeypatch.delenv("FFUSE_GROUP_BARRIER")


@pytest.mark.gpu
def test_the_default_call_and_its_two_launches():
    """The model's choice for a decode layer is this kernel; the comparison path runs it one phase per launch, to the bit."""
    w, host, dev = _case(7, 1288, 3080, 1288, "bf16", True)
    ref = gu.oracle_rows(w, host)
    Y = gu.run(w, dev)
    assert ff.ffuse_last_plan().bk == 128
    gu.check(Y, ref, "bf16", what="default call")
    assert torch.equal(Y, gu.run(w, dev, unfused=True))


@pytest.mark.gpu
@pytest.mark.parametrize("gated", [False, True])
def test_infinities_stay_in_their_rows(gated):
    """An infinity meets the zeros past K, past N1 and past the last rows' end: its row is not finite, no other changes."""
    w, host, dev = _case(20, 72, 136, 72, "bf16", gated, act=ACT_RELU)
    clean = gu.run(w, dev, plan=_plan(32, 2))
    dev["X"][3, 71] = float("inf")
    y = gu.run(w, dev, plan=_plan(32, 2))
    keep = [r for r in range(20) if r != 3]
    assert torch.equal(y[keep], clean[keep]) and not bool(torch.isfinite(y[3]).all())


@pytest.mark.gpu
def test_changing_inputs_replays_and_an_expired_wait():
    """Call after call on one workspace with other families between, from a graph with the input overwritten in place, and
    after a barrier wait that was made to expire from the host."""
    variants = []
    for i in range(3):
        w, host, dev = _case(12, 264, 1304, 520, "bf16", False, cfg_id=1210 + i)
        variants.append((w, dev, gu.oracle_rows(w, host)))
    other = ff.make_plan(ff.FAMILY_REDUCE, bm=16, bh=64, bk=32, splits=5)
    plan = _plan(16, 3)
    for n in range(8):
        w, dev, ref = variants[n % 3]
        gu.check(gu.run(w, dev, plan=other if n % 4 == 3 else plan), ref, "bf16", what=f"call {n}")
    w, dev, ref = variants[0]
    X, Y = dev["X"].clone(), torch.zeros((w.M, w.N2), dtype=torch.bfloat16, device="cuda")
    side = torch.cuda.Stream()
    ff.ffuse_force_plan(plan)
    try:
        # the weights differ between the variants as well: replays keep the first one's
        with torch.cuda.stream(side):
            ff.ffuse_ffn(X, dev["W1"], None, dev["W2"], w.act, Y)
            side.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=side):
                ff.ffuse_ffn(X, dev["W1"], None, dev["W2"], w.act, Y)
        torch.cuda.synchronize()
        for rep in range(5):
            src = variants[rep % 3][1]["X"]
            X.copy_(src)
            ff.ffuse_force_plan(other if rep % 2 else plan)
            want = torch.empty_like(Y)
            ff.ffuse_ffn(src, dev["W1"], None, dev["W2"], w.act, want)
            Y.fill_(float("nan"))
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            # (the other family sums in another order: two bf16 roundings of the intermediate apart)
            assert torch.equal(Y, want) if rep % 2 == 0 else float((Y - want).float().abs().max()) <= 2.0 ** -6 * float(want.float().abs().max())
        ff.ffuse_force_plan(plan)
        ff.ffuse_debug_barrier(1, 64)
        try:
            assert ff.ffuse_ffn(dev["X"], dev["W1"], None, dev["W2"], w.act, Y, check=False) == 0
            assert ff.ffuse_sync_status(check=False) == -9
        finally:
            ff.ffuse_debug_barrier(0, 1 << 24)
        Y.fill_(float("nan"))
        ff.ffuse_ffn(dev["X"], dev["W1"], None, dev["W2"], w.act, Y)
        assert ff.ffuse_sync_status(check=False) == 0
        gu.check(Y, ref, "bf16", what="after the expired wait")
    finally:
        ff.ffuse_force_plan(None)


def test_where_the_chooser_takes_it():
    """Up to 32 rows, at most one 64-column slice a workgroup, weights of some MB to 512 MB."""
    def chosen(M, K, N1, N2, gated):
        return ff.ffuse_choose_plan(ff.DT_BF16, 3 if gated else 2, gated, M, K, N1, N2)
    for shape, gated in (((1, 4096, 11008, 4096), True), ((16, 4096, 11008, 4096), True), ((32, 4096, 11008, 4096), True),
                         ((6, 1688, 5760, 1688), False), ((13, 5000, 13000, 5000), False), ((9, 4608, 16128, 4608), False)):
        p = chosen(*shape, gated)
        assert p.family == ff.FAMILY_TWOPHASE and p.bk == 128 and p.bm == (16 if shape[0] <= 16 else 32), (shape, p.as_dict())
    for shape, gated in (((33, 4096, 11008, 4096), True), ((9, 2304, 27704, 2304), False), ((16, 8192, 28672, 8192), True),
                         ((5, 312, 864, 312), False), ((31, 384, 2560, 384), False)):
        assert chosen(*shape, gated).bk != 128, shape


def test_group_local_barrier_condition():
    """As for the other plans of the family: true exactly where every second-phase item (64 output columns) of a group reads
    slices of the intermediate (64 columns) that the group wrote."""
    def independent(N1, N2, splits):
        ksplit = (-(-N1 // splits) + 63) // 64 * 64
        ranges, ns, ncb = -(-N1 // ksplit), -(-N1 // 64), -(-N2 // 64)
        per1, per2 = -(-ns // 8), -(-(ncb * ranges) // 8)
        for v in range(ncb * ranges):
            sp = v // ncb
            for s in range(sp * ksplit // 64, -(-min(N1, (sp + 1) * ksplit) // 64)):
                if s // per1 != v // per2:
                    return False
        return True
    rng, seen = random.Random(9), set()
    cases = [(4096, 4096, 8), (11008, 4096, 4), (2048, 64, 8)] + [(8 * rng.randint(1, 2000), 8 * rng.randint(1, 600), rng.choice([1, 2, 3, 4, 8, 16])) for _ in range(60)]
    for N1, N2, splits in cases:
        got = ff.ffuse_plan_group_local(_plan(16, splits), ff.DT_BF16, False, 16, 1024, N1, N2)
        assert got == independent(N1, N2, splits), (N1, N2, splits)
        seen.add(got)
    assert seen == {True, False}
    # what the kernel does not run: more rows than the block, separate branches
    t = ff.Traffic()
    split = _plan(16, 2)
    split.gate_split = 1
    assert ff.lib().ffuse_traffic_model(ctypes.byref(_plan(16, 2)), ff.DT_BF16, 0, 17, 64, 64, 64, ctypes.byref(t)) == -8
    assert ff.lib().ffuse_traffic_model(ctypes.byref(split), ff.DT_BF16, 1, 16, 64, 64, 64, ctypes.byref(t)) == -8
