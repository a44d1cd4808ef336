"""Which plan runs in a workspace of a given size: the best-ranked of those that fit, on every path, so that a
workspace is refused only where no plan for the problem fits it."""
import pytest
import torch

from paper_2512_12949_amd import binding as ff
from paper_2512_12949_amd import inputs
from paper_2512_12949_amd.inputs import ACT_GELU_TANH, ACT_RELU, ACT_SILU

import gpu_util as gu
import oracle

pytestmark = pytest.mark.gpu


def plan_bytes(p, M, N1, N2):
    """Workspace of a 16-bit plan, from the families' layouts."""
    up = lambda v: (v + 255) // 256 * 256
    if p.family == ff.FAMILY_ROWS:
        return 0
    if p.family == ff.FAMILY_REDUCE and p.bm > 32:
        return 4 * M * N2
    if p.family == ff.FAMILY_REDUCE:                       # whole slices of 64 hidden columns per range
        ns = -(-N1 // 64)
        slices = -(-ns // min(p.splits, ns))
        return up(4 * M * N2 * -(-ns // slices))
    if p.family == ff.FAMILY_TWOPHASE:
        ksplit = -(-(-(-N1 // p.splits)) // 64) * 64
        planes = -(-N1 // ksplit)
        return (up(4 * M * N2 * planes) if planes > 1 else 0) + (1 + p.gate_split) * up(2 * M * N1) + 1024
    return 1 << 62                                         # (the exchange family is never a second choice)


def _problem(M, K, N1, N2, gated, cfg_id):
    w = inputs.custom("ws", M, K, N1, N2, dtype="bf16", act=ACT_SILU if gated else ACT_GELU_TANH, gated=gated, cfg_id=cfg_id)
    host = inputs.make(w)
    return w, gu.oracle_rows(w, host), {k: gu.to_device(v, "bf16") for k, v in host.items()}


@pytest.mark.parametrize("M,K,N1,N2,gated", [(64, 264, 1304, 520, True), (128, 384, 1536, 384, False), (300, 264, 1304, 520, True),
                                             (600, 264, 1304, 520, False), (700, 264, 2056, 520, False)])
def test_the_best_plan_that_fits_runs(M, K, N1, N2, gated):
    w, ref, dev = _problem(M, K, N1, N2, gated, 1101)
    ranked = [(p, plan_bytes(p, M, N1, N2)) for p, _ in ff.ffuse_rank_plans(ff.DT_BF16, w.act, gated, M, K, N1, N2, 1024)]
    model = lambda p: ff.ffuse_traffic_model(p, ff.DT_BF16, gated, M, K, N1, N2)
    sizes = sorted({b for _, b in ranked if 0 < b < 1 << 40})
    Y = torch.empty((M, N2), dtype=torch.bfloat16, device="cuda")
    for nbytes in sorted({sizes[0], sizes[len(sizes) // 3], sizes[len(sizes) // 2], sizes[-1]}, reverse=True):
        first = next(p for p, b in ranked if b <= nbytes)
        ws = torch.full((nbytes,), 0xA5, dtype=torch.uint8, device="cuda")
        for registered in (False, True):
            print(f"{(M, K, N1, N2)} gated={gated} workspace {nbytes} registered={registered}", flush=True)
            Y.fill_(float("nan"))
            if registered:
                gu.Workspace.buf = None
                ff.ffuse_set_workspace(ws)
                ff.FUSED["bf16"](dev["X"], dev["W1"], dev["W3"], dev["W2"], w.act, Y)
            else:
                ff.ffuse_ffn_ws(ff.DT_BF16, dev["X"], dev["W1"], dev["W3"], dev["W2"], w.act, Y, ws)
            ff.ffuse_sync_status()
            gu.check(Y, ref, "bf16", what=f"workspace of {nbytes}")
            last = ff.ffuse_last_plan()
            if last.as_dict() != first.as_dict():      # a near-tie goes to the plan with at most half the bytes
                a, b = model(first), model(last)
                assert plan_bytes(last, M, N1, N2) <= nbytes and b.t_pred <= 1.06 * a.t_pred and b.fabric_bytes <= 0.5 * a.fabric_bytes
    ff.ffuse_set_workspace(None)
    if gated:      # (without a gate the rows family needs no workspace at all)
        assert ff.ffuse_ffn_ws(ff.DT_BF16, dev["X"], dev["W1"], dev["W3"], dev["W2"], w.act, Y, ws[: (sizes[0] - 256) // 16 * 16], check=False) == -5
        assert ff.ffuse_ffn_ws(ff.DT_BF16, dev["X"], dev["W1"], dev["W3"], dev["W2"], w.act, Y, None, check=False) == -5


@pytest.mark.parametrize("M,K,N1,N2,gated", [(64, 264, 1304, 520, True), (333, 1016, 2744, 1016, False), (700, 264, 2056, 520, False)])
def test_the_two_launch_path_takes_the_best_plan_that_fits(M, K, N1, N2, gated):
    w, ref, dev = _problem(M, K, N1, N2, gated, 1102)
    ranked = [p for p, _ in ff.ffuse_rank_plans(ff.DT_BF16, w.act, gated, M, K, N1, N2, 1024) if p.family == ff.FAMILY_TWOPHASE]
    sizes = sorted({plan_bytes(p, M, N1, N2) for p in ranked})
    Y = torch.empty((M, N2), dtype=torch.bfloat16, device="cuda")
    for nbytes in (sizes[-1], sizes[len(sizes) // 2], sizes[0]):
        print(f"two launches {(M, K, N1, N2)} gated={gated} workspace {nbytes}", flush=True)
        ws = torch.full((nbytes,), 0xA5, dtype=torch.uint8, device="cuda")
        Y.fill_(float("nan"))
        ff.ffuse_ffn_unfused_ws(ff.DT_BF16, dev["X"], dev["W1"], dev["W3"], dev["W2"], w.act, Y, ws)
        torch.cuda.synchronize()
        gu.check(Y, ref, "bf16", what=f"two launches, workspace of {nbytes}")
        # the same bits as the fused call in the plan that should have run
        first = next(p for p in ranked if plan_bytes(p, M, N1, N2) <= nbytes)
        assert torch.equal(Y, gu.run(w, dev, plan=first))
    assert ff.ffuse_ffn_unfused_ws(ff.DT_BF16, dev["X"], dev["W1"], dev["W3"], dev["W2"], w.act, Y, ws[: sizes[0] - 256], check=False) == -5


def test_a_3x3_chain_forgets_a_small_workspace():
    """A plan picked because a small workspace was registered does not stay when a larger one is."""
    w = inputs.ConvWorkload("ws3", 1, 14, 14, 64, 256, 256, 3, 1, "bf16", ACT_RELU, 610)
    host = inputs.make_conv(w)
    ref = oracle.conv_chain(host["X"], host["W1"], host["W2"], ACT_RELU, bf16=True)
    dev = {k: gu.to_device(v, "bf16") for k, v in host.items()}
    M, K = 14 * 14, 9 * 64
    gu.Workspace.buf = None
    seen = {}
    for step, nbytes in enumerate((4 * M * 256 + 4096, 64 << 20, 4 * M * 256 + 4096, 64 << 20)):
        ws = torch.full((nbytes // 256 * 256,), 0xA5, dtype=torch.uint8, device="cuda")
        ff.ffuse_set_workspace(ws)
        Y = torch.full((1, 14, 14, 256), float("nan"), dtype=torch.bfloat16, device="cuda")
        ff.ffuse_conv_chain(dev["X"], dev["W1"], dev["W2"], ACT_RELU, Y)
        ff.ffuse_sync_status()
        gu.check(Y.reshape(M, 256), ref.reshape(M, 256), "bf16", what=f"step {step}, workspace of {nbytes}")
        last = ff.ffuse_last_plan()
        assert plan_bytes(last, M, 256, 256) <= ws.numel()
        assert seen.setdefault(nbytes, last.as_dict()) == last.as_dict(), f"step {step}"
    assert len({tuple(p.items()) for p in seen.values()}) == 2
    # the plan of the large workspace is the ranking's first among the loader's plans
    first = next(p for p, _ in ff.ffuse_rank_plans(ff.DT_BF16, ACT_RELU, False, M, K, 256, 256, 1024)
                 if (p.family == ff.FAMILY_TWOPHASE and p.bm <= 128 and p.bk != 32) or (p.family == ff.FAMILY_REDUCE and p.bm <= 32))
    assert seen[64 << 20] == first.as_dict()
    ff.ffuse_set_workspace(None)
