"""GPU parity of the gate backward (moe_route_bwd) against the float64 oracle."""
import numpy as np
import pytest
import torch

import moe_workloads as wl
import paper_2510_19470_amd as moe
from oracle import moe_oracle as orc
from gpu_common import TOL, nerr, to_device, to_host_f32, vals

pytestmark = pytest.mark.gpu


def _case(cfg, renorm, T=None):
    T = T or cfg.T
    inp = wl.make_inputs(cfg, experts="none")
    x, Wg = inp.x[:T], inp.Wg
    rng = np.random.default_rng(cfg.seed + 5)
    dw = rng.standard_normal((T, cfg.k)).astype(np.float32)
    dx0 = wl.store(rng.standard_normal((T, cfg.d)).astype(np.float32), cfg.dtype)
    ctx = moe.moe_create(T_max=T, d=cfg.d, E=cfg.E, k=cfg.k, f=cfg.f, R=cfg.R, local_rank=0,
                         dtype=moe.MOE_BF16 if cfg.dtype == "bf16" else moe.MOE_F32,
                         renormalize=int(renorm))
    dx_ = to_device(x, cfg.dtype)
    dWg_ = to_device(Wg, cfg.dtype)
    bias = None if inp.bias is None else torch.from_numpy(inp.bias.astype(np.float32)).cuda()
    idx, w, logits = moe.moe_route(ctx, dx_, dWg_, bias, want_logits=True)
    ddx = to_device(dx0, cfg.dtype)
    dl, dWg, db = moe.moe_route_bwd(ctx, dx_, dWg_, idx, w, torch.from_numpy(dw).cuda(),
                                    logits=logits, dx=ddx, want_dbias=True)
    torch.cuda.synchronize()
    # the oracle takes the GPU's own logits and selection (the selection is checked elsewhere)
    L = logits.cpu().numpy().astype(np.float64)
    oL, oW, ob, ox = orc.route_bwd(vals(x, cfg.dtype), vals(Wg, cfg.dtype), L,
                                   idx.cpu().numpy(), dw.astype(np.float64), renorm)
    assert nerr(dl.cpu().numpy(), oL) <= 1e-5
    assert nerr(dWg.cpu().numpy(), oW) <= 1e-4
    assert nerr(db.cpu().numpy(), ob) <= 1e-4
    assert nerr(to_host_f32(ddx), vals(dx0, cfg.dtype) + ox) <= TOL[cfg.dtype]
    # the added part alone, against its own scale (dx0 is O(1), the gate term can be smaller)
    got_gate = to_host_f32(ddx).astype(np.float64) - vals(dx0, cfg.dtype)
    ulp = 2.0 ** -8 if cfg.dtype == "bf16" else 2.0 ** -23
    assert np.max(np.abs(got_gate - ox)) <= 4 * ulp * np.max(np.abs(vals(dx0, cfg.dtype))) + 1e-4 * np.max(np.abs(ox))
    moe.moe_destroy(ctx)


@pytest.mark.parametrize("renorm", [True, False])
def test_tiny_f32(renorm):
    _case(wl.CONFIGS["tiny"], renorm)


@pytest.mark.parametrize("renorm", [True, False])
def test_bf16_ragged_T(renorm):
    _case(wl.scaled(wl.CONFIGS["small"], T=1000, d=512, E=16), renorm)


def test_finegrained_shape_bias_and_many_experts():
    _case(wl.scaled(wl.CONFIGS["finegrained"], T=2048), True)
    _case(wl.scaled(wl.CONFIGS["finegrained"], T=700), False)


def test_mixtral_full_size():
    _case(wl.CONFIGS["mixtral"], True)


def test_determinism_and_empty():
    cfg = wl.scaled(wl.CONFIGS["small"], T=777, d=512)
    inp = wl.make_inputs(cfg, experts="none")
    ctx = moe.moe_create(T_max=cfg.T, d=cfg.d, E=cfg.E, k=cfg.k, f=cfg.f, R=cfg.R, local_rank=0,
                         dtype=moe.MOE_BF16, renormalize=1)
    x, Wg = to_device(inp.x, "bf16"), to_device(inp.Wg, "bf16")
    idx, w, _ = moe.moe_route(ctx, x, Wg, None)
    dw = torch.randn(cfg.T, cfg.k, device="cuda")
    a = moe.moe_route_bwd(ctx, x, Wg, idx, w, dw)
    b = moe.moe_route_bwd(ctx, x, Wg, idx, w, dw)
    torch.cuda.synchronize()
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    # T = 0: defined outputs, no launch
    e = moe.moe_route_bwd(ctx, x[:0], Wg, idx[:0], w[:0], dw[:0], want_dbias=True)
    torch.cuda.synchronize()
    assert e[0].shape == (0, cfg.E) and float(e[1].abs().sum()) == 0.0 and float(e[2].abs().sum()) == 0.0
    moe.moe_destroy(ctx)


@pytest.mark.parametrize("renorm", [True, False])
@pytest.mark.parametrize("dtype,T,d,E,k", [
    ("bf16", 1, 8, 2, 1),        # one token of a step of four, one column group of sixteen
    ("bf16", 131, 136, 17, 3),   # a second chunk of 3 tokens, second column block, second expert group
    ("bf16", 163, 1160, 65, 6),  # steps of 32 tokens and single ones; experts of a second lane group
    ("bf16", 40, 256, 256, 8),   # as many experts as there can be
    ("bf16", 70, 1032, 40, 12),  # more than eight experts of a token, two pieces of a row and a bit
    ("f32", 33, 72, 16, 2),      # 64 columns a wavefront
    ("f32", 130, 520, 200, 4),
])
def test_tile_edges(dtype, T, d, E, k, renorm):
    _case(wl.MoEConfig("edges", 91 + T + d, dtype, T=T, d=d, E=E, k=k, f=8, R=1), renorm)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_x_aligned_to_its_elements_only(dtype):
    T, d, E, k = 150, 136, 20, 2
    ctx = moe.moe_create(T_max=T, d=d, E=E, k=k, f=8, R=1, local_rank=0, renormalize=1,
                         dtype=moe.MOE_BF16 if dtype == torch.bfloat16 else moe.MOE_F32)
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn(T, d, device="cuda", generator=g).to(dtype)
    Wg = torch.randn(E, d, device="cuda", generator=g).to(dtype)
    idx, w, _ = moe.moe_route(ctx, x, Wg, None)
    dw = torch.randn(T, k, device="cuda", generator=g)
    off = torch.empty(T * d + 1, dtype=dtype, device="cuda")[1:].view(T, d)
    off.copy_(x)
    a = moe.moe_route_bwd(ctx, x, Wg, idx, w, dw)
    b = moe.moe_route_bwd(ctx, off, Wg, idx, w, dw)
    torch.cuda.synchronize()
    assert off.data_ptr() % 16 != 0 and torch.equal(a[1], b[1])
    moe.moe_destroy(ctx)


@pytest.mark.parametrize("renorm", [1, 0])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_gradients_that_are_not_finite_show_in_both_outputs(bad, renorm):
    """dWg = dlogits^T x for what is no number, too: a token whose dtopk_w is not finite has no finite logit gradient."""
    T, d, E, k = 200, 136, 40, 2
    ctx = moe.moe_create(T_max=T, d=d, E=E, k=k, f=8, R=1, dtype=moe.MOE_BF16, renormalize=renorm)
    g = torch.Generator(device="cuda").manual_seed(4)
    x, Wg = (torch.randn(n, d, device="cuda", generator=g).bfloat16() for n in (T, E))
    idx, w, logits = moe.moe_route(ctx, x, Wg, None, want_logits=True)
    dw = torch.randn(T, k, device="cuda", generator=g)
    dw[150, 0] = bad
    dl, dWg, _ = moe.moe_route_bwd(ctx, x, Wg, idx, w, dw, logits=logits)
    torch.cuda.synchronize()
    assert not torch.isfinite(dl[150]).any() and torch.isfinite(dl[:150]).all() and torch.isfinite(dl[151:]).all()
    assert not torch.isfinite(dWg).any()
    moe.moe_destroy(ctx)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("T,d,E,k", [
    (131, 136, 17, 1), (260, 520, 64, 2),   # one piece of a row or a bit of it (f32: two and a bit)
    (77, 1160, 65, 4), (64, 2056, 40, 7), (33, 1032, 256, 16),
])
def test_one_launch_and_two_give_the_same(dtype, T, d, E, k):
    """The logit gradients beside the weight gradient's sums or before them, with and without dx; and a routing that
    names experts that do not exist."""
    ctx = moe.moe_create(T_max=T, d=d, E=E, k=k, f=8, R=1, renormalize=1,
                         dtype=moe.MOE_BF16 if dtype == torch.bfloat16 else moe.MOE_F32)
    g = torch.Generator(device="cuda").manual_seed(7 + T)
    x, Wg, dx = (torch.randn(n, d, device="cuda", generator=g).to(dtype) for n in (T, E, T))
    idx, w, _ = moe.moe_route(ctx, x, Wg, None)
    idx[T // 2, 0], idx[T // 3, k - 1] = E, -1
    dw = torch.randn(T, k, device="cuda", generator=g)
    got = {}
    for joint in (1, 2):
        moe.load_library().moe_internal_gate_joint(ctx.handle, joint)
        out = dx.clone()
        dl, dWg, db = moe.moe_route_bwd(ctx, x, Wg, idx, w, dw, dx=out, want_dbias=True)
        only = moe.moe_route_bwd(ctx, x, Wg, idx, w, dw)
        torch.cuda.synchronize()
        assert torch.equal(only[0], dl) and torch.equal(only[1], dWg)
        got[joint] = (dl, dWg, db, out)
    for a, b in zip(got[1], got[2]):
        assert torch.equal(a, b)
    moe.moe_destroy(ctx)
