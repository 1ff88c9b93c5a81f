"""GPU parity of the expert FFN, forward and backward, at the edges of the tiled kernels: sizes
that no tile divides (one and several k-steps, a partial and a rounded-up last step, a last
column block of 8 columns), next to sizes that it does.  bf16 and fp32."""
import numpy as np
import pytest
import torch

import moe_workloads as wl
from oracle import moe_oracle as orc

pytestmark = pytest.mark.gpu


def _f64(ws, dtype):
    return [None if w is None else wl.stored_to_f32(w, dtype).astype(np.float64) for w in ws]


@pytest.mark.parametrize("gated", [True, False])
@pytest.mark.parametrize("dtype,T,d,E,k,f", [
    ("bf16", 200, 8, 4, 2, 8),          # one partial k-step, the second one all padding
    ("bf16", 300, 72, 4, 2, 136),       # the last k-step holds 8 of 64
    ("bf16", 515, 136, 6, 3, 264),      # three k-steps and a padding one; 8 columns in a block
    ("bf16", 300, 320, 3, 2, 2888),     # K-split parts of the down GEMM, the last one partial
    ("bf16", 700, 1160, 4, 2, 384),     # f a multiple of 128 only
    ("bf16", 260, 512, 3, 1, 1408),
    ("f32", 50, 8, 4, 2, 8),            # one partial contraction step, 32x32 tiles
    ("f32", 515, 136, 6, 3, 264),
    ("f32", 900, 72, 80, 2, 520),       # more experts than a wavefront has lanes
    ("f32", 8000, 200, 3, 2, 1032),     # 64x64 tiles, all sides ragged
])
def test_forward_and_backward_match_oracle(dtype, T, d, E, k, f, gated):
    from gpu_common import DEV, TOL, moe, nerr, vals, to_device, to_host_f32, layer_from_inputs, say
    say(f"[ffn sizes] {dtype} T={T} d={d} E={E} k={k} f={f} gated={gated}")
    cfg = wl.MoEConfig("sizes", 31 + T + d, dtype, T=T, d=d, E=E, k=k, f=f, R=1, gated=gated)
    inp = wl.make_inputs(cfg)
    lay = layer_from_inputs(inp)
    idx = wl.random_routing(T, E, k, seed=T + 1, skew=0.6)
    cnt, off, _, _, s2r, r2s = orc.dispatch_maps(idx, inp.dest_rank, cfg.R)
    xp_st = orc.pack_rows(inp.x, r2s, k)
    dy_st = wl.store(np.random.default_rng(T).standard_normal((cfg.S, d)).astype(np.float32), dtype)
    xp, dy = to_device(xp_st, dtype), to_device(dy_st, dtype)
    cnt_d, off_d = torch.from_numpy(cnt).to(DEV), torch.from_numpy(off).to(DEV)
    y, G, U = moe.moe_expert_ffn(lay.ctx, xp, cnt_d, off_d, lay.W1, lay.W3, lay.W2, save=True)
    dxp, dW1, dW3, dW2 = moe.moe_expert_ffn_bwd(lay.ctx, dy, xp, G, U, cnt_d, off_d, lay.W1,
                                                lay.W3, lay.W2)
    torch.cuda.synchronize()
    W1, W2 = _f64(inp.W1, dtype), _f64(inp.W2, dtype)
    xv, dyv = vals(xp_st, dtype), vals(dy_st, dtype)
    tol = TOL[dtype]
    # the backward is checked from the GPU's saves (themselves checked): the two-matrix expert
    # takes a yes/no decision on them
    Gg = to_host_f32(G).astype(np.float64)
    if gated:
        W3 = _f64(inp.W3, dtype)
        yo, Go, Uo = orc.expert_ffn(xv, cnt, off, W1, W3, W2)
        assert nerr(to_host_f32(U), Uo) <= tol
        Ug = to_host_f32(U).astype(np.float64)
        dxo, g1, g3, g2 = orc.expert_ffn_bwd(dyv, xv, Gg, Ug, cnt, off, W1, W3, W2)
    else:
        yo, Go = orc.expert_ffn2(xv, cnt, off, W1, W2)
        dxo, g1, g2 = orc.expert_ffn2_bwd(dyv, xv, Gg, cnt, off, W1, W2)
        g3 = None
    assert nerr(Gg, Go) <= tol
    errs = dict(y=nerr(to_host_f32(y), yo), dx=nerr(to_host_f32(dxp), dxo))
    for name, got, want in (("dW1", dW1, g1), ("dW3", dW3, g3), ("dW2", dW2, g2)):
        if want is None:
            continue
        scale = max(np.max(np.abs(w)) for w in want)   # experts with few rows: the layer's largest
        errs[name] = max(float(np.max(np.abs(g.cpu().numpy() - w))) for g, w in zip(got, want)) / scale
    say("    " + ", ".join(f"{n}={v:.2e}" for n, v in errs.items()))
    bad = {n: v for n, v in errs.items() if not v <= tol}
    assert not bad, bad
    lay.close()


@pytest.mark.parametrize("gated", [True, False])
@pytest.mark.parametrize("T,d,E,k,f,skew", [
    (1, 8, 4, 2, 8, 0.0),          # a single chunk of the contraction, 8 of 16 weight rows
    (7, 72, 4, 2, 136, 0.6),       # a partial unit after a whole one
    (16, 520, 8, 2, 1032, 0.0),    # one unit for each wavefront and a partial one
    (20, 2048, 8, 2, 4104, 3.0),   # several rounds of units
    (33, 2048, 8, 2, 4104, 3.0),   # too many token rows through L2 for that: the tiles
    (150, 1160, 16, 2, 520, 0.6),  # more tokens than one pass takes rows: the tiles
    (256, 320, 24, 2, 264, 4.0),
    (2, 64, 256, 4, 64, 0.0),      # as many experts as there can be
])
def test_few_rows_per_expert_match_oracle(T, d, E, k, f, skew, gated):
    from gpu_common import DEV, TOL, moe, nerr, vals, to_device, to_host_f32, layer_from_inputs, say
    say(f"[few rows] T={T} d={d} E={E} k={k} f={f} gated={gated}")
    cfg = wl.MoEConfig("few", 77 + T + d, "bf16", T=T, d=d, E=E, k=k, f=f, R=1, gated=gated)
    inp = wl.make_inputs(cfg)
    lay = layer_from_inputs(inp)
    idx = wl.random_routing(T, E, k, seed=T + 1, skew=skew)
    cnt, off, _, _, s2r, r2s = orc.dispatch_maps(idx, inp.dest_rank, cfg.R)
    xp_st = orc.pack_rows(inp.x, r2s, k)
    cnt_d, off_d = torch.from_numpy(cnt).to(DEV), torch.from_numpy(off).to(DEV)
    y, G, U = moe.moe_expert_ffn(lay.ctx, to_device(xp_st, "bf16"), cnt_d, off_d, lay.W1, lay.W3,
                                 lay.W2, save=True)
    torch.cuda.synchronize()
    W1, W2 = _f64(inp.W1, "bf16"), _f64(inp.W2, "bf16")
    if gated:
        yo, Go, Uo = orc.expert_ffn(vals(xp_st, "bf16"), cnt, off, W1, _f64(inp.W3, "bf16"), W2)
        assert nerr(to_host_f32(U), Uo) <= TOL["bf16"]
    else:
        yo, Go = orc.expert_ffn2(vals(xp_st, "bf16"), cnt, off, W1, W2)
    assert nerr(to_host_f32(G), Go) <= TOL["bf16"]
    assert nerr(to_host_f32(y), yo) <= TOL["bf16"]
    lay.close()


# rows: of each expert, given by hand; more rows on one expert than there are tokens need another pass
# over its weights (no routing does that, a caller's counts may)
@pytest.mark.parametrize("gated", [True, False])
@pytest.mark.parametrize("T,d,E,k,f,rows", [
    (16, 2048, 8, 2, 2056, [16, 1, 0, 15, 0, 0, 0, 0]),       # four units of the contraction in flight
    (64, 2048, 8, 2, 1032, [17, 32, 33, 0, 16, 1, 29, 0]),    # 16, 32 and 64 rows a pass
    (64, 1160, 8, 2, 520, [0, 63, 0, 65, 0, 0, 0, 0]),        # a second pass for one row
    (64, 320, 8, 3, 264, [0, 0, 192, 0, 0, 0, 0, 0]),         # three whole passes
])
def test_few_rows_per_expert_by_given_counts(T, d, E, k, f, rows, gated):
    from gpu_common import DEV, TOL, moe, nerr, vals, to_device, to_host_f32, layer_from_inputs, say
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    assert moe.load_library().moe_internal_ffn_few_rows(T, d, f, E, k, E, int(gated), n_cu)
    say(f"[few rows, given] T={T} d={d} E={E} k={k} f={f} rows={rows} gated={gated}")
    cfg = wl.MoEConfig("given", 5 + T + d, "bf16", T=T, d=d, E=E, k=k, f=f, R=1, gated=gated)
    inp = wl.make_inputs(cfg)
    lay = layer_from_inputs(inp)
    cnt = np.array(rows, np.int32)
    off = (np.cumsum(cnt) - cnt).astype(np.int32)
    xp_st = wl.store(np.random.default_rng(d).standard_normal((T * k, d)).astype(np.float32), "bf16")
    y0 = torch.full((T * k, d), 3.0, dtype=torch.bfloat16, device=DEV)
    y, G, U = moe.moe_expert_ffn(lay.ctx, to_device(xp_st, "bf16"), torch.from_numpy(cnt).to(DEV),
                                 torch.from_numpy(off).to(DEV), lay.W1, lay.W3, lay.W2, y_packed=y0, save=True)
    torch.cuda.synchronize()
    n = int(cnt.sum())
    W1, W2 = _f64(inp.W1, "bf16"), _f64(inp.W2, "bf16")
    if gated:
        yo, Go, Uo = orc.expert_ffn(vals(xp_st, "bf16"), cnt, off, W1, _f64(inp.W3, "bf16"), W2)
        assert nerr(to_host_f32(U)[:n], Uo[:n]) <= TOL["bf16"]
    else:
        yo, Go = orc.expert_ffn2(vals(xp_st, "bf16"), cnt, off, W1, W2)
    assert nerr(to_host_f32(G)[:n], Go[:n]) <= TOL["bf16"]
    assert nerr(to_host_f32(y)[:n], yo[:n]) <= TOL["bf16"]
    assert torch.all(y[n:] == 3.0)      # rows of no expert are left alone
    lay.close()
