"""GPU parity of the bf16 expert FFN, forward and backward, for given rows per expert, in 128-row and in
256-row tiles: the edges of the row blocks and their 32-row parts, of the 16-row slices and the ring of
seven that the weight gradients run ahead, of k-steps and column blocks, and cut contractions."""
import numpy as np
import pytest
import torch

import moe_workloads as wl
from oracle import moe_oracle as orc

pytestmark = pytest.mark.gpu


def _f64(ws):
    return [None if w is None else wl.stored_to_f32(w, "bf16").astype(np.float64) for w in ws]


@pytest.mark.parametrize("tile", [128, 256])
@pytest.mark.parametrize("gated", [True, False])
@pytest.mark.parametrize("d,f,rows", [
    (512, 256, [1, 0, 15, 16, 17, 31, 32, 33]),        # whole tiles of the weight gradients
    (264, 520, [63, 64, 65, 0, 96, 97, 1, 2]),         # every last block 8 columns wide
    (256, 1032, [111, 112, 113, 127, 128, 129, 0, 5]), # one more and one less than the ring holds
    (1160, 264, [257, 0, 255, 256, 0, 385, 0, 17]),
    (8, 8, [1, 33, 0, 130]),                           # one partial k-step
    (72, 136, [300, 0, 65, 31]),                       # 8 of 64 in the last k-step, 8 columns in a block
    (136, 2888, [100, 200, 0, 1]),                     # several parts per contraction, the last one partial
    (520, 4096, [0, 64, 0, 0]),                        # eight parts, one expert
])
def test_given_rows_match_oracle(d, f, rows, gated, tile):
    _check_given_rows(d, f, rows, gated, tile)


# The kernel for few rows takes 32 weight rows a block in calls of at most 16 tokens and contractions of at most 2048,
# of two matrices 768, where there are blocks enough (the first GEMM here, the second, both, neither); counts may hold
# more rows of an expert than there are tokens.
@pytest.mark.parametrize("gated", [True, False])
@pytest.mark.parametrize("d,f,rows", [
    (2048, 2056, [16, 0, 1, 9]), (2056, 2048, [20, 3, 0, 9]), (520, 40, [17, 15]), (2056, 2064, [32, 0]),
    (768, 4104, [16, 0, 1, 9]), (776, 2048, [3, 20, 0, 9]), (4104, 2048, [5, 4, 3, 20]),
])
def test_few_rows_match_oracle(d, f, rows, gated):
    _check_given_rows(d, f, rows, gated, 16)


# The schedule gives dH to the 128-row tiles (one round of theirs against one; two against one:
# the larger ones), whatever serves the other GEMMs.
@pytest.mark.parametrize("gated", [True, False])
@pytest.mark.parametrize("d,f,rows", [(264, 520, [130, 0, 65, 257]), (72, 4096, [2200, 0, 65]), (72, 4096, [17, 400])])
def test_dh_in_either_tiles_matches_oracle(d, f, rows, gated):
    _check_given_rows(d, f, rows, gated, 384)


# A block's tiles follow one another without a stop: the next one's first copies are under way while the
# outputs of the last are stored.  512 blocks serve the 128-row tiles, 256 the 256-row ones (here 816 and 264
# tiles or more in each of the four GEMMs), and tiles that follow one another differ in the rows they hold.
@pytest.mark.parametrize("tile", [128, 256])
@pytest.mark.parametrize("gated", [True, False])
@pytest.mark.parametrize("d,f", [(648, 648), (768, 768)])
def test_several_tiles_per_block_match_oracle(d, f, gated, tile):
    rows = [1, 33, 129, 161, 300, 385, 20, 257] * 8
    for n in (d, f):
        n_tiles = sum(-(-r // tile) for r in rows) * -(-n // tile)
        assert n_tiles > (2 if tile == 128 else 1) * torch.cuda.get_device_properties(0).multi_processor_count
    _check_given_rows(d, f, rows, gated, tile)


def _check_given_rows(d, f, rows, gated, tile):
    from gpu_common import DEV, TOL, moe, nerr, vals, to_device, to_host_f32, layer_from_inputs, say
    say(f"[row edges] d={d} f={f} rows={rows} gated={gated} tile={tile}")
    E, k = len(rows), 2
    cnt = np.array(rows, np.int32)
    T = -(-int(cnt.sum()) // k)
    cfg = wl.MoEConfig("rows", 3 + d + f, "bf16", T=T, d=d, E=E, k=k, f=f, R=1, gated=gated)
    inp = wl.make_inputs(cfg)
    lay = layer_from_inputs(inp)
    moe.load_library().moe_internal_ffn_tile_rows(lay.ctx.handle, tile)
    off = (np.cumsum(cnt) - cnt).astype(np.int32)
    n = int(cnt.sum())
    rng = np.random.default_rng(d)
    xp_st = wl.store(rng.standard_normal((T * k, d)).astype(np.float32), "bf16")
    dy_st = wl.store(rng.standard_normal((T * k, d)).astype(np.float32), "bf16")
    xp, dy = to_device(xp_st, "bf16"), to_device(dy_st, "bf16")
    cnt_d, off_d = torch.from_numpy(cnt).to(DEV), torch.from_numpy(off).to(DEV)
    y, G, U = moe.moe_expert_ffn(lay.ctx, xp, cnt_d, off_d, lay.W1, lay.W3, lay.W2, save=True)
    dxp, dW1, dW3, dW2 = moe.moe_expert_ffn_bwd(lay.ctx, dy, xp, G, U, cnt_d, off_d, lay.W1,
                                                lay.W3, lay.W2)
    torch.cuda.synchronize()
    W1, W2 = _f64(inp.W1), _f64(inp.W2)
    xv, dyv = vals(xp_st, "bf16"), vals(dy_st, "bf16")
    # the backward from the GPU's saves, which are checked themselves
    Gg = to_host_f32(G).astype(np.float64)
    if gated:
        W3 = _f64(inp.W3)
        yo, Go, Uo = orc.expert_ffn(xv, cnt, off, W1, W3, W2)
        Ug = to_host_f32(U).astype(np.float64)
        assert nerr(Ug[:n], Uo[:n]) <= TOL["bf16"]
        dxo, g1, g3, g2 = orc.expert_ffn_bwd(dyv, xv, Gg, Ug, cnt, off, W1, W3, W2)
    else:
        yo, Go = orc.expert_ffn2(xv, cnt, off, W1, W2)
        dxo, g1, g2 = orc.expert_ffn2_bwd(dyv, xv, Gg, cnt, off, W1, W2)
        g3 = None
    # every expert by itself: a wrong tile, a row too many or too few shows where there are few
    yg, dxg = to_host_f32(y), to_host_f32(dxp)
    for e in range(E):
        seg = slice(int(off[e]), int(off[e] + cnt[e]))
        if cnt[e] > 0:
            assert nerr(Gg[seg], Go[seg]) <= TOL["bf16"], ("G", e, rows[e])
            assert nerr(yg[seg], yo[seg]) <= TOL["bf16"], ("y", e, rows[e])
            assert nerr(dxg[seg], dxo[seg]) <= TOL["bf16"], ("dX", e, rows[e])
    for got, want in ((dW1, g1), (dW3, g3), (dW2, g2)):
        for e in range(E if want is not None else 0):
            assert nerr(got[e].cpu().numpy(), want[e]) <= TOL["bf16"], (e, rows[e])
    lay.close()


@pytest.mark.parametrize("tile", [128, 256, 384])
def test_counts_that_do_not_fit_compute_nothing(tile):
    """A segment outside the buffers, a negative count, a negative offset: no output is written, the weight
    gradients are zero."""
    from gpu_common import DEV, moe, to_device, layer_from_inputs
    E, k, T, d, f = 4, 2, 64, 136, 264
    cfg = wl.MoEConfig("bad", 9, "bf16", T=T, d=d, E=E, k=k, f=f, R=1)
    inp = wl.make_inputs(cfg)
    lay = layer_from_inputs(inp)
    moe.load_library().moe_internal_ffn_tile_rows(lay.ctx.handle, tile)
    xp = to_device(wl.store(np.ones((T * k, d), np.float32), "bf16"), "bf16")
    G, U = (torch.ones((T * k, f), dtype=torch.bfloat16, device=DEV) for _ in range(2))
    for cnt, off in (([10, 120, 0, 0], [0, 10, 0, 0]), ([10, -1, 0, 0], [0, 10, 0, 0]),
                     ([128, 10, 0, 0], [0, -1, 0, 0])):
        c = torch.tensor(cnt, dtype=torch.int32, device=DEV)
        o = torch.tensor(off, dtype=torch.int32, device=DEV)
        y = torch.full((T * k, d), 3.0, dtype=torch.bfloat16, device=DEV)
        moe.moe_expert_ffn(lay.ctx, xp, c, o, lay.W1, lay.W3, lay.W2, y_packed=y)
        dxp = torch.full((T * k, d), 5.0, dtype=torch.bfloat16, device=DEV)
        _, dW1, _, dW2 = moe.moe_expert_ffn_bwd(lay.ctx, xp, xp, G, U, c, o, lay.W1, lay.W3, lay.W2,
                                                dx_packed=dxp)
        torch.cuda.synchronize()
        assert torch.all(y == 3.0) and torch.all(dxp == 5.0)
        assert all(torch.all(w == 0) for w in dW1 + dW2)
    lay.close()


def test_dh_is_computed_by_either_tiles_where_segments_overlap():
    """Experts that share their rows: more 128-row blocks than a call of these tokens can have, not more 256-row
    ones.  The schedule offers dH to the smaller tiles only where they take it.  (All experts have the same weights:
    whoever writes a shared row writes the same.)"""
    from gpu_common import DEV, moe
    E, k, T, d, f = 4, 2, 128, 136, 264
    g = torch.Generator(device=DEV).manual_seed(5)
    one = lambda r, c: [(torch.randn(r, c, device=DEV, generator=g) * c ** -0.5).bfloat16()] * E
    W1, W3, W2 = one(f, d), one(f, d), one(d, f)
    x, dy = (torch.randn(T * k, d, device=DEV, generator=g).bfloat16() for _ in range(2))
    G, U = (torch.randn(T * k, f, device=DEV, generator=g).bfloat16() for _ in range(2))
    cnt = torch.full((E,), T * k, dtype=torch.int32, device=DEV)
    off = torch.zeros(E, dtype=torch.int32, device=DEV)
    got = {}
    for tile in (256, 384):
        ctx = moe.moe_create(T_max=T, d=d, E=E, k=k, f=f, R=1, dtype=moe.MOE_BF16)
        moe.load_library().moe_internal_ffn_tile_rows(ctx.handle, tile)
        # other rows first: what a dH that is left out would leave behind
        moe.moe_expert_ffn_bwd(ctx, x, dy, U, G, torch.full_like(cnt, 64), off + 64 * torch.arange(E, device=DEV).int(),
                               W1, W3, W2)
        dxp, dW1, dW3, dW2 = moe.moe_expert_ffn_bwd(ctx, dy, x, G, U, cnt, off, W1, W3, W2)
        torch.cuda.synchronize()
        got[tile] = [dxp] + dW1 + dW3 + dW2
        moe.moe_destroy(ctx)
    assert float(got[256][0].abs().sum()) > 0
    for a, b in zip(got[256], got[384]):
        assert torch.equal(a, b)


@pytest.mark.parametrize("few", [128, 256])
@pytest.mark.parametrize("d,f", [(256, 512), (288, 352), (264, 520)])   # whole tiles; whole lines; neither
def test_weight_gradients_wherever_they_lie(d, f, few):
    """Gradients that begin inside a 128-byte line are stored by another kernel: the same bits, and nothing
    beside them is written."""
    from gpu_common import DEV, moe, to_device, layer_from_inputs
    E, k, T = 3, 2, 100
    cfg = wl.MoEConfig("lines", 5, "bf16", T=T, d=d, E=E, k=k, f=f, R=1)
    inp = wl.make_inputs(cfg)
    lay = layer_from_inputs(inp)
    moe.load_library().moe_internal_wgrad_rows(lay.ctx.handle, few)
    rng = np.random.default_rng(d)
    xp, dy = (to_device(wl.store(rng.standard_normal((T * k, d)).astype(np.float32), "bf16"), "bf16") for _ in range(2))
    cnt = torch.tensor([90, 33, 77], dtype=torch.int32, device=DEV)
    off = torch.tensor([0, 90, 123], dtype=torch.int32, device=DEV)
    y, G, U = moe.moe_expert_ffn(lay.ctx, xp, cnt, off, lay.W1, lay.W3, lay.W2, save=True)

    def grads(shift):   # [E] views, `shift` floats into a 128-byte line, and the buffers they lie in
        flat = [torch.full((rows * cols + 64,), 7.0, device=DEV) for rows, cols in ((f, d), (f, d), (d, f)) for _ in range(E)]
        views = [b[shift:shift + f * d].view(*((d, f) if i >= 2 * E else (f, d))) for i, b in enumerate(flat)]
        moe.moe_expert_ffn_bwd(lay.ctx, dy, xp, G, U, cnt, off, lay.W1, lay.W3, lay.W2, dW1=views[:E],
                               dW3=views[E:2 * E], dW2=views[2 * E:])
        torch.cuda.synchronize()
        assert all(torch.all(b[:shift] == 7.0) and torch.all(b[shift + f * d:] == 7.0) for b in flat)
        return views

    for a, b in zip(grads(0), grads(4)):
        assert torch.equal(a, b)
    lay.close()


@pytest.mark.parametrize("d,f,rows,parts", [
    (128, 4096, [40], 8), (1024, 1408, [64], 4), (1024, 4096, [128] * 10, 3), (2048, 2048, [100] * 8, 2),
    (1536, 5888, [100] * 4, 5), (1280, 5888, [70] * 4, 6), (1152, 5888, [40] * 4, 7),   # a node without a neighbour
])
def test_joined_parts_are_the_same_bits_every_time(d, f, rows, parts):
    """Which of two neighbouring parts is added by which block depends on who comes first; the sum and the counters
    for the next call do not."""
    from gpu_common import DEV, moe
    lib, n, T = moe.load_library(), len(rows), sum(rows)
    slots = 2 * torch.cuda.get_device_properties(0).multi_processor_count // 8 * 8
    assert lib.moe_internal_tile128_parts(sum(-(-r // 128) for r in rows) * -(-d // 128), slots, -(-f // 64)) == parts
    ctx = moe.moe_create(T_max=T, d=d, E=n, k=1, f=f, R=1, dtype=moe.MOE_BF16)
    lib.moe_internal_ffn_tile_rows(ctx.handle, 128)
    g = torch.Generator(device=DEV).manual_seed(d + f)
    W = lambda r, c: [(torch.randn(r, c, device=DEV, generator=g) * c ** -0.5).bfloat16() for _ in rows]
    W1, W2 = W(f, d), W(d, f)
    x = torch.randn(T, d, device=DEV, generator=g).bfloat16()
    cnt = torch.tensor(rows, dtype=torch.int32, device=DEV)
    off = (torch.cumsum(cnt, 0) - cnt).int()
    first = None
    for _ in range(20):
        y, _, _ = moe.moe_expert_ffn(ctx, x, cnt, off, W1, None, W2)
        torch.cuda.synchronize()
        first = y if first is None else first
        assert torch.equal(y, first)
    for e, r in enumerate(rows):
        s = slice(int(off[e]), int(off[e]) + r)
        h = torch.relu(x[s].float() @ W1[e].float().t().contiguous())
        want = h.bfloat16().float() @ W2[e].float().t().contiguous()
        assert float((first[s].float() - want).norm() / want.norm()) <= 1e-2   # bf16 output and H: 2^-8 each
    moe.moe_destroy(ctx)


def test_cut_gate_up_saves_the_same_bits_every_time():
    """The gated expert's first GEMM in four parts, two accumulator halves of 32 rows and a bit: H, G and U."""
    from gpu_common import DEV, moe
    lib, d, f, T = moe.load_library(), 2048, 512, 65
    slots = 2 * torch.cuda.get_device_properties(0).multi_processor_count // 8 * 8
    assert lib.moe_internal_tile128_parts(-(-f // 64), slots, -(-d // 64)) >= 4
    ctx = moe.moe_create(T_max=T, d=d, E=1, k=1, f=f, R=1, dtype=moe.MOE_BF16)
    lib.moe_internal_ffn_tile_rows(ctx.handle, 128)
    g = torch.Generator(device=DEV).manual_seed(11)
    W1, W3 = ([(torch.randn(f, d, device=DEV, generator=g) * d ** -0.5).bfloat16()] for _ in range(2))
    W2 = [(torch.randn(d, f, device=DEV, generator=g) * f ** -0.5).bfloat16()]
    x = torch.randn(T, d, device=DEV, generator=g).bfloat16()
    cnt, off = torch.tensor([T], dtype=torch.int32, device=DEV), torch.zeros(1, dtype=torch.int32, device=DEV)
    first = None
    for _ in range(20):
        got = moe.moe_expert_ffn(ctx, x, cnt, off, W1, W3, W2, save=True)
        torch.cuda.synchronize()
        first = got if first is None else first
        assert all(torch.equal(a, b) for a, b in zip(got, first))
    y, G, U = first
    for got, w in ((G, W1[0]), (U, W3[0])):
        want = x.float() @ w.float().t().contiguous()
        assert float((got.float() - want).norm() / want.norm()) <= 4e-3      # bf16 output: 2^-8 at most
    h = (torch.nn.functional.silu(G.float()) * U.float()).bfloat16().float()
    want = h @ W2[0].float().t().contiguous()
    assert float((y.float() - want).norm() / want.norm()) <= 1e-2   # bf16 output, H, G and U: 2^-8 each
    moe.moe_destroy(ctx)
