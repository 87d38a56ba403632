"""GPU parity of the lm_head variant (logits never materialised) and of its MFMA product."""
import sys

import numpy as np
import pytest
import torch

import paper_2507_19766_amd as ulorl
import ulorl_inputs as ui
from parity import params_for, run_lmhead_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def say(msg):
    print(msg, file=sys.stderr, flush=True)


@pytest.mark.parametrize("M,N,K", [(128, 128, 64), (130, 70, 72), (257, 300, 2048), (1000, 520, 8), (64, 33, 136)])
def test_gemm_tn_bf16_against_fp64(M, N, K):
    g = torch.Generator(device=DEV).manual_seed(M * 1000 + N)
    a = torch.randn(M, K, generator=g, device=DEV).to(torch.bfloat16)
    b = torch.randn(N, K, generator=g, device=DEV).to(torch.bfloat16)
    c = ulorl.gemm_tn_bf16(a, b)
    ref = a.double() @ b.double().T
    bound = 1e-6 * (a.double().abs() @ b.double().abs().T) + 1e-30
    assert torch.all((c.double() - ref).abs() <= bound), float(((c.double() - ref).abs() / bound).max())
    # strided operands (leading dimension > K)
    big = torch.zeros(M, K + 16, device=DEV, dtype=torch.bfloat16)
    big[:, :K] = a
    c2 = ulorl.gemm_tn_bf16(big[:, :K], b)
    assert torch.equal(c, c2)
    # strided result whose pitch allows 16-byte stores while N itself may end inside a vector:
    # same values, and the columns beyond N stay untouched
    ldc = (N + 3) // 4 * 4 + 4
    wide = torch.full((M, ldc), -7.0, device=DEV, dtype=torch.float32)
    ulorl.gemm_tn_bf16(a, b, out=wide[:, :N])
    assert torch.equal(wide[:, :N], c)
    assert torch.all(wide[:, N:] == -7.0)


@pytest.mark.parametrize("tile,group_m", [(0, 0), (1, 0), (0, 1), (0, 7), (1, 64)])
def test_every_compiled_tile_shape(tile, group_m):
    """Every tile of the plain product (large, small, and the one for a ragged K) and other walks of the tile
    grid give the same answers; the lm_head case is one of few rows and a short hidden size, which takes the
    small tile whatever is asked for (its large tiles: test_walks_of_large_tiles_in_both_calls)."""
    launch = ulorl.Launch(gemm_tile=tile, gemm_group_m=group_m)
    g = torch.Generator(device=DEV).manual_seed(tile)
    for (M, N, K) in ((300, 520, 192), (256, 256, 72), (1300, 700, 128)):     # K = 72 exercises the ragged-K fallback
        a = torch.randn(M, K, generator=g, device=DEV).to(torch.bfloat16)
        b = torch.randn(N, K, generator=g, device=DEV).to(torch.bfloat16)
        c = ulorl.gemm_tn_bf16(a, b, launch=launch)
        ref = a.double() @ b.double().T
        bound = 1e-6 * (a.double().abs() @ b.double().abs().T) + 1e-30
        assert torch.all((c.double() - ref).abs() <= bound)
    w = ui.shrink(ui.config(5), [150, 120], V=1544, hidden=128, seg_len=64, name="lmhead_tile%d" % tile)
    run_lmhead_parity(w, params_for(w, gate_mode=ulorl.GATE_ALWAYS, tau=0.05), chunk=512, launch=launch)


@pytest.mark.parametrize("tile", [0, 1])
@pytest.mark.parametrize("n,V,hidden", [(256, 512, 64), (257, 520, 128), (63, 256, 192), (129, 264, 256), (1, 8, 8), (320, 1096, 72)])
def test_tile_edges_of_every_product(tile, n, V, hidden):
    """One to four K tiles of the small tile (all of these shapes take it, by their size or by request), tiles
    one row or one vector past an edge, and shapes whose weight is padded or whose last columns are taken apart
    (hidden or vocabulary no multiple of 64); the tolerances are those of every lm_head case.  The large
    tile: test_large_tiles_of_every_width and test_large_tiles_of_the_backward."""
    launch = ulorl.Launch(gemm_tile=tile)
    w = ui.shrink(ui.config(5), [n], V=V, hidden=hidden, seg_len=64, name="lmhead_edges")
    for dense in (False, True):
        launch.dense_rows = dense
        run_lmhead_parity(w, params_for(w, gate_mode=ulorl.GATE_NEVER), chunk=320, launch=launch)


@pytest.mark.parametrize("n,V,hidden", [(512, 65536 + 192, 64),     # eighteen chunks, the last shorter than the three parts of the dHidden contraction
                                        (300, 9000, 320),             # three chunks of three parts
                                        (2049, 264, 64),              # live rows counted by three workgroups in one launch
                                        (33000, 64, 64)])             # ... and by the three-launch scan
def test_backward_partitions(n, V, hidden):
    """Where the backward pass is cut: vocabulary chunks, parts of the dHidden contraction, and the two
    ways the live rows are counted (clipped tokens are not live)."""
    w = ui.shrink(ui.config(5), [n - 1, 1], V=V, hidden=hidden, seg_len=64, name="lmhead_parts")
    res, tt = run_lmhead_parity(w, params_for(w, gate_mode=ulorl.GATE_NEVER), chunk=64)
    assert 0 < tt.n_clip_inactive < n


@pytest.mark.parametrize("n,V,hidden", [(1300, 64, 320), (1300, 136, 320), (1408, 264, 384), (1409, 1096, 392), (1537, 200, 512)])
def test_many_rows_and_few_columns(n, V, hidden):
    """More than a thousand rows and few columns, with 20, 128, 129 and 1 rows beyond a multiple of 256, hidden sizes whose last
    tile is half empty too, and contractions of one to four K tiles in the dHidden product.  (Small tiles, too few
    for large ones, which are below.)"""
    w = ui.shrink(ui.config(5), [n - 7, 7], V=V, hidden=hidden, seg_len=64, name="lmhead_halves")
    for dense in (False, True):
        run_lmhead_parity(w, params_for(w, gate_mode=ulorl.GATE_NEVER), chunk=8192, launch=ulorl.Launch(dense_rows=dense))


# Large tiles share the tokens evenly, in units of 32 columns.
LARGE_IN_FORWARD = [(257, 30000, 1024),     # one of 160 and one of 128, whose second half is empty
                    (288, 30000, 1024),     # the same, full
                    (290, 30000, 1024),     # two of 160, the last with empty columns
                    (353, 30000, 1024),     # two of 192
                    (450, 20048, 1024)]     # 256 and 224
LARGE_IN_BOTH = [(257, 22008, 2048), (300, 22008, 2048), (353, 22008, 2048),      # the first ones' widths
                 (513, 20048, 1024),        # 192, 192, 160
                 (545, 20048, 1024)]        # three of 192


@pytest.mark.parametrize("n,V,hidden", LARGE_IN_FORWARD + LARGE_IN_BOTH)
def test_large_tiles_of_every_width(n, V, hidden):
    """The vocabularies leave a rest of 48 or 80 columns, or 248."""
    w = ui.shrink(ui.config(5), [n - 7, 7], V=V, hidden=hidden, seg_len=64, name="lmhead_widths")
    run_lmhead_parity(w, params_for(w, gate_mode=ulorl.GATE_NEVER), chunk=8192)


LARGE_BACKWARD = [(1300, 9536, 320, 8192),     # last hidden tile a quarter full
                  (1409, 9544, 392, 8192),     # hidden and vocabulary no multiple of 64: padded copies
                  (1281, 9480, 448, 1024),     # three chunks, the last columns apart; a last tile of tokens with empty columns
                  (1537, 9472, 512, 8192)]


@pytest.mark.parametrize("n,V,hidden,chunk", LARGE_BACKWARD)
def test_large_tiles_of_the_backward(n, V, hidden, chunk):
    """Few K tiles of the dz product (5 to 8) and 21 to 25 of the dW product."""
    w = ui.shrink(ui.config(5), [n - 7, 7], V=V, hidden=hidden, seg_len=64, name="lmhead_large_bwd")
    for dense in (False, True):
        run_lmhead_parity(w, params_for(w, gate_mode=ulorl.GATE_NEVER), chunk=chunk, launch=ulorl.Launch(dense_rows=dense))


@pytest.mark.parametrize("n_live", [0, 1, 64, 65, 128, 129, 257])
@pytest.mark.parametrize("hidden,V", [(320, 9536), (392, 9480)])
def test_large_tiles_of_the_backward_with_few_live_rows(n_live, hidden, V):
    """The dW product over none, one, two, three and five K tiles of the large tile, in narrow and whole ones."""
    w = ui.shrink(ui.config(5), [1290, 10], V=V, hidden=hidden, seg_len=64, name="lmhead_large_few")
    d, keep = _few_live(w, n_live)
    p = params_for(w, gate_mode=ulorl.GATE_NEVER, eps_low=10.0, eps_high=10.0)
    res, _ = run_lmhead_parity(w, p, chunk=8192, data=d)
    assert int((res.gcoef != 0).sum()) == n_live
    assert bool((res.d_hidden[~keep] == 0).all())


@pytest.mark.parametrize("n,V,hidden", [(1500, 50000, 512), (400, 151936, 256)])
def test_chunks_where_the_accumulators_do_not_fit_beside_all_columns(n, V, hidden):
    """Shapes whose workspace holds dZ of all columns but few of the dHidden accumulators: in chunks (large and
    small tile); d_hidden and d_weight against products of the library's own dlogits."""
    g = torch.Generator(device=DEV).manual_seed(n)
    h, w = torch.randn(n, hidden, generator=g, device=DEV).bfloat16(), (torch.randn(hidden, V, generator=g, device=DEV) * 0.05).bfloat16()
    y = torch.randint(0, V, (n,), generator=g, device=DEV, dtype=torch.int32)
    lse = ulorl.lmhead_token_loss_fwd(h, w, y, None, None).lse
    coef = torch.randn(n, generator=g, device=DEV) / n
    dh, dw = ulorl.lmhead_token_loss_bwd(h, w, y, lse, coef)
    dz = -coef[:, None].double() * torch.exp(h.double() @ w.double() - lse[:, None].double())
    dz[torch.arange(n, device=DEV), y.long()] += coef.double()
    for got, ref in ((dh, dz @ w.double().T), (dw, h.double().T @ dz)):
        assert float((got.double() - ref).norm() / ref.norm()) <= 4e-3          # bf16 roundings of dz and of the result: 2^-9 each


@pytest.mark.parametrize("n", [300, 1300])
def test_backward_in_one_chunk_of_eight_parts(n):
    w = ui.shrink(ui.config(5), [n - 1, 1], V=9000, hidden=320, seg_len=64, name="lmhead_eight_parts")
    run_lmhead_parity(w, params_for(w, gate_mode=ulorl.GATE_NEVER), chunk=8192)


@pytest.mark.parametrize("n,V", [(8191, 264), (8192, 264), (8200, 4096), (8200, 4104)])
def test_backward_of_many_rows_and_few_columns(n, V):
    """Around the line from which a d_W of few tiles (at most 32 of 256 x 256) is cut into small ones."""
    w = ui.shrink(ui.config(5), [n - 1, 1], V=V, hidden=320, seg_len=64, name="lmhead_many_rows")
    run_lmhead_parity(w, params_for(w, gate_mode=ulorl.GATE_NEVER), chunk=8192)


def _few_live(w, n_live):
    """The workload's inputs with an advantage in n_live rows only, and parameters that neither clip nor mask."""
    d = ui.generate(w, DEV)
    keep = torch.zeros(w.N, dtype=torch.bool, device=DEV)
    keep[torch.randperm(w.N, generator=torch.Generator().manual_seed(n_live))[:n_live].to(DEV)] = True
    d["advantages"] = torch.where(keep, torch.full_like(d["advantages"], 0.75), torch.zeros_like(d["advantages"]))
    return d, keep


@pytest.mark.parametrize("n_live", [0, 1, 64, 65, 128, 129, 257])
@pytest.mark.parametrize("hidden,V", [(320, 328), (512, 256), (392, 1096)])
def test_many_rows_with_few_live_ones(n_live, hidden, V):
    """A batch of 1300 rows with few that carry a gradient: the d_W product, both operands transposed, contracts over none, one,
    two, three and five K tiles, in whole and half empty tiles; against the oracle.  (Small tiles, by the number of columns; the
    large ones: test_large_tiles_of_the_backward_with_few_live_rows.)"""
    w = ui.shrink(ui.config(5), [1290, 10], V=V, hidden=hidden, seg_len=64, name="lmhead_large_few")
    d, keep = _few_live(w, n_live)
    p = params_for(w, gate_mode=ulorl.GATE_NEVER, eps_low=10.0, eps_high=10.0)
    res, _ = run_lmhead_parity(w, p, chunk=8192, data=d)
    assert int((res.gcoef != 0).sum()) == n_live
    assert bool((res.d_hidden[~keep] == 0).all())
    if n_live == 0:
        assert bool((res.d_weight == 0).all())


@pytest.mark.parametrize("group_m", [1, 7, 64])
def test_walks_of_many_rows_and_few_columns(group_m):
    """1320 rows and 1544 columns in several chunks.  (Small tiles; the large ones in the next test.)"""
    w = ui.shrink(ui.config(5), [1200, 120], V=1544, hidden=320, seg_len=64, name="lmhead_large_walk")
    run_lmhead_parity(w, params_for(w, gate_mode=ulorl.GATE_ALWAYS, tau=0.05), chunk=512, launch=ulorl.Launch(gemm_group_m=group_m))


@pytest.mark.parametrize("group_m", [1, 7, 64])
def test_walks_of_large_tiles_in_both_calls(group_m):
    w = ui.shrink(ui.config(5), [500, 45], V=20048, hidden=1024, seg_len=64, name="lmhead_large_walks")
    run_lmhead_parity(w, params_for(w, gate_mode=ulorl.GATE_NEVER), chunk=8192, launch=ulorl.Launch(gemm_group_m=group_m))


def test_lengths_that_a_kernel_cannot_read_are_refused():
    """As the logits path refuses them; a stats-only pass reads none."""
    w = ui.shrink(ui.config(5), [20, 13], V=520, hidden=64, seg_len=16, name="lmhead_lengths")
    d = ui.generate(w, DEV)
    rest = (d["advantages"], d["old_logp"], params_for(w, gate_mode=ulorl.GATE_NEVER))
    for cu in (d["cu_seqlens"].cpu(), d["cu_seqlens"].long(), d["cu_seqlens"].repeat_interleave(2)[::2]):
        for call in (ulorl.lmhead_token_loss_fwd, ulorl.autograd.lmhead_token_loss):
            with pytest.raises(ValueError, match="cu_seqlens"):
                call(d["hidden"], d["weight"], d["token_ids"], cu, *rest)
    with pytest.raises(ulorl.UlorlError):
        ulorl.lmhead_token_loss_fwd(d["hidden"], d["weight"], d["token_ids"], None, *rest)
    res = ulorl.lmhead_token_loss_fwd(d["hidden"], d["weight"], d["token_ids"], d["cu_seqlens"].cpu(), None)
    ref = ulorl.lmhead_token_loss_fwd(d["hidden"], d["weight"], d["token_ids"], None, None)
    assert torch.equal(res.lse, ref.lse)


def test_lmhead_small_ragged_chunks():
    w = ui.shrink(ui.config(5), [120, 83], V=2056, hidden=136, seg_len=32, name="lmhead_small")
    d = ui.generate(w, DEV)
    for mode in (ulorl.GATE_ALWAYS, ulorl.GATE_NEVER):
        run_lmhead_parity(w, params_for(w, gate_mode=mode, tau=0.05), chunk=512, data=d)
    run_lmhead_parity(w, params_for(w, gate_mode=ulorl.GATE_PER_RESPONSE, sigma=100.0, tau=0.05,
                                    is_mode=ulorl.IS_POIS), chunk=8192, data=d, grad_out=-1.5)


def test_lmhead_config5_reduced_rows():
    # the full hidden size and vocabulary of configuration 5, 2 x 512 rows
    w = ui.shrink(ui.config(5), [512, 512], seg_len=256, name="cfg5_reduced")
    res, tt = run_lmhead_parity(w, params_for(w, gate_mode=ulorl.GATE_ALWAYS), chunk=8192, say=say)
    assert tt.n_clip_inactive > 0


def test_lmhead_mpt_mask_fires():
    """A labelled extra case: full hidden size and vocabulary of configuration 5, 2 x 384 rows, a
    third of the hidden rows aligned with one column of W (scaled so that the sampled token's
    probability spreads from ~0.93 to ~1) -- with hidden ~ N(0, 1) . W ~ N(0, 0.02) alone no token
    comes near tau = 0.99 and the mask of Eq. MPTS / I_msk (Sec. 3.2.2) would never be set.
    Mask bit-exact outside |p - tau| < 1e-6, masked tokens carry a zero coefficient and contribute
    exactly nothing to d_hidden (checked in run_lmhead_parity), d_W against the oracle."""
    from dataclasses import replace
    w = replace(ui.shrink(ui.config(5), [384, 384], seg_len=192), align_frac=0.35, name="cfg5_mpt_fires")
    p = params_for(w, gate_mode=ulorl.GATE_ALWAYS)
    res, tt = run_lmhead_parity(w, p, chunk=8192, say=say)
    mask = res.mpt_mask.cpu().numpy().astype(bool)
    assert tt.n_masked >= 20 and int(res.counters[0]) > 0, tt.n_masked
    # some aligned tokens stay below the threshold, and the negative-advantage response is never masked
    prob = np.exp(res.logp.cpu().numpy())
    assert ((prob > 0.9) & (prob < 0.99) & ~mask).sum() >= 5
    assert not mask[384:].any() and mask[:384].any()
    assert bool((res.gcoef[torch.as_tensor(mask, device=DEV)] == 0).all())
    assert bool((res.d_hidden[torch.as_tensor(mask, device=DEV)] == 0).all())
    # the same batch under the per-response gate with sigma between the two responses' mean entropies:
    # only one response's MPTs are masked
    hb = np.sort(tt.resp_entropy)
    if hb[1] - hb[0] > 2e-3:
        sigma = float(0.5 * (hb[0] + hb[1]))
        d = ui.generate(w, DEV)
        r2, tt2 = run_lmhead_parity(w, params_for(w, gate_mode=ulorl.GATE_PER_RESPONSE, sigma=sigma), chunk=8192, data=d)
        assert int(tt2.resp_gate.sum()) == 1


@pytest.mark.parametrize("lengths,V,hidden,chunk", [([300, 212], 4096 + 1544, 256, 1024), ([64], 8192 + 8, 64, 64),
                                                    ([1000, 24], 1544, 128, 2048),
                                                    # several chunks: last columns apart, W padded for V < 2 n, padded along hidden
                                                    ([693, 7], 8392, 64, 64), ([1500, 1], 3000, 64, 64), ([893, 7], 6000, 72, 64),
                                                    ([1299, 1], 5000, 320, 64), ([1400], 2760, 328, 64)])
def test_workspace_is_never_overrun(lengths, V, hidden, chunk):
    """Guard bytes behind the workspace stay untouched by the forward and the backward call (shapes
    with few token tiles and many vocabulary tiles ask for the most vocabulary slices)."""
    w = ui.shrink(ui.config(5), lengths, V=V, hidden=hidden, seg_len=64, name="lmhead_guard")
    d = ui.generate(w, DEV)
    p = ulorl.Params(gate_mode=ulorl.GATE_ALWAYS, seg_len=w.seg_len)
    need = ulorl.lmhead_workspace_bytes(w.N, w.hidden, w.V, w.R, chunk)
    guard = 1 << 20
    buf = torch.full((need + guard,), 0xA5, dtype=torch.uint8, device=DEV)
    ws = buf[:need]
    out = ulorl.lmhead_token_loss_fwd(d["hidden"], d["weight"], d["token_ids"], d["cu_seqlens"], d["advantages"],
                                      d["old_logp"], p, vocab_chunk=chunk, workspace=ws)
    ulorl.lmhead_token_loss_bwd(d["hidden"], d["weight"], d["token_ids"], out.lse, out.gcoef, 1.0, vocab_chunk=chunk,
                                workspace=ws)
    torch.cuda.synchronize()
    assert bool((buf[need:] == 0xA5).all())


def test_lmhead_stats_only_pass():
    """advantages = None: only lse, logp and entropy are produced (how a caller records the
    behaviour policy's log-probs), identical to those of the full forward."""
    w = ui.shrink(ui.config(5), [150, 120], V=1544, hidden=128, seg_len=64, name="lmhead_stats_only")
    d = ui.generate(w, DEV)
    p = ulorl.Params(gate_mode=ulorl.GATE_ALWAYS, seg_len=w.seg_len)
    full = ulorl.lmhead_token_loss_fwd(d["hidden"], d["weight"], d["token_ids"], d["cu_seqlens"], d["advantages"],
                                       d["old_logp"], p, vocab_chunk=512)
    only = ulorl.lmhead_token_loss_fwd(d["hidden"], d["weight"], d["token_ids"], None, None, vocab_chunk=512)
    assert only.loss is None and only.gcoef is None
    for name in ("lse", "logp", "entropy"):
        assert torch.equal(getattr(only, name), getattr(full, name)), name


def _lmhead_bwd_pair(d, w, p, chunk):
    """(forward result, (d_hidden, d_W) over the live rows, the same with every row in the products)"""
    fwd = ulorl.lmhead_token_loss_fwd(d["hidden"], d["weight"], d["token_ids"], d["cu_seqlens"], d["advantages"],
                                      d["old_logp"], p, vocab_chunk=chunk)
    live = ulorl.lmhead_token_loss_bwd(d["hidden"], d["weight"], d["token_ids"], fwd.lse, fwd.gcoef, 1.0, vocab_chunk=chunk)
    dense = ulorl.lmhead_token_loss_bwd(d["hidden"], d["weight"], d["token_ids"], fwd.lse, fwd.gcoef, 1.0, vocab_chunk=chunk,
                                        launch=ulorl.Launch(dense_rows=True))
    torch.cuda.synchronize()
    return fwd, live, dense


def _assert_dw_same_up_to_rounding(a, b):
    a, b = a.float(), b.float()
    # different grouping of the same fp32 terms, then one rounding to bf16: at most an ulp of the larger entries
    assert float((a - b).abs().max()) <= 2.0 ** -7 * float(torch.maximum(a.abs(), b.abs()).max())
    assert float((a - b).abs().mean()) <= 2.0 ** -9 * float(a.abs().mean()) + 1e-30


def test_backward_runs_over_the_live_rows_only():
    """The backward pass gathers the rows with a non-zero coefficient (Sec. 3.2.2: a masked token
    contributes no gradient) and runs its products over those; ULORL_LAUNCH_DENSE_ROWS runs them
    over every row.  Both against the oracle, and against each other: d_hidden bit for bit (a row's
    sums do not depend on which other rows are present), d_W up to the rounding of regrouped sums."""
    from dataclasses import replace
    w = replace(ui.shrink(ui.config(5), [300, 212], V=4096 + 8, hidden=256, seg_len=64), align_frac=0.5,
                name="lmhead_live_rows")
    d = ui.generate(w, DEV)
    p = params_for(w, gate_mode=ulorl.GATE_ALWAYS)
    res, tt = run_lmhead_parity(w, p, chunk=1024, data=d)
    res2, _ = run_lmhead_parity(w, p, chunk=1024, data=d, launch=ulorl.Launch(dense_rows=True))
    dead = int((res.gcoef == 0).sum())
    say("live rows: %d of %d" % (w.N - dead, w.N))
    assert 20 <= dead < w.N - 20
    assert torch.equal(res.d_hidden, res2.d_hidden)
    _assert_dw_same_up_to_rounding(res.d_weight, res2.d_weight)


@pytest.mark.parametrize("n_live", [0, 1, 65])
def test_backward_with_few_or_no_live_rows(n_live):
    """Degenerate live counts: no row at all (every advantage zero: both gradients exactly zero), one
    row, one row more than a 64-column block of the contraction."""
    w = ui.shrink(ui.config(5), [200, 150], V=2056, hidden=128, seg_len=64, name="lmhead_few_live")
    d = ui.generate(w, DEV)
    keep = torch.zeros(w.N, dtype=torch.bool, device=DEV)
    if n_live:
        keep[torch.randperm(w.N, generator=torch.Generator().manual_seed(5))[:n_live].to(DEV)] = True
    d["advantages"] = torch.where(keep, torch.full_like(d["advantages"], 0.75), torch.zeros_like(d["advantages"]))
    p = ulorl.Params(gate_mode=ulorl.GATE_NEVER, seg_len=w.seg_len, eps_low=10.0, eps_high=10.0)
    fwd, (dH, dW), (dH2, dW2) = _lmhead_bwd_pair(d, w, p, chunk=512)
    assert int((fwd.gcoef != 0).sum()) == n_live
    assert torch.equal(dH, dH2)
    assert bool((dH[~keep] == 0).all())
    if n_live == 0:
        assert bool((dH == 0).all()) and bool((dW == 0).all()) and bool((dW2 == 0).all())
    else:
        assert bool((dH[keep].float().abs().sum(dim=1) > 0).all())
        _assert_dw_same_up_to_rounding(dW, dW2)


@pytest.mark.parametrize("n,Hd", [(200, 320), (300, 320), (300, 2048)])        # the small tile twice, and the large one
def test_forward_statistics_of_large_logits(n, Hd):
    """Logits far beyond the range a model produces still have a log-sum-exp and an entropy: +-2^20 with
    the maxima of one slice's tiles on both sides of it, 1.25 2^28 in steps of 32, 2^29 times small numbers
    of either sign (maxima on both sides of the point where the statistics change their exponents; the
    softmax is shared by the ties at the top) and 2^32 (all equal in fp32).  Two non-zero hidden dimensions keep every sum exact, so the reference is that of the
    fp32 logits; what is left is the fp32 resolution of lse and of a difference of logits."""
    V = 65536 + 8                                 # up to three tiles of 256 columns to a slice
    g = torch.Generator(device=DEV).manual_seed(n)
    w = torch.zeros(Hd, V, device=DEV)
    w[0] = 1024.0
    w[7] = torch.randint(-127, 128, (V,), generator=g, device=DEV) / 8.0
    first = (torch.arange(V, device=DEV) // 256) % 3 == 0
    w[7] -= torch.where(first, 16.0, 0.0)         # multiples of 1/8 up to 32: 8 bits
    h = torch.zeros(n, Hd, device=DEV)
    kind = torch.arange(n, device=DEV) % 6
    h[:, 0] = torch.tensor([1024.0, -1024.0, 0.0, 2.0 ** 22, 0.0, 1.25 * 2.0 ** 18], device=DEV)[kind]
    h[:, 7] = torch.tensor([1.0, 1.0, 2.0 ** 29, 1.0, -2.0 ** 29, 256.0], device=DEV)[kind]
    h, w = h.bfloat16(), w.bfloat16()
    y = torch.randint(0, V, (n,), generator=g, device=DEV, dtype=torch.int32)
    res = ulorl.lmhead_token_loss_fwd(h, w, y, None, None)
    z = (h[:, :8].double() @ w[:8].double()).float().double()
    lse = torch.logsumexp(z, 1)
    logp = z - lse[:, None]
    ent = -(logp.exp() * torch.where(logp > -700, logp, 0.0)).sum(1)
    at = logp.gather(1, y[:, None].long())[:, 0]
    assert torch.all((res.lse.double() - lse).abs() <= 2.0 ** -23 * lse.abs() + 2e-6)
    assert torch.all((res.entropy.double() - ent).abs() <= 2e-5 * ent + 2e-5), float((res.entropy.double() - ent).abs().max())
    assert torch.all((res.logp.double() - at).abs() <= 1e-6 * at.abs() + 2e-6 + 2e-6 * ent)


@pytest.mark.parametrize("V", [1 << 25, (1 << 25) + 8])        # the widest weight of the large tile, and the small tile beyond
def test_forward_of_a_very_wide_vocabulary(V):
    """Offsets into the weight of more than 2^31 bytes.  All columns are zero but for blocks at the start, in the
    middle and at the end.  The 1024 terms of a logit add up to at most about 15; their independent roundings in
    fp32 to 32 x 15 x 2^-24 = 3e-5 at the very most, a typical row to a fifth of it."""
    n, Hd = 260, 1024
    g = torch.Generator(device=DEV).manual_seed(7)
    w = torch.zeros(Hd, V, dtype=torch.bfloat16, device=DEV)
    cols = torch.cat([torch.arange(0, 300), torch.arange(V // 2 - 200, V // 2 + 100), torch.arange(V - 300, V)]).to(DEV)
    w[:, cols] = (torch.randn(Hd, 900, generator=g, device=DEV) * 0.1).bfloat16()
    h = torch.randn(n, Hd, generator=g, device=DEV).bfloat16()
    y = cols[torch.randint(0, 900, (n,), generator=g, device=DEV)].int()
    res = ulorl.lmhead_token_loss_fwd(h, w, y, None, None)
    z = h.double() @ w[:, cols].double()
    lse = torch.logsumexp(torch.cat([z, torch.full((n, 1), float(np.log(V - 900)), dtype=torch.float64, device=DEV)], 1), 1)
    at = (h.double() * w[:, y.long()].double().T).sum(1)
    assert float((res.lse - lse).abs().max()) <= 2e-5
    assert float((res.logp - (at - lse)).abs().max()) <= 4e-5


# The vocabulary in several chunks (vocab_chunk = 64 and more rows than hidden columns, so that the workspace
# has no room for wide ones), the last one narrower and no multiple of 64; W with its last columns apart
# (hidden a multiple of 64), padded for having few columns (V < 2 n) and padded along hidden.
LARGE_IN_CHUNKS = [(1300, 9480, 320), (3000, 5000, 832), (1404, 9544, 328)]       # the same three with the large tile


@pytest.mark.parametrize("n,V,hidden", [(700, 8392, 64), (1501, 3000, 64), (900, 6000, 72), (90, 56, 64),
                                        (1300, 5000, 320), (1400, 2760, 320), (1300, 5000, 328)] + LARGE_IN_CHUNKS)
@pytest.mark.parametrize("dense", [False, True])
def test_backward_over_several_ragged_chunks(n, V, hidden, dense):
    w = ui.shrink(ui.config(5), [n - 7, 7], V=V, hidden=hidden, seg_len=64, name="lmhead_chunks")
    run_lmhead_parity(w, params_for(w, gate_mode=ulorl.GATE_NEVER), chunk=64, launch=ulorl.Launch(dense_rows=dense))


@pytest.mark.parametrize("n,most,V,hidden", [(300, 400, 2056, 128), (1300, 1313, 5000, 320), (1300, 4288, 5000, 72)])
def test_workspace_of_a_larger_batch(n, most, V, hidden):
    """A workspace sized for the longest batch takes a shorter one, with the bits of its own workspace."""
    w = ui.shrink(ui.config(5), [n - 7, 7], V=V, hidden=hidden, seg_len=64, name="lmhead_reuse")
    d = ui.generate(w, DEV)
    p = ulorl.Params(gate_mode=ulorl.GATE_ALWAYS, seg_len=w.seg_len)
    got = []
    for rows in (n, most):
        ws = torch.full((ulorl.lmhead_workspace_bytes(rows, hidden, V, 2, 512),), 0xA5, dtype=torch.uint8, device=DEV)
        f = ulorl.lmhead_token_loss_fwd(d["hidden"], d["weight"], d["token_ids"], d["cu_seqlens"], d["advantages"], d["old_logp"], p,
                                        vocab_chunk=512, workspace=ws)
        got.append((f.loss, f.lse, f.entropy) + ulorl.lmhead_token_loss_bwd(d["hidden"], d["weight"], d["token_ids"], f.lse, f.gcoef, 1.0,
                                                                            vocab_chunk=512, workspace=ws))
    for a, b in zip(*got):
        assert torch.equal(a, b)
