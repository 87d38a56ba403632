"""GPU parity of the small neighbours of the token loss: segment-rollout pool update,
advantage preparation and per-segment diagnostics."""
import numpy as np
import pytest
import torch

import oracle
import paper_2507_19766_amd as ulorl
import ulorl_inputs as ui
from parity import params_for

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("G,unbiased", [(8, False), (4, True), (1, False)])
def test_advantage_prep_matches_the_oracle(G, unbiased):
    rs = np.random.RandomState(G)
    R = 8 * 40
    lengths = rs.randint(1, 300, size=R)
    lengths[5] = 0                                          # an empty response is legal
    cu = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    rewards = (rs.rand(R) < 0.45).astype(np.float32)
    rewards[:G] = 1.0                                       # one all-correct group
    rewards[G:2 * G] = 0.0                                  # one all-wrong group
    trunc = (rs.rand(R) < 0.1).astype(np.uint8)
    resp, keep, tok, kept = ulorl.advantage_prep(torch.tensor(rewards, device=DEV), torch.tensor(cu, device=DEV), G,
                                                 truncated=torch.tensor(trunc, device=DEV), eps=1e-6, unbiased=unbiased)
    o_resp, o_keep, o_tok, o_kept = oracle.advantages(rewards, cu, G, truncated=trunc, eps=float(np.float32(1e-6)),
                                                      unbiased=unbiased)
    np.testing.assert_array_equal(keep.cpu().numpy(), o_keep)
    assert int(kept.item()) == o_kept
    np.testing.assert_allclose(resp.cpu().numpy(), o_resp, rtol=1e-6, atol=0)
    np.testing.assert_allclose(tok.cpu().numpy(), o_tok, rtol=1e-6, atol=0)
    assert np.all(resp.cpu().numpy()[o_resp == 0.0] == 0.0)
    if G > 1:
        assert 0 < o_keep.sum() < len(o_keep)


@pytest.mark.parametrize("G", [31, 32, 33, 96])
def test_advantage_prep_in_one_or_two_launches(G):
    """Around the group size up to which the tokens' advantages are formed in the same launch as the
    responses'; lengths that leave the last workgroup of tokens partly filled."""
    rs = np.random.RandomState(G)
    R = 3 * G
    cu = np.concatenate([[0], np.cumsum(rs.randint(0, 40, size=R))]).astype(np.int32)
    cu[-1] += 1                                              # at least one token
    rewards = (rs.rand(R) < 0.4).astype(np.float32)
    rewards[:G] = 1.0                                        # a dropped group
    trunc = (rs.rand(R) < 0.1).astype(np.uint8)
    trunc[:G] = 0
    resp, keep, tok, kept = ulorl.advantage_prep(torch.from_numpy(rewards).to(DEV), torch.from_numpy(cu).to(DEV), G,
                                                 truncated=torch.from_numpy(trunc).to(DEV))
    ref = oracle.advantages(rewards, cu, G, truncated=trunc)
    np.testing.assert_allclose(resp.cpu().numpy(), ref[0], rtol=1e-6, atol=1e-7)
    assert torch.equal(tok.cpu(), resp.cpu()[torch.from_numpy(np.repeat(np.arange(R), np.diff(cu)))])
    assert keep.cpu().tolist() == [0, 1, 1] and int(kept.item()) == ref[3]


@pytest.mark.parametrize("N", [(1 << 19) - 1, 1 << 19, (1 << 19) + 1, 3 << 19])
def test_advantage_prep_around_the_token_count_of_one_launch(N):
    """Up to 2^19 tokens their advantages are formed in the launch of the responses', beyond by a second one."""
    G, R = 8, 64
    rs = np.random.RandomState(N % 1000)
    cu = np.sort(np.concatenate([[0, N], rs.randint(0, N, size=R - 1)])).astype(np.int32)
    rewards = (rs.rand(R) < 0.4).astype(np.float32)
    rewards[:G] = 1.0
    resp, keep, tok, kept = ulorl.advantage_prep(torch.from_numpy(rewards).to(DEV), torch.from_numpy(cu).to(DEV), G)
    ref = oracle.advantages(rewards, cu, G)
    np.testing.assert_allclose(resp.cpu().numpy(), ref[0], rtol=1e-6, atol=1e-7)
    assert torch.equal(tok.cpu(), resp.cpu()[torch.from_numpy(np.repeat(np.arange(R), np.diff(cu)))])
    assert int(kept.item()) == ref[3]


def test_prepared_advantages_feed_the_token_loss():
    """rewards -> advantages -> loss, all on the device, against the oracle chain."""
    w = ui.shrink(ui.config(2), [60, 45, 80, 30, 50, 50, 20, 70], V=4096, seg_len=32, name="chain")
    d = ui.generate(w, DEV)
    rewards = np.array([1, 0, 0, 1, 1, 1, 1, 1], np.float32)         # second group is all-correct: dropped
    cu = w.cu_seqlens
    resp, keep, tok, kept = ulorl.advantage_prep(torch.tensor(rewards, device=DEV), d["cu_seqlens"], 4, eps=0.0)
    p = params_for(w, gate_mode=ulorl.GATE_ALWAYS, denominator=float(kept.item()))
    res = ulorl.token_loss_fwd(d["logits"], d["token_ids"], d["cu_seqlens"], tok, d["old_logp"], p)
    _, _, o_tok, o_kept = oracle.advantages(rewards, cu, 4, eps=0.0)
    assert o_kept == 60 + 45 + 80 + 30
    lse, logp, H = oracle.row_stats(ui.to_numpy_logits(d["logits"]), d["token_ids"].cpu().numpy())
    tt = oracle.token_terms(logp, H, cu, o_tok.astype(np.float32), d["old_logp"].cpu().numpy(), seg_len=32,
                            gate_mode=oracle.GATE_ALWAYS, denominator=float(o_kept), eps_low=float(np.float32(0.2)),
                            eps_high=float(np.float32(0.2)), tau=float(np.float32(0.99)))
    np.testing.assert_allclose(res.loss.item(), tt.loss, rtol=2e-5, atol=1e-7)
    assert torch.all(res.gcoef[215:] == 0)                           # dropped group: no gradient


def test_segment_diagnostics_match_the_oracle():
    w = ui.shrink(ui.config(4), [3000], V=4096, seg_len=400, name="diag")          # 8 segments, growing staleness
    d = ui.generate(w, DEV)
    p = params_for(w, gate_mode=ulorl.GATE_ALWAYS, tau=0.5)
    res = ulorl.token_loss_fwd(d["logits"], d["token_ids"], d["cu_seqlens"], d["advantages"], d["old_logp"], p)
    K = 8
    g = ulorl.segment_diagnostics(res, d["advantages"], d["old_logp"], K)
    g2 = ulorl.segment_diagnostics(res, d["advantages"], d["old_logp"], K)
    for k in g:
        assert torch.equal(g[k], g2[k])                                             # reproducible
    # the oracle side is computed from the oracle's own per-token quantities (never from GPU outputs)
    lse, logp, H = oracle.row_stats(ui.to_numpy_logits(d["logits"]), d["token_ids"].cpu().numpy())
    adv = d["advantages"].cpu().numpy()
    old = d["old_logp"].cpu().numpy()
    f32 = lambda x: float(np.float32(x))
    tt = oracle.token_terms(logp, H, w.cu_seqlens, adv, old, seg_len=400, gate_mode=oracle.GATE_ALWAYS,
                            eps_low=f32(0.2), eps_high=f32(0.2), tau=f32(0.5))
    o = oracle.segment_diagnostics(tt.seg, tt.ratio, logp, old, H, tt.mask, adv, K, eps_low=f32(0.2), eps_high=f32(0.2))
    near_edge = int(((np.abs(tt.ratio - 0.8) < 1e-5) | (np.abs(tt.ratio - 1.2) < 1e-5)).sum())
    near_tau = int((np.abs(np.exp(logp) - 0.5) < 1e-6).sum())
    np.testing.assert_array_equal(g["count"].cpu().numpy(), o["count"])
    assert np.abs(g["clipped"].cpu().numpy() - o["clipped"]).sum() <= near_edge
    assert np.abs(g["masked"].cpu().numpy() - o["masked"]).sum() <= near_tau
    assert o["masked"].sum() > 0 and o["clipped"].sum() > 0
    for name in ("ratio_sum", "ent_sum"):
        np.testing.assert_allclose(g[name].cpu().numpy(), o[name], rtol=2e-5)
    np.testing.assert_allclose(g["kl_sum"].cpu().numpy(), o["kl_sum"], rtol=2e-5, atol=2e-6 * 400)
    np.testing.assert_allclose(g["ratio_max"].cpu().numpy(), o["ratio_max"], rtol=2e-5)
    assert int(g["out_of_range"].item()) == 0 and o["count"].sum() == 3000
    # later segments are staler: their mean |log ratio| grows (0.02 * segment index of noise)
    mean_ratio = o["ratio_sum"] / o["count"]
    assert abs(mean_ratio[0] - 1.0) < 1e-5 and o["clipped"][7] >= o["clipped"][1]
    # ids outside [0, K) are counted and ignored; POIS has no old log-probs
    g3 = ulorl.segment_diagnostics(res, d["advantages"], None, 4)
    assert int(g3["out_of_range"].item()) == 3000 - 1600 and float(g3["kl_sum"].abs().sum()) == 0.0
    np.testing.assert_array_equal(g3["count"].cpu().numpy(), o["count"][:4])


def test_segment_diagnostics_take_what_a_kernel_can_read():
    """Each tensor where the ids are, of its type and as long; a mask of either one-byte type and a column are as good."""
    n, K = 70, 3
    f = torch.rand(n, device=DEV)
    t = dict(ratio=f + 0.5, logp=-f, old=-f * 1.1, entropy=f, mask=(f > 0.5).to(torch.uint8), adv=f - 0.5,
             ids=torch.arange(n, device=DEV, dtype=torch.int32) % K)

    def call(**change):
        x = dict(t, **change)
        res = ulorl.FwdResult(None, x["logp"], x["entropy"], x["logp"], ratio=x["ratio"], segment_out=x["ids"], mpt_mask=x["mask"])
        return ulorl.segment_diagnostics(res, x["adv"], x["old"], K)
    ref = call()
    for same in (dict(mask=t["mask"].bool()), dict(adv=t["adv"][:, None]), dict(logp=torch.cat([t["logp"], f]))):
        got = call(**same)
        assert all(torch.equal(got[k], ref[k]) for k in ref)
    for name in ("ratio", "logp", "old", "entropy", "mask", "adv"):
        for bad in (t[name].cpu(), t[name].double(), t[name][:-1], t[name].repeat(2)[::2]):
            with pytest.raises(ValueError):
                call(**{name: bad})
    with pytest.raises(ValueError):
        call(ids=t["ids"].long())
    with pytest.raises(ulorl.UlorlError):
        call(ratio=None)


@pytest.mark.parametrize("case", ["logits_two_call", "logits_one_call", "lmhead", "explicit_ids_pois", "many_segments"])
def test_segment_diagnostics_as_a_by_product_of_the_forward_calls(case):
    """The forward calls hand out the per-segment diagnostics in the same pass as the token terms;
    the numbers carry the bits of the standalone call on the stored outputs (which the test above
    holds against the oracle), and the other outputs do not change."""
    K = 1024 if case == "many_segments" else 6
    pois = case in ("explicit_ids_pois", "many_segments")
    if case == "lmhead":
        w = ui.shrink(ui.config(5), [700, 1500, 30], V=1544, hidden=128, seg_len=300, name="diag_lmhead")
        d = ui.generate(w, DEV)
        p = params_for(w, gate_mode=ulorl.GATE_ALWAYS, tau=0.001)
        plain = ulorl.lmhead_token_loss_fwd(d["hidden"], d["weight"], d["token_ids"], d["cu_seqlens"], d["advantages"],
                                            d["old_logp"], p, vocab_chunk=512)
        res = ulorl.lmhead_token_loss_fwd(d["hidden"], d["weight"], d["token_ids"], d["cu_seqlens"], d["advantages"],
                                          d["old_logp"], p, vocab_chunk=512, segments=K)
        old, ids = d["old_logp"], None
    else:
        w = ui.shrink(ui.config(4), [1100, 2050, 1, 37], V=4096, seg_len=400, name="diag_fused")   # ids 0..5, ragged blocks
        d = ui.generate(w, DEV)
        p = params_for(w, gate_mode=ulorl.GATE_ALWAYS, tau=0.5, is_mode=ulorl.IS_POIS if pois else ulorl.IS_SAIS,
                       seg_len=0 if pois else 400)
        old = None if pois else d["old_logp"]
        # arbitrary ids, some outside [0, K): many distinct ids inside one wave
        ids = ((torch.arange(w.N, device=DEV) * 7) % 9 - 1).to(torch.int32) if pois else None
        if case == "many_segments":     # the largest table the kernels take, every id present, a few outside
            ids = ((torch.arange(w.N, device=DEV) * 5) % 1030 - 3).to(torch.int32)
        args = (d["logits"], d["token_ids"], d["cu_seqlens"], d["advantages"], old, p)
        if case == "logits_one_call":
            plain, _ = ulorl.token_loss_fwd_bwd(*args)
            res, _ = ulorl.token_loss_fwd_bwd(*args, segments=K)
        else:
            plain = ulorl.token_loss_fwd(*args, segment_ids=ids)
            res = ulorl.token_loss_fwd(*args, segment_ids=ids, segments=K)
    for name in ("loss", "logp", "entropy", "lse", "gcoef", "mpt_mask", "ratio", "segment_out", "counters"):
        assert torch.equal(getattr(res, name), getattr(plain, name)), name
    alone = ulorl.segment_diagnostics(res, d["advantages"], old, K)
    fused = res.segment_stats
    for name in ("count", "ratio_sum", "ratio_max", "clipped", "kl_sum", "ent_sum", "masked", "out_of_range"):
        a, b = fused[name], alone[name]
        assert torch.equal(a.view(torch.int64) if a.dtype == torch.float64 else a,
                           b.view(torch.int64) if b.dtype == torch.float64 else b), name
    n_in = int(((res.segment_out >= 0) & (res.segment_out < K)).sum())
    assert int(fused["count"].sum()) == n_in and int(fused["out_of_range"]) == w.N - n_in
    if pois:
        assert int(fused["out_of_range"]) > 0 and float(fused["kl_sum"].abs().sum()) == 0.0
        assert bool((fused["ratio_sum"] == fused["count"].double()).all())       # POIS: every ratio is 1


@pytest.mark.parametrize("B", [1, 63, 1024, 1025, 5000])
def test_segment_pool_step_matches_the_oracle(B):
    rng = np.random.default_rng(B)
    seg, mx = 64, 640
    prev = (rng.integers(0, mx // seg, B) * seg).astype(np.int32)
    room = np.minimum(seg, mx - prev)
    kind = rng.integers(0, 3, B)
    new = np.where(kind == 1, rng.integers(1, room + 1), room).astype(np.int32)
    eos = (kind >= 1).astype(np.uint8)
    # a few inconsistent samples: short without a reason, too long, negative, end flag without a token
    for j, (p, n, e) in enumerate([(0, 5, 0), (0, seg + 1, 0), (-3, 4, 1), (64, 0, 1), (mx, 1, 0)]):
        if j * 7 < B:
            prev[j * 7], new[j * 7], eos[j * 7] = p, n, e
    ref = oracle.pool_step(prev, new, eos, seg, mx)
    out = ulorl.segment_pool_step(torch.from_numpy(prev).to(DEV), torch.from_numpy(new).to(DEV),
                                  torch.from_numpy(eos).to(DEV), seg, mx)
    got = {k: v.cpu().numpy() for k, v in out.items()}
    nu, ne = int(ref["counts"][0]), int(ref["counts"][1])
    assert got["counts"].tolist() == ref["counts"].tolist()
    for k in ("state", "total_len", "segments"):
        assert np.array_equal(got[k], ref[k]), k
    assert np.array_equal(got["unfinished_idx"][:nu], ref["unfinished_idx"])
    assert np.array_equal(got["experience_idx"][:ne], ref["experience_idx"])
    assert np.array_equal(got["exp_cu_seqlens"][:ne + 1].astype(np.int64), ref["exp_cu_seqlens"])
    assert np.array_equal(got["exp_truncated"][:ne], ref["exp_truncated"])


def test_segment_pool_step_takes_lengths_that_int_takes():
    prev, new = (torch.tensor(x, device=DEV, dtype=torch.int32) for x in ([0, 16, 48], [16, 5, 16]))
    eos = torch.tensor([0, 1, 0], device=DEV, dtype=torch.uint8)
    a, b = ulorl.segment_pool_step(prev, new, eos, 16, 64), ulorl.segment_pool_step(prev, new, eos, 16.0, np.float32(64))
    for name in ("state", "total_len", "segments", "counts"):
        assert torch.equal(a[name], b[name])


def test_rollout_model_takes_the_same_path_on_the_gpu():
    """Forty steps of the segment-rollout loop driven by the GPU pool update and by the oracle:
    identical pools at every step."""
    import rollout_sim as rm

    L = rm.synthetic_lengths(3000, 4096, 5)
    a = rm.simulate(rm.gpu_pool_step, L, batch=96, segments=4, max_len=4096, steps=40)
    b = rm.simulate(oracle.pool_step, L, batch=96, segments=4, max_len=4096, steps=40)
    assert a["records"] == b["records"]
    assert a["done"] == b["done"]


def test_pool_step_feeds_advantages_and_token_loss():
    """The experience pool's cu_seqlens and truncation flags go straight into the next two calls."""
    seg, mx = 32, 128
    prev = torch.tensor([0, 32, 96, 0, 64, 96, 0, 32], dtype=torch.int32, device=DEV)
    new = torch.tensor([20, 32, 32, 32, 9, 32, 32, 5], dtype=torch.int32, device=DEV)
    eos = torch.tensor([1, 0, 0, 0, 1, 1, 1, 1], dtype=torch.uint8, device=DEV)
    out = ulorl.segment_pool_step(prev, new, eos, seg, mx)
    cnt = out["counts"].cpu().tolist()
    ne, ntok = cnt[1], cnt[3]
    assert cnt[:3] == [2, 6, 1] and ntok == 20 + 128 + 73 + 128 + 32 + 37
    cu = out["exp_cu_seqlens"][:ne + 1].contiguous()
    trunc = out["exp_truncated"][:ne].contiguous()
    rewards = torch.tensor([1, 1, 0, 1, 0, 1], dtype=torch.float32, device=DEV)
    resp, keep, tok_adv, kept = ulorl.advantage_prep(rewards, cu, 6, truncated=trunc)
    ref = oracle.advantages(rewards.cpu().numpy(), cu.cpu().numpy(), 6, truncated=trunc.cpu().numpy())
    assert np.allclose(resp.cpu().numpy(), ref[0], rtol=1e-6, atol=1e-7)
    assert int(kept.item()) == ref[3] == ntok
    V = 512
    g = torch.Generator(device=DEV).manual_seed(1)
    logits = torch.randn(ntok, V, generator=g, device=DEV)
    y = torch.randint(0, V, (ntok,), generator=g, device=DEV, dtype=torch.int32)
    p = ulorl.Params(is_mode=ulorl.IS_POIS, gate_mode=ulorl.GATE_NEVER, seg_len=seg)
    res = ulorl.token_loss_fwd(logits, y, cu, tok_adv, None, p)
    assert int(res.counters[3].item()) == 0
    seg_ids = res.segment_out.cpu().numpy()
    cu_h = cu.cpu().numpy()
    assert seg_ids[cu_h[1]:cu_h[2]].max() == 3 and seg_ids[cu_h[0]:cu_h[1]].max() == 0


@pytest.mark.parametrize("N,K", [(1, 1), (65, 3), (1024, 64), (5000, 5), (5000, 70), (9000, 1024), (70000, 9)])
def test_segment_diagnostics_of_ids_in_any_order(N, K):
    """Ids without order: up to 64 distinct ones in a wave (several passes of four), shared by all waves or by
    none, some out of range; sums against 64 bits, and again with the same bits."""
    g = torch.Generator(device=DEV).manual_seed(N + K)
    seg = torch.randint(-1, K + 1, (N,), generator=g, device=DEV, dtype=torch.int32)
    ratio, logp, old, ent = (torch.rand(N, generator=g, device=DEV) * 1.5 for _ in range(4))
    mask = (torch.rand(N, generator=g, device=DEV) < 0.3).to(torch.uint8)
    adv = torch.where(torch.rand(N, generator=g, device=DEV) < 0.5, 1.5, -0.65).float()
    res = ulorl.FwdResult(None, logp, ent, logp, mpt_mask=mask, ratio=ratio, segment_out=seg)
    got, again = (ulorl.segment_diagnostics(res, adv, old, K) for _ in range(2))
    ok = (seg >= 0) & (seg < K)
    at = seg[ok].long()
    zero = torch.zeros(K, dtype=torch.float64, device=DEV)
    r = ratio.double()
    lo, hi = 1.0 - float(np.float32(0.2)), 1.0 + float(np.float32(0.2))
    clipped = r * adv.double() > r.clamp(lo, hi) * adv.double()
    ref = dict(count=zero.index_add(0, at, torch.ones_like(r)[ok]), ratio_sum=zero.index_add(0, at, r[ok]),
               ratio_max=zero.scatter_reduce(0, at, r[ok], "amax"), clipped=zero.index_add(0, at, clipped.double()[ok]),
               kl_sum=zero.index_add(0, at, (old.double() - logp.double())[ok]), ent_sum=zero.index_add(0, at, ent.double()[ok]),
               masked=zero.index_add(0, at, mask.double()[ok]))
    for name, want in ref.items():
        assert torch.equal(got[name], again[name]), name
        # sums of up to N doubles below 1.5 in another order
        assert torch.all((got[name].double() - want).abs() <= 1.5 * N * N * 2.0 ** -53), name
    assert int(got["out_of_range"]) == int((~ok).sum())
