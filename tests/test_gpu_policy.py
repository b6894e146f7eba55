"""Candidate counts per sequence (Section 1, Equation 1 used inside the loop; Section 3.2.2 reports a different best
count per task): the draft / verify / commit calls with per-sequence counts against the oracle run sequence by
sequence with the same counts, and the device-side choice of the counts against the host function."""
import numpy as np
import pytest
import torch

import oracle
from paper_2505_08600_amd import api
from paper_2505_08600_amd import datagen as dg

import sdharness as H

pytestmark = pytest.mark.gpu


def _run(pair, prompts, G, T, n_steps, seed, gamma_fn, dtype):
    """Teacher-forced lockstep of a batch whose sequences use their own candidate counts: gamma_fn(step, history) ->
    counts for this step (history: per sequence, the oracle's (n_acc, gamma) of earlier steps).  Returns the number of
    flagged sequence-steps and the counts used."""
    B, V = len(prompts), pair.shape_t.vocab
    caps = [len(p) + n_steps * (G + 1) + 8 for p in prompts]
    tseqs = [pair.ot.new_seq(c) for c in caps]
    dseqs = [pair.od.new_seq(c) for c in caps]
    ctxs = [[int(t) for t in p] for p in prompts]
    for b in range(B):
        oracle.prefill(tseqs[b], ctxs[b])
        oracle.prefill(dseqs[b], ctxs[b])
    ctx = api.Context(caps)
    ctx.attach(pair.gt)
    ctx.attach(pair.gd)
    H.gpu_prefill(ctx, [pair.gt, pair.gd], [list(p) for p in prompts])
    cand_g = torch.zeros((B, G), dtype=torch.int32, device="cuda")
    q_g = torch.zeros((B, G, V), dtype=torch.float32, device="cuda")
    na_g = torch.zeros(B, dtype=torch.int32, device="cuda")
    nx_g = torch.zeros(B, dtype=torch.int32, device="cuda")
    history = [[] for _ in range(B)]
    flagged, used = 0, []
    for k in range(n_steps):
        gam = gamma_fn(k, history, ctx)
        used.append(list(gam))
        ud = np.stack([dg.make_uniforms(seed, dg.DRAFT_STREAM, b, k, G) for b in range(B)])
        uv = np.stack([dg.make_uniforms(seed, dg.VERIFY_STREAM, b, k, G + 1) for b in range(B)])
        # ---- oracle, sequence by sequence, each with its own count
        recs = []
        for b in range(B):
            g = int(gam[b])
            n0 = len(ctxs[b])
            if g > 0:
                cand, q, mgd = dseqs[b].draft(ctxs[b], g, T, ud[b, :g])
            else:
                cand, q, mgd = np.zeros(0, np.int32), (np.zeros((0, V), np.float32) if T > 0 else None), np.zeros(0)
            r_na, r_nx, mgv, lg = tseqs[b].verify(ctxs[b], g, T, cand, q, uv[b, :g + 1], want_logits=True)
            oracle.loop.commit(ctxs[b], tseqs[b], dseqs[b], cand, r_na, r_nx)
            recs.append(oracle.StepRecord(n0, cand, q, ud[b, :g], uv[b, :g + 1], r_na, r_nx, mgd, mgv, lg))
            history[b].append((r_na, g))
        # ---- HIP path: one draft call, one verify call for the whole batch
        cand_g.fill_(-1)
        q_g.fill_(-1.0)
        api.sd_draft(pair.gd, ctx, None, B, G, T, H.dev(ud) if T > 0 else None, cand_g, q_g if T > 0 else None)
        cg, qg = cand_g.cpu().numpy(), q_g.cpu().numpy()
        refeed = []
        for b in range(B):
            g = int(gam[b])
            assert (cg[b, g:] == -1).all(), "candidates beyond the sequence's count must stay untouched"
            if T > 0:
                assert (qg[b, g:] == -1.0).all()
            if g > 0:
                f, first_bad, _ = H.check_draft_step(recs[b], cg[b, :g], qg[b, :g] if T > 0 else None, T, dtype, V)
                flagged += int(f)
                if first_bad is not None:
                    refeed.append((b, recs[b].n_ctx - 1 + first_bad))
        cand_in = np.zeros((B, G), np.int32)
        q_in = np.zeros((B, G, V), np.float32)
        for b in range(B):
            g = int(gam[b])
            cand_in[b, :g] = recs[b].cand
            if T > 0 and g > 0:
                q_in[b, :g] = recs[b].q
        cand_d = H.dev(cand_in)
        api.sd_verify(pair.gt, ctx, None, B, G, T, cand_d, H.dev(q_in) if T > 0 else None, H.dev(uv) if T > 0 else None,
                      na_g, nx_g, commit=False)
        lg_g = pair.gt.last_logits().cpu().numpy().reshape(B, G + 1, V)
        na_h, nx_h = na_g.cpu().numpy(), nx_g.cpu().numpy()
        for b in range(B):
            g = int(gam[b])
            f, _ = H.check_verify_step(recs[b], int(na_h[b]), int(nx_h[b]), lg_g[b, :g + 1], T, dtype, V)
            flagged += int(f)
        api.sd_commit(ctx, None, B, G, cand_d, H.dev(np.array([r.n_acc for r in recs], np.int32)),
                      H.dev(np.array([r.next_token for r in recs], np.int32)))
        for b, keep in refeed:
            torch.cuda.synchronize()
            ctx.truncate(pair.gd, b, keep)
            api.sd_prefill(pair.gd, ctx, H.dev(np.array([b], np.int32)), 1, G + 2)
    nt, kv = ctx.sync(pair.gt)
    for b in range(B):
        assert nt[b] == len(ctxs[b]) and kv[b] == nt[b] - 1
        assert list(ctx.get_tokens(b)) == ctxs[b]
    on, g_dev, acc, exam = ctx.policy_read()
    for b in range(B):   # the device's acceptance history is the oracle's
        assert acc[b] == sum(a for a, g in history[b])
        assert exam[b] == sum(a + 1 if a < g else g for a, g in history[b])
    ctx.close()
    return flagged, used


@pytest.mark.parametrize("T", [0.0, 1.0])
def test_fixed_counts_per_sequence_match_oracle(T):
    """Counts 0 (a plain autoregressive sequence), 1, 3 and the full 4 in one batch, changing from step to step."""
    print(f"per-sequence candidate counts, fp32 tiny pair, T={T}", flush=True)
    st, sd_ = dg.SHAPES["tiny_target"], dg.SHAPES["tiny_draft"]
    wt = dg.make_weights(st, 51, 20.0)
    pair = H.Pair(st, st, 51, target_weights=wt, draft_weights=dg.perturbed_copy(wt, st, seed=52, rel=0.1), max_rows=32)
    prompts = [dg.make_prompt(51, b, 9 + 5 * b, st.vocab) for b in range(4)]
    table = [[0, 1, 3, 4], [4, 0, 2, 1], [2, 4, 0, 3], [0, 0, 4, 4], [3, 3, 3, 0], [1, 4, 4, 2]]
    state = {}

    def gamma_fn(k, history, ctx):
        ctx.policy_set(table[k % len(table)])
        return table[k % len(table)]

    flagged, used = _run(pair, prompts, 4, T, 12, 51, gamma_fn, dg.FP32)
    print(f"  flagged={flagged}", flush=True)
    assert flagged <= 1
    pair.close()


@pytest.mark.parametrize("shapes,dtype,T", [(("tiny_target", "tiny_draft"), dg.FP32, 1.0),
                                            (("small_target_bf16", "small_draft_bf16"), dg.BF16, 0.7)])
def test_counts_follow_equation_1_step_by_step(shapes, dtype, T):
    """The counts are chosen on the device before every step from the running acceptance estimate; the host function
    sd_choose_gamma on the oracle's own history must give the same counts, and every step must still match the
    oracle run with those counts.  A draft close to the target earns long drafts, an independent draft short ones."""
    print(f"Equation 1 in the loop: {shapes} T={T}", flush=True)
    st, sd_ = dg.SHAPES[shapes[0]], dg.SHAPES[shapes[1]]
    G, c_ratio, alpha0, B, n_steps = 6, 0.05, 0.5, 5, 14
    scale = 20.0 if dtype == dg.FP32 else 4.0
    wt = dg.make_weights(st, 61, scale)
    # the draft: a slightly perturbed copy of the target (high acceptance) - except that two of the five sequences
    # get prompts from another seed, which changes nothing about the model but gives varied histories
    pair = H.Pair(st, st, 61, target_weights=wt, draft_weights=dg.perturbed_copy(wt, st, seed=62, rel=0.1 if dtype == dg.FP32 else 0.3),
                  max_rows=64,
                  max_pos=256)
    prompts = [dg.make_prompt(61 + (b % 2), b, 8 + 3 * b, st.vocab) for b in range(B)]
    gam_dev = torch.zeros(B, dtype=torch.int32, device="cuda")

    def gamma_fn(k, history, ctx):
        ctx.policy_choose(None, B, c_ratio, G, alpha0, gam_dev)
        got = gam_dev.cpu().numpy()
        want = []
        for b in range(B):
            acc = sum(a for a, g in history[b])
            exam = sum(a + 1 if a < g else g for a, g in history[b])
            alpha = acc / exam if exam > 0 else alpha0
            want.append(api.choose_gamma(alpha, c_ratio, G)[0])
        assert list(got) == want, (k, list(got), want)
        on, g_all, _, _ = ctx.policy_read()
        assert on and list(g_all) == want
        return want

    flagged, used = _run(pair, prompts, G, T, n_steps, 61, gamma_fn, dtype)
    print(f"  flagged={flagged} counts per step: {used}", flush=True)
    assert flagged <= 1
    assert len({g for row in used for g in row}) >= 2, "the history should move the counts"
    pair.close()


@pytest.mark.parametrize("V,B,G", [(32772, 4, 3), (1024, 52, 4)])
def test_counts_in_wide_rows_and_in_large_batches(V, B, G):
    """Counts per sequence in the other two forms of the acceptance rule: rows above 32768 columns, whose slices follow the
    call's row slots and not the sequence's own count, and more than 256 rows, where one block per sequence draws."""
    import dataclasses
    print(f"per-sequence counts V={V} B={B} gamma={G}", flush=True)
    st = dataclasses.replace(dg.SHAPES["tiny_target"], vocab=V, n_layers=1, name=f"policy_{V}")
    wt = dg.make_weights(st, 81, 20.0)
    pair = H.Pair(st, st, 81, target_weights=wt, draft_weights=dg.perturbed_copy(wt, st, seed=82, rel=0.1), max_rows=B * (G + 1))
    prompts = [dg.make_prompt(81, b, 3 + b % 7, V) for b in range(B)]

    def gamma_fn(k, history, ctx):
        counts = [(b + k) % (G + 1) for b in range(B)]
        ctx.policy_set(counts)
        return counts

    flagged, used = _run(pair, prompts, G, 1.0, 2, 81, gamma_fn, dg.FP32)
    print(f"  flagged={flagged}", flush=True)
    assert flagged <= 1 + B // 50
    pair.close()


def test_policy_argument_errors():
    ctx = api.Context([32, 32])
    L = api.lib()
    assert L.sd_policy_set(None, None) == api.SD_EINVAL
    with pytest.raises(api.SdError):
        ctx.policy_set([1, 16])
    with pytest.raises(api.SdError):
        ctx.policy_choose(None, 3, 0.1, 5, 0.5)
    with pytest.raises(api.SdError):
        ctx.policy_choose(None, 2, -0.1, 5, 0.5)
    with pytest.raises(api.SdError):
        ctx.policy_choose(None, 2, 0.1, 16, 0.5)
    on, g, a, e = ctx.policy_read()
    assert not on and (a == 0).all() and (e == 0).all()
    ctx.policy_set([2, 3])
    assert ctx.policy_read()[0] and list(ctx.policy_read()[1]) == [2, 3]
    ctx.policy_set(None)
    assert not ctx.policy_read()[0]
    ctx.close()
