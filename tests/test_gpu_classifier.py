"""GPU parity of the prompt classifier (Sections 2.4, 3.3.3) against the fp64 oracle."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import mamba
from paper_2505_08600_amd import api
from paper_2505_08600_amd import datagen as dg

pytestmark = pytest.mark.gpu

# fp32 kernel against an fp64 oracle: sums of at most a few hundred terms and a recurrence of at
# most a few hundred steps whose decay is below one, so the error stays within a small multiple
# of 2^-24 times the number of terms; 1e-4 of the row's largest logit is the stated bar.
LOGIT_RTOL = 1e-4

WIDE = dg.ClassifierShape("classifier_wide", vocab=501, d_model=300, d_inner=192, d_state=16, dt_rank=16, d_conv=4,
                          n_classes=64)
ONE_TAP = dataclasses.replace(dg.CLASSIFIER_TINY, name="classifier_one_tap", d_conv=1, d_state=1, dt_rank=1,
                              n_classes=1)


def _run(shape, weights, tokens, lens, want_logits=True, **options):
    cls = api.Classifier(shape, weights)
    n = tokens.shape[0]
    t = torch.from_numpy(tokens).cuda()
    l = torch.from_numpy(lens).cuda()
    ids = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    logits = torch.full((n, shape.n_classes), float("nan"), device="cuda") if want_logits else None
    cls.route(t, l, ids, logits, **options)
    torch.cuda.synchronize()
    cls.close()
    return ids.cpu().numpy(), (logits.cpu().numpy() if want_logits else None)


def _check(shape, weights, tokens, lens, ids, logits):
    max_len = tokens.shape[1]
    close = 0
    for i in range(tokens.shape[0]):
        L = int(np.clip(lens[i], 0, max_len))
        ref, label = mamba.classify(weights, tokens[i, :L])
        scale = np.abs(ref).max()
        assert np.abs(logits[i] - ref).max() <= LOGIT_RTOL * scale, (i, L, logits[i], ref)
        top = np.sort(ref)
        if shape.n_classes > 1 and top[-1] - top[-2] <= 2 * LOGIT_RTOL * scale:
            close += 1      # a tie within the tolerance: either of the two is right
            assert ref[ids[i]] >= top[-2]
        else:
            assert ids[i] == label, (i, L, ids[i], label)
    return close


@pytest.mark.parametrize("shape,n,max_len,seed", [(dg.CLASSIFIER_TINY, 37, 40, 1), (ONE_TAP, 9, 20, 2),
                                                  (WIDE, 24, 50, 3), (dg.ClassifierShape(), 400, 128, 4)],
                         ids=lambda v: getattr(v, "name", None))
def test_labels_and_logits_match_oracle(shape, n, max_len, seed):
    print(f"classifier parity {shape.name} n={n} max_len={max_len}", flush=True)
    w = dg.make_classifier(shape, seed)
    tokens, lens = dg.make_classifier_prompts(seed, n, shape.vocab, max_len)
    edge = [0, 1, 7, 8, 9, 16, 17, max_len, max_len + 5]        # empty, chunk boundaries, full, over-long (clamped)
    lens[:len(edge)] = edge[:min(len(edge), n)]
    tokens = dg._rng(seed, 52).integers(0, shape.vocab, size=tokens.shape, dtype=np.int32)   # no zero padding
    ids, logits = _run(shape, w, tokens, lens)
    close = _check(shape, w, tokens, lens, ids, logits)
    assert close <= n // 20
    if shape.n_classes > 1 and n >= 37:
        assert len(set(ids.tolist())) > 1
    ids2, _ = _run(shape, w, tokens, lens, want_logits=False)
    assert np.array_equal(ids, ids2)


@pytest.mark.parametrize("d_inner,d_state,dt_rank,d_conv,d_model,n_classes", [
    (64, 16, 16, 4, 512, 64), (64, 1, 1, 1, 1, 2), (128, 5, 7, 2, 40, 3), (192, 16, 6, 4, 96, 4), (192, 3, 16, 3, 7, 33), (256, 4, 2, 4, 24, 5)])
def test_every_channel_count_and_rank_matches_oracle(d_inner, d_state, dt_rank, d_conv, d_model, n_classes):
    """Both sides of the line between the kernels (192 and 256 channels), every wave count of the four-threads-per-channel
    kernel, the smallest and largest state, rank, taps, output and class counts, prompts that end on and beside its chunks."""
    shape = dg.ClassifierShape("classifier_edge", vocab=61, d_model=d_model, d_inner=d_inner, d_state=d_state, dt_rank=dt_rank,
                               d_conv=d_conv, n_classes=n_classes)
    print(f"classifier d_inner={d_inner} d_state={d_state}", flush=True)
    w = dg.make_classifier(shape, 31)
    lens = np.array([0, 1, 2, 3, 4, 5, 15, 16, 17, 31, 32, 33, 48, 49, 70, 77], np.int32)   # (the last one is clamped to 70)
    tokens = dg._rng(31, 52).integers(0, shape.vocab, size=(len(lens), 70), dtype=np.int32)
    ids, logits = _run(shape, w, tokens, lens)
    assert _check(shape, w, tokens, lens, ids, logits) <= 1


def test_padding_is_ignored_and_batch_position_does_not_matter():
    shape = dg.CLASSIFIER_TINY
    w = dg.make_classifier(shape, 5)
    tokens, lens = dg.make_classifier_prompts(5, 16, shape.vocab, 32)
    ids, logits = _run(shape, w, tokens, lens)
    junk = tokens.copy()
    junk[np.arange(32)[None, :] >= lens[:, None]] = 96
    perm = np.random.default_rng(0).permutation(16)
    ids2, logits2 = _run(shape, w, junk[perm], lens[perm])
    assert np.array_equal(ids[perm], ids2) and np.array_equal(logits[perm], logits2)


@pytest.mark.parametrize("d_inner", [64, 192])
def test_batch_invariant_logits_are_the_same_bits_in_any_batch(d_inner):
    """60 prompts of up to 300 tokens, which the default call cuts: with batch_invariant a prompt's logits do not change with the
    order of the batch or with who else is in it; without it they agree to the stated bar."""
    shape = dg.ClassifierShape("classifier_invariant", vocab=97, d_model=24, d_inner=d_inner, d_state=16, dt_rank=6, d_conv=4, n_classes=5)
    w = dg.make_classifier(shape, 49)
    rng = dg._rng(49, 71)
    n, max_len = 60, 300
    tokens = rng.integers(0, shape.vocab, size=(n, max_len), dtype=np.int32)
    lens = rng.integers(0, max_len + 1, size=n).astype(np.int32)
    ids, logits = _run(shape, w, tokens, lens, batch_invariant=True)
    perm = np.random.default_rng(3).permutation(n)
    ids2, logits2 = _run(shape, w, tokens[perm], lens[perm], batch_invariant=True)
    assert np.array_equal(ids[perm], ids2) and np.array_equal(logits[perm], logits2)
    for part in (slice(0, 1), slice(7, 9), slice(20, 60)):
        ids3, logits3 = _run(shape, w, tokens[part], lens[part], batch_invariant=True)
        assert np.array_equal(ids[part], ids3) and np.array_equal(logits[part], logits3)
    _, cut = _run(shape, w, tokens, lens)
    assert np.abs(cut - logits).max() <= LOGIT_RTOL * np.abs(logits).max()


@pytest.mark.parametrize("d_inner,n,max_len", [(192, 1, 700), (192, 400, 128), (128, 300, 60), (64, 40, 200), (192, 30, 33), (192, 6000, 80), (192, 520, 16), (64, 3, 2000)])
def test_runs_of_chunks_that_cut_prompts(d_inner, n, max_len):
    """Batches dealt out in runs of chunks that start inside prompts: one prompt over many workgroups, runs of one, several and
    many chunks (more than are laid out at a time), prompts of one chunk; a sample of the batch against the oracle, in the batch,
    alone and in the batch permuted; the entry without a workspace; an id out of range in the last token of a prompt."""
    print(f"classifier batches d_inner={d_inner} n={n} max_len={max_len}", flush=True)
    shape = dg.ClassifierShape("classifier_cut", vocab=97, d_model=24, d_inner=d_inner, d_state=16, dt_rank=6, d_conv=4, n_classes=5)
    w = dg.make_classifier(shape, 41)
    rng = dg._rng(41, 53)
    tokens = rng.integers(0, shape.vocab, size=(n, max_len), dtype=np.int32)
    lens = rng.integers(0, max_len + 1, size=n).astype(np.int32)
    edge = [max_len, 0, 33, 32, 16, 17, 64, 65, 31]
    lens[:len(edge)] = edge[:n]
    lens = np.minimum(lens, max_len).astype(np.int32)
    bad = min(6, n - 1)
    if n > 1:
        tokens[bad, lens[bad] - 1] = shape.vocab   # in the last of its segments
    ids, logits = _run(shape, w, tokens, lens)
    perm = np.random.default_rng(1).permutation(n)
    ids2, logits2 = _run(shape, w, tokens[perm], lens[perm])
    assert np.abs(logits[perm] - logits2).max() <= LOGIT_RTOL * np.abs(logits).max()
    top = np.sort(logits, 1)
    clear = top[:, -1] - top[:, -2] > 2 * LOGIT_RTOL * np.abs(logits).max()   # (elsewhere two classes tie to rounding)

    def same_ids(a, b):
        assert np.array_equal(a == -1, b == -1) and np.array_equal(a[clear], b[clear])

    assert np.array_equal(np.flatnonzero(ids == -1), [bad] if n > 1 else [])
    same_ids(ids, ids2[np.argsort(perm)])
    some = [0] + list(range(1, min(n, 12))) + [n - 1]
    for i in some:
        one, lone = _run(shape, w, tokens[i:i + 1], lens[i:i + 1])
        assert np.abs(lone[0] - logits[i]).max() <= LOGIT_RTOL * np.abs(logits[i]).max(), i
        assert (one[0] == -1) == (ids[i] == -1)
    if n > 1:
        assert ids[bad] == -1
    keep = [i for i in some if n == 1 or i != bad]
    _check(shape, w, tokens[keep], lens[keep], ids[keep], logits[keep])
    cls = api.Classifier(shape, w)   # the entry without a workspace
    t, l = torch.from_numpy(tokens).cuda(), torch.from_numpy(lens).cuda()
    ids3 = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    logits3 = torch.full((n, 5), float("nan"), device="cuda")
    assert api.lib().sd_route_classifier(cls.h, t.data_ptr(), l.data_ptr(), n, max_len, logits3.data_ptr(), ids3.data_ptr(), None) == api.SD_OK
    torch.cuda.synchronize()
    cls.close()
    ids3, logits3 = ids3.cpu().numpy(), logits3.cpu().numpy()
    same_ids(ids, ids3)
    _check(shape, w, tokens[keep], lens[keep], ids3[keep], logits3[keep])
    assert np.abs(logits3 - logits).max() <= LOGIT_RTOL * np.abs(logits).max()   # (both paths within the bar of the oracle)


@pytest.mark.parametrize("d_inner,n,lo,hi", [(192, 250, 50, 70), (128, 200, 60, 64), (64, 256, 1, 17), (192, 31, 33, 40)])
def test_batches_of_nearly_equal_lengths_are_not_cut(d_inner, n, lo, hi):
    """Lengths within a chunk of each other on up to 256 workgroups: a workgroup per prompt in the call with a workspace too, so the
    logits do not depend on the batch bit for bit; an empty prompt and an invalid last id among them."""
    print(f"classifier uncut d_inner={d_inner} n={n} of {lo} to {hi}", flush=True)
    shape = dg.ClassifierShape("classifier_uncut", vocab=97, d_model=24, d_inner=d_inner, d_state=16, dt_rank=6, d_conv=4, n_classes=5)
    w = dg.make_classifier(shape, 45)
    rng = dg._rng(45, 67)
    tokens = rng.integers(0, shape.vocab, size=(n, hi), dtype=np.int32)
    lens = rng.integers(lo, hi + 1, size=n).astype(np.int32)
    lens[3], lens[4], lens[n - 1] = 0, hi, hi
    tokens[4, hi - 1] = -5
    ids, logits = _run(shape, w, tokens, lens)
    assert np.flatnonzero(ids == -1).tolist() == [4]
    some = [0, 1, 2, 3, 5, n // 2, n - 1]
    _check(shape, w, tokens[some], lens[some], ids[some], logits[some])
    perm = np.random.default_rng(2).permutation(n)
    ids2, logits2 = _run(shape, w, tokens[perm], lens[perm])
    assert np.array_equal(ids[perm], ids2) and np.array_equal(logits[perm], logits2)


@pytest.mark.parametrize("d_inner", [64, 192])
def test_an_invalid_id_in_any_part_of_a_cut_prompt_is_flagged(d_inner):
    """Three prompts of 1300 to 2000 tokens over some 200 workgroups (runs of two chunks): an id out of range in the part a prompt
    starts in, in runs that lie inside it, in its last chunk and behind its end; exactly the prompts that hold one get -1, and
    the others keep their logits."""
    shape = dg.ClassifierShape("classifier_parts", vocab=97, d_model=24, d_inner=d_inner, d_state=16, dt_rank=6, d_conv=4, n_classes=5)
    w = dg.make_classifier(shape, 43)
    rng = dg._rng(43, 59)
    tokens = rng.integers(0, shape.vocab, size=(3, 2000), dtype=np.int32)
    lens = np.array([1777, 2000, 1300], np.int32)
    ids, logits = _run(shape, w, tokens, lens)
    assert (ids >= 0).all()
    for i in range(3):
        L = int(lens[i])
        for at in (0, 15, 16, 40, L // 2, L - 40, L - 17, L - 1, L):
            if at == tokens.shape[1]:
                continue
            print(f"invalid id d_inner={d_inner} prompt {i} token {at}", flush=True)
            t = tokens.copy()
            t[i, at] = (-1, shape.vocab, 2 ** 31 - 1)[at % 3]
            got, lg = _run(shape, w, t, lens)
            want = ids.copy()
            if at < L:
                want[i] = -1
            assert np.array_equal(got, want), (i, at, got)
            others = [k for k in range(3) if k != i or at >= L]
            assert np.array_equal(lg[others], logits[others])


def test_workspaces_hold_anything_and_calls_on_several_streams_keep_apart():
    """The same batch with workspaces of zeros, ones, NaN, of a call of another batch and at an address that is no multiple of 8, on
    four streams at once: the same bits in every call; and captured into a graph whose replays see other lengths and ids."""
    shape = dg.ClassifierShape("classifier_streams", vocab=97, d_model=24, d_inner=128, d_state=16, dt_rank=6, d_conv=4, n_classes=5)
    w = dg.make_classifier(shape, 47)
    rng = dg._rng(47, 61)
    n, max_len, L = 37, 300, api.lib()
    cls = api.Classifier(shape, w)
    batches = []
    for k in range(4):
        t = torch.from_numpy(rng.integers(0, shape.vocab, size=(n, max_len), dtype=np.int32)).cuda()
        l = torch.from_numpy((rng.integers(0, max_len + 1, size=n) if k else np.full(n, max_len)).astype(np.int32)).cuda()
        batches.append((t, l))
    need = L.sd_classifier_workspace(cls.h, n, max_len)

    def call(t, l, ws):
        ids = torch.full((n,), -7, dtype=torch.int32, device="cuda")
        lg = torch.full((n, 5), float("nan"), device="cuda")
        api._check(L.sd_route_classifier_ws(cls.h, t.data_ptr(), l.data_ptr(), n, max_len, lg.data_ptr(), ids.data_ptr(), ws.data_ptr(), api._stream()))
        return ids, lg

    ref = [call(t, l, torch.zeros(need, dtype=torch.uint8, device="cuda")) for t, l in batches]
    torch.cuda.synchronize()
    for fill in (0, 1, 255):
        ws = torch.full((need + 8,), fill, dtype=torch.uint8, device="cuda")
        for k, (t, l) in enumerate(batches):   # (the second call finds the first one's workspace)
            for at in (0, 4):
                ids, lg = call(t, l, ws[at:])
                assert torch.equal(ids, ref[k][0]) and torch.equal(lg, ref[k][1])
    streams = [torch.cuda.Stream() for _ in batches]
    spaces = [torch.full((need,), 255, dtype=torch.uint8, device="cuda") for _ in batches]
    torch.cuda.synchronize()
    got = []
    for _ in range(25):
        for k, s in enumerate(streams):
            with torch.cuda.stream(s):
                got.append((k,) + call(*batches[k], spaces[k]))
    torch.cuda.synchronize()
    assert all(torch.equal(ids, ref[k][0]) and torch.equal(lg, ref[k][1]) for k, ids, lg in got)
    t, l = (x.clone() for x in batches[0])
    ids, lg = torch.empty(n, dtype=torch.int32, device="cuda"), torch.empty((n, 5), device="cuda")
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        cls.route(t, l, ids, lg)
    for rep in range(3):
        for k in (1, 0, 2, 3):
            t.copy_(batches[k][0])
            l.copy_(batches[k][1])
            graph.replay()
            assert torch.equal(ids, ref[k][0]) and torch.equal(lg, ref[k][1]), (rep, k)
            cls.route(*batches[(k + 1) % 4], torch.empty_like(ids))   # the program's own calls in between
            torch.cuda.synchronize()
    cls.close()


def test_more_chunks_than_32_bits_number_take_no_workspace():
    """Up to 2^30 chunks of 16 tokens are dealt out; more could wrap the numbers the blocks count them with: a block per prompt."""
    shape = dg.CLASSIFIER_TINY
    cls = api.Classifier(shape, dg.make_classifier(shape, 6))
    need = lambda n, max_len: api.lib().sd_classifier_workspace(cls.h, n, max_len)
    assert need(2 ** 31 - 1, 17) == 0 and need(2 ** 31 - 1, 2 ** 31 - 1) == 0
    assert need(2 ** 30, 16) > 0 and need(2 ** 29, 32) > 0 and need(2 ** 29 + 1, 32) == 0
    cls.close()


def test_out_of_range_token_is_flagged_not_read():
    shape = dg.CLASSIFIER_TINY
    w = dg.make_classifier(shape, 6)
    tokens, lens = dg.make_classifier_prompts(6, 6, shape.vocab, 16)
    lens[:] = [16, 10, 4, 16, 9, 12]
    tokens[1, 9] = shape.vocab
    tokens[3, 0] = -1
    tokens[4, 12] = 1 << 30         # beyond the prompt's length: never looked at
    ids, logits = _run(shape, w, tokens, lens)
    assert ids[1] == -1 and ids[3] == -1 and np.isfinite(logits).all()
    good = [0, 2, 4, 5]
    _check(shape, w, tokens[good], lens[good], ids[good], logits[good])


def test_shapes_outside_the_kernel_limits_are_rejected():
    w = dg.make_classifier(dg.CLASSIFIER_TINY, 1)
    for bad in (dict(d_inner=96), dict(d_inner=32), dict(d_inner=576), dict(d_state=17), dict(dt_rank=0), dict(d_conv=5),
                dict(n_classes=65), dict(d_model=513), dict(vocab=0)):
        with pytest.raises(api.SdError) as ei:
            api.Classifier(dataclasses.replace(dg.CLASSIFIER_TINY, **bad), w)
        assert ei.value.code == api.SD_EINVAL, bad
    big = dg.ClassifierShape("too_big_for_lds", vocab=10, d_model=64, d_inner=512, d_state=16, dt_rank=16)
    with pytest.raises(api.SdError) as ei:
        api.Classifier(big, dg.make_classifier(big, 1))
    assert ei.value.code == api.SD_EINVAL and "LDS" in str(ei.value)
