"""GPU parity of the acceptance rule as a call of its own (sd_accept; Section 3.1) against the oracle's
orc_accept on the same fp32 logits, draft distributions, candidates and uniforms."""
import numpy as np
import pytest
import torch

import oracle
from paper_2505_08600_amd import api
from paper_2505_08600_amd import datagen as dg

pytestmark = pytest.mark.gpu


def synthetic_case(seed, B, gamma, V, rho, T):
    """Config-5 style inputs without a model: target logits N(0, 3), q = softmax(rho * logits + (1 - rho) * 4 N(0,1)),
    candidates drawn from q by the oracle's own inverse CDF, uniforms on the 2^-24 grid."""
    logits = np.stack([3.0 * dg.make_logit_noise(seed, b, 100 + i, V) for b in range(B) for i in range(gamma + 1)])
    logits = logits.reshape(B, gamma + 1, V).astype(np.float32)
    q = np.zeros((B, max(gamma, 1), V), np.float32)
    cand = np.zeros((B, max(gamma, 1)), np.int32)
    for b in range(B):
        ud = dg.make_uniforms(seed, dg.DRAFT_STREAM, b, 0, max(gamma, 1))
        for i in range(gamma):
            z = rho * logits[b, i] + (1.0 - rho) * 4.0 * dg.make_logit_noise(seed, b, i, V)
            q[b, i] = oracle.softmax_T(z.astype(np.float32), T if T > 0 else 1.0)
            cand[b, i] = oracle.sample_cdf(q[b, i].astype(np.float64), float(ud[i]))[0]
    u = np.stack([dg.make_uniforms(seed, dg.VERIFY_STREAM, b, 0, gamma + 1) for b in range(B)])
    return logits, q[:, :gamma], cand[:, :gamma], u


def check_against_oracle(logits, q, cand, u, T, na, nx, thr=1e-5):
    """Bit-exact decisions, unless the oracle's own margin is below the fp32 threshold.  -> flagged count"""
    B, rows, V = logits.shape
    gamma = rows - 1
    flagged = 0
    for b in range(B):
        r_na, r_nx, mg = oracle.accept(logits[b], q[b] if gamma and T > 0 else None, cand[b], u[b], T)
        if (int(na[b]), int(nx[b])) == (r_na, r_nx):
            continue
        flagged += 1
        if int(na[b]) != r_na:
            i = min(int(na[b]), r_na)
            lim = thr if T > 0 else thr * float(np.abs(logits[b, i]).max())
            assert mg[i] < lim, (b, int(na[b]), r_na, mg)
        elif T > 0:
            w = oracle.next_weights(logits[b], q[b] if gamma else None, r_na, T)
            assert oracle.cdf_distance(w, float(u[b, gamma]), int(nx[b])) < thr, (b, int(nx[b]), r_nx)
        else:
            assert mg[gamma] < thr * float(np.abs(logits[b, r_na]).max())
    return flagged


@pytest.mark.parametrize("V,gamma,T,rho", [(32000, 8, 1.0, 0.5), (32000, 8, 0.7, 0.9), (32000, 5, 1.0, 0.0),
                                           (32000, 5, 0.0, 0.9), (50000, 3, 1.0, 0.5), (1024, 4, 1.0, 0.5),
                                           (32000, 0, 1.0, 0.0), (262144, 2, 1.0, 0.5)])
def test_accept_alone_matches_oracle(V, gamma, T, rho):
    print(f"sd_accept V={V} gamma={gamma} T={T} rho={rho}", flush=True)
    B = 6
    logits, q, cand, u = synthetic_case(91, B, gamma, V, rho, T)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    na = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    nx = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    ws = torch.full((3 * B * (gamma + 1),), float("nan"), device="cuda")   # contents on entry must not matter
    api.sd_accept(dev(logits), gamma, T, dev(cand) if gamma else None, dev(q) if gamma and T > 0 else None,
                  dev(u) if T > 0 else None, na, nx, ws)
    torch.cuda.synchronize()
    na_h, nx_h = na.cpu().numpy(), nx.cpu().numpy()
    flagged = check_against_oracle(logits, q, cand, u, T, na_h, nx_h)
    print(f"  n_acc={na_h.tolist()} flagged={flagged}", flush=True)
    assert flagged <= 1
    if gamma >= 5 and 0 < rho < 1 and T > 0:
        assert len(set(na_h.tolist())) >= 2   # the case exercises accept, reject and the residual draw


@pytest.mark.parametrize("V,gamma,T", [(32772, 15, 1.0), (32772, 1, 0.7), (65536, 0, 1.0), (100004, 7, 1.0), (262144, 1, 0.7),
                                       (131072, 4, 0.0)])
def test_rows_beyond_a_blocks_registers(V, gamma, T):
    """Rows of more than 32768 columns: one vector past the boundary, slices of unequal length, a single slice (gamma 0),
    slices whose columns are all masked (-inf, and the lowest float), up to 16 slices; residual draws and draws from p."""
    print(f"wide rows V={V} gamma={gamma} T={T}", flush=True)
    B = 5
    logits, q, cand, u = synthetic_case(37, B, gamma, V, 0.9, T)
    if T > 0:
        logits[:, :, V // 3:V // 2] = -np.inf
        logits[:, :, V - 4:] = np.float32(-3.4028235e38)
        logits[1, :, V // 4:] = -np.inf          # everything after the first quarter: the later slices have no mass
        logits[2, :, :3 * V // 4] = -np.inf      # everything before the last quarter
        if gamma:
            q = np.stack([np.stack([oracle.softmax_T(logits[b, i] * np.float32(0.9), T) for i in range(gamma)]) for b in range(B)])
            q[3] = np.stack([oracle.softmax_T(logits[3, i], T) for i in range(gamma)])   # q = p: everything is accepted
            cand = np.stack([[oracle.sample_cdf(q[b, i].astype(np.float64), 0.37 + 0.05 * i / 16)[0] for i in range(gamma)] for b in range(B)]).astype(np.int32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    na, nx = (torch.full((B,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    ws = torch.full((3 * B * (gamma + 1),), float("nan"), device="cuda")
    for _ in range(2):   # the workspace holds the first call's slice masses when the second starts
        api.sd_accept(dev(logits), gamma, T, dev(cand) if gamma else None, dev(q) if gamma and T > 0 else None,
                      dev(u) if T > 0 else None, na, nx, ws)
        torch.cuda.synchronize()
        na_h, nx_h = na.cpu().numpy(), nx.cpu().numpy()
        assert check_against_oracle(logits, q, cand, u, T, na_h, nx_h) <= 1
        assert all(np.isfinite(logits[b, na_h[b], nx_h[b]]) and logits[b, na_h[b], nx_h[b]] > -1e38 for b in range(B))
    print(f"  n_acc={na_h.tolist()}", flush=True)


@pytest.mark.parametrize("T", [1.0, 0.0])
def test_wide_rows_in_blocks_of_512_threads(T):
    """512 rows and more above 32768 columns, two blocks to a compute unit: 129 sequences of 4 rows over 33004 columns, with
    rejections, residual draws, a masked range and everything accepted, against the oracle (sequences repeat five
    cases with uniforms of their own)."""
    V, gamma, n = 33004, 3, 5
    print(f"512-thread blocks V={V} T={T}", flush=True)
    logits, q, cand, u = synthetic_case(43, n, gamma, V, 0.9, T)
    logits[:, :, V // 3:V // 2] = -np.inf
    if T > 0:
        q = np.stack([np.stack([oracle.softmax_T(logits[b, i] * np.float32(0.9 if b else 1.0), T) for i in range(gamma)]) for b in range(n)])
        cand = np.stack([[oracle.sample_cdf(q[b, i].astype(np.float64), 0.37 + 0.05 * i)[0] for i in range(gamma)] for b in range(n)]).astype(np.int32)
    else:
        cand[0] = logits[0, :gamma].argmax(-1)
        cand[1, 0] = logits[1, 0].argmax(-1)
    B = 129
    pick = np.arange(B) % n
    logits, q, cand = logits[pick], q[pick], cand[pick]
    u = np.stack([dg.make_uniforms(43, dg.VERIFY_STREAM, b, 1, gamma + 1) for b in range(B)])
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    na, nx = (torch.full((B,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    ws = torch.full((3 * B * (gamma + 1),), float("nan"), device="cuda")
    api.sd_accept(dev(logits), gamma, T, dev(cand), dev(q) if T > 0 else None, dev(u) if T > 0 else None, na, nx, ws)
    torch.cuda.synchronize()
    na_h, nx_h = na.cpu().numpy(), nx.cpu().numpy()
    assert check_against_oracle(logits, q, cand, u, T, na_h, nx_h) <= 2
    assert len(set(na_h.tolist())) >= 3


@pytest.mark.parametrize("V,gamma,n_trials", [(2772, 0, 1500), (2772, 1, 1500), (32000, 0, 900), (32000, 1, 600),
                                              (50000, 0, 450), (262144, 0, 99)])
def test_next_token_for_uniforms_on_the_boundaries_of_the_cdf(V, gamma, n_trials):
    """The next token is the first index whose inclusive sum of weights exceeds u * Z (Section 3.1: a draw from p, or
    from the normalised max(p - q, 0) after a rejection).  The kernels add those sums in parallel - per thread of four
    consecutive weights, per wave, per segment - so the places where rounding can make two partial sums disagree are the
    ends of those groups.  Here every trial is one sequence with the same logits row and a uniform that sits on such an
    end of the exact CDF, or one or two float32 steps beside it: the token returned must always be one of the two that
    meet there (within the fp32 band of the decision rule), never one from elsewhere in the row."""
    print(f"boundary uniforms V={V} gamma={gamma} trials={n_trials}", flush=True)
    T = 1.0
    rng = np.random.default_rng(V + gamma)
    row = (3.0 * dg.make_logit_noise(17, 0, 0, V)).astype(np.float32)
    logits1 = np.stack([row] + [(3.0 * dg.make_logit_noise(17, 0, 1 + i, V)).astype(np.float32) for i in range(gamma)])
    q1 = cand1 = None
    if gamma:   # a candidate that is certainly rejected: q puts ten times the target's mass on it
        p0 = oracle.softmax_T(row, T).astype(np.float64)
        c = int(np.argsort(-p0)[3])
        q1 = oracle.softmax_T((0.5 * row + 2.0 * dg.make_logit_noise(17, 1, 0, V)).astype(np.float32), T).astype(np.float64)
        q1[c] = min(0.9, 10.0 * p0[c] + 0.05)
        q1 = (q1 / q1.sum()).astype(np.float32)[None]
        cand1 = np.array([c], np.int32)
    w = np.asarray(oracle.next_weights(logits1, q1, 0, T), np.float64)
    assert (w > 0).sum() > V // 8
    cdf = np.cumsum(w) / w.sum()
    # ends of a thread's four weights, of a wave's 256, of a segment's 4096; a third of the trials each
    ends = np.concatenate([rng.choice(np.arange(3, V - 4, 4), n_trials // 9, replace=False),
                           rng.choice(np.arange(255, V - 4, 256), n_trials // 9),
                           rng.choice(np.arange(4095, V - 4, 4096), n_trials // 9) if V > 8192 else
                           rng.choice(np.arange(3, V - 4, 4), n_trials // 9, replace=False)])
    us = []
    for k in ends:
        u0 = np.float32(cdf[k])
        us += [u0, np.nextafter(u0, np.float32(0)), np.nextafter(u0, np.float32(1))]
    us = np.clip(np.array(us, np.float32), np.float32(2.0 ** -24), np.float32(1.0 - 2.0 ** -24))
    us = np.concatenate([us, np.array([0.0, 2.0 ** -24, 1.0 - 2.0 ** -24], np.float32)])   # and the ends of the grid
    B = len(us)
    u = np.full((B, gamma + 1), 0.999, np.float32)   # (the candidate's own test: u = 0.999 against p / q <= 0.1)
    u[:, gamma] = us
    logits = np.broadcast_to(logits1, (B, gamma + 1, V)).copy()
    q = np.broadcast_to(q1, (B, gamma, V)).copy() if gamma else None
    cand = np.broadcast_to(cand1, (B, gamma)).copy() if gamma else None
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    na = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    nx = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    ws = torch.zeros(3 * B * (gamma + 1), device="cuda")
    api.sd_accept(dev(logits), gamma, T, dev(cand) if gamma else None, dev(q) if gamma else None, dev(u), na, nx, ws)
    torch.cuda.synchronize()
    na_h, nx_h = na.cpu().numpy(), nx.cpu().numpy()
    assert (na_h == 0).all()
    other = 0
    for b in range(B):
        ref = oracle.sample_cdf(w, float(us[b]))[0]
        if int(nx_h[b]) != ref:
            other += 1
            assert 0 <= nx_h[b] < V and w[nx_h[b]] > 0, (b, int(nx_h[b]), ref)
            d = oracle.cdf_distance(w, float(us[b]), int(nx_h[b]))
            assert d < 1e-5, (b, float(us[b]), int(nx_h[b]), ref, d)
    print(f"  {B} uniforms, {other} resolved to the neighbouring token", flush=True)


def row_verdict_case(V, gamma):
    """One sequence per place of the first rejection (none for the last); the rows behind it hold candidates that would be
    accepted, rejected or lie outside the vocabulary.  From gamma 2 on, two sequences reject a row whose q is twice p."""
    rng = np.random.default_rng(17 + V)
    B = gamma + 2
    logits = rng.normal(0, 2, (B, gamma + 1, V)).astype(np.float32)
    logits[:, :, V // 3] = -np.inf
    q = np.zeros((B, gamma, V), np.float32)
    cand = np.zeros((B, gamma), np.int32)
    u = np.full((B, gamma + 1), 0.25, np.float32)
    u[:, gamma] = dg.make_uniforms(23, dg.VERIFY_STREAM, 0, 0, B)
    for b in range(B):
        for i in range(gamma):
            p = oracle.softmax_T(logits[b, i], 1.0)
            c = int(np.argmax(p))
            q[b, i] = oracle.softmax_T((logits[b, i] + rng.normal(0, 1, V)).astype(np.float32), 1.0)
            q[b, i, c] = p[c] * np.float32(4.0 if i == b else 2.0)   # accepted below 1/4 or 1/2
            cand[b, i] = c
            if i == b:
                u[b, i] = 0.75
            elif i > b:
                cand[b, i] = (c, V, -1)[i % 3]
                u[b, i] = 0.9 if i % 2 else 0.25
    expect = [min(b, gamma) for b in range(B)]
    if gamma >= 2:
        for b, i in ((gamma, 0), (gamma + 1, 1)):
            q[b, i] = 2.0 * oracle.softmax_T(logits[b, i], 1.0)
            u[b, i] = 0.75
            expect[b] = i
    return logits, q, cand, u, expect


@pytest.mark.parametrize("V,gamma", [(4, 2), (1024, 15), (1028, 2), (2048, 4), (2052, 2), (4096, 3), (4100, 1), (8192, 2), (8196, 2), (16384, 2), (16388, 2),
                                     (32000, 5), (32768, 3)])
def test_every_row_of_a_sequence_decides_for_itself(V, gamma):
    """Rows that fit a block's registers: the verdicts of the rows behind the first rejection must not matter, and a
    rejection without residual mass draws from p."""
    print(f"row verdicts V={V} gamma={gamma}", flush=True)
    logits, q, cand, u, expect = row_verdict_case(V, gamma)
    B = len(expect)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    na, nx = (torch.full((B,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    ws = torch.full((3 * B * (gamma + 1),), float("nan"), device="cuda")
    api.sd_accept(dev(logits), gamma, 1.0, dev(cand), dev(q), dev(u), na, nx, ws)
    torch.cuda.synchronize()
    na_h, nx_h = na.cpu().numpy(), nx.cpu().numpy()
    assert na_h.tolist() == expect
    assert check_against_oracle(logits, q, cand, u, 1.0, na_h, nx_h) <= 1   # (a uniform next to an edge of the CDF)


@pytest.mark.parametrize("V,gamma,copies", [(32772, 15, 1), (40960, 4, 1), (40964, 4, 1), (65536, 3, 1), (65540, 3, 1), (131072, 3, 1), (131076, 3, 1),
                                            (131076, 1, 1), (66000, 3, 26), (64000, 3, 26), (44204, 3, 38)])
def test_wide_rows_decide_by_the_sign_of_their_sums(V, gamma, copies):
    """Rows of more than 32768 columns: verdicts of every row, candidates outside the vocabulary, an empty residual; slices of
    2048, 4096 and 8192 vectors and one more (the pick's register forms and the form without), more than 128 MB of logits
    (the nontemporal pass, in blocks of 256 threads at 520 and at 760 rows) and just less."""
    print(f"wide verdicts V={V} gamma={gamma} x{copies}", flush=True)
    logits, q, cand, u, expect = row_verdict_case(V, gamma)
    tile = lambda a: np.ascontiguousarray(np.concatenate([a] * copies))
    logits, q, cand, u, expect = tile(logits), tile(q), tile(cand), tile(u), expect * copies
    B = len(expect)
    u[:, gamma] = dg.make_uniforms(31, dg.VERIFY_STREAM, 0, 0, B)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    na, nx = (torch.full((B,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    ws = torch.full((3 * B * (gamma + 1),), float("nan"), device="cuda")
    api.sd_accept(dev(logits), gamma, 1.0, dev(cand), dev(q), dev(u), na, nx, ws)
    torch.cuda.synchronize()
    na_h, nx_h = na.cpu().numpy(), nx.cpu().numpy()
    assert na_h.tolist() == expect
    assert check_against_oracle(logits, q, cand, u, 1.0, na_h, nx_h) <= 1 + B // 50


@pytest.mark.parametrize("V,B,T", [(33000, 160, 1.1), (33000, 270, 1.3), (33000, 270, 0.6), (128000, 100, 1.0), (128000, 150, 1.1), (128000, 150, 2.0),
                                      (66004, 257, 1.1), (128000, 300, 0.7), (44004, 383, 1.3)])
def test_wide_rows_sum_their_exponentials_without_a_bias(V, B, T):
    """The sums wide rows leave in the workspace, against 64 bits at the factor 1 / T the kernel has (rounded to 32): their mean
    error over 2 B rows (above 128 MB of logits in blocks of 512 threads up to 511 rows, of 256 from 513 to 767).
    Roundings of the sums and of each exponential's argument have no preferred sign: 1e-7 rms a row and less, 6e-9 in the mean
    of 300 rows.  A factor log2(e) / T rounded once would put the same sign on every column, up to 2^-24
    of the mean of |x - max| / T weighted by the exponentials, 4 to 6 here: 7e-8 at T = 1.1, 3e-8 at 1.3."""
    print(f"wide sums V={V} B={B} T={T}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    x = 2.0 * torch.randn((B, 2, V), device="cuda", generator=g)
    cand, q = torch.zeros((B, 1), dtype=torch.int32, device="cuda"), torch.full((B, 1, V), 1.0 / V, device="cuda")
    na, nx = (torch.zeros(B, dtype=torch.int32, device="cuda") for _ in range(2))
    ws = torch.zeros(6 * B, device="cuda")
    api.sd_accept(x, 1, T, cand, q, torch.rand((B, 2), device="cuda", generator=g), na, nx, ws)
    s = float(np.float32(1.0) / np.float32(T))
    rows = x.view(2 * B, V)
    ref = torch.stack([torch.exp((r.double() - r.max().double()) * s).sum() for r in rows])
    err = ws.view(2 * B, 3)[:, 1].abs().double() / ref - 1.0
    assert float(err.square().mean().sqrt()) < 1.5e-7 and abs(float(err.mean())) < 2e-8, (err.square().mean().sqrt(), err.mean())


@pytest.mark.parametrize("V,gamma,copies", [(1024, 15, 1), (1028, 15, 1), (4096, 15, 1), (8192, 15, 1), (16384, 2, 22), (32000, 15, 1),
                                            (32768, 2, 22), (8192, 1, 44), (16384, 1, 44)])
def test_more_rows_than_compute_units(V, gamma, copies):
    """257 rows and more: from two candidates on one block per sequence draws behind the rows' tests, with one candidate
    every row draws for itself (both read q late).  Verdicts and draws of every sequence against the oracle."""
    print(f"many rows V={V} gamma={gamma}", flush=True)
    logits, q, cand, u, expect = row_verdict_case(V, gamma)
    tile = lambda a: np.ascontiguousarray(np.concatenate([a] * copies))
    logits, q, cand, u, expect = tile(logits), tile(q), tile(cand), tile(u), expect * copies
    B = len(expect)
    assert B * (gamma + 1) > 256
    u[:, gamma] = dg.make_uniforms(29, dg.VERIFY_STREAM, 0, 0, B)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    na, nx = (torch.full((B,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    ws = torch.full((3 * B * (gamma + 1),), float("nan"), device="cuda")
    api.sd_accept(dev(logits), gamma, 1.0, dev(cand), dev(q), dev(u), na, nx, ws)
    torch.cuda.synchronize()
    na_h, nx_h = na.cpu().numpy(), nx.cpu().numpy()
    assert na_h.tolist() == expect
    assert check_against_oracle(logits, q, cand, u, 1.0, na_h, nx_h) <= 1 + B // 50


@pytest.mark.parametrize("V", [1024, 1028, 32000, 32772, 100004])
def test_infinite_temperature_draws_from_the_uniform_distribution(V):
    """T = inf is the limit of the rule: p = 1 / V whatever the logits are, in rows that fit a block's registers and in
    wider ones.  Candidate i carries q = 2 / V or 8 / V against u = 1/4 (accepted, rejected); sequence b rejects at place b."""
    print(f"infinite temperature V={V}", flush=True)
    gamma, T = 3, float("inf")
    B = gamma + 2
    rng = np.random.default_rng(V)
    logits = rng.normal(0, 3, (B, gamma + 1, V)).astype(np.float32)
    cand = rng.integers(0, V, (B, gamma)).astype(np.int32)
    q = np.zeros((B, gamma, V), np.float32)
    u = np.full((B, gamma + 1), 0.25, np.float32)
    u[:, gamma] = [0.011, 0.27, 0.5003, 0.713, 0.986]
    for b in range(B):
        for i in range(gamma):
            q[b, i] = oracle.softmax_T(rng.normal(0, 1, V).astype(np.float32), 1.0)
            q[b, i, cand[b, i]] = np.float32((8.0 if i == b else 2.0) / V)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    na, nx = (torch.full((B,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    ws = torch.zeros(3 * B * (gamma + 1), device="cuda")
    api.sd_accept(dev(logits), gamma, T, dev(cand), dev(q), dev(u), na, nx, ws)
    torch.cuda.synchronize()
    na_h, nx_h = na.cpu().numpy(), nx.cpu().numpy()
    assert na_h.tolist() == [min(b, gamma) for b in range(B)]
    check_against_oracle(logits, q, cand, u, T, na_h, nx_h)
    # masked columns stay out of it: a draw from the first half alone, index u V / 2 (sums of V terms: 1e-6 of them)
    half = V // 2
    logits[:, 0, half:] = -np.inf
    api.sd_accept(dev(logits[:, :1]), 0, T, None, None, dev(u[:, gamma:]), na, nx, ws)
    torch.cuda.synchronize()
    assert np.abs(nx.cpu().numpy() - np.floor(u[:, gamma].astype(np.float64) * half)).max() <= 1 + 1e-6 * V


@pytest.mark.parametrize("T", [0.05, 0.7, 1.0, 40.0])
@pytest.mark.parametrize("V", [4, 260, 1028, 4096, 8192, 16384, 32764, 32772, 66000])
def test_masked_columns_carry_no_weight(V, T):
    """Rows whose columns are masked with -inf, the lowest float or -3e38: nothing masked is drawn,
    accepted or counted, and the draws agree with the oracle's on the same rows."""
    print(f"masked columns V={V} T={T}", flush=True)
    B, gamma = 6, 1
    rng = np.random.default_rng(V)
    logits = rng.normal(0, 2, (B, gamma + 1, V)).astype(np.float32)
    keep = rng.random((B, V)) < 0.4
    keep[:, V // 2] = True
    for b, mask in enumerate([-np.inf, np.finfo(np.float32).min, -3.0e38] * 2):
        logits[b, :, ~keep[b]] = mask
    cand = np.array([[int(np.flatnonzero(~keep[b])[0]) if b % 2 and not keep[b].all() else V // 2] for b in range(B)], np.int32)
    q = np.full((B, gamma, V), 1.0 / V, np.float32)
    u = np.stack([dg.make_uniforms(77, dg.VERIFY_STREAM, b, 0, gamma + 1) for b in range(B)])
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    na, nx = (torch.full((B,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    api.sd_accept(dev(logits), gamma, T, dev(cand), dev(q), dev(u), na, nx, torch.zeros(3 * B * (gamma + 1), device="cuda"))
    torch.cuda.synchronize()
    na_h, nx_h = na.cpu().numpy(), nx.cpu().numpy()
    for b in range(B):
        assert keep[b, nx_h[b]], (b, nx_h[b])
        assert na_h[b] == 0 or keep[b, cand[b, 0]]
    low = np.float32(-1.0e30)  # (the oracle's masks: far below everything else, and finite in its differences)
    assert check_against_oracle(np.maximum(logits, low), q, cand, u, T, na_h, nx_h) <= 1


@pytest.mark.parametrize("V,gamma,B", [(4, 1, 6), (1028, 1, 6), (20000, 1, 6), (1028, 1, 140), (20000, 1, 140), (1028, 2, 100), (20000, 2, 100)])
def test_a_negative_q_in_the_last_columns_adds_no_weight_past_the_row(V, gamma, B):
    """q = -0.5 in the last four columns: the token comes from max(0, p - q) over the row alone, in rows that read q early, late
    and in the draw per sequence, with most of the residual's mass in the row's last vector."""
    print(f"negative q V={V} gamma={gamma} B={B}", flush=True)
    rng = np.random.default_rng(V + B)
    logits = rng.normal(0, 2, (B, gamma + 1, V)).astype(np.float32)
    q = np.full((B, gamma, V), 1.0 / V, np.float32)
    q[:, :, V - 4:] = -0.5
    q[:, :, 0] = 1.0
    cand = np.zeros((B, gamma), np.int32)
    u = np.full((B, gamma + 1), 0.9999, np.float32)   # (above p / q of column 0: rejected)
    u[:, gamma] = rng.random(B).astype(np.float32)
    u[0, gamma], u[1, gamma] = 1.0 - 2.0 ** -24, 0.0
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    na, nx = (torch.full((B,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    api.sd_accept(dev(logits), gamma, 1.0, dev(cand), dev(q), dev(u), na, nx, torch.zeros(3 * B * (gamma + 1), device="cuda"))
    torch.cuda.synchronize()
    na_h, nx_h = na.cpu().numpy(), nx.cpu().numpy()
    assert (na_h == 0).all() and ((0 <= nx_h) & (nx_h < V)).all()
    assert check_against_oracle(logits, q, cand, u, 1.0, na_h, nx_h) <= 1


@pytest.mark.parametrize("dtype", [dg.FP32, dg.BF16])
def test_draft_at_infinite_temperature_is_uniform(dtype):
    """The samplers of the draft phase at T = inf: q = 1 / V and the candidate at u V, in both data types."""
    print(f"draft at infinite temperature dtype={dtype}", flush=True)
    shape = dg.ModelShape("t_inf", 1, 128, 2, 64, 384, 2048, dtype)
    m = api.Model(shape, dg.make_weights(shape, 3, 1.0), max_rows=16, max_pos=64)
    ctx = api.Context([32])
    ctx.attach(m)
    ctx.set_tokens([[5, 9, 77]])
    api.sd_prefill(m, ctx, None, 1, 2)
    u = np.array([[0.1, 0.77]], np.float32)
    cand = torch.zeros((1, 2), dtype=torch.int32, device="cuda")
    q = torch.zeros((1, 2, shape.vocab), device="cuda")
    api.sd_draft(m, ctx, None, 1, 2, float("inf"), torch.from_numpy(u).cuda(), cand, q)
    ctx.sync()
    assert np.abs(q.cpu().numpy() * shape.vocab - 1.0).max() < 1e-5
    assert np.abs(cand.cpu().numpy() - np.floor(u * shape.vocab)).max() <= 1
    ctx.close()
    m.close()


@pytest.mark.parametrize("V", [1024, 32000, 50000])
def test_greedy_rows_with_equal_maxima_take_the_lowest_index(V):
    """T = 0: every logits row holds its largest value two to four times, at positions in different threads, waves
    and 4096-column segments of the kernels' reductions; the arg max is the lowest of them (the oracle's rule), so
    a candidate equal to a later copy is rejected and the next token is the first copy."""
    print(f"greedy ties V={V}", flush=True)
    B, gamma = 12, 3
    rng = np.random.default_rng(V)
    logits = rng.standard_normal((B, gamma + 1, V)).astype(np.float32)
    cand = np.zeros((B, gamma), np.int32)
    first = np.zeros((B, gamma + 1), np.int64)
    for b in range(B):
        for i in range(gamma + 1):
            k = int(rng.integers(2, 5))
            lo = int(rng.integers(0, V - 1))
            pos = {lo, min(V - 1, lo + int(rng.choice([1, 3, 4, 255, 256, 4095, 4096])))}
            while len(pos) < k:
                pos.add(int(rng.integers(lo, V)))
            pos = sorted(pos)
            logits[b, i, pos] = 9.0
            first[b, i] = pos[0]
            if i < gamma:   # even sequences propose the first copy (accepted), odd ones a later copy (rejected)
                cand[b, i] = pos[0] if (b + i) % 2 == 0 else pos[-1]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    na = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    nx = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    ws = torch.zeros(3 * B * (gamma + 1), device="cuda")
    api.sd_accept(dev(logits), gamma, 0.0, dev(cand), None, None, na, nx, ws)
    torch.cuda.synchronize()
    na_h, nx_h = na.cpu().numpy(), nx.cpu().numpy()
    for b in range(B):
        r_na, r_nx, _ = oracle.accept(logits[b], None, cand[b], np.zeros(gamma + 1, np.float32), 0.0)
        want_na = next((i for i in range(gamma) if cand[b, i] != first[b, i]), gamma)
        assert (r_na, r_nx) == (want_na, int(first[b, want_na]))          # the oracle follows the stated rule
        assert (int(na_h[b]), int(nx_h[b])) == (r_na, r_nx), (b, int(na_h[b]), int(nx_h[b]), r_na, r_nx)
    assert len(set(na_h.tolist())) >= 2


def test_accept_argument_errors():
    L = api.lib()
    x = torch.zeros(8, device="cuda")
    i = torch.zeros(8, dtype=torch.int32, device="cuda")
    p = lambda t: t.data_ptr()
    assert L.sd_accept(None, 1, 1, 8, 1.0, p(i), p(x), p(x), p(i), p(i), p(x), None) == api.SD_EINVAL
    assert L.sd_accept(p(x), 1, 16, 8, 1.0, p(i), p(x), p(x), p(i), p(i), p(x), None) == api.SD_ECAP
    assert L.sd_accept(p(x), 1, 1, 6, 1.0, p(i), p(x), p(x), p(i), p(i), p(x), None) == api.SD_EINVAL
    assert L.sd_accept(p(x), 1, 1, 8, 1.0, p(i), None, p(x), p(i), p(i), p(x), None) == api.SD_EINVAL
    assert L.sd_accept(p(x), 1, 1, 8, 1.0, p(i), p(x), p(x), p(i), p(i), None, None) == api.SD_EINVAL


@pytest.mark.parametrize("nt", [1, 0])
def test_stream_read_probe_reads_every_word_exactly_once(nt):
    """In its checking mode the read probe folds every 32-bit word it reads into the scratch word with XOR: the
    result equals the XOR of the buffer iff both patterns cover every 16-byte vector exactly once, for sizes on
    and off the grid's granularity; and in measuring mode the word is left alone."""
    print(f"stream read probe, nontemporal pattern = {nt}", flush=True)
    try:
        rng = np.random.default_rng(7)
        for n_words in (4, 4 * 255, 4 * 2048 + 4, 4 * 65536 * 3 + 12, 1 << 22):
            w = rng.integers(0, 1 << 32, n_words, dtype=np.uint64).astype(np.uint32)
            buf = torch.from_numpy(w.view(np.int32)).cuda()
            word = torch.zeros(1, dtype=torch.int32, device="cuda")
            api.set_option("stream_read_nt", nt + 2)
            api.stream_read(buf, word)
            torch.cuda.synchronize()
            assert int(word.item()) & 0xffffffff == int(np.bitwise_xor.reduce(w)), f"{n_words} words: a vector was skipped or read twice"
            api.set_option("stream_read_nt", nt)
            word.zero_()
            api.stream_read(buf, word)
            torch.cuda.synchronize()
            assert int(word.item()) == 0
    finally:
        api.set_option("stream_read_nt", 1)


@pytest.mark.parametrize("rows,V", [(257, 131076), (511, 66004), (512, 66004), (513, 66004), (767, 44004), (768, 44004)])
def test_wide_greedy_rows_at_the_edges_of_each_block_shape(rows, V):
    """More than 128 MB of logits, row counts on both sides of the block shapes' limits: the first of equal maxima is taken, also
    where they lie in different threads, waves and loads of a row, in its first and its last vector."""
    print(f"wide greedy rows={rows} V={V}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(11)
    x = torch.randn((rows, 1, V), device="cuda", generator=g)
    at = torch.randint(0, V, (rows, 3), device="cuda", generator=g)
    at[0, 0], at[1, :], at[2, 0] = 0, V - 1, 1023
    x[:, 0].scatter_(1, at, 9.0)
    x[3, 0] = -1.0e30
    na, nx = (torch.full((rows,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    ws = torch.full((3 * rows,), float("nan"), device="cuda")
    api.sd_accept(x, 0, 0.0, None, None, None, na, nx, ws)
    expect = at.min(dim=1).values
    expect[3] = 0
    assert (na == 0).all() and (nx.long() == expect).all()
