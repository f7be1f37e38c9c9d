"""GPU parity of the accept/reject kernels and the device Philox stream against the oracle, fed
identical logits and uniforms through the C ABI."""
import numpy as np
import pytest

import synth
from oracle import philox as ophilox, spec as ospec

pytestmark = pytest.mark.gpu


def _logits(B, k, V, seed, agree=0.6):
    rng = np.random.default_rng(seed)
    p = (rng.standard_normal((B, k + 1, V)) * 2.0).astype(np.float32)
    q = (p[:, :k] + rng.standard_normal((B, k, V)).astype(np.float32) * 1.0).astype(np.float32)
    d = np.argmax(p[:, :k], axis=-1).astype(np.int32)
    flip = rng.random((B, k)) > agree
    d[flip] = rng.integers(0, V, flip.sum())
    return p, q, d


# vocabularies of up to 32768 ids that are a multiple of 4 take the register-resident kernels (each row
# read once); 33 and 40000 take the general ones
@pytest.mark.parametrize("B,k,V", [(7, 4, 512), (3, 8, 32000), (1, 1, 33), (5, 0, 100), (64, 6, 32768),
                                   (4, 3, 40000), (3, 2, 12), (5, 16, 32768), (3, 16, 1001), (300, 2, 256),
                                   (300, 6, 4096), (300, 6, 4095)])
def test_accept_greedy(B, k, V):
    import torch
    import paper_2505_10259_amd as P
    from gpu_common import dev
    p, _, d = _logits(B, k, V, seed=B * 100 + k)
    if k > 0 and B > 2:                          # exact ties: lowest id must win on both sides
        p[0, 0, 5] = p[0, 0].max() + 1; p[0, 0, 9] = p[0, 0, 5]; d[0, 0] = 5
        p[1, 0, 11] = p[1, 0].max() + 1; p[1, 0, 3] = p[1, 0, 11]; d[1, 0] = 11
    n = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    nx = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    P.spec_accept(dev(p), None, dev(d) if k else None, None, None, 1.0, 0, 0, 0, B, k, V, n, nx)
    torch.cuda.synchronize()
    exp = [ospec.accept_greedy(p[b], d[b]) for b in range(B)]
    assert n.cpu().tolist() == [e[0] for e in exp]
    assert nx.cpu().tolist() == [e[1] for e in exp]


@pytest.mark.parametrize("B,k,V,tau", [(16, 4, 512, 0.8), (6, 6, 32000, 0.8), (4, 1, 17, 1.3), (32, 3, 1000, 0.5),
                                       (8, 3, 32768, 0.8), (4, 2, 40000, 0.8), (5, 1, 256, 1.0),
                                       (4, 16, 32768, 0.8), (4, 16, 1001, 0.9)])
def test_accept_sample_given_uniforms(B, k, V, tau):
    import torch
    import paper_2505_10259_amd as P
    from gpu_common import dev
    p, q, _ = _logits(B, k, V, seed=7 * B + k)
    ud = synth.make_uniforms((B, k), seed=1)
    ua = synth.make_uniforms((B, k), seed=2)
    ur = synth.make_uniforms((B, k + 1), seed=3)
    # candidates are genuine draws from the draft rows
    d = np.array([[ospec.sample_inverse_cdf(ospec.softmax_t(q[b, i], tau), ud[b, i]) for i in range(k)]
                  for b in range(B)], dtype=np.int32)
    if B >= 4:
        q[0] = p[0, :k]                          # q == p: everything kept, bonus token from p_k
        d[0] = [ospec.sample_inverse_cdf(ospec.softmax_t(q[0, i], tau), ud[0, i]) for i in range(k)]
    n = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    nx = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    P.spec_accept(dev(p), dev(q), dev(d), dev(ua), dev(ur), tau, 0, 0, 0, B, k, V, n, nx)
    torch.cuda.synchronize()
    n, nx = n.cpu().numpy(), nx.cpu().numpy()
    exempt = 0
    for b in range(B):
        margins = []
        en, enx = ospec.accept_sample(p[b], q[b], d[b], ua[b], ur[b], tau, margins=margins)
        if n[b] != en:
            assert min(margins) < 1e-4, f"kept count differs at row {b} without a near-tie"
            exempt += 1
            continue
        if nx[b] != enx:
            # only a CDF-boundary near-tie may move the draw, and then only to a neighbouring id
            pr = ospec.softmax_t(p[b, en], tau)
            r = np.maximum(0, pr - ospec.softmax_t(q[b, en], tau)) if en < k else pr
            if r.sum() <= 0:
                r = pr
            c = np.cumsum(r) / r.sum()
            assert np.abs(c - ur[b, en]).min() < 1e-5, f"next token differs at row {b} away from a CDF edge"
            exempt += 1
    assert exempt <= max(1, B // 8)
    if B >= 4:
        assert n[0] == k


def test_accept_sample_internal_philox_matches_oracle_stream():
    import torch
    import paper_2505_10259_amd as P
    from gpu_common import dev
    B, k, V, tau, seed, rnd, base = 9, 5, 700, 0.8, 0x1234567ABCDEF, 3, 40
    out = torch.zeros((B, k + 1, 3), dtype=torch.float32, device="cuda")
    P.spec_philox_uniforms(seed, rnd, base, B, k, out)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    for b in range(B):
        ud, ua, ur = ophilox.round_uniforms(seed, rnd, base + b, k)
        assert np.array_equal(got[b, :, 0], ud.astype(np.float32))
        assert np.array_equal(got[b, :, 1], ua.astype(np.float32))
        assert np.array_equal(got[b, :, 2], ur.astype(np.float32))
    p, q, _ = _logits(B, k, V, seed=5)
    d = np.zeros((B, k), dtype=np.int32)
    exp = []
    for b in range(B):
        ud, ua, ur = ophilox.round_uniforms(seed, rnd, base + b, k)
        d[b] = [ospec.sample_inverse_cdf(ospec.softmax_t(q[b, i], tau), ud[i + 1]) for i in range(k)]
        exp.append(ospec.accept_sample(p[b], q[b], d[b], ua[1:], ur, tau))
    n = torch.zeros(B, dtype=torch.int32, device="cuda")
    nx = torch.zeros(B, dtype=torch.int32, device="cuda")
    P.spec_accept(dev(p), dev(q), dev(d), None, None, tau, seed, rnd, base, B, k, V, n, nx)
    torch.cuda.synchronize()
    agree = sum(int(a == e[0] and c == e[1]) for a, c, e in zip(n.cpu().tolist(), nx.cpu().tolist(), exp))
    assert agree >= B - 1


def test_accept_sample_distribution_chi_square():
    """Tiny vocabulary, context-free p and q, device Philox: emitted tokens follow the target."""
    import torch
    from scipy import stats
    import paper_2505_10259_amd as P
    from gpu_common import dev
    V, k, tau, B = 12, 4, 0.8, 20000
    rng = np.random.default_rng(1)
    pz, qz = rng.standard_normal(V) * 1.5, rng.standard_normal(V) * 1.5
    pr, qr = ospec.softmax_t(pz, tau), ospec.softmax_t(qz, tau)
    p = np.tile(pz.astype(np.float32), (B, k + 1, 1))
    q = np.tile(qz.astype(np.float32), (B, k, 1))
    d = rng.choice(V, size=(B, k), p=ospec.softmax_t(qz.astype(np.float32), tau)).astype(np.int32)
    n = torch.zeros(B, dtype=torch.int32, device="cuda")
    nx = torch.zeros(B, dtype=torch.int32, device="cuda")
    P.spec_accept(dev(p), dev(q), dev(d), None, None, tau, 99, 0, 0, B, k, V, n, nx)
    torch.cuda.synchronize()
    n, nx = n.cpu().numpy(), nx.cpu().numpy()
    emitted = np.concatenate([np.concatenate([d[b, :n[b]], [nx[b]]]) for b in range(B)])
    obs = np.bincount(emitted, minlength=V)
    chi2, pval = stats.chisquare(obs, pr * len(emitted))
    assert pval > 0.01, (chi2, pval)
    alpha = np.minimum(pr, qr).sum()
    assert abs((n + 1).mean() - ospec.expected_generated(alpha, k)) < 4 * (n + 1).std() / np.sqrt(B)


@pytest.mark.parametrize("V", [512, 40000])        # register-resident and general kernels
def test_candidate_outside_the_vocabulary_is_rejected(V):
    """An id that is no token (V, a negative number) must never index the probability rows: the
    sampling rule treats it as rejected at its position, the greedy rule as a mismatch."""
    import torch
    import paper_2505_10259_amd as P
    from gpu_common import dev
    B, k, tau = 4, 3, 0.8
    p, q, _ = _logits(B, k, V, seed=V)
    q[:] = p[:, :k]                              # q == p: every genuine candidate is kept
    ud = synth.make_uniforms((B, k), seed=11)
    d = np.array([[ospec.sample_inverse_cdf(ospec.softmax_t(q[b, i], tau), ud[b, i]) for i in range(k)]
                  for b in range(B)], dtype=np.int32)
    d[0, 1], d[1, 0], d[2, 2] = V, -7, V + 12345
    ua = synth.make_uniforms((B, k), seed=12)
    ur = synth.make_uniforms((B, k + 1), seed=13)
    for q_dev in (dev(q), None):
        n = torch.full((B,), -1, dtype=torch.int32, device="cuda")
        nx = torch.full((B,), -1, dtype=torch.int32, device="cuda")
        if q_dev is None:
            dd = np.argmax(p[:, :k], axis=-1).astype(np.int32)      # greedy: the target's own choices ...
            dd[0, 1], dd[1, 0], dd[2, 2] = V, -7, V + 12345         # ... except the invalid ids
            P.spec_accept(dev(p), None, dev(dd), None, None, 1.0, 0, 0, 0, B, k, V, n, nx)
        else:
            P.spec_accept(dev(p), q_dev, dev(d), dev(ua), dev(ur), tau, 0, 0, 0, B, k, V, n, nx)
        torch.cuda.synchronize()
        assert n.cpu().tolist() == [1, 0, 2, 3]
        assert all(0 <= t < V for t in nx.cpu().tolist())


# candidates tested one workgroup each and one after the other, on either side of the lines between the two and between
# the kernels for short and long rows; rows at every alignment
# (V mod 4 = 0..3), one id short of and past a run of the inverse-CDF search, runs of more than one granule per lane
@pytest.mark.parametrize("B,k,V,tau", [(4, 2, 65537, 0.8), (4, 3, 300001, 0.8), (4, 2, 262142, 0.8), (4, 2, 262147, 1.0),
                                       (100, 3, 512, 0.8), (90, 4, 1001, 0.8), (64, 4, 1003, 0.8), (5, 16, 4098, 0.8),
                                       (260, 1, 64, 0.8), (4, 1, 3, 0.8), (4, 2, 1, 0.8), (5, 2, 3071, 0.8), (5, 2, 3073, 0.8),
                                       (5, 6, 2047, 0.8), (5, 6, 2049, 0.8), (3, 6, 6143, 0.8), (3, 6, 6145, 0.8), (4, 3, 262147, 1.0),
                                       (200, 4, 1021, 0.8), (100, 1, 512, 0.8), (101, 1, 512, 0.8), (100, 2, 8190, 0.8),
                                       (101, 2, 8190, 0.8), (4, 16, 32000, 0.8), (3, 1, 8191, 0.8)])
def test_accept_sample_wide_rows_and_both_test_orders(B, k, V, tau):
    import torch
    import paper_2505_10259_amd as P
    from gpu_common import dev
    test_accept_sample_given_uniforms(B, k, V, tau)
    # without n_accepted the candidates are tested in turn: same next tokens
    p, q, d = _logits(B, k, V, seed=3 * B + V)
    p, q, d = dev(p), dev(q), dev(d)
    out = []
    for n in (torch.full((B,), -1, dtype=torch.int32, device="cuda"), None):
        nx = torch.full((B,), -1, dtype=torch.int32, device="cuda")
        P.spec_accept(p, q, d, None, None, tau, 5, 1, 0, B, k, V, n, nx)
        torch.cuda.synchronize()
        out.append(nx)
    assert torch.equal(out[0], out[1])


# edges of the row kernels: granules that the row ends in, one wavefront's and one workgroup's granules and one id more, workgroups of 256 and
# 512 threads (at once 8192 ids, in turn 24576), rows at once and in turn (3072 ids, four candidates, 32 and 128 sequences)
@pytest.mark.parametrize("B,k,V,tau", [(4, 2, 4, 0.8), (4, 2, 5, 0.8), (4, 2, 7, 0.8), (4, 2, 257, 0.8), (4, 2, 1023, 0.8), (4, 2, 1025, 0.8),
                                       (4, 2, 4097, 0.8), (4, 3, 24576, 0.8), (4, 3, 24577, 0.8), (4, 2, 24579, 0.8), (4, 2, 131073, 0.8),
                                       (127, 3, 130, 0.8), (128, 3, 130, 0.8), (128, 4, 130, 0.8),
                                       (4, 5, 4, 0.8), (4, 5, 5, 0.8), (4, 5, 7, 0.8), (4, 5, 257, 0.8), (4, 5, 1023, 0.8), (4, 5, 1025, 0.8),
                                       (31, 5, 130, 0.8), (32, 5, 130, 0.8), (8, 5, 3072, 0.8), (8, 4, 3073, 0.8), (127, 4, 3074, 0.8),
                                       (128, 4, 3074, 0.8), (128, 5, 3074, 0.8), (4, 3, 8192, 0.8), (4, 3, 8193, 0.8)])
def test_accept_sample_row_kernels(B, k, V, tau):
    test_accept_sample_wide_rows_and_both_test_orders(B, k, V, tau)


# greedy rows at once (from 4097 ids and three candidates on, over 32768 ids two; up to 8 M ids) and, without n_accepted, in turn
@pytest.mark.parametrize("B,k,V", [(5, 2, 4097), (5, 2, 4098), (5, 2, 4100), (5, 3, 8195), (3, 2, 65537), (5, 1, 8195), (40, 16, 4100),
                                   (300, 16, 4112), (5, 3, 4097), (5, 3, 4098), (5, 3, 4099), (5, 3, 4100), (3, 2, 32768), (3, 2, 32769),
                                   (120, 16, 4112), (121, 16, 4112)])
def test_accept_greedy_at_once_and_in_turn(B, k, V):
    import torch
    import paper_2505_10259_amd as P
    from gpu_common import dev
    test_accept_greedy(B, k, V)
    p, _, d = _logits(B, k, V, seed=V, agree=0.9)
    p[:, :, V - 1] = p.max(-1) * (np.arange(B) % 3 == 0)[:, None]              # the last id, of equal value, wins over none
    exp = [ospec.accept_greedy(p[b], d[b]) for b in range(B)]
    p, d = dev(p), dev(d)
    for n in (torch.full((B,), -1, dtype=torch.int32, device="cuda"), None):
        nx = torch.full((B,), -1, dtype=torch.int32, device="cuda")
        P.spec_accept(p, None, d, None, None, 1.0, 0, 0, 0, B, k, V, n, nx)
        torch.cuda.synchronize()
        assert nx.cpu().tolist() == [e[1] for e in exp]
        if n is not None:
            assert n.cpu().tolist() == [e[0] for e in exp]


# rows at once (from three candidates on), a wavefront per row (1001) and, without n_accepted or of one or two candidates, in turn
@pytest.mark.parametrize("bad", [float("nan"), -float("inf")])
@pytest.mark.parametrize("B,k,V", [(9, 2, 4097), (9, 3, 4097), (9, 16, 4097), (9, 2, 32000), (9, 16, 32000), (9, 3, 65537), (9, 1, 32000), (9, 4, 1001)])
def test_greedy_row_without_a_number_keeps_nothing(B, k, V, bad):
    """A row that is -inf or not-a-number throughout keeps no candidate, whatever the rows behind it say, and its token is 0."""
    import torch
    import paper_2505_10259_amd as P
    g = torch.Generator("cuda").manual_seed(V + k)
    p = torch.randn(B, k + 1, V, device="cuda", generator=g)
    p[:, :, 0] = -5.0                            # (no other row's choice)
    d = p[:, :k].argmax(-1).to(torch.int32).contiguous()
    tokens = p.argmax(-1)
    row = [0, k // 2, k - 1, k, None]            # the bad row of each sequence: first, middle, last candidate's, the one behind them, none
    exp = []
    for b in range(B):
        r = row[b % 5]
        if r is not None:
            p[b, r] = bad
        if b == 8:                               # no good row at all
            p[b], r = bad, 0
        if b == 5:                               # the bad row's candidate is the number that says so inside the kernels
            d[b, 0] = 0x7fffffff
        exp.append((k, tokens[b, k].item()) if r is None else (r, 0))
    for n in (torch.full((B,), -1, dtype=torch.int32, device="cuda"), None):
        nx = torch.full((B,), -1, dtype=torch.int32, device="cuda")
        P.spec_accept(p, None, d, None, None, 1.0, 0, 0, 0, B, k, V, n, nx)
        torch.cuda.synchronize()
        assert nx.cpu().tolist() == [e[1] for e in exp]
        if n is not None:
            assert n.cpu().tolist() == [e[0] for e in exp]


@pytest.mark.parametrize("vocab", [512, 4100])
def test_greedy_round_of_a_model_without_numbers_commits_tokens_of_the_vocabulary(vocab):
    """An LM head of not-a-numbers: every round of both models commits one token 0 per sequence and counts no kept candidate."""
    import paper_2505_10259_amd as P
    from gpu_common import GpuDecode, host_model_pinned
    from synth import ModelShape
    hm = host_model_pinned(ModelShape(2, 256, 4, 4, 64, 512, vocab, dtype="f32"))
    hm.globals()["head"][:] = np.nan
    prompts = synth.make_prompts(3, (5, 9), vocab, seed=1)
    g = GpuDecode(hm, 1, False, prompts, 4, 6)
    rounds = g.run(want_logits=False)
    stats = P.spec_get_stats(g.s.ctx)
    assert all((r["draft"] == 0).all() and (r["n_acc"] == 0).all() and (r["next"] == 0).all() for r in rounds)
    # (the first of the 6 tokens may come with the prefill)
    assert g.generated() == [[0] * 6] * 3
    assert sum(stats["accept_hist"][1:]) == 0
    g.close()


# rows at once, in turn (without n_accepted) and, for fewer than four ids, a thread per sequence
@pytest.mark.parametrize("V,B", [(3, 4096), (4, 4096), (8, 4096), (32, 4096), (1001, 512), (9001, 256), (32000, 256), (65537, 128)])
@pytest.mark.parametrize("tau", [0.8, 1.0])
def test_draw_from_rows_that_are_equal_up_to_rounding(V, B, tau):
    """The draft's row is the target's plus a constant, or with one logit a unit in the last place up: the residual is rounding, or nothing
    at all.  A candidate outside the vocabulary forces the draw, which must give an id of positive target probability, and for one
    pair of rows must not fall while u rises."""
    import torch
    import paper_2505_10259_amd as P
    g = torch.Generator("cuda").manual_seed(V)
    masked = torch.arange(V, device="cuda") % 3 == 0          # id 0 among them
    for same in (False, True):                                # a pair of rows each; one pair for all
        p = (torch.randn(1 if same else B, 1, V, device="cuda", generator=g) * 2).masked_fill(masked, -float("inf"))
        up = p.clone()
        up[:, 0, V - 1 - int(masked[V - 1])] = torch.nextafter(p[:, 0, V - 1 - int(masked[V - 1])], torch.tensor(9.0, device="cuda"))
        for q in (p + 0.37, p + torch.rand(p.shape[0], 1, 1, device="cuda", generator=g) * 3, up):
            pb = p.expand(B, 1, V).repeat(1, 2, 1).contiguous()
            qb = q.expand(B, 1, V).contiguous()
            d = torch.full((B, 1), V, dtype=torch.int32, device="cuda")
            ua = torch.full((B, 1), 0.5, device="cuda")
            ur = ((torch.arange(B, device="cuda") + 0.5) / B).reshape(B, 1).repeat(1, 2).contiguous()
            for n in (torch.full((B,), -1, dtype=torch.int32, device="cuda"), None):
                nx = torch.full((B,), -1, dtype=torch.int32, device="cuda")
                P.spec_accept(pb, qb, d, ua, ur, tau, 0, 0, 0, B, 1, V, n, nx)
                torch.cuda.synchronize()
                t = nx.cpu().long()
                assert ((t >= 0) & (t < V)).all() and not masked.cpu()[t].any(), (V, tau, same)
                if n is not None:
                    assert (n == 0).all()
                if same:
                    assert (t[1:] >= t[:-1]).all(), (V, tau)


@pytest.mark.parametrize("V", [512, 4096, 40001])
def test_weights_below_the_smallest_normal_number_are_drawn(V):
    """A bonus row whose first id has the weight exp(x), subnormal, and whose last has 1, a long way behind: id 0 is drawn exactly while
    u < exp(x) (the total is 1 in f32).  u half and twice the weight."""
    import torch
    import paper_2505_10259_amd as P
    B = 64
    x = torch.linspace(-101.0, -87.5, B, dtype=torch.float64).float()
    p = torch.full((B, 2, V), -float("inf"), device="cuda")
    p[:, 0, 1] = 0.0                             # the candidate, token 1, is certain on both sides: kept
    q = p[:, :1].contiguous()
    p[:, 1, 0], p[:, 1, V - 1] = x.cuda(), 0.0
    d = torch.ones(B, 1, dtype=torch.int32, device="cuda")
    ua = torch.full((B, 1), 0.5, device="cuda")
    for factor, token in ((0.5, 0), (2.0, V - 1)):
        u = (x.double().exp() * factor).float().cuda().reshape(B, 1).repeat(1, 2).contiguous()
        for n in (torch.zeros(B, dtype=torch.int32, device="cuda"), None):
            nx = torch.full((B,), -1, dtype=torch.int32, device="cuda")
            P.spec_accept(p, q, d, ua, u, 1.0, 0, 0, 0, B, 1, V, n, nx)
            torch.cuda.synchronize()
            assert nx.cpu().tolist() == [token] * B, factor


@pytest.mark.parametrize("rows", ["random", "far"])
@pytest.mark.parametrize("tau", [0.8, 1.0, 1.3])
@pytest.mark.parametrize("V", [300, 4097, 32000, 65537, 131073])
def test_normaliser_error_at_any_length(V, tau, rows):
    """1 / normaliser as in test_normaliser_error, of random rows and of rows of one large logit and many equal ones far below it.  Bound in
    units of 2^-24, of the value: an exponential (1.8, the library's), four levels of sums inside a step, one rounding of the thread's sum and its
    corrections, an exponential and a product where threads and wavefronts meet (twice), six levels of lanes, the wavefronts one behind the other,
    one for the division and one for the quotient that u is compared with: whatever the length.  On average (of 64) rounding takes no more than
    a sixth of that."""
    import torch
    import paper_2505_10259_amd as P
    B = 64
    g = torch.Generator("cuda").manual_seed(V)
    if rows == "random":
        p = torch.randn(B, 2, V, device="cuda", generator=g) * 3
    else:
        p = (-torch.rand(B, 1, 1, device="cuda", generator=g) * 4 - float(np.log(V)) + 1).expand(B, 2, V).contiguous()
        p[:, :, V // 3] = 0.0
    d = p[:, :1].argmax(-1).to(torch.int32).contiguous()
    q = torch.full((B, 1, V), -float("inf"), device="cuda").scatter_(2, d.long().unsqueeze(-1), 0.0)
    n = torch.empty(B, dtype=torch.int32, device="cuda")
    nx = torch.empty(B, dtype=torch.int32, device="cuda")
    ur = torch.full((B, 2), 0.5, device="cuda")
    lo = torch.zeros(B, dtype=torch.int32, device="cuda")
    hi = torch.full((B,), 0x3f800000, dtype=torch.int32, device="cuda")
    for _ in range(31):
        mid = lo + (hi - lo) // 2
        P.spec_accept(p, q, d, mid.view(torch.float32).reshape(B, 1).contiguous(), ur, tau, 0, 0, 0, B, 1, V, n, nx)
        torch.cuda.synchronize()
        lo, hi = torch.where(n == 1, mid, lo), torch.where(n == 1, hi, mid)
    z = p[:, 0].double()                         # (torch's softmax of doubles is off by several units of 2^-24 itself)
    ref = 1.0 / torch.exp((z - z.max(-1, keepdim=True).values) * float(np.float32(1.0) / np.float32(tau))).sum(-1)
    err = (hi.view(torch.float32).double() / ref - 1).abs() * 2 ** 24
    bound = 1.8 + 4 + 1 + 2 * 2.8 + 6 + 8 + 2
    assert err.max().item() <= bound and err.mean().item() <= bound / 6, (err.max().item(), err.mean().item())


# each at most 0.7 of its time at once
@pytest.mark.parametrize("B,k,V,greedy", [(64, 4, 1001, False), (256, 4, 32000, False), (64, 8, 32000, True), (24, 5, 65537, True), (100, 2, 9001, True)])
def test_drafts_of_which_nothing_is_kept_cost_what_their_first_rows_cost(B, k, V, greedy):
    """Calls that rows at once slow down most where the first candidate is rejected are as fast as in turn (without n_accepted): a quarter of
    the time is left for the clock."""
    import torch
    import paper_2505_10259_amd as P
    g = torch.Generator("cuda").manual_seed(V)
    p = torch.randn(B, k + 1, V, device="cuda", generator=g)
    best = p[:, :k].argmax(-1).to(torch.int32)
    d = ((best + 1) % V).to(torch.int32) if greedy else best
    q = None if greedy else p[:, :k].contiguous().scatter_(2, d.long().unsqueeze(-1), 40.0)
    ua = None if greedy else torch.full((B, k), 0.9999, device="cuda")
    ur = None if greedy else torch.rand(B, k + 1, device="cuda", generator=g)
    nx = torch.zeros(B, dtype=torch.int32, device="cuda")
    n = torch.zeros(B, dtype=torch.int32, device="cuda")
    st = torch.cuda.Stream()
    us = {}
    for key, count in (("rule", n), ("turn", None)):
        call = lambda: P.spec_accept(p, q, d, ua, ur, 1.0, 0, 0, 0, B, k, V, count, nx, st.cuda_stream)
        torch.cuda.synchronize()
        call()
        st.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            for _ in range(20):
                call()
        times = []
        for _ in range(6):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            with torch.cuda.stream(st):
                e0.record()
                graph.replay()
                e1.record()
            st.synchronize()
            times.append(e0.elapsed_time(e1))
        us[key] = min(times) * 50
    assert (n == 0).all()
    assert us["rule"] <= 1.25 * us["turn"], us


@pytest.mark.parametrize("V,ahead", [(300, True), (9001, True), (24577, True), (65537, True), (9001, False)])
def test_normaliser_error(V, ahead):
    """With a draft row of one id the candidate is kept exactly while u < p(c), so bisecting u gives p(c) to the bit; the id of the largest
    logit makes it 1 / normaliser.  Bound in units of 2^-24: a sum behind another in a thread (16 ids a step) and in the reduction over
    lanes and wavefronts, each rounded once, three levels inside a step, half a unit for the rounded exponent of weights that average
    over the row, one for the division."""
    import torch
    import paper_2505_10259_amd as P
    B, T = 8, 256 if V <= 24576 else 512
    g = torch.Generator("cuda").manual_seed(V)
    p = torch.randn(B, 2, V, device="cuda", generator=g) * 3
    d = p[:, :1].argmax(-1).to(torch.int32).contiguous()
    q = torch.full((B, 1, V), -float("inf"), device="cuda").scatter_(2, d.long().unsqueeze(-1), 0.0)
    n = torch.empty(B, dtype=torch.int32, device="cuda") if ahead else None
    nx = torch.empty(B, dtype=torch.int32, device="cuda")
    ur = torch.full((B, 2), 0.5, device="cuda")
    # (in turn there is no count: behind a kept candidate the draw is of a row that is all token 0, behind a rejected one never token 0)
    p[:, 1] = -float("inf")
    p[:, 1, 0] = 0.0
    p[:, 0, 0] = -float("inf")
    lo = torch.zeros(B, dtype=torch.int32, device="cuda")
    hi = torch.full((B,), 0x3f800000, dtype=torch.int32, device="cuda")
    for _ in range(31):
        mid = lo + (hi - lo) // 2
        P.spec_accept(p, q, d, mid.view(torch.float32).reshape(B, 1).contiguous(), ur, 0.8, 0, 0, 0, B, 1, V, n, nx)
        torch.cuda.synchronize()
        kept = n == 1 if ahead else nx == 0
        lo, hi = torch.where(kept, mid, lo), torch.where(kept, hi, mid)
    got = hi.view(torch.float32).double()
    ref = torch.softmax(p[:, 0].double() * float(np.float32(1.0) / np.float32(0.8)), -1).max(-1).values
    bound = -(-V // (16 * T)) + 6 + (T // 64) + 3 + 0.5 + 1
    assert ((got / ref - 1).abs() * 2 ** 24).max().item() <= bound


@pytest.mark.parametrize("V", [512, 4000, 40001])        # (512: in turn)
def test_accept_at_once_under_capture(V):
    """The outputs are the meeting point of the workgroups of a sequence: every replay starts it afresh, whatever they hold."""
    import torch
    import paper_2505_10259_amd as P
    from gpu_common import dev
    B, k = 7, 4
    p, q, d = (dev(x) for x in _logits(B, k, V, seed=0))
    n = torch.zeros(B, dtype=torch.int32, device="cuda")
    nx = torch.zeros_like(n)
    n1, nx1 = torch.zeros_like(n), torch.zeros_like(n)
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        P.spec_accept(p, q, d, None, None, 0.8, 5, 1, 0, B, k, V, n, nx, torch.cuda.current_stream().cuda_stream)
    for seed in range(4):
        for t, x in zip((p, q, d), _logits(B, k, V, seed=seed)):
            t.copy_(dev(x))
        n.fill_(12345)
        nx.fill_(seed - 2)
        P.spec_accept(p, q, d, None, None, 0.8, 5, 1, 0, B, k, V, None, nx1)          # in turn
        P.spec_accept(p, q, d, None, None, 0.8, 5, 1, 0, B, k, V, n1, nx1)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(n, n1) and torch.equal(nx, nx1)
        assert 0 <= n.min().item() and n.max().item() <= k


@pytest.mark.parametrize("V", [40001, 1002, 512])
def test_accept_sample_masked_and_infinite_rows(V):
    """Ids masked with -inf are never emitted; a target row with one finite id emits it; rows of -inf or with a
    not-a-number still give an id of the vocabulary."""
    import torch
    import paper_2505_10259_amd as P
    B, k = 6, 2
    g = torch.Generator("cuda").manual_seed(V)
    p = torch.randn(B, k + 1, V, device="cuda", generator=g)
    q = torch.randn(B, k, V, device="cuda", generator=g)
    keep = torch.arange(V, device="cuda") % 7 == 3
    p[:, :, ~keep] = -float("inf")
    p[1] = -float("inf"); p[1, :, V // 2] = 0.0
    p[2] = -float("inf")
    p[3, :, 5] = float("nan")
    p[4, :, 3] = float("inf")
    d = torch.full((B, k), 4, dtype=torch.int32, device="cuda")      # masked: rejected at once
    for n in (torch.zeros(B, dtype=torch.int32, device="cuda"), None):
        nx = torch.full((B,), -1, dtype=torch.int32, device="cuda")
        P.spec_accept(p, q, d, None, None, 0.8, 7, 1, 0, B, k, V, n, nx)
        torch.cuda.synchronize()
        t = nx.cpu().tolist()
        assert all(0 <= x < V for x in t)
        assert t[0] % 7 == 3 and t[5] % 7 == 3 and t[1] == V // 2
        if n is not None:
            assert n.cpu().tolist()[:2] == [0, 0] and n[5].item() == 0


# register-resident kernel (8) and general ones (5, 40001)
@pytest.mark.parametrize("V,B", [(8, 16384), (5, 16384), (40001, 512)])
def test_weights_have_the_error_of_the_library_exponential(V, B):
    """A bonus row [x, 0, -inf, ...] draws id 0 exactly while u < exp(x): for x < -17.4 the normaliser and the total are 1
    in f32, so bisecting u over the floats gives the kernel's exp(x) to the bit.  Bound: 1 ulp, the documented error of
    expf (a rounded product x log2 e in front of exp2 alone is off by up to 2.3), subnormal results included."""
    import torch
    import paper_2505_10259_amd as P
    inf = float("inf")
    x = torch.linspace(-103.0, -17.5, B, dtype=torch.float64).float()
    p = torch.full((B, 2, V), -inf, device="cuda")
    p[:, 0, 1] = 0.0                             # the candidate, token 1, is certain on both sides: kept
    q = p[:, :1].contiguous()
    p[:, 1, 0], p[:, 1, 1] = x.cuda(), 0.0
    d = torch.ones(B, 1, dtype=torch.int32, device="cuda")
    ua = torch.full((B, 1), 0.5, device="cuda")
    lo = torch.zeros(B, dtype=torch.int32, device="cuda")                     # bits of the largest u that draws id 0
    hi = torch.full((B,), 0x34000000, dtype=torch.int32, device="cuda")       # (2^-23: id 1)
    nx = torch.empty(B, dtype=torch.int32, device="cuda")
    for _ in range(31):
        mid = lo + (hi - lo) // 2
        ur = mid.view(torch.float32).reshape(B, 1).repeat(1, 2).contiguous()
        P.spec_accept(p, q, d, ua, ur, 1.0, 0, 0, 0, B, 1, V, None, nx)
        torch.cuda.synchronize()
        assert ((nx == 0) | (nx == 1)).all()
        lo, hi = torch.where(nx == 0, mid, lo), torch.where(nx == 0, hi, mid)
    got = hi.cpu().view(torch.float32).double()  # exp(x) is the first float that u does not stay below
    ref = x.double().exp()
    ulp = torch.exp2(ref.log2().floor().clamp(min=-126) - 23)
    err = (got - ref).abs() / ulp
    assert err.max().item() <= 1.0, (err.max().item(), x[err.argmax()].item())


# every value that one thread of the general kernel holds of the row is not a number: a granule of four where a
# thread takes one (4001), ten granules 4096 ids apart (40001)
@pytest.mark.parametrize("V", [1001, 4001, 40001, 4096])
@pytest.mark.parametrize("side", ["p", "q"])
def test_not_a_number_anywhere_in_a_row_rejects(V, side):
    """A row with a not-a-number has no normaliser: whatever the candidate's own value, it is not kept."""
    import torch
    import paper_2505_10259_amd as P
    B, k = 8, 1
    g = torch.Generator("cuda").manual_seed(V)
    p = torch.randn(B, k + 1, V, device="cuda", generator=g)
    q = p[:, :k].clone().contiguous()
    p[:, 0, 7], q[:, 0, 7] = 30.0, 30.0          # certain on both sides: kept but for the not-a-numbers
    d = torch.full((B, k), 7, dtype=torch.int32, device="cuda")
    ua = torch.full((B, k), 0.5, device="cuda")
    ur = torch.full((B, k + 1), 0.5, device="cuda")

    def kept():
        n = torch.full((B,), -1, dtype=torch.int32, device="cuda")
        nx = torch.full((B,), -1, dtype=torch.int32, device="cuda")
        P.spec_accept(p, q, d, ua, ur, 0.8, 0, 0, 0, B, k, V, n, nx)
        torch.cuda.synchronize()
        assert all(0 <= t < V for t in nx.cpu().tolist())
        return n.cpu().tolist()

    assert kept() == [1] * B
    t = p if side == "p" else q
    for b in range(1, B):
        row = t[b, 0]
        off = (row.data_ptr() // 4) % 4          # granules lie at 16-byte boundaries
        for first in range(64 - off, V - 3, 4096):
            row[first:first + 4] = float("nan")
    assert kept() == [1] + [0] * (B - 1)


@pytest.mark.parametrize("V", [512, 1001, 4001, 32000, 40001])
def test_infinite_temperature_is_uniform(V):
    """1 / temperature = 0: every id is as likely as the next, on the rows' padding as little as before."""
    import torch
    import paper_2505_10259_amd as P
    B, k = 33, 2
    g = torch.Generator("cuda").manual_seed(V)
    p = torch.randn(B, k + 1, V, device="cuda", generator=g) * 5
    q = torch.randn(B, k, V, device="cuda", generator=g) * 5
    d = torch.randint(0, V, (B, k), device="cuda", generator=g, dtype=torch.int32)
    ids = torch.linspace(0, V - 1, B).long()
    ua = torch.full((B, k), 0.99, device="cuda")
    ur = ((ids + 0.5) / V).float().cuda().reshape(B, 1).repeat(1, k + 1).contiguous()
    n = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    nx = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    P.spec_accept(p, q, d, ua, ur, float("inf"), 0, 0, 0, B, k, V, n, nx)
    torch.cuda.synchronize()
    assert n.cpu().tolist() == [k] * B
    assert nx.cpu().tolist() == ids.tolist()
