"""GPU parity of the ratio acceptance rule for sampled draft tokens (spec_k_accept_qratio, spec_k_sample_children,
through the C ABI) against oracle/qratio.py: the same counter-based random numbers on both sides, so the same
decisions.  The oracle evaluates probabilities in fp64, the kernel in fp32: draws whose decision sits within
1e-4 (relative) of the boundary are set aside (the oracle reports that margin); the rest must agree exactly.
A chi-square test on the kernel's own output checks the property the rule exists for."""
import numpy as np
import pytest
import scipy.stats

from oracle import qratio

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2408_15766_amd as P
    assert torch.cuda.is_available()
    return torch, P


def make_tree(g, q_logits, temperature, branching, seed, cycle):
    """Two-level tree with sampled children: `branching[0]` children of the root, `branching[1]` of each of those."""
    token, parent = [0], [-1]
    level = [0]
    for width in branching:
        nxt = []
        for node in level:
            for tok in qratio.sample_children(q_logits[node], temperature, width, seed, cycle, node):
                token.append(tok); parent.append(node); nxt.append(len(token) - 1)
        level = nxt
    return np.array(token, dtype=np.int32), np.array(parent, dtype=np.int32)


@pytest.mark.parametrize("vocab,branching,temperature,trials", [(50, (3, 2), 1.0, 150), (1000, (4, 1), 0.8, 60), (32000, (2, 2), 1.0, 12)])
def test_accept_qratio_matches_oracle_decisions(env, vocab, branching, temperature, trials):
    torch, P = env
    g = np.random.default_rng(vocab)
    n_nodes = 1 + branching[0] + branching[0] * branching[1]
    compared = accepted_some = 0
    for cycle in range(trials):
        p_logits = (g.standard_normal((n_nodes, vocab)) * 2).astype(np.float32)
        q_logits = (p_logits + g.standard_normal((n_nodes, vocab)) * 1.0).astype(np.float32)   # a draft near the target
        token, parent = make_tree(g, q_logits, temperature, branching, 77, cycle)
        want_acc, want_next, margin = qratio.accept_qratio(token, parent, p_logits, q_logits, temperature, 77, cycle)
        got_acc, got_tok = P.spec_k_accept_qratio(torch.from_numpy(p_logits).cuda(), torch.from_numpy(q_logits).cuda(),
                                                  torch.from_numpy(token).cuda(), torch.from_numpy(parent).cuda(), temperature, 77, cycle)
        if margin < 1e-4:
            continue
        compared += 1
        accepted_some += bool(want_acc)
        assert got_acc == want_acc, (cycle, got_acc, want_acc)
        assert got_tok == [int(token[c]) for c in want_acc] + [want_next], (cycle, got_tok, want_next)
    assert compared >= trials * 0.9 and 0 < accepted_some < compared


@pytest.mark.parametrize("vocab,branching,temperature,trials,masked", [(4096, (3, 2), 1.0, 24, False), (9001, (4, 2), 0.8, 24, False), (32000, (2, 2), 1.0, 16, False),
                                                                       (270001, (2, 1), 1.0, 4, False), (16500, (3, 2), 1.0, 24, True)])
def test_accept_qratio_from_row_statistics_matches_oracle_decisions(env, vocab, branching, temperature, trials, masked):
    """The engine's form: draft rows only for nodes with children, in another order than the nodes, and every row's statistics from
    slices of 4096 tokens (one, several, more than 64, a ragged last one).  The level of every (row, slice) is its own, so that
    statistics of another row or slice change probabilities by factors; masked: whole slices without probability."""
    torch, P = env
    g = np.random.default_rng(vocab + 1)
    n_nodes = 1 + branching[0] + branching[0] * branching[1]
    n_exp = 1 + branching[0]
    n_slices = (vocab + 4095) // 4096
    compared = accepted_some = rejected_some = 0
    for cycle in range(trials):
        level = np.repeat(g.standard_normal((n_nodes, n_slices)) * 2, 4096, axis=1)[:, :vocab]
        if masked:
            for row in level:
                row.reshape(-1)[4096 * int(g.integers(1, n_slices)):][:4096] = -np.inf
        p_logits = (g.standard_normal((n_nodes, vocab)) * 2 + level).astype(np.float32)
        q_logits = (p_logits + g.standard_normal((n_nodes, vocab)) * 1.0).astype(np.float32)
        token, parent = make_tree(g, q_logits, temperature, branching, 78, cycle)
        want_acc, want_next, margin = qratio.accept_qratio(token, parent, p_logits, q_logits, temperature, 78, cycle)
        place = g.permutation(n_exp).astype(np.int32)          # node -> row
        q_rows = np.empty((n_exp, vocab), np.float32)
        q_rows[place] = q_logits[:n_exp]
        qrow_of = np.concatenate([place, np.full(n_nodes - n_exp, -1, np.int32)])
        cu = lambda a: torch.from_numpy(a).cuda()
        got_acc, got_tok = P.spec_k_accept_qratio_rows(cu(p_logits), cu(q_rows), cu(qrow_of), cu(token), cu(parent), temperature, 78, cycle)
        if margin < 1e-4:
            continue
        compared += 1
        accepted_some += bool(want_acc)
        rejected_some += want_acc[:1] != [1]
        assert got_acc == want_acc, (cycle, got_acc, want_acc)
        assert got_tok == [int(token[c]) for c in want_acc] + [want_next], (cycle, got_tok, want_next)
    assert compared >= trials * 0.9 and accepted_some and rejected_some


@pytest.mark.parametrize("vocab,m", [(50, 3), (1000, 16), (32000, 10), (128256, 4)])
def test_sample_children_matches_oracle(env, vocab, m):
    torch, P = env
    g = np.random.default_rng(vocab + m)
    logits = (g.standard_normal(vocab) * 2).astype(np.float32)
    dl = torch.from_numpy(logits).cuda()
    for cycle in range(20):
        want = qratio.sample_children(logits, 0.9, m, 5, cycle, 3)
        got = P.spec_k_sample_children(dl, 0.9, m, 5, cycle, qratio.DRAFT_NODE_BASE + 3)
        assert got == want and len(set(got)) == m


def test_gpu_rule_is_lossless_chi_square(env):
    # children sampled on the GPU from a draft that disagrees with the target, accepted on the GPU:
    # the first emitted token must follow the target distribution (Sec. 2, third step)
    torch, P = env
    g = np.random.default_rng(3)
    vocab, m, n = 7, 2, 12000
    p_logits = (g.standard_normal((1 + m, vocab)) * 1.5).astype(np.float32)
    q_logits = (g.standard_normal((1 + m, vocab)) * 1.5).astype(np.float32)
    dp, dq = torch.from_numpy(p_logits).cuda(), torch.from_numpy(q_logits).cuda()
    parent = torch.tensor([-1] + [0] * m, dtype=torch.int32, device="cuda")
    counts = np.zeros(vocab)
    for cycle in range(n):
        kids = P.spec_k_sample_children(dq[0], 1.0, m, 11, cycle, qratio.DRAFT_NODE_BASE)
        token = torch.tensor([0] + kids, dtype=torch.int32, device="cuda")
        _, toks = P.spec_k_accept_qratio(dp, dq, token, parent, 1.0, 11, cycle)
        counts[toks[0]] += 1
    e = np.exp(p_logits[0].astype(np.float64) - p_logits[0].max())
    pval = scipy.stats.chisquare(counts, e / e.sum() * n)[1]
    assert pval > 0.01, (pval, counts)


def test_qratio_error_paths(env):
    torch, P = env
    z = torch.zeros((2, 10), dtype=torch.float32, device="cuda")
    tok = torch.zeros(2, dtype=torch.int32, device="cuda")
    par = torch.tensor([-1, 0], dtype=torch.int32, device="cuda")
    with pytest.raises(P.SpecError):
        P.spec_k_accept_qratio(z, z, tok, par, 0.0, 1, 1)      # temperature must be positive
    with pytest.raises(P.SpecError):
        P.spec_k_sample_children(z[0], 1.0, 17, 1, 1, 0)       # more children than the limit
    with pytest.raises(P.SpecError):
        P.spec_k_sample_children(z[0], 1.0, 11, 1, 1, 0)       # more children than tokens
