"""GPU parity of the Top-K distillation loss (spec_topk_loss, through the C ABI: LM-head GEMM + loss kernels)
against oracle/distill.py on the same seeded inputs.

Tolerance.  Inputs are exact in the storage type, products are exact in fp32 and accumulated in fp32 over d
terms, the loss kernels work in fp32: the logits differ from the fp64 oracle's by ~1e-6 relative, the losses
(O(1..10)) by well under 2e-4.  Membership of the top-K set is an integer decision taken on fp32 logits here
and on fp64 logits in the oracle: where the K-th and (K+1)-th target logits are closer than 1e-4 either
choice is accepted (the oracle is asked for both)."""
import ctypes as C

import numpy as np
import pytest

import workload as wl
from oracle import distill

pytestmark = pytest.mark.gpu

TOL = dict(rtol=2e-4, atol=2e-4)


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2408_15766_amd as P
    assert torch.cuda.is_available()
    return torch, P


def run_gpu(torch, P, ft, fd, w, k, dtype):
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    dev = lambda x: torch.from_numpy(x).cuda().to(tdt)
    head = P.spec_pack_weight(dev(w))
    topk, ce, tot = P.spec_topk_loss(dev(ft), dev(fd), head, k)
    torch.cuda.synchronize()
    return topk.cpu().numpy().astype(np.float64), ce.cpu().numpy().astype(np.float64), tot.cpu().numpy().astype(np.float64)


def oracle_losses(ft, fd, w, k, rows=None):
    f64 = lambda x: x.astype(np.float64)
    if rows is not None:
        ft, fd = ft[rows], fd[rows]
    zq, zp = f64(ft) @ f64(w).T, f64(fd) @ f64(w).T
    want = distill.topk_distill_loss(zq, zp, k)
    alt = want.copy()
    if k < w.shape[0]:                                         # near-tie at the boundary: the other admissible set
        for r in range(zq.shape[0]):
            order = distill.topk_set(zq[r], k + 1)
            if zq[r, order[k - 1]] - zq[r, order[k]] < 1e-4:
                logq = zq[r] - np.log(np.exp(zq[r] - zq[r].max()).sum()) - zq[r].max()
                logp = zp[r] - np.log(np.exp(zp[r] - zp[r].max()).sum()) - zp[r].max()
                om = np.concatenate([order[:k - 1], order[k:k + 1]])
                alt[r] = -(np.exp(logq[om]) * logp[om]).sum()
    return want, alt, distill.soft_cross_entropy(zq, zp)


def check(got_topk, got_ce, want, alt, want_ce):
    assert np.isfinite(got_topk).all() and np.isfinite(got_ce).all()
    ok = np.isclose(got_topk, want, **TOL) | np.isclose(got_topk, alt, **TOL)
    assert ok.all(), f"rows {np.nonzero(~ok)[0][:5]}: got {got_topk[~ok][:5]} want {want[~ok][:5]}"
    np.testing.assert_allclose(got_ce, want_ce, **TOL)


CASES = [
    # dtype, rows, d, vocab, k
    ("fp32", 37, 256, 1000, 10),        # one ragged slice
    ("fp32", 5, 128, 9000, 1),          # three slices, the target's best token only
    ("fp32", 33, 256, 9000, 16),
    ("fp32", 20, 128, 9000, 100),       # the largest K of the paper's ablation
    ("fp32", 9, 128, 4097, 128),        # the entry point's K limit; a slice of one token
    ("bf16", 130, 512, 32000, 10),      # the paper's K on the LLaMA2 vocabulary
    ("bf16", 600, 256, 5000, 5),        # two row chunks (512 + 88)
    ("bf16", 40, 256, 128256, 10),      # LLaMA3 vocabulary: 32 slices
    ("bf16", 12, 256, 128256, 128),     # 4096 candidates in the merge
    ("bf16", 17, 264, 1000, 3),         # both sides' rows in one token tile of the LM head, the boundary inside a 32-row block
    ("bf16", 64, 256, 1000, 3),         # ... the largest such pair
    ("bf16", 65, 256, 1000, 3),         # ... and one row more per side: tiled, each side its own tiles
    ("fp32", 45, 200, 7000, 5),         # fp32 rows enough for the tiled LM head: each side its own 32-row tiles, ragged ones
    ("fp32", 129, 512, 9000, 16),       # ... eight tiles of k
    ("fp32", 100, 260, 9000, 16),       # ... five, the last one of four k
    ("fp32", 33, 8, 32000, 10),         # ... one ragged tile of k
    ("fp32", 33, 192, 9000, 3),         # ... one row in a side's last tile; three tiles of k
    ("fp32", 200, 64, 9090, 5),         # ... a ragged weight block in the last workgroup
    ("fp32", 520, 132, 9000, 4),        # ... two chunks of positions, the second in the other kernel
    ("bf16", 1, 256, 100, 100),         # K = V: Eq. (1) becomes the cross-entropy (vocabulary smaller than one slice)
]


@pytest.mark.parametrize("dtype,rows,d,vocab,k", CASES)
def test_topk_loss_matches_oracle(env, dtype, rows, d, vocab, k):
    torch, P = env
    ft, fd, w = wl.make_distill_inputs(21, rows, d, vocab, dtype)
    got_topk, got_ce, tot = run_gpu(torch, P, ft, fd, w, k, dtype)
    want, alt, want_ce = oracle_losses(ft, fd, w, k)
    check(got_topk, got_ce, want, alt, want_ce)
    np.testing.assert_allclose(tot, [got_topk.sum(), got_ce.sum()], rtol=1e-5)


@pytest.mark.parametrize("rows", [330, 260])
def test_lm_head_in_whole_and_half_tiles(env, rows):
    # both sides' rows through one launch whose token tiles end raggedly (74 and 4 rows) and whose last round runs in half tiles
    torch, P = env
    assert P.spec_k_gemm_plan(rows, (37000 + 31) // 32, 264, sets=2) == (0, 32, 38)
    ft, fd, w = wl.make_distill_inputs(28, rows, 264, 37000, "bf16")
    got_topk, got_ce, _ = run_gpu(torch, P, ft, fd, w, 5, "bf16")
    want, alt, want_ce = oracle_losses(ft, fd, w, 5)
    check(got_topk, got_ce, want, alt, want_ce)


def test_whole_small_vocabulary_equals_cross_entropy(env):
    torch, P = env
    ft, fd, w = wl.make_distill_inputs(22, 7, 128, 100, "fp32")
    got_topk, got_ce, _ = run_gpu(torch, P, ft, fd, w, 100, "fp32")
    np.testing.assert_allclose(got_topk, got_ce, rtol=1e-5)
    _, _, want_ce = oracle_losses(ft, fd, w, 100)
    np.testing.assert_allclose(got_ce, want_ce, **TOL)


def test_exact_ties_take_the_lower_token_id(env):
    # every logit occurs twice (the LM head's second half repeats the first): an odd K must split a pair,
    # and which member is kept changes nothing in q but is fixed by the reading (lower id) for the set
    torch, P = env
    ft, fd, w = wl.make_distill_inputs(23, 16, 128, 6000, "fp32", tie_halves=True)
    for k in (1, 7):
        got_topk, got_ce, _ = run_gpu(torch, P, ft, fd, w, k, "fp32")
        want, alt, want_ce = oracle_losses(ft, fd, w, k)
        check(got_topk, got_ce, want, want, want_ce)          # no alternative: the tie is exact on both sides


def test_all_equal_target_logits(env):
    # a zero target feature gives the same logit for every token: Omega-hat is then tokens 0 .. K-1 (lower id first),
    # and far more than 64 values tie at the top of every wavefront (the selection's general path)
    torch, P = env
    ft, fd, w = wl.make_distill_inputs(26, 6, 128, 9000, "fp32")
    ft[1] = 0.0
    ft[4] = 0.0
    for k in (3, 10, 70):
        got_topk, got_ce, _ = run_gpu(torch, P, ft, fd, w, k, "fp32")
        want, alt, want_ce = oracle_losses(ft, fd, w, k)
        assert distill.topk_set(np.zeros(9000), k).tolist() == list(range(k))
        check(got_topk, got_ce, want, want if k < 9000 else alt, want_ce)


@pytest.mark.parametrize("vocab,k", [(4096, 1), (4100, 64), (9000, 65), (9000, 100), (33000, 124), (131072, 128)])
def test_large_logits_next_to_each_other(env, vocab, k):
    # target logits that fall with the token id: the largest sit in neighbouring registers of few threads, so that far more
    # than k of them pass a bound made from one value per thread; a row of scattered logits and a rising one beside it
    torch, P = env
    ft, fd, w = wl.make_distill_inputs(27, 3, 128, vocab, "fp32")
    w[:, 0] = np.linspace(4.0, -4.0, vocab, dtype=np.float32)
    ft[0] = 0.0
    ft[0, 0] = 1.0
    ft[2] = 0.0
    ft[2, 0] = -1.0
    got_topk, got_ce, _ = run_gpu(torch, P, ft, fd, w, k, "fp32")
    want, alt, want_ce = oracle_losses(ft, fd, w, k)
    check(got_topk, got_ce, want, alt, want_ce)


@pytest.mark.parametrize("vocab,k", [(4096, 40), (9000, 30), (12288, 100), (4097, 55)])
def test_candidates_of_one_wavefront_and_of_all(env, vocab, k):
    # tokens above the bound: all in the first wavefront's quarter of a slice (more than it has places for, or fewer), and
    # spread over the four so that their lists are read one behind the other
    torch, P = env
    ft, fd, w = wl.make_distill_inputs(29, 4, 128, vocab, "fp32")
    tok = np.arange(vocab)
    w[:, 0] = np.where(tok % 1024 < 256, 4.0, -4.0) - tok * (2.0 / vocab)
    w[:, 1] = np.where(tok % 16 < 3, 4.0, -4.0) - tok * (2.0 / vocab)
    for r in (0, 1):
        ft[r] = 0.0
        ft[r, r] = 1.0
    got_topk, got_ce, _ = run_gpu(torch, P, ft, fd, w, k, "fp32")
    want, alt, want_ce = oracle_losses(ft, fd, w, k)
    check(got_topk, got_ce, want, alt, want_ce)


def test_infinite_and_nan_logits(env):
    # tokens ruled out on both sides have no weight (their product 0 * inf makes the whole-vocabulary term NaN, as it did);
    # NaN logits show in that position's losses and in no other's
    torch, P = env
    ft, fd, w = wl.make_distill_inputs(30, 5, 128, 9000, "fp32")
    keep = np.arange(9000) % 3 > 0
    ft[:, 0] = fd[:, 0] = 1.0
    w[:, 0] = 0.0
    want, alt, _ = oracle_losses(ft, fd, w[keep], 20)
    w[~keep, 0] = -np.inf
    got_topk, got_ce, _ = run_gpu(torch, P, ft, fd, w, 20, "fp32")
    assert (np.isclose(got_topk, want, **TOL) | np.isclose(got_topk, alt, **TOL)).all()
    assert np.isnan(got_ce).all()
    w[~keep, 0] = 0.0
    clean = run_gpu(torch, P, ft, fd, w, 20, "fp32")
    ft[3] = np.nan
    fd[1] = np.nan
    got = run_gpu(torch, P, ft, fd, w, 20, "fp32")
    for g, c in zip(got[:2], clean[:2]):
        assert np.isnan(g[[1, 3]]).all()
        np.testing.assert_array_equal(g[[0, 2, 4]], c[[0, 2, 4]])


@pytest.mark.parametrize("value,factor", [("lowest", 1.0), ("lowest", 3.0), ("-inf", 2.0)])
@pytest.mark.parametrize("rows", [40, 129])
def test_ruled_out_tokens_in_the_tiled_head(env, rows, value, factor):
    # a column takes every third token to the lowest value, past it (an overflow) or to -inf; beside the ruled out tokens the logits are those of a
    # head without them
    torch, P = env
    ft, fd, w = wl.make_distill_inputs(36, rows, 130 * 2, 9000, "fp32")
    out = np.arange(9000) % 3 == 0
    ft[:, 5] = fd[:, 5] = factor
    w[:, 5] = 0.0
    kept = w[~out]
    w[out, 5] = float(torch.finfo(torch.float32).min) if value == "lowest" else -np.inf
    got_topk, got_ce, _ = run_gpu(torch, P, ft, fd, w, 20, "fp32")
    want, alt, want_ce = oracle_losses(ft, fd, kept, 20)
    if value == "lowest" and factor == 1.0:
        check(got_topk, got_ce, want, alt, want_ce)            # weight 0 times a finite logit
    else:
        assert (np.isclose(got_topk, want, **TOL) | np.isclose(got_topk, alt, **TOL)).all()
        assert np.isnan(got_ce).all()                          # 0 * -inf, as the definition has it


@pytest.mark.parametrize("dtype,d,vocab", [("fp32", 512, 9000), ("fp32", 132, 32000), ("fp32", 64, 1000), ("bf16", 1096, 33000), ("bf16", 136, 9000)])
def test_losses_of_a_position_have_the_same_bits_in_any_call(env, dtype, d, vocab):
    # few positions and many, whole chunks of 512 and short ones (bf16: 188 rows a side join at 33000 tokens): the ways of the LM head add up a logit in the same order
    torch, P = env
    rows = 520 if dtype == "fp32" else 700
    ft, fd, w = wl.make_distill_inputs(41, rows, d, vocab, dtype)
    topk, ce, _ = run_gpu(torch, P, ft, fd, w, 10, dtype)
    for lo, hi in ((0, 1), (100, 116), (0, 33), (30, 94), (391, 520), (512, 520), (512, rows)):
        a, b, _ = run_gpu(torch, P, np.ascontiguousarray(ft[lo:hi]), np.ascontiguousarray(fd[lo:hi]), w, 10, dtype)
        assert np.array_equal(a, topk[lo:hi]) and np.array_equal(b, ce[lo:hi])


@pytest.mark.parametrize("rows", [4, 40, 129, 512])
def test_fp32_logits_of_one_product_are_rounded_once(env, rows):
    # Target logits of one product each, 4096 * s^2 for even tokens and 4096 * s * (1 + 2^-7) for odd ones, where s has its bits in three groups of
    # eight: an LM head that leaves out part of a product moves the even logits against the odd ones, and the draft's 3 for even tokens shows it in
    # the losses.  Rounded once a logit has 2^-24 of itself, which is in the expected value; what the losses add to that is 1e-6.
    torch, P = env
    vocab, d = 9000, 512
    s = np.float32(1 + 2.0 ** -7 - 2.0 ** -15 + 2.0 ** -16 - 2.0 ** -22)
    even = np.arange(vocab) % 2 == 0
    ft, fd, w = np.zeros((rows, d), np.float32), np.zeros((rows, d), np.float32), np.zeros((vocab, d), np.float32)
    ft[:, 5], fd[:, 5], fd[:, 6] = 64 * s, 1, 1
    w[:, 5], w[:, 6] = np.where(even, 64 * s, np.float32(64 * (1 + 2.0 ** -7))), np.where(even, 3, 0)
    zq = (ft[0, 5] * w[:, 5]).astype(np.float64)
    zp = w[:, 5].astype(np.float64) + w[:, 6]
    want = -(np.exp(zq - zq.max()) / np.exp(zq - zq.max()).sum() * (zp - zp.max() - np.log(np.exp(zp - zp.max()).sum()))).sum()
    _, ce, _ = run_gpu(torch, P, ft, fd, w, 10, "fp32")
    np.testing.assert_allclose(ce, want, rtol=1e-5)


@pytest.mark.parametrize("lo,hi", [(0, 4096), (4096, 8192), (8192, 9000)])
def test_slices_without_any_probability(env, lo, hi):
    # all logits of a 4096-token slice -inf: on the target's side (the product overflows) they have no weight; on both sides the top-K loss
    # is the remaining tokens', and the whole-vocabulary term is 0 * inf
    torch, P = env
    ft, fd, w = wl.make_distill_inputs(34, 5, 128, 9000, "fp32")
    keep = np.ones(9000, bool)
    keep[lo:hi] = False
    ft[:, 0] = fd[:, 0] = 0.0
    zq, zp = ft.astype(np.float64) @ w.astype(np.float64).T, fd.astype(np.float64) @ w.astype(np.float64).T
    zq[:, ~keep] = -np.inf
    ft[:, 0] = 2.0
    w[:, 0] = np.where(keep, 0.0, -3e38)
    got_topk, got_ce, _ = run_gpu(torch, P, ft, fd, w, 20, "fp32")
    want = distill.topk_distill_loss(zq, zp, 20)
    check(got_topk, got_ce, want, want, distill.soft_cross_entropy(zq, zp))
    fd[:, 0] = 2.0
    got_topk, got_ce, _ = run_gpu(torch, P, ft, fd, w, 20, "fp32")
    np.testing.assert_allclose(got_topk, distill.topk_distill_loss(zq[:, keep], zp[:, keep], 20), **TOL)
    assert np.isnan(got_ce).all()


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("side", ["target", "both"])
def test_tokens_ruled_out_by_the_lowest_value(env, dtype, side):
    # a column of the LM head takes every third token to the type's lowest value, on the target's side or on both: finite
    # differences that overflow when scaled, tokens without weight, finite losses
    torch, P = env
    ft, fd, w = wl.make_distill_inputs(32, 6, 128, 9000, dtype)
    lowest = float(torch.finfo(torch.float32 if dtype == "fp32" else torch.bfloat16).min)
    ft[:, 0], fd[:, 0] = 1.0, 1.0 if side == "both" else 0.0
    w[:, 0] = np.where(np.arange(9000) % 3 == 0, lowest, 0.0)
    got_topk, got_ce, _ = run_gpu(torch, P, ft, fd, w, 20, dtype)
    want, alt, want_ce = oracle_losses(ft, fd, w, 20)
    check(got_topk, got_ce, want, alt, want_ce)


@pytest.mark.parametrize("lo,hi", [(0, 4096), (4096, 8192), (8192, 9000)])
@pytest.mark.parametrize("dtype,side", [("fp32", "target"), ("bf16", "target"), ("fp32", "draft"), ("bf16", "draft"), ("fp32", "both"), ("bf16", "both")])
def test_slices_ruled_out_by_the_lowest_value(env, dtype, side, lo, hi):
    # a whole 4096-token slice, or the ragged one: its 4096 draft logits add up to more than the type holds.  On the draft's side alone the
    # losses are the slice's target weight times 3.4e38
    torch, P = env
    ft, fd, w = wl.make_distill_inputs(35, 6, 128, 9000, dtype)
    ft[:, 0], fd[:, 0] = float(side != "draft"), float(side != "target")
    w[:, 0] = 0.0
    w[lo:hi, 0] = float(torch.finfo(torch.float32 if dtype == "fp32" else torch.bfloat16).min)
    got_topk, got_ce, _ = run_gpu(torch, P, ft, fd, w, 20, dtype)
    want, alt, want_ce = oracle_losses(ft, fd, w, 20)
    check(got_topk, got_ce, want, alt, want_ce)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_draft_rules_tokens_out_by_the_lowest_value(env, dtype):
    # three tokens that the target gives about 1e-13 of its best token's weight: the whole-vocabulary loss is that weight times
    # 3.4e38 there, the top-K loss does not see them
    torch, P = env
    ft, fd, w = wl.make_distill_inputs(33, 6, 128, 9000, dtype)
    tok = [17, 4095, 8191]
    ft[:, 0], fd[:, 0], ft[:, 1], fd[:, 1] = 0.0, 1.0, 1.0, 0.0
    w[:, 0] = w[:, 1] = 0.0
    w[tok, 0] = float(torch.finfo(torch.float32 if dtype == "fp32" else torch.bfloat16).min)
    w[tok, 1] = -30.0
    got_topk, got_ce, _ = run_gpu(torch, P, ft, fd, w, 20, dtype)
    want, alt, want_ce = oracle_losses(ft, fd, w, 20)
    check(got_topk, got_ce, want, alt, want_ce)


@pytest.mark.parametrize("rows,vocab,k", [(1100, 32000, 128), (1537, 4096, 3), (600, 128256, 40)])
def test_one_merge_for_several_chunks(env, rows, vocab, k):
    # two chunks' slices merged at a time, then a ragged rest; all four in one merge; one chunk a merge.  A scratch with room
    # for one chunk's only is merged chunk by chunk, with the same bits.
    torch, P = env
    ft, fd, w = wl.make_distill_inputs(31, rows, 64, vocab, "bf16")
    dev = lambda x: torch.from_numpy(x).cuda().bfloat16()
    dft, dfd, head = dev(ft), dev(fd), P.spec_pack_weight(dev(w))
    n = P.spec_topk_loss_scratch_bytes(rows, vocab, k)
    up = lambda x: (x + 63) // 64 * 64
    cand = lambda r: up(r * ((vocab + 4095) // 4096) * (8 + 3 * k))
    least = 4 * (2 * up(512 * up(vocab)) + 2 * up(rows) + cand(512))
    assert least <= n <= max(least, 4 * (2 * up(512 * up(vocab)) + 2 * up(rows)) + (16 << 20))
    out = [P.spec_topk_loss(dft, dfd, head, k, scratch=torch.empty(b, dtype=torch.uint8, device="cuda")) for b in (n, least)]
    for a, b in zip(*out):
        assert torch.equal(a, b)
    with pytest.raises(P.SpecError):
        P.spec_topk_loss(dft, dfd, head, k, scratch=torch.empty(least - 256, dtype=torch.uint8, device="cuda"))
    sel = np.array([0, 511, 512, 513, rows - 77, rows - 76, rows - 1] + ([1023, 1024] if rows > 1024 else []))
    want, alt, want_ce = oracle_losses(ft, fd, w, k, rows=sel)
    got = [o.cpu().numpy().astype(np.float64) for o in out[0]]
    check(got[0][sel], got[1][sel], want, alt, want_ce)


def test_topk_loss_full_size_sampled_rows(env):
    # the benchmark's launch: 4096 positions (batch 2 x 2048), LLaMA2-7B widths; the oracle takes 24 sampled rows
    torch, P = env
    ft, fd, w = wl.make_distill_inputs(24, 4096, 4096, 32000, "bf16")
    got_topk, got_ce, tot = run_gpu(torch, P, ft, fd, w, 10, "bf16")
    rows = np.array([0, 1, 127, 128, 511, 512, 513, 1023, 2047, 2048, 3000, 3583, 3584, 4000, 4094, 4095] + list(range(700, 708)))
    want, alt, want_ce = oracle_losses(ft, fd, w, 10, rows=rows)
    check(got_topk[rows], got_ce[rows], want, alt, want_ce)
    assert np.isfinite(got_topk).all() and (got_topk > 0).all() and (got_topk <= got_ce + 1e-3).all()
    np.testing.assert_allclose(tot, [got_topk.sum(), got_ce.sum()], rtol=1e-5)


def test_topk_loss_error_paths_and_optional_outputs(env):
    torch, P = env
    ft, fd, w = wl.make_distill_inputs(25, 8, 128, 500, "fp32")
    dev = lambda x: torch.from_numpy(x).cuda()
    head = P.spec_pack_weight(dev(w))
    dft, dfd = dev(ft), dev(fd)
    for bad_k in (0, 129, 501):
        assert P.spec_topk_loss_scratch_bytes(8, 500, bad_k) == 0
        with pytest.raises(P.SpecError):
            P.spec_topk_loss(dft, dfd, head, bad_k)
    n = P.spec_topk_loss_scratch_bytes(8, 500, 10)
    small = torch.empty(n - 256, dtype=torch.uint8, device="cuda")
    with pytest.raises(P.SpecError):
        P.spec_topk_loss(dft, dfd, head, 10, scratch=small)
    # only the totals wanted: the per-position outputs may be NULL
    scratch = torch.empty(n, dtype=torch.uint8, device="cuda")
    tot = torch.zeros(2, dtype=torch.float32, device="cuda")
    rc = P.lib.spec_topk_loss(0, dft.data_ptr(), dfd.data_ptr(), 8, 128, head.data_ptr(), 500, 10, scratch.data_ptr(), n,
                              None, None, tot.data_ptr(), C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    torch.cuda.synchronize()
    want, _, want_ce = oracle_losses(ft, fd, w, 10)
    np.testing.assert_allclose(tot.cpu().numpy(), [want.sum(), want_ce.sum()], rtol=2e-4)


@pytest.mark.parametrize("rows,d,vocab,tile", [
    (144, 64, 22000, (256, 192)), (188, 136, 33000, (128, 256)), (192, 64, 22016, (256, 192)),
    (300, 72, 16500, (256, 256)), (188, 1096, 32000, (256, 256)), (257, 1024, 40000, (256, 256)), (310, 1096, 20000, (256, 256)),   # ragged ends beside whole tiles
    (700, 64, 22000, (256, 192)), (700, 1096, 33000, (128, 256)),                                    # 512 apart, then 188
])
def test_both_sides_rows_as_one_set_of_tiles(env, rows, d, vocab, tile):
    """Where the sides' rows take fewer tiles together, one launch runs over them as one set: the border inside a 32-row block, inside a tile and (192 rows) at
    the end of a half tile, either side first in memory, a second chunk behind one that is not joined, every tile, one to sixteen tiles of k.  The losses have
    the bits of two sets of tiles (sides too far apart in memory for one), and fp64's value."""
    torch, P = env
    m, blocks = rows % 512 or 512, (vocab + 31) // 32
    assert (2 * m + 127) // 128 < 2 * ((m + 127) // 128) and P.spec_k_gemm_tile(2 * m, blocks, d) == tile
    _, whole, tiles = P.spec_k_gemm_plan(m, blocks, d, sets=2)
    assert (0, whole, tiles) == P.spec_k_gemm_plan(2 * m, blocks, d)
    if tile == (256, 256):
        assert whole == tiles > 0 and 0 < 2 * m % 256 <= 128
    ft, fd, w = wl.make_distill_inputs(5, rows, d, vocab, "bf16")
    packed = P.spec_pack_weight(torch.from_numpy(w).cuda().to(torch.bfloat16))
    ft, fd = (torch.from_numpy(x).cuda().to(torch.bfloat16) for x in (ft, fd))
    memory = torch.empty((1 << 29) + 2 * rows * d, dtype=torch.bfloat16, device="cuda")
    got = []
    for far in (False, True):
        low, high = memory[:rows * d].view(rows, d), memory[1 << 29 if far else rows * d:][:rows * d].view(rows, d)
        for a, b in ((low, high), (high, low)):
            a.copy_(ft), b.copy_(fd)
            assert (abs(a.data_ptr() - b.data_ptr()) < 1 << 30) != far
            got.append([t.cpu() for t in P.spec_topk_loss(a, b, packed, 7)[:2]])
    for topk, ce in got[1:]:
        assert torch.equal(topk, got[0][0]) and torch.equal(ce, got[0][1])
    head = torch.from_numpy(w).to(torch.bfloat16).double()
    zq, zp = ft.cpu().double() @ head.T, fd.cpu().double() @ head.T
    want = -(torch.softmax(zq, -1) * torch.log_softmax(zp, -1)).sum(-1)
    np.testing.assert_allclose(got[0][1].numpy(), want.numpy(), rtol=2e-4, atol=2e-4)      # as the oracle's cases
