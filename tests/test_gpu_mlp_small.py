"""The small-batch form of the BF16 and FP8 predictors equals the large-batch one."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2601_03187_amd import synth, train
from paper_2601_03187_amd import tang as T
from tests._gpu import mlp_dev, torch_cuda

pytestmark = pytest.mark.gpu

LARGE = 32769   # past every size that takes the small form


@pytest.mark.parametrize("topk", [1, 2])
@pytest.mark.parametrize("space", ["narrow", "wide", "all"])
@pytest.mark.parametrize("hidden", [128, 256])
@pytest.mark.parametrize("prec", ["bf16", "fp8"])
def test_small_form_equals_large_form_bit_for_bit(prec, hidden, space, topk):
    """Scores and candidates of a header at the edges of the small form's tiles and size
    rules are those of a large batch, bit for bit (k_mlp's are checked against the oracle in
    test_gpu_mlp); tied scores and NaN scores too."""
    torch_cuda()
    rules = synth.make_rules(3000, seed=111, wide=space == "wide", all_lengths=space == "all")
    rs = T.tang_ruleset_create(0, rules)
    try:
        C = T.tang_ruleset_num_tuples(rs)
        Ws, bs = train.random_weights(C, hidden, seed=5)
        Ws[2][7] = Ws[2][3]         # two classes with equal scores
        bs[2][7] = bs[2][3]
        bs[2][11] = np.nan
        hdr = synth.make_packets(rules, 83, seed=112, frac_in=0.7)
        sc = train.act_scales(Ws, bs, train.feature_bits_torch(hdr)) if prec == "fp8" else None
        T.tang_model_load(rs, Ws, bs, prec, topk=topk, act_scales=sc)
        big, bc = mlp_dev(rs, hdr[np.arange(LARGE) % len(hdr)], C, topk=topk)
        logits, cand = big[:83], bc[:83]
        finite = np.arange(C) != 11
        want = orc.mlp_forward(orc.feature_bits(hdr), Ws, bs, prec, act_scales=sc)[:, finite]
        got = logits[:, finite]
        assert np.median(np.abs(got - want).max(axis=1) / np.abs(want).max(axis=1)) < 2.0 ** -8
        for n in (1, 15, 17, 83, 4096, 4097, 16384, 16385, 32768):
            at = np.arange(n) % len(hdr)
            small, sc_ = mlp_dev(rs, hdr[at], C, topk=topk)
            assert np.array_equal(small, logits[at], equal_nan=True), n
            assert np.array_equal(sc_, cand[at]), n
    finally:
        T.tang_ruleset_destroy(rs)


@pytest.mark.parametrize("C", [33, 48, 49, 64, 65])
@pytest.mark.parametrize("hidden", [128, 256])
@pytest.mark.parametrize("prec", ["bf16", "fp8"])
def test_class_tile_edges(prec, hidden, C):
    """Class counts at the edges of the 16-class tiles and 32-class blocks, large form: the
    candidates are the best of the scores, ties to the lower class, and the scores are within
    the type's rounding of the oracle's (the median header within 2^-8, as above)."""
    torch_cuda()
    rules = synth.make_rules(6000, seed=113, all_lengths=True)
    pair = 33 * rules["sip_len"].astype(np.int64) + rules["dip_len"]
    rules = rules[np.isin(pair, np.unique(pair)[:C])]
    rs = T.tang_ruleset_create(0, rules)
    try:
        assert T.tang_ruleset_num_tuples(rs) == C
        Ws, bs = train.random_weights(C, hidden, seed=6)
        Ws[2][C - 1] = Ws[2][C - 2]     # the last two classes tie, and beat most others
        bs[2][C - 1] = bs[2][C - 2] = np.abs(bs[2]).max()
        hdr = synth.make_packets(rules, 83, seed=114, frac_in=0.7)
        sc = train.act_scales(Ws, bs, train.feature_bits_torch(hdr)) if prec == "fp8" else None
        want = orc.mlp_forward(orc.feature_bits(hdr), Ws, bs, prec, act_scales=sc)
        for topk in (1, 2, 4):
            T.tang_model_load(rs, Ws, bs, prec, topk=topk, act_scales=sc)
            logits, cand = mlp_dev(rs, hdr[np.arange(LARGE) % len(hdr)], C, topk=topk)
            best = np.argsort(-logits[:83], axis=1, kind="stable")[:, :topk]
            assert np.array_equal(cand[:83].reshape(83, topk), best), topk
            assert np.array_equal(cand, cand[np.arange(LARGE) % len(hdr)])
            assert np.median(np.abs(logits[:83] - want).max(axis=1) / np.abs(want).max(axis=1)) < 2.0 ** -8
    finally:
        T.tang_ruleset_destroy(rs)


@pytest.mark.parametrize("topk", [2, 3, 4])
@pytest.mark.parametrize("hidden", [128, 256])
@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp8"])
def test_best_classes_of_all_waves(prec, hidden, topk):
    """Many classes, spread over the waves: the candidates are the best of the scores whatever
    waves hold them, ties to the lower class (four classes of different tiles that tie, above
    most others), a NaN score last."""
    torch_cuda()
    rules = synth.make_rules(6000, seed=115, wide=True)
    rs = T.tang_ruleset_create(0, rules)
    try:
        C = T.tang_ruleset_num_tuples(rs)
        assert C > 128
        Ws, bs = train.random_weights(C, hidden, seed=8)
        for c in (60, 77, C - 1):
            Ws[2][c] = Ws[2][5]
            bs[2][c] = bs[2][5]
        bs[2][[5, 60, 77, C - 1]] = np.sort(np.abs(bs[2]))[-3]
        hdr = synth.make_packets(rules, 131, seed=116, frac_in=0.7)
        sc = train.act_scales(Ws, bs, train.feature_bits_torch(hdr)) if prec == "fp8" else None
        bs[2][90] = np.nan
        T.tang_model_load(rs, Ws, bs, prec, topk=topk, act_scales=sc)
        for n in (1, 16, 131, 4099):
            at = np.arange(n) % len(hdr)
            logits, cand = mlp_dev(rs, hdr[at], C, topk=topk)
            known = np.where(np.isnan(logits), -np.inf, logits)
            assert np.isnan(logits[:, 90]).all()
            assert np.array_equal(cand, np.argsort(-known, axis=1, kind="stable")[:, :topk]), n
    finally:
        T.tang_ruleset_destroy(rs)
