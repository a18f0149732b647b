"""The FP32 predictor on BF16 planes: every tile form, and the weights that keep the FP32
instructions."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2601_03187_amd import synth, train
from paper_2601_03187_amd import tang as T
from tests._gpu import mlp_dev, torch_cuda

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def _setup(space, hidden, seed):
    rules = synth.make_rules(3000, seed=101, wide=space == "wide", all_lengths=space == "all")
    rs = T.tang_ruleset_create(0, rules)
    C = T.tang_ruleset_num_tuples(rs)
    Ws, bs = train.random_weights(C, hidden, seed=seed)
    return rules, rs, C, Ws, bs


@pytest.mark.parametrize("topk", [1, 2])
@pytest.mark.parametrize("space", ["narrow", "wide", "all"])
@pytest.mark.parametrize("hidden", [128, 256])
def test_tile_forms_agree_bit_for_bit(hidden, space, topk):
    """A header's scores and candidates do not depend on its batch: sizes at the edges of
    the tiles and of the size rule, against the first 61 headers alone; those within the
    bound of test_gpu_mlp (4 K u m) of the oracle."""
    torch_cuda()
    rules, rs, C, Ws, bs = _setup(space, hidden, 7)
    try:
        T.tang_model_load(rs, Ws, bs, "fp32", topk=topk)
        hdr = synth.make_packets(rules, 61, seed=102, frac_in=0.7)
        logits, cand = mlp_dev(rs, hdr, C, topk=topk)
        X = orc.feature_bits(hdr)
        mag = orc.mlp_abs_forward(X, Ws, bs)[-1]
        assert (np.abs(logits - orc.mlp_forward(X, Ws, bs, "fp32")) <= 4 * (104 + 2 * hidden) * U * mag).all()
        assert np.array_equal(cand, np.argsort(-logits, axis=1, kind="stable")[:, :topk])
        sizes = [1, 31, 33, 8192, 8193, 16384, 16385]
        if space == "narrow":
            sizes += [(1 << 18) - 1, (1 << 18) + 1]
        for n in sizes:
            at = np.arange(n) % len(hdr)
            got, gc = mlp_dev(rs, hdr[at], C, topk=topk)
            assert np.array_equal(got, logits[at]), n
            assert np.array_equal(gc, cand[at]), n
    finally:
        T.tang_ruleset_destroy(rs)


@pytest.mark.parametrize("hidden", [128, 256])
def test_weights_out_of_the_planes_range(hidden):
    """Weights whose outputs may pass 1e30 run on the FP32 instructions and stay within the
    same bound; with an infinite weight the scores of untouched classes stay finite."""
    torch_cuda()
    rules, rs, C, Ws, bs = _setup("narrow", hidden, 9)
    try:
        hdr = synth.make_packets(rules, 300, seed=103, frac_in=0.7)
        X = orc.feature_bits(hdr)
        big = [Ws[0] * np.float32(1e12), Ws[1] * np.float32(1e12), Ws[2] * np.float32(1e8)]
        for W in (Ws, big):
            T.tang_model_load(rs, W, bs, "fp32")
            logits, _ = mlp_dev(rs, hdr, C)
            mag = orc.mlp_abs_forward(X, W, bs)[-1]
            assert (np.abs(logits - orc.mlp_forward(X, W, bs, "fp32")) <= 4 * (104 + 2 * hidden) * U * mag).all()
        odd = [W.copy() for W in Ws]
        odd[2][3, 5] = np.inf
        T.tang_model_load(rs, odd, bs, "fp32")
        logits, cand = mlp_dev(rs, hdr, C)
        keep = np.arange(C) != 3
        T.tang_model_load(rs, Ws, bs, "fp32")
        plain, _ = mlp_dev(rs, hdr, C)
        mag = orc.mlp_abs_forward(X, Ws, bs)[-1]
        assert (np.abs(logits[:, keep] - plain[:, keep]) <= 8 * (104 + 2 * hidden) * U * mag[:, keep]).all()
        assert not np.isfinite(logits[:, 3]).all() and (cand < C).all()
    finally:
        T.tang_ruleset_destroy(rs)


@pytest.mark.parametrize("layer", [1, 2])
@pytest.mark.parametrize("hidden", [128, 256])
def test_weights_below_the_planes_range(hidden, layer):
    """A hidden layer scaled by 2^-116 and the next by 2^116: ordinary scores from values
    whose planes would vanish. The error over the scores stays that of FP32 sums: a random
    walk of K roundings, 4 sqrt(K) u at most (two planes alone would give 2^-17)."""
    torch_cuda()
    rules, rs, C, _, _ = _setup("narrow", hidden, 11)
    try:
        rng = np.random.default_rng(12)
        dims = [104, hidden, hidden, C]
        Ws = [(rng.uniform(0.5, 1.0, (o, i)) * rng.choice([-1, 1], (o, i)) / np.sqrt(i)).astype(np.float32)
              for i, o in zip(dims, dims[1:])]
        bs = [np.full(o, v, np.float32) for o, v in zip(dims[1:], (4.0, 4.0, 0.5))]   # few inputs near zero
        small, large = np.float32(2.0 ** -116), np.float32(2.0 ** 116)
        if layer == 1:      # the hidden layer's weights and outputs
            Ws[1], bs[1], Ws[2] = Ws[1] * small, bs[1] * small, Ws[2] * large
        else:               # the output layer's weights alone, its scores 2^-116 of the ordinary
            Ws[2], bs[2] = Ws[2] * small, bs[2] * small
        hdr = synth.make_packets(rules, 500, seed=104, frac_in=0.7)
        T.tang_model_load(rs, Ws, bs, "fp32")
        logits, _ = mlp_dev(rs, hdr, C)
        a = orc.feature_bits(hdr).astype(np.float64)
        for k in range(3):
            a = a @ Ws[k].astype(np.float64).T + bs[k]
            a = np.maximum(a, 0) if k < 2 else a
        err = np.linalg.norm(logits - a) / np.linalg.norm(a)
        assert err <= 4 * np.sqrt(104 + 2 * hidden) * U, err
    finally:
        T.tang_ruleset_destroy(rs)
