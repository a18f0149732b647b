"""What is timed: the work a user of this framework has it do, through its public calls.

A case is a dict of plain values; its "kind" says which call it stands for:

* ``classify``  headers in device memory -> rule ids (``tang_classify``), with a plain
  predictor (``prec`` and ``hidden``, trained for the ruleset) or with none;
* ``logits``    the predictor's scores of every header (``tang_mlp_forward``), plain
  network or the paper-size residual one (``prec`` "resnet": 6 blocks of 512);
* ``update``    one round of a changing ruleset: insert rules, look a batch up, delete
  those rules again;
* ``serve``     a burst of requests from host memory through the serving loop.

Rulesets and headers follow the framework's own workloads: ``space`` names the tuple
space ("narrow": five prefix lengths per address, "wide": twelve, "all": every length),
``mix`` the share of wildcard-heavy rules, ``inside`` the share of headers that lie in a
rule (the others are uniform random), ``zipf`` whether rule popularity is Zipf(1).
"""
import numpy as np
import torch

from paper_2601_03187_amd import synth, train
from paper_2601_03187_amd import tang as T

MAX_HEADERS = 1 << 24


def _case(name, kind, rules, n, prec="bf16", hidden=256, topk=1, space="narrow", mix=0.0, inside=0.8,
          zipf=False, order="specificity"):
    return dict(name=name, kind=kind, rules=rules, n=n, prec=prec, hidden=hidden, topk=topk, space=space,
                mix=mix, inside=inside, zipf=zipf, order=order)


def listed():
    return [
        # one small request's worth of packets looked up by itself: latency
        _case("packets_64", "classify", 10_000, 64),
        # an access list of a thousand rules and a batch of ten thousand packets, full precision
        _case("acl_1k_fp32", "classify", 1024, 10_000, prec="fp32", hidden=128, inside=0.7),
        # a firewall with many wildcards, a million packets, full precision
        _case("fw_64k_fp32", "classify", 65_536, 1_000_000, prec="fp32", mix=0.25),
        # the serving loop: 48 requests of 32 to 65,536 headers, two resident rulesets
        _case("serve_burst", "serve", 100_000, 48),
        # a core router's ruleset and a large batch of skewed traffic, the default precision
        _case("core_512k_bf16", "classify", 524_288, MAX_HEADERS, inside=1.0, zipf=True),
        # the same kind of batch at 100,000 rules, ragged, in the fastest precision with two candidates
        _case("core_100k_fp8", "classify", 100_000, 5_000_003, prec="fp8", topk=2),
        # search alone: no predictor loaded
        _case("search_512k", "classify", 524_288, 4_194_304, prec="none", inside=1.0, zipf=True),
        # 144 prefix-length pairs, with a predictor
        _case("wide_144_bf16", "classify", 524_288, 2_097_152, space="wide", inside=1.0, zipf=True),
        # every prefix length, 387 pairs, no predictor
        _case("wide_387", "classify", 524_288, 1_048_576, prec="none", space="all", inside=1.0, zipf=True),
        # the predictor's scores for inspection and training checks, ragged batch
        _case("scores_bf16", "logits", 10_000, 1_000_003),
        # the paper-size residual predictor's scores
        _case("scores_resnet", "logits", 10_000, 262_144, prec="resnet"),
        # an update round: 100 rules in, a lookup of a million packets, the rules out again
        _case("update_512k", "update", 524_288, 1_000_000),
    ]


def draw(rng):
    case = _drawn(rng)
    del case["name"]
    return case


def _drawn(rng):
    def size(lo, hi):
        return int(round(lo * (hi / lo) ** rng.random()))

    kind = rng.choices(["classify", "logits", "update", "serve"], [8, 3, 1, 1])[0]
    if kind == "serve":
        return _case("", kind, size(10_000, 100_000), rng.randint(8, 64))
    if kind == "update":
        return _case("", kind, size(10_000, 524_288), size(10_000, 1_000_000), mix=rng.choice([0.0, 0.25]))
    space = rng.choices(["narrow", "wide", "all"], [6, 2, 2])[0]
    prec = rng.choice(["fp32", "bf16", "fp8", "resnet"] if kind == "logits" else ["none", "bf16", "fp8", "fp32"])
    hidden = rng.choice([128, 256])
    most = {"resnet": 200_000, "fp32": 1_000_000}.get(prec, 4_000_000)
    if kind == "logits":
        rules, most = 10_000, min(most, 1_000_000)
    else:
        rules = size(1024, 524_288)
        most = min(most, {"narrow": 4_000_000, "wide": 2_000_000, "all": 700_000}[space])
    topk = rng.choice([1, 1, 2]) if space == "all" else rng.choice([1, 1, 2, 4])
    return _case("", kind, rules, size(32, most), prec=prec, hidden=hidden, topk=topk, space=space,
                 mix=rng.choice([0.0, 0.0, 0.25]), inside=rng.choice([0.5, 0.8, 1.0]), zipf=rng.random() < 0.5,
                 order=rng.choice(["specificity", "specificity", "literal"]))


# --- inputs -----------------------------------------------------------------------------

def _rules(case, seed, n=None):
    return synth.make_rules(n or case["rules"], seed=seed * 7 + 1, ordering=case["order"], mix=case["mix"],
                            wide=case["space"] == "wide", all_lengths=case["space"] == "all")


def _headers(case, rules, seed, n=None):
    """[n, 4] int32 header words on the GPU, drawn like ``synth.make_packets``."""
    n = n or case["n"]
    g = torch.Generator(device="cuda").manual_seed(seed * 7 + 2)

    def uniform(hi, count=n):
        return torch.randint(0, hi, (count,), generator=g, device="cuda", dtype=torch.int64)

    def column(name):
        return torch.from_numpy(rules[name].astype(np.int64)).cuda()

    sip, dip, sp, dp, proto = uniform(1 << 32), uniform(1 << 32), uniform(65536), uniform(65536), uniform(256)
    r = len(rules)
    if case["zipf"]:
        cdf = torch.cumsum(1.0 / torch.arange(1, r + 1, device="cuda", dtype=torch.float64), 0)
        u = torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * cdf[-1]
        src = torch.randperm(r, generator=g, device="cuda")[torch.searchsorted(cdf, u).clamp_(max=r - 1)]
    else:
        src = uniform(r)
    inside = torch.rand(n, generator=g, device="cuda") < case["inside"]
    for v, name in ((sip, "sip"), (dip, "dip")):
        ln = column(name + "_len")
        host = ((1 << (32 - ln)) - 1)[src]
        v.copy_(torch.where(inside, column(name)[src] | (v & host), v))
    for v, name in ((sp, "sp"), (dp, "dp")):
        lo, hi = column(name + "_lo")[src], column(name + "_hi")[src]
        v.copy_(torch.where(inside, lo + v % (hi - lo + 1), v))
    proto = torch.where(inside & (column("proto_mask")[src] != 0), column("proto")[src], proto)
    h = torch.stack([sip, dip, sp | (dp << 16), proto], 1)
    return torch.where(h >= 1 << 31, h - (1 << 32), h).to(torch.int32).contiguous()


def _weights(case, seed, n_out):
    """Layers [out][in] with biases, as an untrained network has them."""
    rng = np.random.default_rng(seed * 7 + 3)
    if case["prec"] == "resnet":
        dims, gain = [7] + [512] * 13 + [n_out], [2.0] + [0.7] * 13
    else:
        dims, gain = [104, case["hidden"], case["hidden"], n_out], [1.0] * 3
    Ws = [(rng.standard_normal((o, i), dtype=np.float32) * np.float32(s / np.sqrt(i)))
          for i, o, s in zip(dims, dims[1:], gain)]
    bs = [rng.standard_normal(o, dtype=np.float32) * np.float32(0.1) for o in dims[1:]]
    return Ws, bs


def _bits(h):
    """[n, 104] header bits, most significant first: SIP, DIP, SP, DP, protocol."""
    words = [(h[:, 0], 32), (h[:, 1], 32), (h[:, 2], 16), (h[:, 2] >> 16, 16), (h[:, 3], 8)]
    return torch.cat([(w[:, None] >> torch.arange(k - 1, -1, -1, device=h.device)) & 1 for w, k in words], 1)


def _scales(Ws, bs, h):
    """FP8 activation scales: each hidden layer's largest output over some headers, / 448."""
    a, out = _bits(h[:4096]).double(), [1.0]
    for W, b in list(zip(Ws, bs))[:2]:
        a = torch.relu(a @ torch.from_numpy(W).cuda().double().T + torch.from_numpy(b).cuda().double())
        out.append(float(a.max()) / 448.0)
    return out


# --- states -----------------------------------------------------------------------------

class _State:
    """A program's handles and buffers; gives the handles back when it goes."""

    def __init__(self, case):
        self.case, self.rulesets, self.server = case, [], None

    def ruleset(self, rules):
        rs = T.tang_ruleset_create(torch.cuda.current_device(), rules)
        self.rulesets.append(rs)
        return rs

    def __del__(self):
        if self.server is not None:
            T.tang_server_destroy(self.server)
        if self.rulesets:
            torch.cuda.synchronize()
        for rs in self.rulesets:
            T.tang_ruleset_destroy(rs)


def _train(rs, case, rules, seed):
    """The plain predictor, fitted to tell the tuple of the rule a header was drawn from."""
    C = T.tang_ruleset_num_tuples(rs)
    number = np.full(33 * 33, 0, dtype=np.int64)
    for t in range(C):
        s, d = T.tang_ruleset_tuple(rs, t)
        number[33 * s + d] = t
    hdr, src = synth.make_packets(rules, 32_768, seed=seed * 7 + 4, frac_in=1.0,
                                  zipf_s=1.0 if case["zipf"] else None, return_src=True)
    y = number[33 * rules["sip_len"][src].astype(np.int64) + rules["dip_len"][src]]
    X = train.feature_bits_torch(hdr, "cuda")
    Ws, bs = train.train_mlp(X, y, C, case["hidden"], steps=100, batch=4096, lr=3e-3, seed=seed, device="cuda")
    T.tang_model_load(rs, Ws, bs, case["prec"], topk=case["topk"],
                      act_scales=train.act_scales(Ws, bs, X) if case["prec"] == "fp8" else None)


def prepare(case, seed):
    st = _State(case)
    if case["kind"] == "serve":
        rng = np.random.default_rng(seed * 7 + 5)
        # log-uniform sizes, the same ones for every seed in another order
        sizes = rng.permutation((32 * 2048 ** ((np.arange(case["n"]) + 0.5) / case["n"])).astype(np.int64))
        st.server = T.tang_server_create(torch.cuda.current_device())
        both = []
        for k, n_rules in enumerate((10_000, case["rules"])):
            rules = _rules(case, 2 * seed + k, n_rules)
            rs = st.ruleset(rules)
            _train(rs, case, rules, seed)
            tag = T.tang_server_add_ruleset(st.server, rs)
            T.tang_server_prepare(st.server, tag)
            both.append((tag, rules))
        st.out = np.full(int(sizes.sum()), 0, dtype=np.uint32)
        st.requests, at = [], 0
        for k, n in enumerate(sizes):
            tag, rules = both[int(rng.integers(2))]
            hdr = synth.make_packets(rules, int(n), seed=seed * 1000 + k, frac_in=case["inside"])
            st.requests.append((tag, hdr, st.out[at:at + n]))
            at += int(n)
        return st
    rules = _rules(case, seed)
    rs = st.rs = st.ruleset(rules)
    st.n = case["n"]
    st.hdr = _headers(case, rules, seed)
    st.out = torch.zeros(st.n, dtype=torch.int32, device="cuda")
    if case["kind"] == "logits":
        st.C = T.tang_ruleset_num_tuples(rs)
        Ws, bs = _weights(case, seed, st.C)
        if case["prec"] == "resnet":
            T.tang_model_load_resnet(rs, Ws, bs)
        else:
            T.tang_model_load(rs, Ws, bs, case["prec"], topk=case["topk"],
                              act_scales=_scales(Ws, bs, st.hdr) if case["prec"] == "fp8" else None)
        st.out = torch.zeros(st.n, st.C, dtype=torch.float32, device="cuda")
    elif case["prec"] != "none":
        _train(rs, case, rules, seed)
    if case["kind"] == "update":
        (st.inserts, _), = synth.make_update_stream(rules, rounds=1, per_round=100, seed=seed * 7 + 6)
    return st


def run(st):
    kind, stream = st.case["kind"], torch.cuda.current_stream()
    if kind == "serve":
        reqs = [T.tang_server_submit(st.server, tag, hdr, out) for tag, hdr, out in st.requests]
        for r in reqs:
            T.tang_server_wait(r)
            T.tang_server_req_free(r)
        return st.out
    if kind == "logits":
        T.tang_mlp_forward(st.rs, st.hdr, st.n, st.out, None, stream)
        return st.out
    if kind == "update":
        stream.synchronize()  # an update is applied between lookups, not beside them
        T.tang_insert(st.rs, st.inserts)
        T.tang_classify(st.rs, st.hdr, st.out, st.n, stream)
        stream.synchronize()
        T.tang_delete(st.rs, st.inserts["id"])
        return st.out
    T.tang_classify(st.rs, st.hdr, st.out, st.n, stream)
    return st.out


# --- what a pass cannot do without -------------------------------------------------------

_TUPLES = {"narrow": 25, "wide": 144, "all": 387}


def work(case):
    n, C = case["n"], _TUPLES[case["space"]]
    if case["kind"] == "serve":
        n = n * 8_600                       # mean of a log-uniform request size
    if case["prec"] == "none":
        flops = 0
    elif case["prec"] == "resnet":
        flops = 2 * (7 * 512 + 12 * 512 * 512 + 512 * C)
    else:
        flops = 2 * (104 * case["hidden"] + case["hidden"] ** 2 + case["hidden"] * C)
    # headers in, ids or scores out, and the rules (28 bytes each) once
    out = 4 * C if case["kind"] == "logits" else 4
    return {"bytes": n * (16 + out) + (0 if case["kind"] == "logits" else 28 * case["rules"]), "flops": n * flops}


# --- the answer in 64 bits ----------------------------------------------------------------

def exact(case, seed):
    """Scores in 64-bit floating point from the unrounded weights; rule ids are whole
    numbers and have no such value."""
    if case["kind"] != "logits":
        return None
    rules = _rules(case, seed)
    h = _headers(case, rules, seed)
    C = len(np.unique(rules["sip_len"].astype(np.int64) * 33 + rules["dip_len"]))
    Ws, bs = _weights(case, seed, C)
    W = [torch.from_numpy(w).cuda().double().T.contiguous() for w in Ws]
    b = [torch.from_numpy(x).cuda().double() for x in bs]
    out = []
    for x in h.split(65_536):
        if case["prec"] == "resnet":
            words = [x[:, 0] >> 16, x[:, 0], x[:, 1] >> 16, x[:, 1], x[:, 2], x[:, 2] >> 16, x[:, 3]]
            a = torch.relu(torch.stack([w & 0xFFFF for w in words], 1).double() / 65535.0 @ W[0] + b[0])
            for k in range(1, len(W) - 1, 2):
                a = torch.relu(torch.relu(a @ W[k] + b[k]) @ W[k + 1] + b[k + 1] + a)
        else:
            a = _bits(x).double()
            for k in range(2):
                a = torch.relu(a @ W[k] + b[k])
        out.append(a @ W[-1] + b[-1])
    return torch.cat(out)
