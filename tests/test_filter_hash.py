"""The bucket filter's hashes on addresses as rulesets have them: uniform, all in one network,
in many networks, consecutive subnets and hosts. Tuples that pass the filter by chance must
not be many more than with independent hash functions in the same table (each costs the
search a slot walk)."""
import ctypes

import numpy as np
import pytest

from paper_2601_03187_amd import synth
from tests import _internal

BODY = """
#include <unordered_set>
static uint64_t mix(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
struct Key {
    uint32_t t, s, d;
    bool operator==(const Key& o) const { return t == o.t && s == o.s && d == o.d; }
};
struct KeyHash {
    size_t operator()(const Key& k) const { return mix(mix(((uint64_t)k.s << 32) | k.d) + k.t); }
};
// Tuples (of lengths sl, dl) per 1000 headers that pass the filter without a bucket, the
// filter as the library builds it (own) or with independent hash functions.
extern "C" double passes(int own, uint32_t C, const uint32_t* sl, const uint32_t* dl, uint32_t n, const uint32_t* t,
                         const uint32_t* sip, const uint32_t* dip, uint32_t nh, const uint32_t* hs, const uint32_t* hd) {
    std::unordered_set<Key, KeyHash> have;
    for (uint32_t i = 0; i < n; ++i) have.insert({t[i], sip[i] & pmask(sl[t[i]]), dip[i] & pmask(dl[t[i]])});
    uint32_t blocks = 1024;
    while (blocks < (have.size() + 1) / 2) blocks *= 2;
    const uint32_t shift = 32 - __builtin_ctz(blocks);
    std::vector<uint32_t> bits(2 * blocks, 0);
    auto place = [&](uint32_t t, uint32_t s, uint32_t d, uint32_t& blk, uint32_t& x, uint32_t& y) {
        const uint32_t gk = group_key_of(sl[t], dl[t]), v = gk & 64u ? d : s, o = gk & 64u ? s : d;
        if (own) {
            blk = filter_block(group_salt(gk), v, shift);
            const uint32_t h = filter_hash(filter_salt(t), o);
            x = filter_pos_x(h);
            y = filter_pos_y(h);
        } else {
            blk = mix(mix(gk) + v) & (blocks - 1);
            const uint64_t h = mix(mix(t + 1000) + o);
            x = h & 31;
            y = (h >> 8) & 31;
        }
    };
    uint32_t b, x, y;
    for (const Key& k : have) {
        if (!sl[k.t] && !dl[k.t]) continue;
        place(k.t, k.s, k.d, b, x, y);
        bits[2 * b] |= 0x80000000u >> x;
        bits[2 * b + 1] |= 0x80000000u >> y;
    }
    uint64_t count = 0;
    for (uint32_t i = 0; i < nh; ++i)
        for (uint32_t k = 0; k < C; ++k) {
            const uint32_t s = hs[i] & pmask(sl[k]), d = hd[i] & pmask(dl[k]);
            if ((!sl[k] && !dl[k]) || have.count({k, s, d})) continue;
            place(k, s, d, b, x, y);
            count += ((bits[2 * b] << x) & (bits[2 * b + 1] << y)) >> 31;
        }
    return 1e3 * count / nh;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = _internal.compile_host(str(tmp_path_factory.mktemp("internal")), BODY)
    so.passes.restype = ctypes.c_double
    return so


def _addresses(kind, n, rng, nets):
    """`kind`: "uniform", "COUNT/LENGTH" (that many random networks), "subnets" (1,024
    consecutive /24s, 20 hosts each) or "hosts" (4,096 consecutive addresses)."""
    r = rng.integers(0, 1 << 32, n)
    if kind == "uniform":
        return r
    if kind == "subnets":
        return 0xC0A80000 + (r % 1024) * 256 + 1 + rng.integers(0, 20, n)
    if kind == "hosts":
        return 0x0A140000 + r % 4096
    count, length = map(int, kind.split("/"))
    low = (1 << (32 - length)) - 1
    base = nets.integers(0, 1 << 32, count) & ~low
    return base[rng.integers(0, count, n)] | (r & low)


@pytest.mark.parametrize("src,dst", [("uniform", "uniform"), ("1/8", "1/8"), ("1/12", "1/12"), ("1/16", "1/24"),
                                     ("200/12", "200/12"), ("1000/16", "40/20"), ("subnets", "subnets"),
                                     ("subnets", "hosts"), ("hosts", "1/8")])
@pytest.mark.parametrize("space,n", [("narrow", 10_000), ("narrow", 65_536), ("wide", 65_536), ("all", 65_536)])
def test_chance_passes_stay_near_independent_hashes(lib, space, n, src, dst):
    """At most twice as many as with independent hashes, plus 0.05 per header (a handful
    among thousands of headers)."""
    shape = synth.make_rules(n, seed=41, wide=space == "wide", all_lengths=space == "all")
    pair = 33 * shape["sip_len"].astype(np.int64) + shape["dip_len"]
    sig, tup = np.unique(pair, return_inverse=True)
    rng, headers = np.random.default_rng(42), 1500
    a, b = (_addresses(k, n + headers, rng, np.random.default_rng(s)) for k, s in ((src, 43), (dst, 44)))
    u = [np.ascontiguousarray(x, dtype=np.uint32)
         for x in (sig // 33, sig % 33, tup, a[:n], b[:n], a[n:], b[n:])]
    p = [x.ctypes.data_as(ctypes.c_void_p) for x in u]
    own, ind = (lib.passes(k, len(sig), p[0], p[1], n, p[2], p[3], p[4], headers, p[5], p[6]) for k in (1, 0))
    assert own <= 2 * ind + 50, (own, ind)
