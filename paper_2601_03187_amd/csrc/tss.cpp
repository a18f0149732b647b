// Host side of the tuple space: construction (Sec. 4.3), restricted insertion and
// deletion (Sec. 5.2.1), and the device deltas they produce.
#include <algorithm>
#include <numeric>

#include "tang_internal.hpp"

namespace tang {

namespace {

uint32_t next_pow2(uint64_t v) {
    uint64_t p = 1;
    while (p < v) p <<= 1;
    return (uint32_t)p;
}

bool key_less(const tang_rule_t& a, const tang_rule_t& b) { return key_of(a) < key_of(b); }

// Slot contents of bucket b: a split marker, or the bucket's list.
Slot slot_value(const tang_ruleset_t* rs, uint32_t b) {
    const auto& bk = rs->buckets[b];
    if (bk.split) return Slot{bk.ms, bk.md, bk.t << kTlShift, kSplit | b};
    return Slot{bk.ms, bk.md, (bk.t << kTlShift) | (uint32_t)bk.members.size(), bk.off};
}

// Linear probing from the hash position to the first empty slot.
uint32_t slot_insert(std::vector<Slot>& slots, const Slot& v) {
    uint32_t mask = (uint32_t)slots.size() - 1;
    uint32_t h = key_hash(v.tl >> kTlShift, v.ms, v.md) & mask;
    while (slots[h].tl != kEmptyTL) h = (h + 1) & mask;
    slots[h] = v;
    return h;
}

bool is_main(const tang_ruleset_t::Bucket& bk) { return (bk.t >> kKindShift) == 0; }

// Sub-list key of rule r inside the split main bucket b of tuple t.
tang_ruleset_t::BKey sub_key_of(uint32_t t, uint32_t b, const tang_rule_t& r) {
    if (r.dp_lo == r.dp_hi) return {t | (kSubDp << kKindShift), b, r.dp_lo};
    if (r.sp_lo == r.sp_hi) return {t | (kSubSp << kKindShift), b, r.sp_lo};
    if (r.proto_mask) return {t | (kSubProto << kKindShift), b, r.proto};
    return {t | (kSubRest << kKindShift), b, 0u};
}
tang_ruleset_t::BKey sub_key(const tang_ruleset_t* rs, uint32_t b, uint32_t h) {
    return sub_key_of(rs->buckets[b].t, b, rs->rules[h].r);
}

// A new sub-list (key (tuple | kind, bucket index, value)) enters its bucket's summary.
uint32_t find_or_add_bucket(tang_ruleset_t* rs, const tang_ruleset_t::BKey& k) {
    auto it = rs->bucket_of.find(k);
    if (it != rs->bucket_of.end()) return it->second;
    const uint32_t b = (uint32_t)rs->buckets.size();
    rs->buckets.push_back({k.t, k.ms, k.md, 0, 0, 0, {}, false});
    rs->bucket_of.emplace(k, b);
    const uint32_t kind = k.t >> kKindShift;
    if (kind) {
        SplitInfo& f = rs->split_info[rs->buckets[k.ms].info];
        const uint32_t d = split_dp_bit(k.md), p = split_sp_bit(k.md);
        if (kind == kSubDp) f.dp[d >> 5] |= 1u << (d & 31u);
        else if (kind == kSubSp) f.sp[p >> 5] |= 1u << (p & 31u);
        else if (kind == kSubProto) f.proto |= 1u << split_proto_bit(k.md);
        else f.proto |= 1u << 31;
    }
    return b;
}

// Moves the rules of main bucket b into its sub-lists (order kept); returns every
// bucket whose contents changed (b itself and the sub-lists).
std::vector<uint32_t> split_bucket(tang_ruleset_t* rs, uint32_t b) {
    std::vector<uint32_t> touched{b};
    std::vector<uint32_t> mem;
    mem.swap(rs->buckets[b].members);
    rs->buckets[b].split = true;
    rs->buckets[b].info = (uint32_t)rs->split_info.size();
    rs->split_info.push_back(SplitInfo{});
    for (uint32_t h : mem) {
        const uint32_t sb = find_or_add_bucket(rs, sub_key(rs, b, h));
        auto& sm = rs->buckets[sb].members;
        auto pos = std::upper_bound(sm.begin(), sm.end(), h, [&](uint32_t a, uint32_t x) {
            return key_of(rs->rules[a].r) < key_of(rs->rules[x].r);
        });
        sm.insert(pos, h);
        rs->rules[h].bucket = sb;
        if (std::find(touched.begin(), touched.end(), sb) == touched.end()) touched.push_back(sb);
    }
    return touched;
}

// Slot table at load <= 1/4 (short walks) and the size of the bucket filter, >= 32 bits per
// bucket (blocks of 64 bits); the device sets the filter's bits from the slots.
void rebuild_slots(tang_ruleset_t* rs) {
    const uint64_t nb = rs->buckets.size();
    rs->slots.assign(next_pow2(std::max<uint64_t>(1024, 4 * nb + 4)), Slot{0, 0, kEmptyTL, 0});
    rs->filter_blocks = next_pow2(std::max<uint64_t>(1024, (nb + 1) / 2));
    for (uint32_t b = 0; b < rs->buckets.size(); ++b) {
        auto& bk = rs->buckets[b];
        bk.slot = slot_insert(rs->slots, slot_value(rs, b));
    }
}

// Restricted insertion (Sec. 5.2.1): identical signature, else the first tuple with the
// largest length sum among those with every length <= the rule's; -1 if none.
int choose_tuple(const std::vector<std::pair<uint8_t, uint8_t>>& sigs, uint8_t sl, uint8_t dl) {
    for (size_t i = 0; i < sigs.size(); ++i)
        if (sigs[i].first == sl && sigs[i].second == dl) return (int)i;
    int best = -1, best_sum = -1;
    for (size_t i = 0; i < sigs.size(); ++i) {
        if (sigs[i].first <= sl && sigs[i].second <= dl) {
            int s = sigs[i].first + sigs[i].second;
            if (s > best_sum) { best = (int)i; best_sum = s; }
        }
    }
    return best;
}

}  // namespace

int validate_rule(const tang_rule_t& r) {
    if (r.sip_len > 32 || r.dip_len > 32) return fail(TANG_EINVAL, "prefix length > 32");
    if (r.sp_lo > r.sp_hi || r.dp_lo > r.dp_hi) return fail(TANG_EINVAL, "port range lo > hi");
    if (r.proto_mask != 0 && r.proto_mask != 0xFF)
        return fail(TANG_EINVAL, "proto_mask must be 0 or 0xFF");
    if (r.id == TANG_NO_MATCH) return fail(TANG_EINVAL, "rule id 0xFFFFFFFF is reserved");
    return TANG_OK;
}

tang_rule_t normalise(const tang_rule_t& r) {
    tang_rule_t n = r;
    n.sip &= pmask(r.sip_len);
    n.dip &= pmask(r.dip_len);
    if (n.proto_mask == 0) n.proto = 0;
    return n;
}

Rec make_rec(const tang_ruleset_t* rs, uint32_t h) {
    const auto& hr = rs->rules[h];
    const tang_rule_t& r = hr.r;
    Rec x;
    x.sip = r.sip;
    x.dip = r.dip;
    x.sp = (uint32_t)r.sp_lo | ((uint32_t)r.sp_hi << 16);
    x.dp = (uint32_t)r.dp_lo | ((uint32_t)r.dp_hi << 16);
    // a rule held by a coarser tuple than its own signature (restricted insertion) has
    // its prefixes checked in the scan; in its own tuple the bucket key implies them
    const auto& sig = rs->sigs[hr.tuple];
    const uint32_t check = (sig.first != r.sip_len || sig.second != r.dip_len) ? 1u : 0u;
    x.meta = meta_pack(r.sip_len, r.dip_len, r.proto, r.proto_mask ? 1u : 0u, hr.tuple, check);
    x.cmask = 0;
    x.prio = r.priority;
    x.id = r.id;
    return x;
}

static BoxDev box_of(const tang_ruleset_s::HRule& hr) {
    const tang_rule_t& r = hr.r;
    return BoxDev{r.sip, r.sip | ~pmask(r.sip_len), r.dip, r.dip | ~pmask(r.dip_len),
                  (uint32_t)r.sp_lo | ((uint32_t)r.sp_hi << 16), (uint32_t)r.dp_lo | ((uint32_t)r.dp_hi << 16),
                  (uint32_t)r.proto | ((r.proto_mask ? 1u : 0u) << 8) | (hr.tuple << 16), hr.pos};
}

static Rec dead_rec() {
    Rec x;
    std::memset(&x, 0, sizeof x);
    x.prio = kDead;
    x.id = kDead;
    return x;
}

TupleTable make_tuple_table(const tang_ruleset_t* rs) {
    TupleTable tt;
    std::memset(&tt, 0, sizeof tt);
    uint32_t n = (uint32_t)rs->sigs.size();
    for (uint32_t t = 0; t < n; ++t) {
        tt.t[t].smask = pmask(rs->sigs[t].first);
        tt.t[t].dmask = pmask(rs->sigs[t].second);
        tt.t[t].best_prio = (uint32_t)(rs->tuple_best[t] >> 32);
        tt.t[t].best_id = (uint32_t)rs->tuple_best[t];
    }
    uint64_t after = ~0ull;
    for (uint32_t t = n; t-- > 0;) {
        after = std::min(after, rs->tuple_best[t]);
        tt.after_prio[t] = (uint32_t)(after >> 32);
        tt.after_id[t] = (uint32_t)after;
    }
    std::vector<uint32_t> ord(n);
    std::iota(ord.begin(), ord.end(), 0u);
    std::stable_sort(ord.begin(), ord.end(),
                     [&](uint32_t a, uint32_t b) { return rs->tuple_best[a] < rs->tuple_best[b]; });
    for (uint32_t i = 0; i < n; ++i) {
        tt.rank_prio[i] = (uint32_t)(rs->tuple_best[ord[i]] >> 32);
        tt.rank_id[i] = (uint32_t)rs->tuple_best[ord[i]];
        for (int w = 0; w < kMaxWords; ++w) tt.prefix[i + 1][w] = tt.prefix[i][w];
        tt.prefix[i + 1][ord[i] >> 5] |= 1u << (ord[i] & 31u);
    }
    tt.n = n;
    for (uint32_t t = 0; t < n; ++t) tt.all_mask[t >> 5] |= 1u << (t & 31u);
    tt.nw = rs->nw;
    // filter groups in order of first appearance over the tuples
    for (uint32_t t = 0; t < n; ++t) {
        const uint32_t ls = rs->sigs[t].first, ld = rs->sigs[t].second;
        if (ls == 0 && ld == 0) {
            tt.tg[t] = TupleGroup{kNoGroup, 0u};
            tt.nogroup[t >> 5] |= 1u << (t & 31u);
            continue;
        }
        const uint32_t gk = group_key_of(ls, ld);
        uint32_t g = 0;
        while (g < tt.ngroups && tt.gkey[g] != gk) ++g;
        if (g == tt.ngroups) tt.gkey[tt.ngroups++] = gk;
        tt.tg[t] = TupleGroup{gk, group_salt(gk)};
        tt.gmask[g][t >> 5] |= 1u << (t & 31u);
    }
    uint32_t ops = 0;
    for (uint32_t g = 0; g < tt.ngroups; ++g) {
        FilterGroup& f = tt.fg[g];
        f.dip = tt.gkey[g] >> 6;
        f.mask = pmask(tt.gkey[g] & 63u);
        f.salt = group_salt(tt.gkey[g]);
        for (uint32_t t = 0; t < n; ++t)
            if (tt.tg[t].gkey == tt.gkey[g]) tt.fop[ops++] = FilterOp{f.dip ? tt.t[t].smask : tt.t[t].dmask, filter_salt(t)};
        f.end = ops;
    }
    tt.slot_mask = rs->slots.empty() ? 0 : (uint32_t)rs->slots.size() - 1;
    tt.filter_shift = 32u - (uint32_t)__builtin_ctz(std::max(rs->filter_blocks, 2u));   // a power of two, 1024 or more
    return tt;
}

int build_host(tang_ruleset_t* rs, const tang_rule_t* rules, size_t n) {
    if (n && !rules) return fail(TANG_EINVAL, "rules is NULL");
    if (n > 0x7FFFFFFFu) return fail(TANG_EINVAL, "too many rules");
    rs->rules.reserve(n);
    rs->id2h.reserve(n * 2 + 16);
    for (size_t i = 0; i < n; ++i) {
        int rc = validate_rule(rules[i]);
        if (rc) return rc;
        if (!rs->id2h.emplace(rules[i].id, (uint32_t)i).second)
            return fail(TANG_EEXIST, "repeated rule id " + std::to_string(rules[i].id));
        rs->rules.push_back({normalise(rules[i]), 0, 0, 0, true});
    }
    rs->n_live = n;

    std::vector<uint32_t> order(n);
    std::iota(order.begin(), order.end(), 0u);
    std::sort(order.begin(), order.end(), [&](uint32_t a, uint32_t b) {
        return key_less(rs->rules[a].r, rs->rules[b].r);
    });

    // Tuples by first appearance in (priority, id) order (Table 1 numbering).
    for (uint32_t h : order) {
        auto& hr = rs->rules[h];
        std::pair<uint8_t, uint8_t> sig(hr.r.sip_len, hr.r.dip_len);
        size_t t = 0;
        while (t < rs->sigs.size() && rs->sigs[t] != sig) ++t;
        if (t == rs->sigs.size()) {
            if (rs->sigs.size() == TANG_MAX_TUPLES)
                return fail(TANG_EINVAL, "more than " + std::to_string(TANG_MAX_TUPLES) +
                                             " distinct (sip_len, dip_len) signatures");
            rs->sigs.push_back(sig);
            rs->tuple_best.push_back(key_of(hr.r));
        }
        hr.tuple = (uint32_t)t;
    }
    rs->nw = words_for(rs->sigs.size());

    // Buckets keyed by (tuple, masked SIP, masked DIP), members in key order.
    for (uint32_t h : order) {
        auto& hr = rs->rules[h];
        uint32_t t = hr.tuple;
        tang_ruleset_s::BKey k{t, hr.r.sip & pmask(rs->sigs[t].first), hr.r.dip & pmask(rs->sigs[t].second)};
        const uint32_t b = find_or_add_bucket(rs, k);
        rs->buckets[b].members.push_back(h);
        hr.bucket = b;
    }
    const size_t n_main = rs->buckets.size();
    for (uint32_t b = 0; b < n_main; ++b)
        if (rs->buckets[b].members.size() > kSplitAt) split_bucket(rs, b);
    // Records: buckets laid out contiguously in creation order (by their best key).
    uint32_t off = 0;
    for (auto& bk : rs->buckets) {
        if (bk.members.size() > kMaxBucketLen) return fail(TANG_ENOMEM, "bucket too long");
        bk.off = off;
        bk.cap = (uint32_t)bk.members.size();
        for (uint32_t i = 0; i < bk.cap; ++i) rs->rules[bk.members[i]].pos = off + i;
        off += bk.cap;
    }
    rs->rec_used = off;
    rs->rec_cap = off + std::max<uint32_t>(65536u, off / 4);
    rebuild_slots(rs);
    rs->touched_in.assign(rs->buckets.size() + rs->buckets.size() / 4 + 1024, 0u);
    return TANG_OK;
}

// ---------------------------------------------------------------------------------------
// Device upload of a freshly built ruleset, with the conflict masks computed on the GPU.

// Fills the whole device slot table from the host mirror, and the (cleared) filter's bits,
// through a staging block that the caller releases once the stream is done.
static hipError_t upload_slots(const tang_ruleset_t* rs, SlotDev* d_slots, uint32_t* d_filter, Slot** d_val,
                               hipStream_t s) {
    hipError_t e = dev_alloc(d_val, rs->slots.size() * sizeof(Slot));
    if (e == hipSuccess)
        e = hipMemcpyAsync(*d_val, rs->slots.data(), rs->slots.size() * sizeof(Slot), hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
        e = launch_fill_slots(d_slots, nullptr, *d_val, (uint32_t)rs->slots.size(), rs->d_recs, rs->d_back,
                              d_filter, rs->d_tt, s);
    std::vector<uint32_t> idx;
    std::vector<SplitInfo> info;
    for (const auto& bk : rs->buckets)
        if (bk.split) {
            idx.push_back(bk.slot);
            info.push_back(rs->split_info[bk.info]);
        }
    uint32_t* d_idx = nullptr;
    SplitInfo* d_info = nullptr;
    if (e == hipSuccess && !idx.empty()) {
        e = dev_alloc(&d_idx, idx.size() * sizeof idx[0]);
        if (e == hipSuccess) e = dev_alloc(&d_info, info.size() * sizeof info[0]);
        if (e == hipSuccess) e = hipMemcpyAsync(d_idx, idx.data(), idx.size() * sizeof idx[0], hipMemcpyHostToDevice, s);
        if (e == hipSuccess) e = hipMemcpyAsync(d_info, info.data(), info.size() * sizeof info[0], hipMemcpyHostToDevice, s);
        if (e == hipSuccess) e = launch_fill_split(d_slots, d_idx, d_info, (uint32_t)idx.size(), s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (d_idx) (void)dev_release(d_idx);
        if (d_info) (void)dev_release(d_info);
    }
    return e;
}

// Makes room for a batch of an update in the device block.
static hipError_t grow_block(tang_ruleset_t* rs, size_t bytes) {
    if (bytes <= rs->upd_dev_cap) return hipSuccess;
    hipError_t e = dev_release(rs->upd_dev);
    rs->upd_dev = nullptr;
    rs->upd_dev_cap = 0;
    const size_t cap = std::max<size_t>(bytes + bytes / 2, kUpdDevMin);
    if (e == hipSuccess) e = dev_alloc(&rs->upd_dev, cap);
    if (e == hipSuccess) rs->upd_dev_cap = cap;
    return e;
}

int upload_all(tang_ruleset_t* rs) {
    TANG_HIP(hipSetDevice(rs->device));
    hipStream_t s = rs->upd_stream;
    TANG_HIP(dev_alloc(&rs->d_slots, rs->slots.size() * sizeof(SlotDev)));
    TANG_HIP(dev_alloc(&rs->d_filter, (size_t)rs->filter_blocks * 8));
    TANG_HIP(hipMemset(rs->d_filter, 0, (size_t)rs->filter_blocks * 8));
    TANG_HIP(dev_alloc(&rs->d_recs, (size_t)rs->rec_cap * sizeof(Rec)));
    if (rs->nw == 1) {
        TANG_HIP(dev_alloc(&rs->d_back, (size_t)rs->rec_cap * sizeof(uint32_t)));
        TANG_HIP(hipMemset(rs->d_back, 0, (size_t)rs->rec_cap * sizeof(uint32_t)));
    } else {
        TANG_HIP(dev_alloc(&rs->d_cmask, (size_t)rs->rec_cap * rs->nw * sizeof(uint32_t)));
        TANG_HIP(hipMemset(rs->d_cmask, 0, (size_t)rs->rec_cap * rs->nw * sizeof(uint32_t)));
    }
    TANG_HIP(dev_alloc(&rs->d_tt, sizeof(TupleTable)));
    TANG_HIP(dev_alloc(&rs->d_stats, kStatCopies * sizeof(StatsDev)));
    // here rather than in the first update
    TANG_HIP(hipHostMalloc(&rs->upd_host, kUpdHost, hipHostMallocDefault));
    TANG_HIP(grow_block(rs, 1));

    std::vector<Rec> recs(rs->rec_cap, dead_rec());
    for (uint32_t h = 0; h < rs->rules.size(); ++h)
        if (rs->rules[h].live) recs[rs->rules[h].pos] = make_rec(rs, h);
    TupleTable tt = make_tuple_table(rs);
    TANG_HIP(hipMemcpy(rs->d_recs, recs.data(), recs.size() * sizeof(Rec), hipMemcpyHostToDevice));
    TANG_HIP(hipMemcpy(rs->d_tt, &tt, sizeof tt, hipMemcpyHostToDevice));

    // Boxes of the live rules in ascending key order for the pairwise mask kernel.
    std::vector<uint32_t> order;
    order.reserve(rs->n_live);
    for (uint32_t h = 0; h < rs->rules.size(); ++h)
        if (rs->rules[h].live) order.push_back(h);
    std::sort(order.begin(), order.end(), [&](uint32_t a, uint32_t b) {
        return key_of(rs->rules[a].r) < key_of(rs->rules[b].r);
    });
    if (!order.empty()) {
        std::vector<BoxDev> boxes(order.size());
        for (size_t i = 0; i < order.size(); ++i) {
            boxes[i] = box_of(rs->rules[order[i]]);
        }
        BoxDev* d_boxes = nullptr;
        TANG_HIP(dev_alloc(&d_boxes, boxes.size() * sizeof(BoxDev)));
        hipError_t e = hipMemcpy(d_boxes, boxes.data(), boxes.size() * sizeof(BoxDev),
                                 hipMemcpyHostToDevice);
        if (e == hipSuccess)
            e = launch_conflict_build(d_boxes, boxes.size(), rs->d_recs, rs->d_cmask, rs->nw,
                                      rs->d_tt->all_mask, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        (void)dev_release(d_boxes);
        if (e != hipSuccess) return hip_fail(e, "conflict-mask build");
    }
    // the slots copy their first records, masks included
    Slot* d_val = nullptr;
    hipError_t e = upload_slots(rs, rs->d_slots, rs->d_filter, &d_val, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (d_val) (void)dev_release(d_val);
    if (e != hipSuccess) return hip_fail(e, "slot table upload");
    return TANG_OK;
}

// ---------------------------------------------------------------------------------------
// Updates.

namespace {

// Arrays laid out one after another (16-byte aligned) in the device block.
struct Packer {
    struct Part {
        const void* p;
        size_t at, bytes;
    };
    std::vector<Part> parts;
    size_t size = 0;
    size_t add(const void* p, size_t bytes) {
        const size_t at = size;
        parts.push_back({p, at, bytes});
        size = (at + bytes + 15) & ~(size_t)15;
        return at;
    }
    template <class T>
    size_t add(const std::vector<T>& v) {
        return add(v.data(), v.size() * sizeof(T));
    }
    // To `dev`, through the pinned staging in one copy where they fit; a large batch goes
    // straight from its arrays (new pinned memory costs the host 0.4 ms a MB in page faults).
    hipError_t copy(char* dev, char* pinned, hipStream_t s) const {
        if (size <= kUpdHost) {
            for (const Part& x : parts)
                if (x.bytes) std::memcpy(pinned + x.at, x.p, x.bytes);
            return size ? hipMemcpyAsync(dev, pinned, size, hipMemcpyHostToDevice, s) : hipSuccess;
        }
        hipError_t e = hipSuccess;
        for (const Part& x : parts)
            if (e == hipSuccess && x.bytes) e = hipMemcpyAsync(dev + x.at, x.p, x.bytes, hipMemcpyHostToDevice, s);
        return e;
    }
};

// A block that a batch larger than the ordinary left behind is given back.
hipError_t trim_block(tang_ruleset_t* rs) {
    if (rs->upd_dev_cap <= kUpdDevKeep) return hipSuccess;
    const hipError_t e = dev_release(rs->upd_dev);
    rs->upd_dev = nullptr;
    rs->upd_dev_cap = 0;
    return e;
}

// Rewrites the given buckets on the device: each keeps its slot, its records are
// re-laid in member order (in place if they fit, else at the end of the record array),
// freed record positions are marked dead, conflict masks of moved rules move with them.
// `fresh` are handles of rules not yet on the device. Then the slot entries, tuple
// table, and the conflict masks of the fresh rules are brought up to date.
int flush(tang_ruleset_t* rs, const std::vector<uint32_t>& dirty, const std::vector<uint32_t>& fresh,
          bool rehash) {
    rs->version++;
    if (rs->device == TANG_HOST_ONLY) return TANG_OK;
    TANG_HIP(hipSetDevice(rs->device));
    hipStream_t s = rs->upd_stream;
    // fresh handles are the newest ones, in order
    auto is_fresh = [&](uint32_t h) { return !fresh.empty() && h >= fresh.front(); };

    std::vector<uint32_t> src, dst;   // src: old position, or kNew | index into newrecs
    std::vector<Rec> newrecs;
    const uint32_t kNew = 0x80000000u;
    std::vector<uint32_t> touched_slots, split_slots;
    std::vector<SplitInfo> split_info;
    uint32_t need_end = rs->rec_used;
    // first pass: capacity planning
    for (uint32_t b : dirty) {
        auto& bk = rs->buckets[b];
        uint32_t len = (uint32_t)bk.members.size();
        if (len > bk.cap) need_end += len + std::max<uint32_t>(4u, len / 2);
    }
    if (need_end > rs->rec_cap) {
        uint32_t ncap = std::max<uint32_t>(need_end + need_end / 2, rs->rec_cap * 2);
        Rec* nrec = nullptr;
        TANG_HIP(dev_alloc(&nrec, (size_t)ncap * sizeof(Rec)));
        TANG_HIP(hipMemcpyAsync(nrec, rs->d_recs, (size_t)rs->rec_used * sizeof(Rec),
                                hipMemcpyDeviceToDevice, s));
        std::vector<Rec> tail(ncap - rs->rec_used, dead_rec());
        TANG_HIP(hipMemcpyAsync(nrec + rs->rec_used, tail.data(), tail.size() * sizeof(Rec),
                                hipMemcpyHostToDevice, s));
        if (rs->nw > 1) {
            uint32_t* nmask = nullptr;
            const size_t row = rs->nw * sizeof(uint32_t);
            TANG_HIP(dev_alloc(&nmask, (size_t)ncap * row));
            TANG_HIP(hipMemsetAsync(nmask, 0, (size_t)ncap * row, s));
            TANG_HIP(hipMemcpyAsync(nmask, rs->d_cmask, (size_t)rs->rec_used * row,
                                    hipMemcpyDeviceToDevice, s));
            TANG_HIP(hipStreamSynchronize(s));
            TANG_HIP(dev_release(rs->d_cmask));
            rs->d_cmask = nmask;
        }
        if (rs->nw == 1) {
            uint32_t* nback = nullptr;
            TANG_HIP(dev_alloc(&nback, (size_t)ncap * sizeof(uint32_t)));
            TANG_HIP(hipMemsetAsync(nback, 0, (size_t)ncap * sizeof(uint32_t), s));
            TANG_HIP(hipMemcpyAsync(nback, rs->d_back, (size_t)rs->rec_used * sizeof(uint32_t),
                                    hipMemcpyDeviceToDevice, s));
            TANG_HIP(hipStreamSynchronize(s));
            TANG_HIP(dev_release(rs->d_back));
            rs->d_back = nback;
        }
        TANG_HIP(hipStreamSynchronize(s));
        TANG_HIP(dev_release(rs->d_recs));
        rs->d_recs = nrec;
        rs->rec_cap = ncap;
    }
    for (uint32_t b : dirty) {
        auto& bk = rs->buckets[b];
        uint32_t len = (uint32_t)bk.members.size();
        uint32_t old_off = bk.off, old_cap = bk.cap;
        if (len > bk.cap) {
            bk.off = rs->rec_used;
            bk.cap = len + std::max<uint32_t>(4u, len / 2);
            rs->rec_used += bk.cap;
            for (uint32_t i = len; i < bk.cap; ++i) {  // new slack: dead
                src.push_back(kNew | (uint32_t)newrecs.size());
                dst.push_back(bk.off + i);
                newrecs.push_back(dead_rec());
            }
        }
        for (uint32_t i = 0; i < len; ++i) {
            uint32_t h = bk.members[i];
            auto& hr = rs->rules[h];
            if (is_fresh(h)) {
                src.push_back(kNew | (uint32_t)newrecs.size());
                newrecs.push_back(make_rec(rs, h));
            } else {
                src.push_back(hr.pos);
            }
            dst.push_back(bk.off + i);
            hr.pos = bk.off + i;
        }
        // vacated positions of the old region
        uint32_t keep_lo = (bk.off == old_off) ? len : 0;
        for (uint32_t i = keep_lo; i < old_cap; ++i) {
            src.push_back(kNew | (uint32_t)newrecs.size());
            dst.push_back(old_off + i);
            newrecs.push_back(dead_rec());
        }
        rs->slots[bk.slot] = slot_value(rs, b);
        touched_slots.push_back(bk.slot);
        // the summary of a split bucket whose sub-lists changed
        const auto& main = is_main(bk) ? bk : rs->buckets[bk.ms];
        if (main.split) {
            split_slots.push_back(main.slot);
            split_info.push_back(rs->split_info[main.info]);
        }
    }

    std::sort(touched_slots.begin(), touched_slots.end());
    touched_slots.erase(std::unique(touched_slots.begin(), touched_slots.end()), touched_slots.end());
    std::vector<Slot> vals(touched_slots.size());
    for (size_t i = 0; i < vals.size(); ++i) vals[i] = rs->slots[touched_slots[i]];
    std::vector<FreshDev> fdev(fresh.size());
    for (size_t i = 0; i < fresh.size(); ++i) {
        const auto& hr = rs->rules[fresh[i]];
        const tang_rule_t& r = hr.r;
        fdev[i] = FreshDev{r.sip, pmask(r.sip_len), r.dip, pmask(r.dip_len), r.proto, r.proto_mask ? 0xFFu : 0u,
                           (uint32_t)r.sp_lo | ((uint32_t)r.dp_lo << 16), (uint32_t)r.sp_hi | ((uint32_t)r.dp_hi << 16),
                           r.priority, r.id, hr.tuple, hr.pos};
    }
    const TupleTable tt = make_tuple_table(rs);

    // The batch in the device block, with scratch behind it; the tuple table has a place of
    // its own, and goes through the end of the staging if there is room.
    Packer pk;
    const size_t o_src = pk.add(src), o_dst = pk.add(dst), o_new = pk.add(newrecs), o_fresh = pk.add(fdev),
                 o_idx = pk.add(touched_slots), o_val = pk.add(vals), o_sidx = pk.add(split_slots),
                 o_info = pk.add(split_info);
    const size_t o_stage = (pk.size + 255) & ~(size_t)255, o_mstage = o_stage + dst.size() * sizeof(Rec);
    hipError_t e = grow_block(rs, o_mstage + (rs->nw > 1 ? dst.size() * rs->nw * sizeof(uint32_t) : 0));
    char* const d = static_cast<char*>(rs->upd_dev);
    auto at = [&](size_t off) { return reinterpret_cast<uint32_t*>(d + off); };
    const size_t tt_bytes = tuple_table_bytes(tt);
    const void* tt_from = &tt;
    if (e == hipSuccess) {
        char* const pinned = static_cast<char*>(rs->upd_host);
        e = pk.copy(d, pinned, s);
        if (pk.size + tt_bytes <= kUpdHost) tt_from = std::memcpy(pinned + pk.size, &tt, tt_bytes);
    }
    if (e == hipSuccess) e = hipMemcpyAsync(rs->d_tt, tt_from, tt_bytes, hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
        e = launch_move_records(rs->d_recs, (const Rec*)(d + o_new), at(o_src), at(o_dst), (uint32_t)dst.size(),
                                (Rec*)(d + o_stage), rs->d_back, s);
    if (e == hipSuccess && rs->nw > 1)
        e = launch_move_masks(rs->d_cmask, rs->nw, at(o_src), at(o_dst), (uint32_t)dst.size(), at(o_mstage), s);
    // conflict masks of fresh rules, and their bit in lower-priority rules they meet
    if (e == hipSuccess)
        e = launch_conflict_update(rs->d_recs, rs->d_cmask, rs->nw, rs->rec_used, (const FreshDev*)(d + o_fresh),
                                   (uint32_t)fdev.size(), rs->d_back, rs->d_slots, s);
    // slots, with their first records as they are now, and the filter bits of new buckets
    if (e == hipSuccess && rehash) {
        SlotDev* ns = nullptr;
        uint32_t* nf = nullptr;
        Slot* d_val = nullptr;
        e = hipStreamSynchronize(s);
        if (e == hipSuccess) e = dev_alloc(&ns, rs->slots.size() * sizeof(SlotDev));
        if (e == hipSuccess) e = dev_alloc(&nf, (size_t)rs->filter_blocks * 8);
        if (e == hipSuccess) e = hipMemsetAsync(nf, 0, (size_t)rs->filter_blocks * 8, s);
        if (e == hipSuccess) e = upload_slots(rs, ns, nf, &d_val, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (d_val) (void)dev_release(d_val);
        if (e == hipSuccess) {
            (void)dev_release(rs->d_slots);
            (void)dev_release(rs->d_filter);
            rs->d_slots = ns;
            rs->d_filter = nf;
        } else {
            if (ns) (void)dev_release(ns);
            if (nf) (void)dev_release(nf);
        }
    } else if (e == hipSuccess) {
        e = launch_fill_slots(rs->d_slots, at(o_idx), (const Slot*)(d + o_val), (uint32_t)vals.size(), rs->d_recs,
                              rs->d_back, rs->d_filter, rs->d_tt, s);
        if (e == hipSuccess)
            e = launch_fill_split(rs->d_slots, at(o_sidx), (const SplitInfo*)(d + o_info),
                                  (uint32_t)split_slots.size(), s);
    }
    hipError_t e2 = hipStreamSynchronize(s);
    if (e2 == hipSuccess) e2 = trim_block(rs);
    if (e != hipSuccess) return hip_fail(e, "update flush");
    if (e2 != hipSuccess) return hip_fail(e2, "update flush sync");
    return TANG_OK;
}

// The host mirror already holds a batch when its device flush runs; if the flush fails
// (an allocation or a HIP call), host and device disagree, so the ruleset refuses every
// later call that reads its device state (tang_ruleset_export still gives the live rules
// a rebuild starts from).
int flush_or_fail(tang_ruleset_t* rs, const std::vector<uint32_t>& dirty,
                  const std::vector<uint32_t>& fresh, bool rehash) {
    const int rc = flush(rs, dirty, fresh, rehash);
    if (rc) {
        rs->failed = true;
        return fail(rc, std::string("update not applied on the device (") + tang_last_error() +
                            "); the ruleset is unusable, rebuild it from tang_ruleset_export");
    }
    return TANG_OK;
}

// The buckets that a batch of an update touches, each once: a bucket carries the number of
// the last batch that did (a set of them takes twice the time of a whole large batch).
void begin_batch(tang_ruleset_t* rs) {
    if (++rs->batch == 0) {
        std::fill(rs->touched_in.begin(), rs->touched_in.end(), 0u);
        rs->batch = 1;
    }
}
bool first_touch(tang_ruleset_t* rs, uint32_t b) {
    if (b >= rs->touched_in.size()) rs->touched_in.resize(rs->buckets.size() + rs->buckets.size() / 2, 0u);
    if (rs->touched_in[b] == rs->batch) return false;
    rs->touched_in[b] = rs->batch;
    return true;
}

}  // namespace

int apply_insert(tang_ruleset_t* rs, const tang_rule_t* rules, size_t n) {
    if (n == 0) return TANG_OK;
    if (!rules) return fail(TANG_EINVAL, "rules is NULL");
    // Validate the whole batch first (all-or-nothing).
    std::unordered_map<uint32_t, int> seen;
    auto sigs = rs->sigs;
    // Every list must stay within what a slot can describe (kMaxBucketLen): each rule's
    // destination list is bounded by its current length plus the batch's rules bound for
    // it (a main bucket that splits during the batch only sheds rules into sub-lists).
    std::unordered_map<tang_ruleset_s::BKey, size_t, tang_ruleset_s::BKeyHash> list_len;
    for (size_t i = 0; i < n; ++i) {
        int rc = validate_rule(rules[i]);
        if (rc) return rc;
        if (rs->id2h.count(rules[i].id) || !seen.emplace(rules[i].id, 1).second)
            return fail(TANG_EEXIST, "rule id " + std::to_string(rules[i].id) + " is live or repeated");
        int t = choose_tuple(sigs, rules[i].sip_len, rules[i].dip_len);
        if (t < 0) {
            if (sigs.size() == tuple_limit(rs->nw))
                return fail(TANG_EINVAL, "insert would need tuple " + std::to_string(sigs.size() + 1) +
                                             " (the ruleset was built with " + std::to_string(rs->nw) +
                                             " conflict-mask words per rule)");
            t = (int)sigs.size();
            sigs.emplace_back(rules[i].sip_len, rules[i].dip_len);
        }
        const tang_rule_t r = normalise(rules[i]);
        tang_ruleset_s::BKey key{(uint32_t)t, r.sip & pmask(sigs[t].first), r.dip & pmask(sigs[t].second)};
        auto mb = rs->bucket_of.find(key);
        if (mb != rs->bucket_of.end() && rs->buckets[mb->second].split)
            key = sub_key_of((uint32_t)t, mb->second, r);
        auto ins = list_len.emplace(key, 0);
        if (ins.second) {
            auto lb = rs->bucket_of.find(key);
            if (lb != rs->bucket_of.end()) ins.first->second = rs->buckets[lb->second].members.size();
        }
        if (++ins.first->second > kMaxBucketLen)
            return fail(TANG_ENOMEM, "insert would make a bucket list longer than " +
                                         std::to_string(kMaxBucketLen) + " rules");
    }
    std::vector<uint32_t> dirty, fresh;
    begin_batch(rs);
    size_t nb_before = rs->buckets.size();
    for (size_t i = 0; i < n; ++i) {
        tang_rule_t r = normalise(rules[i]);
        int t = choose_tuple(rs->sigs, r.sip_len, r.dip_len);
        if (t < 0) {
            t = (int)rs->sigs.size();
            rs->sigs.emplace_back(r.sip_len, r.dip_len);
            rs->tuple_best.push_back(key_of(r));
        }
        uint32_t h = (uint32_t)rs->rules.size();
        rs->rules.push_back({r, (uint32_t)t, 0, 0, true});
        rs->id2h[r.id] = h;
        rs->n_live++;
        if (rs->sigs[t] != std::make_pair(r.sip_len, r.dip_len)) rs->n_coarse++;
        rs->tuple_best[t] = std::min(rs->tuple_best[t], key_of(r));
        tang_ruleset_s::BKey k{(uint32_t)t, r.sip & pmask(rs->sigs[t].first),
                               r.dip & pmask(rs->sigs[t].second)};
        const uint32_t mb = find_or_add_bucket(rs, k);
        const uint32_t b = rs->buckets[mb].split ? find_or_add_bucket(rs, sub_key(rs, mb, h)) : mb;
        auto& mem = rs->buckets[b].members;
        auto pos = std::upper_bound(mem.begin(), mem.end(), h, [&](uint32_t a, uint32_t x) {
            return key_of(rs->rules[a].r) < key_of(rs->rules[x].r);
        });
        mem.insert(pos, h);
        rs->rules[h].bucket = b;
        std::vector<uint32_t> changed{b};
        if (b == mb && mem.size() > kSplitAt) changed = split_bucket(rs, mb);
        for (uint32_t c : changed)
            if (first_touch(rs, c)) dirty.push_back(c);
        fresh.push_back(h);
    }
    // new buckets need slots; grow the table when it would pass half full
    bool rehash = false;
    if (rs->buckets.size() != nb_before) {
        // keep the slot table at most 1/3 full and the filter at >= half its bits per bucket
        if (3 * rs->buckets.size() + 3 > rs->slots.size() ||
            rs->buckets.size() > 4 * (size_t)rs->filter_blocks) {
            rebuild_slots(rs);
            rehash = true;
        } else {
            for (size_t b = nb_before; b < rs->buckets.size(); ++b) {
                auto& bk = rs->buckets[b];
                bk.slot = slot_insert(rs->slots, Slot{bk.ms, bk.md, bk.t << kTlShift, 0});
            }
        }
    }
    return flush_or_fail(rs, dirty, fresh, rehash);
}

int apply_delete(tang_ruleset_t* rs, const uint32_t* ids, size_t n) {
    if (n == 0) return TANG_OK;
    if (!ids) return fail(TANG_EINVAL, "ids is NULL");
    std::unordered_map<uint32_t, int> seen;
    for (size_t i = 0; i < n; ++i) {
        if (!rs->id2h.count(ids[i]) || !seen.emplace(ids[i], 1).second)
            return fail(TANG_ENOTFOUND, "rule id " + std::to_string(ids[i]) + " is not live");
    }
    std::vector<uint32_t> dirty;
    begin_batch(rs);
    for (size_t i = 0; i < n; ++i) {
        uint32_t h = rs->id2h[ids[i]];
        auto& hr = rs->rules[h];
        auto& mem = rs->buckets[hr.bucket].members;
        mem.erase(std::find(mem.begin(), mem.end(), h));
        hr.live = false;
        rs->id2h.erase(ids[i]);
        rs->n_live--;
        if (rs->sigs[hr.tuple] != std::make_pair(hr.r.sip_len, hr.r.dip_len)) rs->n_coarse--;
        if (first_touch(rs, hr.bucket)) dirty.push_back(hr.bucket);
    }
    return flush_or_fail(rs, dirty, {}, false);
}

}  // namespace tang
