// Internal declarations of the gfx950 packet classifier: device data layout, the slot
// hash, the ruleset object and the kernel launchers.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <cstring>
#include <memory>
#include <mutex>
#include <string>
#include <unordered_map>
#include <vector>

#include "../../include/tang.h"

namespace tang {

// ---------------------------------------------------------------------------------------
// Device layout.
//
// Slot (16 B): one bucket of the global open-addressing table. The key is the full
// (tuple, SIP & mask_t, DIP & mask_t), so an answer never depends on the hash function.
//   tl = tuple << 20 | bucket length; kEmptyTL marks a never-used slot.
//   off = first record of the bucket in the record array.
struct alignas(16) Slot {
    uint32_t ms, md, tl, off;
};
constexpr uint32_t kEmptyTL = 0xFFFFFFFFu;
constexpr uint32_t kTlShift = 20;
constexpr uint32_t kMaxBucketLen = (1u << kTlShift) - 1u;

// Long buckets are split. A bucket that would hold more than kSplitAt rules keeps its
// slot only as a marker (len 0, off = kSplit | bucket index); its rules move to four
// sub-lists stored in the same table under keys (tuple | kind << 9, bucket index, value):
//   kSubDp    rules with an exact DP, value = that DP
//   kSubSp    rules with an exact SP (DP not exact), value = that SP
//   kSubProto rules with an exact protocol and no exact port, value = the protocol
//   kSubRest  every other rule, value 0
// A header reads the four lists its own DP, SP and protocol select; each list is in
// (priority, id) order, so the first match of each is its best and the minimum of the
// four is the bucket's best. Rules that cannot match the header are never scanned.
constexpr uint32_t kSplit = 0x80000000u;
constexpr uint32_t kSplitAt = 16;
enum : uint32_t { kSubDp = 1, kSubSp = 2, kSubProto = 3, kSubRest = 4 };
constexpr uint32_t kKindShift = 9;   // tuples < 512; tuple | kind << 9 fits the slot's 12 bits

// Conflict masks: one word per rule (in the record) for rulesets of at most 32 tuples;
// wider ones keep a side array indexed like the records, kMaskWords words per rule for
// at most 256 tuples and kMaxWords for more (up to TANG_MAX_TUPLES).
constexpr int kMaskWords = 8;
constexpr int kMaxWords = TANG_MAX_TUPLES / 32;
// Mask words for a tuple count, and the tuple limit of a mask width.
inline uint32_t words_for(size_t tuples) {
    return tuples <= 32 ? 1u : tuples <= 32u * kMaskWords ? (uint32_t)kMaskWords : (uint32_t)kMaxWords;
}
inline size_t tuple_limit(uint32_t nw) { return 32u * (size_t)nw; }
// Candidate tuples in the predictor's output word: one byte each up to 256 tuples (at
// most 4 candidates), 16 bits each above (at most 2).
__host__ __device__ inline uint32_t cand_bits(int n_tuples) { return n_tuples > 256 ? 16u : 8u; }
inline int max_topk(int n_tuples) {
    const int k = n_tuples > 256 ? 2 : TANG_MAX_TOPK;
    return k < n_tuples ? k : n_tuples;
}

// Rec (32 B): one rule as the bucket scan reads it, hot half first: ports, priority and the
// protocol/length word, which decide a match for a rule held by its own tuple. The second
// half matters for a match (its id and conflict mask), a priority tie (the id breaks it), or
// a rule held by a coarser tuple than its own signature (its prefixes must be checked). A
// step of the search loads both halves; long lists are passed over by their first ones.
//   sp, dp   : lo | hi << 16 (inclusive)
//   prio     : priority; (prio, id) is the key, kDead in both marks a vacated record
//   meta     : proto (bits 0-7) | exact-proto (8) | prefix check (9) | sip_len (10-15)
//              | dip_len (16-21) | tuple (22-31)
//   sip, dip : prefix values, bits beyond the length zeroed
//   id       : rule id
//   cmask    : conflict tuples of a ruleset of at most 32 tuples (wider ones: side
//              array) -- tuples that hold a higher-priority rule whose box meets this
//              rule's box (a superset after deletes)
struct alignas(16) Rec {
    uint32_t sp, dp, prio, meta, sip, dip, id, cmask;
};
constexpr uint32_t kDead = 0xFFFFFFFFu;

// A slot on the device (64 B): the slot and a copy of its list's first record, so that a
// probe costs one line where it took one for the slot and one for the record. Most lists
// hold one rule. The copy is refreshed whenever the slot, the record or (rulesets of at
// most 32 tuples) the record's conflict mask changes.
struct alignas(64) SlotDev {
    Slot s;
    Rec first;
    uint32_t pad[4];
};
// In place of a first record, the slot of a split bucket says which of its sub-lists may
// exist: a bit per exact DP value (128 of them, in the record's first half), per exact SP
// value (96) and per protocol (31), and whether there is a rest list. A header then walks
// only to the lists it may find.
struct alignas(16) SplitInfo {
    uint32_t dp[4], sp[3], proto;   // proto: bit 31 the rest list
};
static_assert(sizeof(SplitInfo) == sizeof(Rec), "the summary takes the record's place");
__host__ __device__ inline uint32_t split_dp_bit(uint32_t dp) { return (dp * 0x9E3779B1u) >> 25; }
__host__ __device__ inline uint32_t split_sp_bit(uint32_t sp) { return ((sp * 0x9E3779B1u) >> 24) * 96u >> 8; }
__host__ __device__ inline uint32_t split_proto_bit(uint32_t proto) { return proto % 31u; }

__host__ __device__ inline uint32_t meta_pack(uint32_t sl, uint32_t dl, uint32_t proto,
                                              uint32_t exact, uint32_t tuple, uint32_t check) {
    return proto | (exact << 8) | (check << 9) | (sl << 10) | (dl << 16) | (tuple << 22);
}
__host__ __device__ inline uint32_t meta_proto(uint32_t m) { return m & 255u; }
__host__ __device__ inline uint32_t meta_exact(uint32_t m) { return (m >> 8) & 1u; }
__host__ __device__ inline uint32_t meta_check(uint32_t m) { return (m >> 9) & 1u; }
__host__ __device__ inline uint32_t meta_sl(uint32_t m) { return (m >> 10) & 63u; }
__host__ __device__ inline uint32_t meta_dl(uint32_t m) { return (m >> 16) & 63u; }
__host__ __device__ inline uint32_t meta_tuple(uint32_t m) { return m >> 22; }

// Prefix mask of length l (0..32): the top l bits; l = 0 gives 0 (no shift by 32).
__host__ __device__ inline uint32_t pmask(uint32_t l) {
    return l == 0 ? 0u : (0xFFFFFFFFu << (32u - l));
}

// Per-tuple data: masks and the smallest (priority, id) key of any rule ever placed in
// the tuple (a lower bound after deletes, used to stop searching tuples early).
struct TupleDev {
    uint32_t smask, dmask, best_prio, best_id;
};
// Filter groups: the tuples whose longer prefix is the SIP (sip_len >= dip_len) share a
// group per SIP length, the others a group per DIP length; tuple (0, 0), whose only
// possible key always has a bucket, has none. At most 64 groups (32 lengths per field).
constexpr int kMaxGroups = 64;
constexpr uint32_t kNoGroup = 0xFFu;
// A group and its tuples as the filter reads them (one scalar load each): the group's own
// field (dip: 0 SIP, 1 DIP) and its mask and salt, and the end of its FilterOps (they begin
// where the group before ends); a tuple's mask on the other field and its salt.
struct alignas(16) FilterGroup {
    uint32_t dip, mask, salt, end;
};
struct alignas(8) FilterOp {
    uint32_t omask, salt;   // the salt's low 9 bits are the tuple
};
constexpr int kOpsAtOnce = 4;   // FilterOps per scalar load; the table has as many to spare
struct alignas(8) FilterOps {
    FilterOp op[kOpsAtOnce];
};
// A tuple's group for a lane that tests one tuple of its own: key (kNoGroup: none) and salt.
struct alignas(8) TupleGroup {
    uint32_t gkey, salt;
};
struct TupleTable {
    TupleDev t[TANG_MAX_TUPLES];
    uint32_t rank_prio[TANG_MAX_TUPLES], rank_id[TANG_MAX_TUPLES];  // best keys in that order
    uint32_t n;                       // number of tuples
    uint32_t all_mask[kMaxWords];     // bits of all tuples
    uint32_t slot_mask;               // slots - 1
    uint32_t filter_shift;            // 32 - log2(filter blocks)
    uint32_t nw;                      // mask words of this ruleset (1, kMaskWords or kMaxWords)
    TupleGroup tg[TANG_MAX_TUPLES];
    // smallest best key among tuples t, t + 1, ...: a probe in tuple order stops there once
    // its answer is better
    uint32_t after_prio[TANG_MAX_TUPLES], after_id[TANG_MAX_TUPLES];
    uint32_t ngroups;
    uint32_t gkey[kMaxGroups];        // side (bit 6: 1 = DIP) | prefix length (bits 0-5)
    uint32_t gmask[kMaxGroups][kMaxWords];  // tuples of each group
    uint32_t nogroup[kMaxWords];      // tuples without a group (always pass)
    FilterGroup fg[kMaxGroups];
    FilterOp fop[TANG_MAX_TUPLES + 2 * kOpsAtOnce];
    // prefix[k]: the k tuples of lowest best key, as mask words; rows past n are not copied
    // to the device
    uint32_t prefix[TANG_MAX_TUPLES + 1][kMaxWords];
};
inline size_t tuple_table_bytes(const TupleTable& tt) {
    return offsetof(TupleTable, prefix) + (tt.n + 1) * sizeof tt.prefix[0];
}

// Key hash: the masked SIP salted by the tuple key, multiplied and folded, then the masked
// DIP, multiplied and folded twice (each stage a bijection, so structured keys -- prefixes
// whose only varying bits are the top byte -- do not collapse). The low bits pick the slot;
// the slot stores the full key, so answers never depend on the hash.
// The bucket filter uses its own hashes (filter_block / filter_hash below).
__host__ __device__ inline uint32_t key_hash(uint32_t t, uint32_t ms, uint32_t md) {
    // a 24-bit product (full rate on the vector units); tuple keys are below 2^12
    const uint32_t salt = ((t + 1u) & 0xFFFFFFu) * 0x9E3779u;
    uint32_t x = (ms ^ salt) * 0x85EBCA6Bu;
    x ^= x >> 15;
    x = (x ^ md) * 0xC2B2AE35u;
    x ^= x >> 15;
    x *= 0x2C1B3C6Du;
    return x ^ (x >> 16);
}
// Bucket filter, blocked by prefix group. A main bucket (t, ms, md) of a tuple with
// lengths (ls, ld) belongs to the tuple's filter group: the SIP group of length ls when
// ls >= ld, else the DIP group of length ld. The group value v (ms or md) picks one
// 64-bit block, filter_block(group_salt, v, shift); the other masked field o (md or ms) and
// the tuple pick two bits in it, filter_hash(filter_salt(t), o) (a blocked Bloom filter with
// two probes: with about two buckets per block a tuple passes by chance 0.3% of the time
// instead of 3% -- it matters when a packet tests a hundred tuples). A header then reads one
// block per group for all the tuples of that group (at most 5 blocks for the 25 tuples of five
// lengths per field), where a bit per tuple took one load each. A clear bit means no
// bucket; a set pair may be a collision, which only costs a slot walk. Placement never
// affects answers.
// Both hashes are made of sums of two 16-bit products and a salt: one instruction at the full
// rate of the vector units, where a 32-bit product takes four times as long. (The key hash
// stays with products: with dot16 the search gained 0 to 4%, but 1,820 rules' headers met 25%
// more slots.) Addresses cluster, so what varies may be any few bits of a field:
//  - the block needs up to 20 bits and is picked once per group: two sums with a fold between
//    them, whose top bits count;
//  - the two positions need ten and are picked once per tuple: bits 14-23 of one sum. Every
//    bit of either half of the field reaches them, and a run of consecutive values fills them
//    evenly, which the top bits do not do (a /8's or a /24's addresses fall on a few of those:
//    with the top bits of one sum for both hashes 65,536 rules of 25 tuples in one /8 let 6.6
//    tuples per header pass by chance, and this lets 0.7, as independent hashes do).
// Over 26 kinds of rulesets (1,000 to 524,288 rules, 9 to 387 tuples; uniform addresses, one
// network of /8 to /24, many networks, consecutive subnets and hosts, nested prefixes) between
// 0.8 and 1.25 times as many tuples pass as with independent hashes; over others at most 1.5.
// Search with the top bits and so, all addresses in one /8: 25 tuples, 65,536 rules, 4,194,304
// headers 419 and 361 us; 144 tuples, 524,288 rules, 1,048,576 headers 336 and 257; 387 tuples,
// 65,536 rules, 524,288 headers 301 and 229. Uniform addresses: 25 tuples alike, 387 tuples,
// 524,288 rules, 1,048,576 headers 567 and 533.
__host__ __device__ inline uint32_t dot16(uint32_t x, uint32_t c, uint32_t add) {
#ifdef __HIP_DEVICE_COMPILE__
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    return __builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, x), __builtin_bit_cast(u16x2, c), add, false);
#else
    return (x & 0xFFFFu) * (c & 0xFFFFu) + (x >> 16) * (c >> 16) + add;
#endif
}
__host__ __device__ inline uint32_t filter_block(uint32_t salt, uint32_t v, uint32_t shift) {
    uint32_t x = dot16(v, 0xAB83A349u, salt);
    x ^= x >> 15;
    return dot16(x, 0xF64DD9EFu, 0u) >> shift;
}
__host__ __device__ inline uint32_t group_salt(uint32_t gkey) { return (gkey + 1u) * 0xCCEA71FFu; }
// (low 9 bits: the tuple)
__host__ __device__ inline uint32_t filter_salt(uint32_t t) { return ((t + 1u) * 0xFD724453u & ~0x1FFu) | t; }
constexpr uint32_t kFilterHashC = 0xC5C78BC9u;
__host__ __device__ inline uint32_t filter_hash(uint32_t salt, uint32_t o) { return dot16(o, kFilterHashC, salt); }
// One bit in each half of the block, counted from the top: shifting each half left by its
// position brings the bit to the sign, so a test is two shifts and an AND. Bit 31 of the
// result: set in both halves.
__host__ __device__ inline uint32_t filter_pos_x(uint32_t h) { return (h >> 19) & 31u; }
__host__ __device__ inline uint32_t filter_pos_y(uint32_t h) { return (h >> 14) & 31u; }
__device__ inline uint32_t filter_has(uint2 blk, uint32_t h) {
    return (blk.x << filter_pos_x(h)) & (blk.y << filter_pos_y(h));
}
__host__ __device__ inline uint32_t group_key_of(uint32_t ls, uint32_t ld) {
    return ls >= ld ? ls : (64u | ld);
}

// Device-side counters for tang_stats_t (kStatCopies copies, summed on the host).
struct StatsDev {
    unsigned long long packets, probes, slots, records, top1, fallbacks, nomatch, filters, steps,
        rounds;
};
constexpr int kStatCopies = 64;

// Updates' staging (see tang_ruleset_s): 800 rules fill the pinned part.
constexpr size_t kUpdHost = (size_t)256 << 10;
constexpr size_t kUpdDevMin = (size_t)512 << 10, kUpdDevKeep = (size_t)16 << 20;

// Rule box used by the conflict-mask kernels (key order), 32 B.
struct alignas(16) BoxDev {
    uint32_t slo, shi, dlo, dhi, sp, dp, pt, pos;  // pt = proto | exact << 8 | tuple << 16
};

// A fresh rule as an update compares it with every record: prefixes with their masks,
// protocol with its mask (0: any), the low and the high bounds of both ports (SP | DP << 16).
struct alignas(16) FreshDev {
    uint32_t sip, sm, dip, dm, proto, pm, lo, hi, prio, id, tuple, pos;
};

// ---------------------------------------------------------------------------------------
// Model on the device.

constexpr int kMaxHidden = 256;
constexpr int kOutPad = 32;   // output classes padded to 2 MFMA tiles
constexpr int kInPad = 128;   // 104 input bits padded to 128

// Weights are loaded ahead of their use, also where a layer or a wave's class tiles have
// ended and nothing follows: such a load takes the last stored piece again. It must not run
// past the end: the scalar offset of a buffer load is not part of its bounds check.
__host__ __device__ constexpr uint32_t stored(uint32_t want, uint32_t count) {
    return want < count ? want : count - 1u;
}
// Plain networks: the 16-class tile of the output layer (stored in pairs) for class tile ct.
__host__ __device__ constexpr uint32_t class_tile(uint32_t ct, uint32_t classes) {
    return stored(ct, 2u * ((classes + 31u) / 32u));
}
// The class tile of a wave's i-th turn when eight waves share `tiles` class tiles for `columns`
// header columns: whole rounds of eight tiles for all columns, then the tiles left, a wave
// taking one column of one (turn_column) per turn.
__host__ __device__ constexpr uint32_t turn_tile(uint32_t i, uint32_t wave, uint32_t tiles, uint32_t columns) {
    const uint32_t rounds = tiles / 8u;
    return i < rounds ? wave + 8u * i : 8u * rounds + (wave + 8u * (i - rounds)) / columns;
}
__host__ __device__ constexpr uint32_t turn_column(uint32_t i, uint32_t wave, uint32_t tiles, uint32_t columns) {
    return (wave + 8u * (i - tiles / 8u)) % columns;
}
// Turns of a wave: its rounds, and its share of the columns of the tiles left.
__host__ __device__ constexpr uint32_t turns(uint32_t wave, uint32_t tiles, uint32_t columns) {
    return tiles / 8u + (tiles % 8u * columns + 7u - wave) / 8u;
}
// Residual network of nb blocks: the byte offset of wave `wave`'s K block kb (4 KB) of block
// layer l, and the bias row (512 floats) of that layer.
__host__ __device__ constexpr uint32_t res_weight_at(uint32_t l, uint32_t wave, uint32_t kb, uint32_t nb) {
    return (stored(l, 2u * nb) * 8u + wave) * 65536u + kb * 4096u;
}
__host__ __device__ constexpr uint32_t res_bias_row(uint32_t l, uint32_t nb) { return 1u + stored(l, 2u * nb); }

struct ModelDev {
    int loaded = 0;
    int kind = 0;     // 0: the plain 104 -> H -> H -> C network; 1: the residual network
    tang_precision_t prec = TANG_FP32;
    int hidden = 0;
    int n_out = 0;    // C
    uint32_t w3frags = 0;  // output-layer weight fragments (classes padded to 32-blocks)
    int topk = 1;
    // Weight fragments for the three layers in MFMA A-operand order, and biases.
    void* w[3] = {nullptr, nullptr, nullptr};
    size_t wbytes[3] = {0, 0, 0};
    // FP32 models: every layer as three BF16 planes (w), or, where weights or outputs are out
    // of the planes' range (split = false), FP32 fragments with W1 as three planes beside
    // them, for the input layer on BF16 MFMAs (its inputs are bits, so products are exact)
    bool split = false;
    void* w1x3 = nullptr;
    float* bias = nullptr;   // [hidden | hidden | 32] floats
    float deq[3] = {1, 1, 1};     // FP8: s_a * s_w per layer
    float inv_a[3] = {1, 1, 1};   // FP8: 1 / s_a per layer (layer 0 unused)
    float rq[2] = {1, 1};         // FP8 hidden layers: 2^-e, e the requantisation exponent
    // Residual network: input layer FP32 [512][8] and BF16 layer weights.
    int n_blocks = 0;
    float* rin = nullptr;
    void* rw = nullptr;
    uint32_t rw_bytes = 0;
    uint32_t cus = 0;   // workgroups of a launch at most
    void* ws = nullptr; // 192 MB that callers' allocators budget for; the kernel needs none of it
    size_t bytes = 0;
};

}  // namespace tang

// ---------------------------------------------------------------------------------------
// The ruleset object behind tang_ruleset_t.

struct tang_ruleset_s {
    struct HRule {
        tang_rule_t r;      // normalised
        uint32_t tuple;
        uint32_t bucket;
        uint32_t pos;       // record index on the device
        bool live;
    };
    struct Bucket {
        uint32_t t, ms, md;             // t | kind << kKindShift (kind 0: main bucket)
        uint32_t slot;
        uint32_t off, cap;
        std::vector<uint32_t> members;  // rule handles in (priority, id) order
        bool split = false;             // main bucket whose rules live in sub-lists
        uint32_t info = 0;              // split: index of its summary
    };
    struct BKey {
        uint32_t t, ms, md;
        bool operator==(const BKey& o) const { return t == o.t && ms == o.ms && md == o.md; }
    };
    struct BKeyHash {
        size_t operator()(const BKey& k) const {
            return (size_t)tang::key_hash(k.t, k.ms, k.md);
        }
    };

    int device = TANG_HOST_ONLY;
    std::vector<HRule> rules;                      // handle-indexed, never shrinks
    std::unordered_map<uint32_t, uint32_t> id2h;   // live id -> handle
    size_t n_live = 0;
    size_t n_coarse = 0;   // live rules held by a tuple coarser than their own signature
    std::vector<std::pair<uint8_t, uint8_t>> sigs; // tuple signatures
    std::vector<uint64_t> tuple_best;              // lower bound on keys per tuple
    std::vector<Bucket> buckets;
    std::unordered_map<BKey, uint32_t, BKeyHash> bucket_of;
    std::vector<tang::Slot> slots;                 // host mirror of the slot table
    std::vector<tang::SplitInfo> split_info;       // summaries of the split buckets' sub-lists
    uint32_t filter_blocks = 0;                    // size of the bucket filter (device only)
    std::vector<uint32_t> touched_in;              // last batch that touched a bucket, and the
    uint32_t batch = 0;                            // number of the present one
    uint32_t rec_used = 0, rec_cap = 0;
    uint32_t nw = 1;   // conflict-mask words per rule (fixed at build: words_for(tuples))

    // device state
    tang::SlotDev* d_slots = nullptr;
    uint32_t* d_back = nullptr;    // nw = 1: slot index + 1 of a list's first record, else 0
    uint32_t* d_filter = nullptr;
    tang::Rec* d_recs = nullptr;
    uint32_t* d_cmask = nullptr;   // nw > 1: nw words per record position
    tang::TupleTable* d_tt = nullptr;
    tang::StatsDev* d_stats = nullptr;
    hipStream_t upd_stream = nullptr;
    // Updates' staging, released with the ruleset: pinned host memory (kUpdHost) that a batch
    // is packed into, and the device block that it is copied to (with scratch behind it; kept
    // up to kUpdDevKeep). One update runs at a time and ends synchronised, so both are free
    // again.
    void* upd_host = nullptr;
    void* upd_dev = nullptr;
    size_t upd_dev_cap = 0;
    tang::ModelDev model;
    std::mutex stats_mu;
    uint64_t version = 0;   // bumped by every change that captured launches depend on
    bool failed = false;    // an update's device flush failed: host and device disagree

    size_t device_bytes() const;
};

namespace tang {

// Error reporting (thread-local message + code).
int fail(int code, const std::string& msg);
int hip_fail(hipError_t e, const char* what);
#define TANG_HIP(call)                                         \
    do {                                                       \
        hipError_t _e = (call);                                \
        if (_e != hipSuccess) return ::tang::hip_fail(_e, #call); \
    } while (0)

// Host tuple space (tss.cpp).
int validate_rule(const tang_rule_t& r);
tang_rule_t normalise(const tang_rule_t& r);
inline uint64_t key_of(const tang_rule_t& r) { return ((uint64_t)r.priority << 32) | r.id; }
int build_host(tang_ruleset_t* rs, const tang_rule_t* rules, size_t n);
int upload_all(tang_ruleset_t* rs);
TupleTable make_tuple_table(const tang_ruleset_t* rs);
Rec make_rec(const tang_ruleset_t* rs, uint32_t h);
int apply_insert(tang_ruleset_t* rs, const tang_rule_t* rules, size_t n);
int apply_delete(tang_ruleset_t* rs, const uint32_t* ids, size_t n);

// Internal device memory: through the caller's allocator when one is set
// (tang_set_allocator), else hipMalloc / hipFree; a block is released through the
// allocator that provided it.
hipError_t dev_alloc(void** p, size_t bytes);
hipError_t dev_release(void* p);
template <class T>
inline hipError_t dev_alloc(T** p, size_t bytes) {
    return dev_alloc(reinterpret_cast<void**>(p), bytes);
}

// Kernel launchers (k_classify.hip, k_build.hip, k_mlp.hip).
// d_live (optional): a device word holding the live header count, read by the kernels at
// their start; lanes and workgroups past min(n, *d_live) do nothing. A launch recorded
// once into a graph for n headers then serves any smaller batch without padding.
hipError_t launch_classify(const tang_ruleset_t* rs, const tang_header_t* d_hdr,
                           uint32_t* d_out, size_t n, int kcand, hipStream_t s, bool stats,
                           const uint32_t* d_live = nullptr);
hipError_t launch_conflict_build(const BoxDev* d_boxes, size_t n, Rec* d_recs, uint32_t* d_cmask,
                                 uint32_t nw, const uint32_t* all_mask,
                                 hipStream_t s);
// back, slots (nw = 1): the mask copies in the slots of records that are their list's first.
hipError_t launch_conflict_update(Rec* d_recs, uint32_t* d_cmask, uint32_t nw, uint32_t rec_used,
                                  const FreshDev* d_fresh, uint32_t n_new, const uint32_t* d_back,
                                  SlotDev* d_slots, hipStream_t s);
// Clears `back` (nw = 1) at every destination.
hipError_t launch_move_records(Rec* d_recs, const Rec* d_src_recs, const uint32_t* d_src,
                               const uint32_t* d_dst, uint32_t n, Rec* d_stage, uint32_t* d_back,
                               hipStream_t s);
// nw > 1: the mask rows move with their records (the same src / dst lists; new sources
// get zero rows), through a stage of n rows.
hipError_t launch_move_masks(uint32_t* d_cmask, uint32_t nw, const uint32_t* d_src,
                             const uint32_t* d_dst, uint32_t n, uint32_t* d_stage, hipStream_t s);
// Writes slots with their first records and sets `back` (nw = 1) and the filter bits of
// main buckets: slot d_idx[i] = d_val[i], or slot i without d_idx.
hipError_t launch_fill_slots(SlotDev* d_slots, const uint32_t* d_idx, const Slot* d_val, uint32_t n,
                             const Rec* d_recs, uint32_t* d_back, uint32_t* d_filter,
                             const TupleTable* d_tt, hipStream_t s);
// Writes the summaries of split buckets into their slots.
hipError_t launch_fill_split(SlotDev* d_slots, const uint32_t* d_idx, const SplitInfo* d_info, uint32_t n,
                             hipStream_t s);
// Largest batch of tang_classify_host_noalloc (its static staging: 5 MiB per GPU).
constexpr size_t kNoAllocMaxHeaders = (size_t)1 << 18;
// tang_classify's body; every launch is on stream s (callers may be capturing it).
// d_live: as for launch_classify (with a plain MLP or no model; not with stats).
int classify_async(tang_ruleset_t* rs, const tang_header_t* d_hdr, uint32_t* d_rule_id, size_t n,
                   hipStream_t s, tang_stats_t* stats, const uint32_t* d_live = nullptr);
hipError_t launch_mlp(const tang_ruleset_t* rs, const tang_header_t* d_hdr, size_t n,
                      uint32_t* d_cand_packed, float* d_logits, uint16_t* d_cand16,
                      hipStream_t s, const uint32_t* d_live = nullptr);
int search_host(const tang_ruleset_t* rs, const tang_header_t* hdr, const uint32_t* cand,
                uint32_t* out, size_t n, uint32_t kcand, uint32_t threads, bool exact,
                tang_stats_t* stats);
int resnet_prepare(tang_ruleset_t* rs, const tang_resnet_desc_t* d, const float* const* W,
                   const float* const* b, tang_precision_t p);
hipError_t launch_resnet(const tang_ruleset_t* rs, const tang_header_t* d_hdr, size_t n,
                         uint32_t* cand, float* logits, uint16_t* cand16, hipStream_t s);
int model_prepare(tang_ruleset_t* rs, const tang_mlp_desc_t* d, const float* const* W,
                  const float* const* b, tang_precision_t p, const float* act_scales);
void model_free(ModelDev& m);

}  // namespace tang
