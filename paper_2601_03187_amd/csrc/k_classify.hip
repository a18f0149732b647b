// Search stage of the two-stage classification (Sec. 5.1.1):
//   1. probe the predicted tuples: truncate SIP/DIP to the tuple's prefix lengths,
//      hash, walk the open-addressing slots to the bucket, and compare the bucket's
//      rules one by one in (priority, id) order -- the first match is the bucket's best;
//   2. certify: if a rule matched, probe the tuples of its conflict mask (the only
//      tuples that can hold a better matching rule); if nothing matched, probe every
//      remaining tuple (the paper's post-verification search, Sec. 5.1.1); in both
//      cases a tuple whose best (lowest) key cannot beat the current answer is skipped.
// Before any slot walk, a bit of the bucket filter rules out a tuple that has no bucket
// for the header's masked addresses. The filter is blocked by prefix group (the tuples
// sharing their longer field's length): one 8-byte block answers every tuple of its
// group, so certification loads one block per group, eight independent loads at a time.
// The headers with tuples left then go through a queue to the wave's lanes, each lane
// running one header's probes. A slot carries a copy of its list's first record, since
// random lines are what the search pays for.
// Candidates come packed in the output word from the MLP (one byte per candidate, 16
// bits above 256 tuples). Tuple spaces of more than 32 tuples use the same steps over
// multiword tuple masks (8 words up to 256 tuples, 16 up to 512), with conflict masks in
// a side array.
#include <algorithm>

#include "tang_internal.hpp"

namespace tang {
namespace {

constexpr uint32_t kNoTuple = 0xFFFFFFFFu;
// Sets of 64 headers per wave, rulesets of at most 32 tuples: two, through a queue, from this
// many headers on, one below. More sets keep a wave's lanes busy longer, fewer make more waves
// (one set and two: 100,000 rules, 600,000 headers 52 and 55 us, 1,048,576 76 and 77,
// 4,194,304 233 and 212; 512k rules with 25% wildcard-heavy rules 79 and 71, 120 and 106, 405
// and 324). Four sets need 36 KB of LDS and leave four waves per SIMD: 1,800 rules, 4.2M
// headers 143 us against 125 with two, 600,000 headers 36 against 28.
constexpr uint32_t kQueueFrom = 1u << 19;
// Long lists are passed over kScan records at a time (4.2M headers, 512k rules in one /8: 3 and
// 4 records 394 and 384 us, 4 and 8 391 and 375; 65,536 rules, 25% wildcard-heavy: 291 and 296,
// 294 and 321), looked for every kScanTry steps (1,800 rules in short lists: every step 209 us,
// every eighth 203, not at all 195).
constexpr uint32_t kScan = 4, kScanTry = 8;

__device__ __forceinline__ bool kless(uint32_t p1, uint32_t i1, uint32_t p2, uint32_t i2) {
    return p1 < p2 || (p1 == p2 && i1 < i2);
}

__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Orders a wave's own LDS accesses: one lane's writes before another lane's reads. The
// hardware runs a wave's LDS instructions in order; this keeps the compiler from moving them.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Lanes of `m` below this one.
__device__ __forceinline__ uint32_t lanes_below(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// A header's search state in LDS: its best answer so far (cm: the answer's conflict mask,
// or its record position where masks are in the side array) and the tuples it still has
// to probe (work: the mask itself, or which words of the wave's `work` rows are not zero).
struct alignas(16) Entry {
    uint32_t prio, id, cm, work;
};

// NW: conflict-mask words (1 for at most 32 tuples, kMaskWords for up to 256, kMaxWords
// above). Tuple sets are NW-word bit masks (word t / 32, bit t % 32). R: sets of 64 headers
// per wave. U: records of a list per step: a small batch lasts as long as its longest list
// scan, so more records in flight pay there, until the registers cost waves.
//
// What bounds it (25 tuples, 512k rules, no predictor, 4.2M Zipf headers: 267 us): vector
// issue, about 190 us of it, and random 128-byte lines beside it: the card serves 265 G
// random accesses/s that hit an L2 and 60 G that miss it, and a header needs about 7.5 and
// 1.1 of them, together 193 us. One header per lane with a slot table, its records and the
// filter each on lines of their own (8.6 and 2.0 accesses) took 396 us, 93% of it vector
// issue: the wave ran its probe loop as long as its busiest lane needed, 25 steps where a
// header needs 3.1 on average.
template <bool STATS, int NW, int R, int U>
__global__ __launch_bounds__(256) void k_classify(const uint4* __restrict__ hdr,
                                                  uint32_t* __restrict__ out, uint32_t n,
                                                  const SlotDev* __restrict__ slots,
                                                  const Rec* __restrict__ recs,
                                                  const uint32_t* __restrict__ cmask_rows,
                                                  const uint2* __restrict__ filter,
                                                  const TupleTable* __restrict__ ttg, int kcand,
                                                  StatsDev* __restrict__ st,
                                                  const uint32_t* __restrict__ live) {
    constexpr uint32_t NT = 32u * NW;
    constexpr uint32_t CB = NW > kMaskWords ? 16u : 8u;   // bits per packed candidate
    constexpr uint32_t NE = 64u * R;                      // entries per wave
    // The largest tables leave out the ranks, which then come from memory: 28 KB of LDS and
    // five waves per SIMD, 32 KB and four with them.
    constexpr bool kRankLds = NW <= kMaskWords;
    __shared__ TupleDev s_t[NT];
    __shared__ uint2 s_after[NT];   // smallest best key from a tuple on
    __shared__ uint2 s_rank[kRankLds ? NT : 1];   // best keys in ascending order
    // with one set a lane keeps its own header, and nothing is queued
    __shared__ uint4 s_hdr[4][R > 1 ? NE : 1];
    __shared__ Entry s_ent[4][R > 1 ? NE : 1];
    __shared__ uint16_t s_queue[4][R > 1 ? NE : 1];
    __shared__ uint32_t s_work[4][NW > 1 ? NW : 1][NW > 1 ? NE : 1];
    __shared__ uint32_t s_prefix[NW == 1 ? NT + 1 : 1];
    __shared__ uint32_t s_tup[4][STATS ? NE : 1];   // the answer's tuple
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (live) n = min(n, *live);
    if (blockIdx.x * 4u * NE >= n) return;   // uniform over the block (a live count below the grid)
    const uint32_t ntup = ttg->n, ngroups = ttg->ngroups;
    const uint32_t slot_mask = ttg->slot_mask, filter_shift = ttg->filter_shift;
    for (uint32_t k = tid; k < ntup; k += 256u) {
        s_t[k] = ttg->t[k];
        s_after[k] = make_uint2(ttg->after_prio[k], ttg->after_id[k]);
        if (kRankLds) s_rank[k] = make_uint2(ttg->rank_prio[k], ttg->rank_id[k]);
    }
    if constexpr (NW == 1)
        if (tid <= NT) s_prefix[tid] = ttg->prefix[tid][0];
    __syncthreads();
    const uint32_t base = (blockIdx.x * 4u + wave) * NE;
    const uint32_t cnt = base < n ? min(n - base, NE) : 0u;   // this wave's headers
    uint4* const hd = s_hdr[wave];
    Entry* const ent = s_ent[wave];
    uint16_t* const queue = s_queue[wave];
    uint4 own_hdr = make_uint4(0u, 0u, 0u, 0u);
    Entry own = Entry{kDead, kDead, 0u, 0u};
    auto header = [&](uint32_t e) -> uint4& { return R > 1 ? hd[e] : own_hdr; };
    auto entry = [&](uint32_t e) -> Entry& { return R > 1 ? ent[e] : own; };
    uint32_t n_probe = 0, n_slots = 0, n_recs = 0, top1 = 0, fb = 0, nm = 0;
    uint32_t n_filter = 0, n_steps = 0, n_rounds = 0;
    // a vector instruction takes one scalar operand: the salt, so this one is held in a vector
    uint32_t hash_c = kFilterHashC;
    asm("" : "+v"(hash_c));

    // Pass 0 probes the predicted tuples, pass 1 certifies.
    for (uint32_t pass = kcand > 0 ? 0u : 1u; pass < 2u; ++pass) {
        uint32_t qn = 0;   // headers with tuples to probe
#pragma unroll 1
        for (uint32_t r = 0; r < (uint32_t)R; ++r) {
            const uint32_t e = r * 64u + lane;
            const bool active = e < cnt;
            uint4 h = make_uint4(0u, 0u, 0u, 0u);
            if (pass == 0 || kcand == 0) {
                if (active) h = hdr[base + e];
                header(e) = h;
                if (STATS) s_tup[wave][e] = kNoTuple;
            } else {
                h = header(e);
            }
            const uint32_t sip = h.x, dip = h.y;
            uint32_t cand = 0;
            if (kcand > 0 && active) cand = out[base + e];
            uint32_t work = 0;   // NW = 1: tuples to probe; else its words that are not zero
            if (pass == 0) {
                if constexpr (NW > 1) {
#pragma unroll
                    for (int w = 0; w < NW; ++w) s_work[wave][w][e] = 0;
                }
                for (int c = 0; c < kcand; ++c) {
                    const uint32_t t = (cand >> (CB * c)) & ((1u << CB) - 1u);
                    if (!active || t >= ntup) continue;
                    const TupleGroup tg = ttg->tg[t];
                    bool pass_f = true;
                    if (tg.gkey != kNoGroup) {
                        const uint32_t ms = sip & s_t[t].smask, md = dip & s_t[t].dmask;
                        const bool by_dip = (tg.gkey & 64u) != 0u;   // the group's field
                        const uint32_t v = by_dip ? md : ms, o = by_dip ? ms : md;
                        const uint2 blk = filter[filter_block(tg.salt, v, filter_shift)];
                        pass_f = filter_has(blk, filter_hash(filter_salt(t), o)) >> 31;
                        if (STATS) ++n_filter;
                    }
                    if (!pass_f) continue;
                    if constexpr (NW == 1) {
                        work |= 1u << t;
                    } else {
                        s_work[wave][t >> 5][e] |= 1u << (t & 31u);
                        work |= 1u << (t >> 5);
                    }
                }
                entry(e) = Entry{kDead, kDead, 0u, work};
            } else {
                Entry b{kDead, kDead, 0u, 0u};
                if (kcand > 0) b = entry(e);
                const bool found = b.id != kDead;
                if (STATS) fb += active && !found;
                // The certification set: the answer's conflict mask, or every tuple after a
                // miss, without the tuples probed in pass 0 and those whose best key cannot
                // beat the answer -- in ascending best-key order the tuples that can form a
                // prefix, found by a binary search.
                uint32_t k = ntup;
                if (__ballot(found)) {
                    k = 0;
#pragma unroll
                    for (uint32_t step = NT; step > 0; step >>= 1)
                        if (k + step <= ntup) {
                            const uint32_t j = k + step - 1u;
                            const uint2 r = kRankLds ? s_rank[j] : make_uint2(ttg->rank_prio[j], ttg->rank_id[j]);
                            if (kless(r.x, r.y, b.prio, b.id)) k += step;
                        }
                }
                uint32_t todo[NW];
                if constexpr (NW == 1) {
                    todo[0] = active ? (found ? b.cm : ~0u) & s_prefix[k] : 0u;
                } else {
#pragma unroll
                    for (int w = 0; w < NW; ++w) todo[w] = active ? ttg->all_mask[w] : 0u;
                    if (active && found) {
                        const uint4* row = reinterpret_cast<const uint4*>(cmask_rows + (size_t)b.cm * NW);
                        const uint4* pre = reinterpret_cast<const uint4*>(ttg->prefix[k]);
#pragma unroll
                        for (int q = 0; q < NW / 4; ++q) {
                            const uint4 m = row[q], p = pre[q];
                            todo[4 * q] = m.x & p.x;
                            todo[4 * q + 1] = m.y & p.y;
                            todo[4 * q + 2] = m.z & p.z;
                            todo[4 * q + 3] = m.w & p.w;
                        }
                    }
                }
                for (int c = 0; c < kcand; ++c) {
                    const uint32_t t = (cand >> (CB * c)) & ((1u << CB) - 1u);
                    if constexpr (NW == 1) {
                        if (t < ntup) todo[0] &= ~(1u << t);
                    } else {
#pragma unroll
                        for (int w = 0; w < NW; ++w)
                            if (t >> 5 == (uint32_t)w) todo[w] &= ~(1u << (t & 31u));
                    }
                }
                // The filter: eight groups at a time, each lane's blocks loaded together, then
                // each group's tuples. Groups and tuples are the same for every lane, so masks
                // and salts are scalars, four tuples to a load, and a test is ten vector
                // instructions without a branch; a lane that does not need a group reads block 0
                // with the others and drops the outcome. This is most of what a wide ruleset's
                // search does: 387 tuples, 1M headers 842 us with one scalar load, a 32-bit
                // product and a branch per tuple, 594 so (548 with the headers in registers, five
                // waves per SIMD instead of four; 484 with long lists passed over and the
                // filter's present hashes).
                uint32_t hits = 0;
                if constexpr (NW == 1) {
                    hits = todo[0] & ttg->nogroup[0];
                } else {
#pragma unroll
                    for (int w = 0; w < NW; ++w) s_work[wave][w][e] = todo[w] & ttg->nogroup[w];
                }
                const bool every = NW > 1 && !__ballot(found);   // no lane can leave a group out
                uint32_t k0 = 0;
                FilterOps ops = *reinterpret_cast<const FilterOps*>(ttg->fop);
                for (uint32_t g0 = 0; g0 < ngroups; g0 += 8u) {
                    uint2 blk[8];
                    if (STATS) n_rounds += active;
#pragma unroll
                    for (uint32_t q = 0; q < 8u; ++q) {
                        blk[q] = make_uint2(0u, 0u);
                        if (g0 + q < ngroups) {
                            const FilterGroup fg = ttg->fg[g0 + q];
                            uint32_t need = active;
                            if (!every) {
                                need = 0;
#pragma unroll
                                for (int w = 0; w < NW; ++w) need |= todo[w] & ttg->gmask[g0 + q][w];
                            }
                            const uint32_t v = (fg.dip ? dip : sip) & fg.mask;
                            blk[q] = filter[need ? filter_block(fg.salt, v, filter_shift) : 0u];
                            if (STATS) n_filter += need != 0;
                        }
                    }
#pragma unroll
                    for (uint32_t q = 0; q < 8u; ++q) {
                        if (g0 + q < ngroups) {
                            const FilterGroup fg = ttg->fg[g0 + q];
                            const uint32_t ov = fg.dip ? sip : dip;
                            // the groups' tuples follow one another; the next four are loaded
                            // while these are tested
                            while (k0 < fg.end) {
                                const uint32_t m = min(fg.end - k0, (uint32_t)kOpsAtOnce);
                                const FilterOps now = ops;
                                k0 += m;
                                ops = *reinterpret_cast<const FilterOps*>(ttg->fop + k0);
#pragma unroll
                                for (uint32_t j = 0; j < (uint32_t)kOpsAtOnce; ++j) {
                                    if (j >= m) break;
                                    const FilterOp op = now.op[j];
                                    const uint32_t has =
                                        filter_has(blk[q], dot16(ov & op.omask, hash_c, op.salt)) >> 31;
                                    if constexpr (NW == 1)
                                        hits |= has << (op.salt & 31u);
                                    else
                                        atomicOr(&s_work[wave][(op.salt & 0x1FFu) >> 5][e], has << (op.salt & 31u));
                                }
                            }
                        }
                    }
                }
                if constexpr (NW == 1) {
                    work = hits & todo[0];
                } else {
#pragma unroll
                    for (int w = 0; w < NW; ++w) {
                        const uint32_t m = s_work[wave][w][e] & todo[w];
                        s_work[wave][w][e] = m;
                        work |= m ? 1u << w : 0u;
                    }
                }
                entry(e) = Entry{b.prio, b.id, b.cm, work};
            }
            if constexpr (R > 1) {
                const unsigned long long has = __ballot(work != 0u);
                if (work) queue[qn + lanes_below(has)] = (uint16_t)e;
                qn += (uint32_t)__popcll(has);
            }
        }
        wave_sync();

        // The probe loop: each lane runs one header's probes as single steps (a slot with its
        // bucket's first record, or a further record), its tuples in index order -- tuples are
        // numbered by first appearance in priority order, so good answers come early --
        // skipping any whose best key can no longer beat the answer. A lane that is done
        // takes the next header of the queue, so the wave's lanes stay busy until the queue
        // is empty.
        enum : uint32_t { P_IDLE = 0, P_NEXT, P_START, P_SLOT, P_REC };
        uint32_t taken = 0;
        uint32_t ps = P_IDLE, e = 0, sip = 0, dip = 0, ports = 0, proto = 0;
        uint32_t bp = kDead, bid = kDead, bcm = 0;   // the lane's header's best
        uint32_t cur = 0, word = 0, nz = 0;   // tuples left (of mask word `word`), words left
        uint32_t ct = 0, tk = 0, k0 = 0, k1 = 0, bi = 0, left = 0;
        uint32_t sub = 0;   // sub-lists of a split bucket still to visit (bit 0 DP, SP, protocol, rest)
        uint32_t at = 0, walk = 0;   // slot or record index; steps of the slot walk
        uint32_t try_scan = kScanTry;
        auto take = [&](uint32_t e) {
            const uint4 h = header(e);
            const Entry b = entry(e);
            sip = h.x;
            dip = h.y;
            ports = h.z;
            proto = h.w & 0xFFu;
            bp = b.prio;
            bid = b.id;
            bcm = b.cm;
            cur = NW == 1 ? b.work : 0u;
            nz = NW == 1 ? 0u : b.work;
        };
        if constexpr (R == 1) {
            e = lane;
            take(e);
            ps = own.work ? P_NEXT : P_IDLE;
        }
        for (;;) {
            if constexpr (R > 1) {
                const unsigned long long idle = __ballot(ps == P_IDLE);
                if (idle && taken < qn) {
                    const uint32_t q = taken + lanes_below(idle);
                    if (ps == P_IDLE && q < qn) {
                        e = queue[q];
                        take(e);
                        ps = P_NEXT;
                    }
                    taken = min(qn, taken + (uint32_t)__popcll(idle));
                }
            }
            if (ps == P_NEXT) {
                ps = P_IDLE;
                for (;;) {
                    if constexpr (NW > 1) {
                        if (!cur && nz) {
                            word = (uint32_t)__builtin_ctz(nz);
                            nz &= nz - 1u;
                            cur = s_work[wave][word][e];
                        }
                    }
                    if (!cur) break;
                    const uint32_t t = 32u * word + (uint32_t)__builtin_ctz(cur);
                    cur &= cur - 1u;
                    const uint2 after = s_after[t];
                    if (!kless(after.x, after.y, bp, bid)) {   // nor any later tuple
                        cur = 0;
                        nz = 0;
                        break;
                    }
                    const TupleDev td = s_t[t];
                    if (kless(td.best_prio, td.best_id, bp, bid)) {
                        ct = t;
                        tk = t;
                        k0 = sip & td.smask;
                        k1 = dip & td.dmask;
                        sub = 0;
                        ps = P_START;
                        if (STATS) ++n_probe;
                        break;
                    }
                }
                if (R > 1 && ps == P_IDLE) ent[e] = Entry{bp, bid, bcm, 0u};   // nothing left to probe
            }
            const unsigned long long busy = __ballot(ps != P_IDLE);
            if (!busy) {
                if (R == 1 || taken >= qn) break;
                continue;
            }
            if (STATS) ++n_steps;
            if (ps == P_START) {
                at = key_hash(tk, k0, k1) & slot_mask;
                walk = 0;
                ps = P_SLOT;
            }
            // one step's loads: the slot (its key and its bucket's first record share a
            // 64-byte line) or the next U records of the list. Every lane loads, an idle one
            // slot 0 with the others, and the step is decided in selects: with a branch per
            // state the copies where the branches meet were a third of the loop's vector
            // instructions.
            const bool slot = ps == P_SLOT, rec = ps == P_REC;
            const uint32_t sp = ports & 0xFFFFu, dp = ports >> 16;
            auto fits = [&](const uint4& b) {   // ports and protocol
                return ((uint32_t)(sp >= (b.x & 0xFFFFu)) & (uint32_t)(sp <= (b.x >> 16)) &
                        (uint32_t)(dp >= (b.y & 0xFFFFu)) & (uint32_t)(dp <= (b.y >> 16)) &
                        ((uint32_t)(meta_exact(b.w) == 0) | (uint32_t)(proto == meta_proto(b.w)))) != 0u;
            };
            // Where most of the wave's busy lanes are in long lists, they first pass over records
            // that cannot matter, kScan at a time, by their first halves (and the one where a lane
            // stops by its own prefixes, if a coarser tuple holds it); the record where a lane
            // stops for good goes through a step. Looked for every kScanTry steps, and every
            // second while it holds. Lists of a record or two do not pay for it (1,800 rules, 4.2M
            // headers 196 us without and 200 with); where headers meet long lists it is most of the
            // time (25 tuples and one list of 4,000 rules that half of the headers go through,
            // 524,288 headers 4.96 and 1.16 ms; 512k rules in one /8 301 and 115 us; 65,536 rules and
            // 17,000 more held by coarser tuples, with the BF16 predictor, 1M headers 1,480 and 1,510
            // Mpps, 1,210 where every step looked and coarse-held records stopped it; every third
            // step 1,530, but the 4,000 rules take 1.49 ms). One word of tuples: at the step's end
            // (before its loads 200 becomes 203); more: before its loads (387 tuples, 1M headers
            // 564, at the end 624).
            auto pass_over = [&]() {
                if (--try_scan != 0) return;
                try_scan = kScanTry;
                bool scan = ps == P_REC && left > kScan;
                while (3u * (uint32_t)__popcll(__ballot(scan)) > 2u * (uint32_t)__popcll(__ballot(ps != P_IDLE))) {
                    try_scan = 2;
                    if (scan) {
                        const uint4* const p = reinterpret_cast<const uint4*>(recs + at);
                        uint4 h[kScan];
#pragma unroll
                        for (uint32_t j = 0; j < kScan; ++j) h[j] = p[2u * j];
                        uint32_t past = 0, at_meta = 0;   // meta of the record where it stops
                        bool on = true;
#pragma unroll
                        for (uint32_t j = 0; j < kScan; ++j) {
                            at_meta = on ? h[j].w : at_meta;
                            on &= !fits(h[j]) & (h[j].z < bp);
                            past += on ? 1u : 0u;
                        }
                        if (!on && meta_check(at_meta)) {   // held by a coarser tuple: its own prefixes
                            const uint4 b = p[2u * past], c = p[2u * past + 1u];
                            on = (b.z < bp) & ((((sip ^ c.x) & pmask(meta_sl(at_meta))) | ((dip ^ c.y) & pmask(meta_dl(at_meta)))) != 0u);
                            past += on ? 1u : 0u;
                        }
                        if (STATS) n_recs += past;
                        at += past;
                        left -= past;
                        scan = on & (left > kScan);
                    }
                }
            };
            if constexpr (NW > 1) pass_over();
            const uint4* const ps_slot = reinterpret_cast<const uint4*>(slots + (slot ? at : 0u));
            const uint4* const p = rec ? reinterpret_cast<const uint4*>(recs + at) : ps_slot + 1;
            const uint4 a = *ps_slot;
            const uint4 b = p[0];   // sp, dp, prio, meta
            const uint4 c = p[1];   // sip, dip, id, cmask
            uint4 xb[U], xc[U];
            if constexpr (U > 1) {
#pragma unroll
                for (uint32_t j = 1; j < (uint32_t)U; ++j) {
                    // the list's last record past its end; an idle or slot lane its own again
                    const uint32_t k = rec ? min(j, left - 1u) : 0u;
                    xb[j] = p[2u * k];
                    xc[j] = p[2u * k + 1u];
                }
            }
            // Records are in (priority, id) order: the first match is the list's best, and the
            // list ends at the first record that cannot beat the answer. True: it ended.
            auto test = [&](bool on, const uint4& b, const uint4& c) {
                if (STATS) n_recs += on;
                bool ok = fits(b);
                const bool better = kless(b.z, c.z, bp, bid);
                bool hit = on & ok & better;
                if (hit && meta_check(b.w)) {   // held by a coarser tuple: its own prefixes
                    ok = (((sip ^ c.x) & pmask(meta_sl(b.w))) | ((dip ^ c.y) & pmask(meta_dl(b.w)))) == 0u;
                    hit = ok;
                }
                bp = hit ? b.z : bp;
                bid = hit ? c.z : bid;
                bcm = hit ? (NW == 1 ? c.w : at) : bcm;
                if (STATS && hit) s_tup[wave][e] = ct;
                at += on ? 1u : 0u;
                left -= on ? 1u : 0u;
                return on & (ok | !better | (left == 0u));
            };
            if (STATS) n_slots += slot;
            const bool empty = slot & (a.z == kEmptyTL);
            // (an empty slot's key is above every tuple's)
            const bool match = slot & (a.x == k0) & (a.y == k1) & ((a.z >> kTlShift) == tk);
            const bool split = match & ((a.w & kSplit) != 0u);
            const bool miss = slot & !empty & !match;
            left = match ? a.z & kMaxBucketLen : left;
            at = match ? a.w : miss ? (at + 1u) & slot_mask : at;
            walk += miss ? 1u : 0u;
            if (split) {
                // a split bucket: the sub-lists the header selects, where the summary in the
                // record's place (SplitInfo) has them
                bi = a.w & ~kSplit;
                const uint32_t d = split_dp_bit(dp), p = split_sp_bit(sp);
                const uint32_t dw = d & 64u ? (d & 32u ? b.w : b.z) : (d & 32u ? b.y : b.x);
                const uint32_t pw = p >= 64u ? c.z : p >= 32u ? c.y : c.x;
                sub = ((dw >> (d & 31u)) & 1u) | ((pw >> (p & 31u)) & 1u) << 1 |
                      ((c.w >> split_proto_bit(proto)) & 1u) << 2 | (c.w >> 31) << 3;
            }
            const bool first = match & !split & (left != 0u);
            // (only a corrupted table has no empty slot to end the walk)
            bool done = empty | (match & !first) | (walk > slot_mask);
            done |= test(rec | first, b, c);
            if constexpr (U > 1) {
#pragma unroll
                for (uint32_t j = 1; j < (uint32_t)U; ++j) done |= test(rec & !done, xb[j], xc[j]);
            }
            ps = first ? P_REC : ps;
            if (done) {
                if (sub) {
                    // the next sub-list of a split bucket
                    const uint32_t q = (uint32_t)__builtin_ctz(sub);
                    sub &= sub - 1u;
                    k1 = q == 0 ? dp : q == 1 ? sp : q == 2 ? proto : 0u;
                    tk = ct | ((q + kSubDp) << kKindShift);
                    k0 = bi;
                    ps = P_START;
                } else if (cur | nz) {
                    ps = P_NEXT;
                } else {
                    ps = P_IDLE;
                    if (R > 1) ent[e] = Entry{bp, bid, bcm, 0u};
                }
            }
            if constexpr (NW == 1) pass_over();
        }
        if constexpr (R == 1) own = Entry{bp, bid, bcm, 0u};
        wave_sync();
    }
#pragma unroll 1
    for (uint32_t e = lane; e < cnt; e += 64u) {
        const uint32_t id = entry(e).id;
        if (STATS) {
            nm += id == kDead;
            if (kcand > 0 && id != kDead) top1 += s_tup[wave][e] == (out[base + e] & ((1u << CB) - 1u));
        }
        out[base + e] = id == kDead ? TANG_NO_MATCH : id;
    }
    if (STATS) {
        // wave sums -> block sums in LDS -> one set of atomics per block, spread over
        // kStatCopies counter copies (summed on the host) to avoid one hot address.
        // Steps are the wave's own count, once for each of its headers.
        constexpr int NS = 10;
        __shared__ unsigned long long s_red[4][NS];
        unsigned long long v[NS] = {lane == 0 ? cnt : 0u, n_probe, n_slots, n_recs, top1, fb, nm, n_filter,
                                    lane == 0 ? (unsigned long long)cnt * n_steps : 0u, n_rounds};
#pragma unroll
        for (int q = 0; q < NS; ++q) v[q] = wave_sum(v[q]);
        if (lane == 0)
#pragma unroll
            for (int q = 0; q < NS; ++q) s_red[wave][q] = v[q];
        __syncthreads();
        if (tid < NS) {
            const unsigned long long sum = s_red[0][tid] + s_red[1][tid] + s_red[2][tid] + s_red[3][tid];
            unsigned long long* dst = reinterpret_cast<unsigned long long*>(st + (blockIdx.x % kStatCopies));
            atomicAdd(dst + tid, sum);
        }
    }
}

}  // namespace

hipError_t launch_classify(const tang_ruleset_t* rs, const tang_header_t* d_hdr, uint32_t* d_out,
                           size_t n, int kcand, hipStream_t s, bool stats, const uint32_t* d_live) {
    const size_t chunk = (size_t)1 << 30;
    if (d_live && n > chunk) return hipErrorInvalidValue;
    for (size_t base = 0; base < n; base += chunk) {
        const uint32_t m = (uint32_t)std::min(chunk, n - base);
        const uint4* h = reinterpret_cast<const uint4*>(d_hdr) + base;
        auto go = [&](auto kern, uint32_t sets) {
            const uint32_t per_block = 256u * sets;
            hipLaunchKernelGGL(kern, dim3((m + per_block - 1) / per_block), dim3(256), 0, s, h, d_out + base, m,
                               rs->d_slots, rs->d_recs, rs->d_cmask,
                               reinterpret_cast<const uint2*>(rs->d_filter), rs->d_tt, kcand, rs->d_stats,
                               d_live);
        };
        // Records per step (U = 1 and 2), 65,536 headers: 100,000 rules 27 and 23 us, 512k with
        // 25% wildcard-heavy rules 31 and 33, 1,800 rules 13 and 15; two sets, 4.2M headers: 100,000
        // rules 212 and 211, 512k 254 and 274, 1,800 125 and 137. 144 tuples, 65,536 headers 39 and
        // 38, 2.1M 253 and 260; 387 tuples, 1M 491 and 514.
        // Wider rulesets take one set: two need LDS for the headers and a second set of work
        // rows, and the waves lost cost more than the fuller lanes give (with the headers in
        // LDS in both forms and records taken one by one, 144 tuples, 2.1M headers: 387 against
        // 476 us; 387 tuples, 1M: 884 against 977).
        if (rs->nw == 1) {
            if (m >= kQueueFrom) {
                if (stats) go(k_classify<true, 1, 2, 1>, 2);
                else go(k_classify<false, 1, 2, 1>, 2);
            } else {
                if (stats) go(k_classify<true, 1, 1, 2>, 1);
                else go(k_classify<false, 1, 1, 2>, 1);
            }
        } else if (rs->nw == kMaskWords) {
            if (stats) go(k_classify<true, kMaskWords, 1, 2>, 1);
            else go(k_classify<false, kMaskWords, 1, 2>, 1);
        } else {
            if (stats) go(k_classify<true, kMaxWords, 1, 1>, 1);
            else go(k_classify<false, kMaxWords, 1, 1>, 1);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace tang
