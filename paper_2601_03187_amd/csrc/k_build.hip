// Build-time and update-time kernels: conflict masks (certification), record moves for
// bucket rewrites, and slot-table scatters.
//
// Conflict mask of rule m: the set of tuples holding a rule r with key(r) < key(m)
// whose 5-field box intersects m's box. If a packet matches m and a better rule r, the
// packet lies in both boxes, so r's tuple is in m's mask; probing those tuples after m
// is found therefore makes the answer exact (the verification the paper leaves to
// future work, Sec. 8). After deletes a mask is a superset, which stays exact.
#include <algorithm>

#include "tang_internal.hpp"

namespace tang {
namespace {

__device__ __forceinline__ bool box_meet(const BoxDev& a, const BoxDev& b) {
    bool ok = (a.slo <= b.shi) & (b.slo <= a.shi) & (a.dlo <= b.dhi) & (b.dlo <= a.dhi);
    ok &= ((a.sp & 0xFFFFu) <= (b.sp >> 16)) & ((b.sp & 0xFFFFu) <= (a.sp >> 16));
    ok &= ((a.dp & 0xFFFFu) <= (b.dp >> 16)) & ((b.dp & 0xFFFFu) <= (a.dp >> 16));
    const uint32_t ea = (a.pt >> 8) & 1u, eb = (b.pt >> 8) & 1u;
    ok &= (ea == 0) | (eb == 0) | ((a.pt & 0xFFu) == (b.pt & 0xFFu));
    return ok;
}

// Mask words of rule at record position p: the record's own word (NW = 1) or a row of
// the side array.
template <int NW>
__device__ __forceinline__ uint32_t* mask_row(Rec* recs, uint32_t* cmask, uint32_t p) {
    if constexpr (NW == 1) return &recs[p].cmask;
    else return cmask + (size_t)p * NW;
}

// One thread per rule i (boxes in ascending key order); rules j < i stream through LDS.
template <int NW>
__global__ __launch_bounds__(256) void k_conflict_build(const BoxDev* __restrict__ boxes,
                                                        uint32_t n, Rec* __restrict__ recs,
                                                        uint32_t* __restrict__ cmask,
                                                        const uint32_t* __restrict__ all_mask) {
    __shared__ BoxDev tile[256];
    const uint32_t base = blockIdx.x * 256u;
    const uint32_t i = base + threadIdx.x;
    const bool valid = i < n;
    BoxDev me = valid ? boxes[i] : BoxDev{0, 0, 0, 0, 0, 0, 0, 0};
    uint32_t mask[NW], full[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        mask[w] = 0;
        full[w] = all_mask[w];
    }
    auto done = [&]() {
        bool f = true;
#pragma unroll
        for (int w = 0; w < NW; ++w) f &= mask[w] == full[w];
        return f;
    };
    const uint32_t j_end = min(n, base + 256u);  // block-uniform
    for (uint32_t j0 = 0; j0 < j_end; j0 += 256u) {
        if (!__syncthreads_or(valid && !done())) break;
        const uint32_t j = j0 + threadIdx.x;
        if (j < n) tile[threadIdx.x] = boxes[j];
        __syncthreads();
        if (valid && !done() && i > j0) {
            const uint32_t cnt = min(256u, i - j0);
            for (uint32_t k = 0; k < cnt; ++k) {
                const uint32_t t = tile[k].pt >> 16;
                const uint32_t tb = 1u << (t & 31u);
                uint32_t& word = mask[NW == 1 ? 0 : t >> 5];
                if (word & tb) continue;
                if (box_meet(me, tile[k])) word |= tb;
            }
        }
        __syncthreads();
    }
    if (valid) {
        uint32_t* row = mask_row<NW>(recs, cmask, me.pos);
#pragma unroll
        for (int w = 0; w < NW; ++w) row[w] = mask[w];
    }
}

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
// max of two packed 16-bit pairs
__device__ __forceinline__ uint32_t pk_max(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a),
                                                                  __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ uint64_t key64(uint32_t prio, uint32_t id) { return ((uint64_t)prio << 32) | id; }

// After inserts: every live record p is compared with each fresh rule q. If they meet,
// the better-keyed one's tuple goes into the other's mask; a record whose mask has the bits
// already is not written. The fresh rules are the same for every lane, so they come through
// scalar loads, and a compare gathers the bits in which the two rules keep apart: prefix bits
// that both fix, the protocol if both fix it, and port bounds the wrong way round, both ports
// in one packed maximum. Bound by issue over the pairs (524,288 rules, 100 fresh: 71 us; 85
// with a compare per bound and the boxes in LDS). Waves of dead records alone (vacated places,
// after large deletes most of the array) compare nothing. A block takes `slice` of the fresh
// rules (blockIdx.y): one after another they cost it the latency of their loads, 0.3 us each.
template <int NW>
__global__ __launch_bounds__(256) void k_conflict_update(Rec* __restrict__ recs,
                                                         uint32_t* __restrict__ cmask, uint32_t used,
                                                         const FreshDev* __restrict__ fresh,
                                                         uint32_t n_new, uint32_t slice,
                                                         const uint32_t* __restrict__ back,
                                                         SlotDev* __restrict__ slots) {
    __shared__ uint32_t qadd[256][NW];
    const uint32_t p = blockIdx.x * 256u + threadIdx.x;
    Rec me = Rec{0u, 0u, kDead, 0u, 0u, 0u, kDead, 0u};
    if (p < used) me = recs[p];
    const bool live = !(me.prio == kDead && me.id == kDead);
    if (!__syncthreads_or(live)) return;
    const bool wave_live = __ballot(live) != 0ull;
    const uint32_t sm = pmask(meta_sl(me.meta)), dm = pmask(meta_dl(me.meta));
    const uint32_t lo = (me.sp & 0xFFFFu) | (me.dp << 16), hi = (me.sp >> 16) | (me.dp & 0xFFFF0000u);
    const uint32_t proto = meta_proto(me.meta), pm = meta_exact(me.meta) ? 0xFFu : 0u;
    const uint64_t key = key64(me.prio, me.id);   // a dead record's is above every rule's
    const uint32_t my_t = meta_tuple(me.meta);
    uint32_t add[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) add[w] = 0;
    const uint32_t end = min(n_new, (blockIdx.y + 1u) * slice);
    for (uint32_t q0 = blockIdx.y * slice; q0 < end; q0 += 256u) {
        const uint32_t cnt = min(256u, end - q0);
#pragma unroll
        for (int w = 0; w < NW; ++w) qadd[threadIdx.x][w] = 0;
        __syncthreads();
#pragma unroll 4
        for (uint32_t k = 0; k < (wave_live ? cnt : 0u); ++k) {
            const FreshDev q = fresh[q0 + k];
            uint32_t apart = (me.sip ^ q.sip) & sm & q.sm;
            apart |= (me.dip ^ q.dip) & dm & q.dm;
            apart |= (proto ^ q.proto) & pm & q.pm;
            apart |= pk_max(lo, q.hi) ^ q.hi;
            apart |= pk_max(hi, q.lo) ^ hi;
            const bool meet = apart == 0u;
            const uint64_t qkey = key64(q.prio, q.id);
            if (meet & (key < qkey)) {
                const uint32_t bit = 1u << (my_t & 31u);
                uint32_t* word = &qadd[k][NW == 1 ? 0 : my_t >> 5];
                if (!(*word & bit)) atomicOr(word, bit);
            }
            const uint32_t bit = meet & (qkey < key) ? 1u << (q.tuple & 31u) : 0u;   // (not q itself)
            if constexpr (NW == 1) {
                add[0] |= bit;
            } else if (bit) {
#pragma unroll
                for (int w = 0; w < NW; ++w)
                    if (q.tuple >> 5 == (uint32_t)w) add[w] |= bit;
            }
        }
        __syncthreads();
        if (threadIdx.x < cnt) {
            uint32_t* row = mask_row<NW>(recs, cmask, fresh[q0 + threadIdx.x].pos);
#pragma unroll
            for (int w = 0; w < NW; ++w)
                if (qadd[threadIdx.x][w]) atomicOr(&row[w], qadd[threadIdx.x][w]);
        }
        __syncthreads();
    }
    if (live) {
        uint32_t* row = mask_row<NW>(recs, cmask, p);
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const uint32_t have = NW == 1 ? me.cmask : add[w] ? row[w] : 0u;
            if (!(add[w] & ~have)) continue;
            atomicOr(&row[w], add[w]);
            // the copy in the slot; slots of fresh rules' lists are written afterwards
            if constexpr (NW == 1) {
                const uint32_t b = back[p];
                if (b) atomicOr(&slots[b - 1u].first.cmask, add[0]);
            }
        }
    }
}

__global__ void k_stage_records(const Rec* __restrict__ recs, const Rec* __restrict__ fresh,
                                const uint32_t* __restrict__ src, uint32_t n,
                                Rec* __restrict__ stage) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t s = src[i];
    stage[i] = (s & 0x80000000u) ? fresh[s & 0x7FFFFFFFu] : recs[s];
}

__global__ void k_place_records(Rec* __restrict__ recs, const Rec* __restrict__ stage,
                                const uint32_t* __restrict__ dst, uint32_t n,
                                uint32_t* __restrict__ back) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    recs[dst[i]] = stage[i];
    if (back) back[dst[i]] = 0u;
}

__global__ void k_stage_masks(const uint32_t* __restrict__ cmask, uint32_t nw,
                              const uint32_t* __restrict__ src, uint32_t n,
                              uint32_t* __restrict__ stage) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * nw) return;
    const uint32_t r = i / nw, w = i % nw, s = src[r];
    stage[i] = (s & 0x80000000u) ? 0u : cmask[(size_t)s * nw + w];
}

__global__ void k_place_masks(uint32_t* __restrict__ cmask, uint32_t nw,
                              const uint32_t* __restrict__ stage, const uint32_t* __restrict__ dst,
                              uint32_t n) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * nw) return;
    cmask[(size_t)dst[i / nw] * nw + i % nw] = stage[i];
}

__global__ void k_fill_slots(SlotDev* __restrict__ slots, const uint32_t* __restrict__ idx,
                             const Slot* __restrict__ val, uint32_t n, const Rec* __restrict__ recs,
                             uint32_t* __restrict__ back, uint32_t* __restrict__ filter,
                             const TupleTable* __restrict__ tt) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t at = idx ? idx[i] : i;
    SlotDev d;
    d.s = val[i];
    d.first = Rec{0u, 0u, kDead, 0u, 0u, 0u, kDead, 0u};
    for (uint32_t& p : d.pad) p = 0u;
    if (d.s.tl != kEmptyTL && !(d.s.off & kSplit) && (d.s.tl & kMaxBucketLen)) {
        d.first = recs[d.s.off];
        if (back) back[d.s.off] = at + 1u;
    }
    slots[at] = d;
    const uint32_t tk = d.s.tl >> kTlShift;
    if (d.s.tl == kEmptyTL || (tk >> kKindShift)) return;
    // a main bucket: its two bits in the block its group value picks (tuple (0, 0) has no
    // group: its one possible key always has a bucket)
    const TupleGroup g = tt->tg[tk];
    if (g.gkey == kNoGroup) return;
    const bool by_dip = (g.gkey & 64u) != 0u;
    const uint32_t v = by_dip ? d.s.md : d.s.ms, o = by_dip ? d.s.ms : d.s.md;
    uint32_t* blk = filter + 2u * filter_block(g.salt, v, tt->filter_shift);
    const uint32_t h = filter_hash(filter_salt(tk), o);
    atomicOr(blk, 0x80000000u >> filter_pos_x(h));
    atomicOr(blk + 1, 0x80000000u >> filter_pos_y(h));
}

__global__ void k_fill_split(SlotDev* __restrict__ slots, const uint32_t* __restrict__ idx,
                             const SplitInfo* __restrict__ info, uint32_t n) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) *reinterpret_cast<SplitInfo*>(&slots[idx[i]].first) = info[i];
}

}  // namespace

hipError_t launch_conflict_build(const BoxDev* d_boxes, size_t n, Rec* d_recs, uint32_t* d_cmask,
                                 uint32_t nw, const uint32_t* all_mask, hipStream_t s) {
    if (!n) return hipSuccess;
    const dim3 g((n + 255) / 256), b(256);
    if (nw == 1)
        hipLaunchKernelGGL(k_conflict_build<1>, g, b, 0, s, d_boxes, (uint32_t)n, d_recs, d_cmask, all_mask);
    else if (nw == kMaskWords)
        hipLaunchKernelGGL(k_conflict_build<kMaskWords>, g, b, 0, s, d_boxes, (uint32_t)n, d_recs,
                           d_cmask, all_mask);
    else
        hipLaunchKernelGGL(k_conflict_build<kMaxWords>, g, b, 0, s, d_boxes, (uint32_t)n, d_recs,
                           d_cmask, all_mask);
    return hipGetLastError();
}

hipError_t launch_conflict_update(Rec* d_recs, uint32_t* d_cmask, uint32_t nw, uint32_t rec_used,
                                  const FreshDev* d_fresh, uint32_t n_new, const uint32_t* d_back,
                                  SlotDev* d_slots, hipStream_t s) {
    if (!n_new || !rec_used) return hipSuccess;
    // Slices of the fresh rules until there are eight blocks per CU, of at least 16 rules, since
    // each slice reads the records again (a whole insert without slices and with them: 1,000
    // rules, 100 fresh 111 and 79 us, 2,000 fresh 1.33 and 0.66 ms; 65,536 rules, 10,000 fresh
    // 8.0 and 6.1 ms).
    const uint32_t blocks = (rec_used + 255) / 256;
    const uint32_t want = std::min(std::max(2048u / blocks, 1u), (n_new + 15) / 16);
    const uint32_t slice = (n_new + want - 1) / want;
    const dim3 g(blocks, (n_new + slice - 1) / slice), b(256);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, g, b, 0, s, d_recs, d_cmask, rec_used, d_fresh, n_new, slice, d_back, d_slots);
    };
    if (nw == 1) go(k_conflict_update<1>);
    else if (nw == kMaskWords) go(k_conflict_update<kMaskWords>);
    else go(k_conflict_update<kMaxWords>);
    return hipGetLastError();
}

hipError_t launch_move_records(Rec* d_recs, const Rec* d_fresh, const uint32_t* d_src,
                               const uint32_t* d_dst, uint32_t n, Rec* d_stage, uint32_t* d_back,
                               hipStream_t s) {
    if (!n) return hipSuccess;
    const dim3 g((n + 255) / 256), b(256);
    hipLaunchKernelGGL(k_stage_records, g, b, 0, s, d_recs, d_fresh, d_src, n, d_stage);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_place_records, g, b, 0, s, d_recs, d_stage, d_dst, n, d_back);
    return hipGetLastError();
}

hipError_t launch_move_masks(uint32_t* d_cmask, uint32_t nw, const uint32_t* d_src,
                             const uint32_t* d_dst, uint32_t n, uint32_t* d_stage, hipStream_t s) {
    if (!n) return hipSuccess;
    const dim3 g((n * nw + 255) / 256), b(256);
    hipLaunchKernelGGL(k_stage_masks, g, b, 0, s, d_cmask, nw, d_src, n, d_stage);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_place_masks, g, b, 0, s, d_cmask, nw, d_stage, d_dst, n);
    return hipGetLastError();
}

hipError_t launch_fill_slots(SlotDev* d_slots, const uint32_t* d_idx, const Slot* d_val, uint32_t n,
                             const Rec* d_recs, uint32_t* d_back, uint32_t* d_filter,
                             const TupleTable* d_tt, hipStream_t s) {
    if (!n) return hipSuccess;
    hipLaunchKernelGGL(k_fill_slots, dim3((n + 255) / 256), dim3(256), 0, s, d_slots, d_idx, d_val, n,
                       d_recs, d_back, d_filter, d_tt);
    return hipGetLastError();
}

hipError_t launch_fill_split(SlotDev* d_slots, const uint32_t* d_idx, const SplitInfo* d_info, uint32_t n,
                             hipStream_t s) {
    if (!n) return hipSuccess;
    hipLaunchKernelGGL(k_fill_split, dim3((n + 255) / 256), dim3(256), 0, s, d_slots, d_idx, d_info, n);
    return hipGetLastError();
}

}  // namespace tang
