// The paper's own tuple predictor: the network of Sec. 6.1 with residual blocks (Eq. 1)
// at the size of Sec. 7.1, on the model input of Sec. 6.2:
//   seven 16-bit header chunks / 65535 -> FC(7 -> 512) + ReLU
//   -> n blocks  x <- relu(relu(x w1 + b1) w2 + b2 + x)
//   -> FC(512 -> C) -> top-k (ties to the lower tuple index).
// About 3.2 M multiply-adds per header with 6.3 MB of BF16 weights. One kernel runs the
// whole network for a tile of headers: the tile's activations stay in LDS, every layer's
// weights stream from L2 straight into the registers of the wave that needs them. The
// input layer (seven inputs) runs in FP32 on the vector ALUs.
//
// MFMA orientation as in the small predictor: weights are the A operand (rows = output
// neurons), headers the B operand (columns). Lane group g supplies elements 8g..8g+7 of
// every 32-wide K block on both sides, so the products pair up whatever the instruction's
// internal K order is. A 16x16 result leaves lane (g, c) holding neurons 4g..4g+3 of
// header c: four consecutive BF16 of that header.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>
#include <vector>

#include "tang_internal.hpp"

namespace tang {
namespace {

constexpr int kW = 512;               // neurons per layer
constexpr int kNoClass = 1 << 20;     // an empty top-k slot (above every class)
// Workspace the public header states for a loaded model: allocated and released with it so
// that a caller's allocator sees the documented size, not read or written (activations stay
// on chip).
constexpr size_t kWorkspace = (size_t)3 * 65536 * kW * 2;

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float fl2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f4 mma(u32x4 a, u32x4 b, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((fl2){a, b}, bf16x2));
}
// ReLU of two packed BF16 as a signed 16-bit max against 0 (RNE keeps signs, so this
// equals rounding after ReLU).
__device__ __forceinline__ uint32_t relu_bf16x2(uint32_t p) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2, p),
                                                                  (s16x2){0, 0}));
}
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}

// Every wave's LDS accesses before this are done before any wave passes it. Weight loads in
// flight stay in flight (__syncthreads would wait for them).
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// The whole network for tiles of 16 NT headers. Workgroup: 8 waves; wave w computes neurons
// 64w..64w+63 (4 row tiles) of every layer for all headers of the tile (NT column tiles).
//
// LDS holds one layer's activations in B-fragment order: fragment (kb, nt) is 1 KB, lane l's
// 16 bytes at 16 l, so a fragment read is one conflict-free 128-bit read, and the four
// neurons a lane holds after a layer are 8 bytes of one fragment of the next. A layer
// overwrites its input in place between two barriers; where it overwrites a block's input,
// each lane keeps its own share of it in registers for the residual sum. Weights are stored
// in A-fragment order per wave, 4 KB per K block, and loaded two K blocks ahead, across
// layer ends too; no wave reads another's weights, so they need no LDS.
//
// What bounds it (262,144 headers, 6 blocks, 25 classes: 1,345 us, 1,230 TFLOP/s; one kernel
// per layer with the activations in memory took 2,780): MFMA issue, 12,288 cycles per layer
// and 96 headers, about 70% of a block's 17.9 us at the clock the chip holds; the rest is
// what a barrier exposes, the epilogue above all. 128 headers per tile leave no registers for
// the block input (kept in memory instead: 1,670 us); 64 take 1,414, since the weights then
// need the whole of a CU's 64 bytes per cycle from L2.
template <int NT>
__global__ __launch_bounds__(512) void k_res(const uint4* __restrict__ hdr, uint32_t n,
                                             const float* __restrict__ win, const float* __restrict__ bias,
                                             const uint16_t* __restrict__ w, uint32_t wbytes, int nb, int C,
                                             int topk, uint32_t* __restrict__ cand,
                                             float* __restrict__ logits, uint16_t* __restrict__ cand16) {
    constexpr uint32_t TH = 16u * NT;   // headers per tile
    constexpr int KB = kW / 32;
    __shared__ u32x4 act[KB * NT * 64];
    __shared__ __attribute__((aligned(16))) float sbias[kW];   // the layer's biases
    const uint32_t tid = threadIdx.x, lane = tid & 63u, g = lane >> 4, r = lane & 15u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const __amdgpu_buffer_rsrc_t rw = rsrc(w, wbytes), rb = rsrc(bias, (uint32_t)(1 + 2 * nb) * kW * 4u);
    // this lane's 8 bytes (neurons 64 wave + 16 mt + 4 g ..) of header column nt, in 8-byte
    // units: own0 + 128 ((mt / 2) NT + nt) + 64 (mt % 2)
    const uint32_t own0 = wave * (256u * NT) + ((g >> 1) * 16u + r) * 2u + (g & 1u);
    u32x2* const act8 = reinterpret_cast<u32x2*>(act);
    const uint32_t tiles = (n + TH - 1) / TH;
    for (uint32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const uint32_t p0 = tile * TH;
        // A fragments of K block kb of layer l (2 nb layers of 512 KB, 64 KB per wave); past
        // the last layer that one's again, not used
        u32x4 A[3][4];
        auto load_a = [&](int buf, int l, int kb) {
            const uint32_t at = res_weight_at((uint32_t)l, wave, (uint32_t)kb, (uint32_t)nb);
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
                A[buf][mt] = __builtin_amdgcn_raw_buffer_load_b128(rw, lane * 16u, at + mt * 1024u, 0);
        };
        load_a(0, 0, 0);
        load_a(1, 0, 1);
        // bias of layer l for neuron tid (past the last not used: the output layer reads its own)
        auto next_bias = [&](int l) {
            return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                 rb, tid * 4u, res_bias_row((uint32_t)l, (uint32_t)nb) * (kW * 4u), 0));
        };
        sbias[tid] = next_bias(0);
        // Input layer: a lane is a header, a wave 64 neurons, so weights are scalars.
#pragma unroll
        for (uint32_t set = 0; set < (TH + 63u) / 64u; ++set) {
            const uint32_t c = set * 64u + lane;
            const uint4 h = c < TH && p0 + c < n ? hdr[p0 + c] : make_uint4(0u, 0u, 0u, 0u);
            // v / 65535 for a 16-bit v: the FP64 product with 1/65535 rounded to FP32 equals
            // the correctly rounded FP32 quotient for every v (checked exhaustively), at three
            // instructions instead of a full-precision division
            auto seg = [](uint32_t v) { return (float)((double)v * (1.0 / 65535.0)); };
            const float s[7] = {seg(h.x >> 16), seg(h.x & 0xFFFFu), seg(h.y >> 16), seg(h.y & 0xFFFFu),
                                seg(h.z & 0xFFFFu), seg(h.z >> 16), seg(h.w & 0xFFu)};
#pragma unroll 2
            for (uint32_t k8 = 0; k8 < 8u; ++k8) {
                const uint32_t n0 = 64u * wave + 8u * k8;
                float v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    float a = bias[n0 + j];
#pragma unroll
                    for (int q = 0; q < 7; ++q) a = __builtin_fmaf(win[(n0 + j) * 8u + q], s[q], a);
                    v[j] = a;
                }
                if (c < TH)
                    act[((n0 >> 5) * NT + (c >> 4)) * 64u + (k8 & 3u) * 16u + (c & 15u)] =
                        (u32x4){relu_bf16x2(pack_bf16(v[0], v[1])), relu_bf16x2(pack_bf16(v[2], v[3])),
                                relu_bf16x2(pack_bf16(v[4], v[5])), relu_bf16x2(pack_bf16(v[6], v[7]))};
            }
        }
        lds_barrier();
        u32x4 x[2][NT];   // the block's input, this lane's share
        // One 512 x 512 layer: out = relu(W in + b [+ block input]), BF16 in and out, FP32
        // accumulation with the bias as the accumulator's start.
        auto layer = [&](int l, auto second) {
            constexpr bool RES = decltype(second)::value;
            f4 acc[4][NT];
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                const f4 bv = *reinterpret_cast<const f4*>(sbias + 64u * wave + 16 * mt + 4 * g);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = bv;
            }
            const float bnext = next_bias(l + 1);
            u32x4 B[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) B[nt] = act[nt * 64 + lane];
            // 16 K blocks in register buffers 0, 1, 2, 0, ..; the next layer's first two are
            // loaded in the last two, into buffers 0 and 1
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                if (kb + 2 < KB) load_a((kb + 2) % 3, l, kb + 2);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
                    for (int mt = 0; mt < 4; ++mt) acc[mt][nt] = mma(A[kb % 3][mt], B[nt], acc[mt][nt]);
                    if (kb + 1 < KB) B[nt] = act[((kb + 1) * NT + nt) * 64 + lane];
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (kb == KB - 2) load_a(1, l + 1, 1);
            }
            load_a(0, l + 1, 0);
            lds_barrier();   // every wave has read the layer's input
            sbias[tid] = bnext;
#pragma unroll
            for (int mp = 0; mp < 2; ++mp) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    u32x2 y[2];
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        f4 v = acc[2 * mp + u][nt];
                        if constexpr (RES) {
                            const uint32_t x0 = x[mp][nt][2 * u], x1 = x[mp][nt][2 * u + 1];
                            v[0] += bf16_lo(x0);
                            v[1] += bf16_hi(x0);
                            v[2] += bf16_lo(x1);
                            v[3] += bf16_hi(x1);
                        }
                        y[u] = (u32x2){relu_bf16x2(pack_bf16(v[0], v[1])), relu_bf16x2(pack_bf16(v[2], v[3]))};
                    }
                    const uint32_t a0 = own0 + (mp * NT + nt) * 128u, a1 = a0 + 64u;
                    if constexpr (!RES) {
                        const u32x2 b0 = act8[a0], b1 = act8[a1];
                        x[mp][nt] = (u32x4){b0[0], b0[1], b1[0], b1[1]};
                    }
                    act8[a0] = y[0];
                    act8[a1] = y[1];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            lds_barrier();
        };
#pragma unroll 1
        for (int k = 0; k < nb; ++k) {
            layer(2 * k, std::false_type{});
            layer(2 * k + 1, std::true_type{});
        }
        // Output layer (C scores, no activation) and top-k, in blocks of 32 classes. Up to two
        // blocks, wave w takes header column w; with more, wave w takes blocks w, w + 8, ..
        // for the whole tile, so that a block's weights are read once per tile (387 classes,
        // 262,144 headers: 2,314 us with the first form, 1,645 with the second).
        // A header's scores of a block sit in the 4 lanes c, c+16, c+32, c+48; each lane
        // keeps a running top-4 of the classes it holds (a strictly larger score displaces,
        // so ties keep the lower class), which contains the lane's share of any top-k
        // (k <= 4); the top-k is then taken across the lanes, ties to the lower class.
        const int ncb = (C + 31) / 32;
        const uint32_t out_at = (uint32_t)nb * (2u * kW * kW * 2u);
        const float* bout = bias + (size_t)(1 + 2 * nb) * kW;
        struct Top {
            float v[4];
            int cl[4];
        };
        auto scores = [&](Top& t, const f4 (&z)[2], int cb, uint32_t pkt) {
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int c = 32 * cb + 16 * mt + 4 * (int)g + q;
                    const float val = z[mt][q];
                    if (logits && pkt < n && c < C) logits[(size_t)pkt * C + c] = val;
                    float x = (c < C && val == val) ? val : -INFINITY;
                    int xc = c;
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        if (x > t.v[s]) {
                            const float tv = t.v[s];
                            const int tc = t.cl[s];
                            t.v[s] = x;
                            t.cl[s] = xc;
                            x = tv;
                            xc = tc;
                        }
                    }
                }
        };
        // the best of the header's four lanes, taken out of them
        auto take = [&](Top& t, float& bv, int& bc) {
            bv = t.v[0];
            bc = t.cl[0];
#pragma unroll
            for (int q = 1; q < 4; ++q)
                if (t.v[q] > bv) { bv = t.v[q]; bc = t.cl[q]; }
#pragma unroll
            for (int o = 16; o <= 32; o <<= 1) {
                const float ov = __shfl_xor(bv, o, 64);
                const int oc = __shfl_xor(bc, o, 64);
                if (ov > bv || (ov == bv && oc < bc)) { bv = ov; bc = oc; }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (t.cl[q] == bc) { t.v[q] = -INFINITY; t.cl[q] = kNoClass; }
        };
        if (ncb <= 2) {
            if (wave < (uint32_t)NT) {
                const uint32_t pkt = p0 + 16u * wave + r;
                Top t;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    t.v[q] = -INFINITY;
                    t.cl[q] = kNoClass;
                }
#pragma unroll 1
                for (int cb = 0; cb < ncb; ++cb) {
                    const uint32_t at = out_at + (uint32_t)cb * (KB * 2048u);
                    f4 z[2];
#pragma unroll
                    for (int mt = 0; mt < 2; ++mt)
                        z[mt] = *reinterpret_cast<const f4*>(bout + 32 * cb + 16 * mt + 4 * g);
#pragma unroll 8
                    for (int kb = 0; kb < KB; ++kb) {
                        const u32x4 b = act[(kb * NT + wave) * 64 + lane];
#pragma unroll
                        for (int mt = 0; mt < 2; ++mt)
                            z[mt] = mma(__builtin_amdgcn_raw_buffer_load_b128(rw, lane * 16u, at + kb * 2048u + mt * 1024u, 0),
                                        b, z[mt]);
                    }
                    scores(t, z, cb, pkt);
                }
                uint32_t packed = 0;
                for (int k = 0; k < topk; ++k) {
                    float bv;
                    int bc;
                    take(t, bv, bc);
                    packed |= (uint32_t)bc << (cand_bits(C) * k);
                    if (cand16 && g == 0 && pkt < n) cand16[(size_t)pkt * topk + k] = (uint16_t)bc;
                }
                if (cand && g == 0 && pkt < n) cand[pkt] = packed;
            }
        } else {
            Top t[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    t[nt].v[q] = -INFINITY;
                    t[nt].cl[q] = kNoClass;
                }
#pragma unroll 1
            for (int cb = (int)wave; cb < ncb; cb += 8) {
                const uint32_t at = out_at + (uint32_t)cb * (KB * 2048u);
                f4 z[NT][2];
#pragma unroll
                for (int mt = 0; mt < 2; ++mt) {
                    const f4 bv = *reinterpret_cast<const f4*>(bout + 32 * cb + 16 * mt + 4 * g);
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) z[nt][mt] = bv;
                }
#pragma unroll 4
                for (int kb = 0; kb < KB; ++kb) {
                    u32x4 a[2];
#pragma unroll
                    for (int mt = 0; mt < 2; ++mt)
                        a[mt] = __builtin_amdgcn_raw_buffer_load_b128(rw, lane * 16u, at + kb * 2048u + mt * 1024u, 0);
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        const u32x4 b = act[(kb * NT + nt) * 64 + lane];
#pragma unroll
                        for (int mt = 0; mt < 2; ++mt) z[nt][mt] = mma(a[mt], b, z[nt][mt]);
                    }
                }
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) scores(t[nt], z[nt], cb, p0 + 16u * nt + r);
            }
            // each wave's top-k of a header to LDS (over the activations), then one lane per
            // header picks from the eight lists
            lds_barrier();
            u32x2* const tops = act8;   // [wave][header][4]
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                for (int k = 0; k < topk; ++k) {
                    float bv;
                    int bc;
                    take(t[nt], bv, bc);
                    if (g == 0) tops[(wave * TH + 16u * nt + r) * 4u + k] = (u32x2){__float_as_uint(bv), (uint32_t)bc};
                }
            lds_barrier();
            const uint32_t pkt = p0 + tid;
            if (tid < TH && pkt < n) {
                uint32_t packed = 0;
                float lv = INFINITY;
                int lc = -1;
                for (int k = 0; k < topk; ++k) {
                    float bv = -INFINITY;
                    int bc = kNoClass;
                    for (uint32_t u = 0; u < 8u * topk; ++u) {
                        const u32x2 x = tops[((u / topk) * TH + tid) * 4u + u % topk];
                        const float v = __uint_as_float(x[0]);
                        const int c = (int)x[1];
                        const bool left = v < lv || (v == lv && c > lc);   // not picked yet
                        if (left && (v > bv || (v == bv && c < bc))) { bv = v; bc = c; }
                    }
                    lv = bv;
                    lc = bc;
                    packed |= (uint32_t)bc << (cand_bits(C) * k);
                    if (cand16) cand16[(size_t)pkt * topk + k] = (uint16_t)bc;
                }
                if (cand) cand[pkt] = packed;
            }
        }
        lds_barrier();   // the next tile's input layer overwrites the activations
    }
}

uint16_t to_bf16(float f) {
    uint32_t u;
    std::memcpy(&u, &f, 4);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0;
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

}  // namespace

int resnet_prepare(tang_ruleset_t* rs, const tang_resnet_desc_t* d, const float* const* W,
                   const float* const* b, tang_precision_t p) {
    if (!d || !W || !b) return fail(TANG_EINVAL, "NULL model argument");
    const int C = (int)rs->sigs.size();
    if (d->width != (uint32_t)kW) return fail(TANG_EINVAL, "residual model width must be 512");
    if (d->n_blocks < 1 || d->n_blocks > 16) return fail(TANG_EINVAL, "n_blocks must be in 1..16");
    if ((int)d->n_out != C || C < 1 || C > TANG_MAX_TUPLES)
        return fail(TANG_EINVAL, "output width must equal the number of tuples (1..256)");
    if (d->topk < 1 || (int)d->topk > max_topk(C))
        return fail(TANG_EINVAL, "topk must be in 1..min(4, C), 1..2 above 256 tuples");
    if (p != TANG_BF16) return fail(TANG_EINVAL, "the residual model runs in BF16");
    const int nb = (int)d->n_blocks, L = 2 + 2 * nb;
    for (int l = 0; l < L; ++l)
        if (!W[l] || !b[l]) return fail(TANG_EINVAL, "NULL weight or bias");

    ModelDev m;
    m.kind = 1;
    m.prec = p;
    m.hidden = kW;
    m.n_out = C;
    m.topk = (int)d->topk;
    m.n_blocks = nb;
    std::vector<float> win((size_t)kW * 8, 0.0f);
    for (int n = 0; n < kW; ++n)
        for (int q = 0; q < 7; ++q) win[(size_t)n * 8 + q] = W[0][(size_t)n * 7 + q];
    // biases: input layer, 2 per block, output (classes padded to 32-blocks, zero past C)
    const int CP = kOutPad * ((C + kOutPad - 1) / kOutPad);
    std::vector<float> bias((size_t)(1 + 2 * nb) * kW + CP, 0.0f);
    for (int l = 0; l < 1 + 2 * nb; ++l)
        for (int n = 0; n < kW; ++n) bias[(size_t)l * kW + n] = b[l][n];
    for (int c = 0; c < C; ++c) bias[(size_t)(1 + 2 * nb) * kW + c] = b[L - 1][c];
    // BF16 weights in A-fragment order (1 KB: 64 lanes of 8 elements): a block layer as
    // [wave][K block][4 row tiles] of 64 neurons per wave, the output layer as [32-class
    // block][K block][2 row tiles]; lane (g, r) holds row r, columns 8g..8g+7
    std::vector<uint16_t> w((size_t)2 * nb * kW * kW + (size_t)CP * kW, 0);
    auto swizzle = [&](uint16_t* dst, const float* src, int rows, int group) {
        for (int r0 = 0; r0 < rows; r0 += group)
            for (int kb = 0; kb < kW / 32; ++kb)
                for (int mt = 0; mt < group / 16; ++mt)
                    for (int lane = 0; lane < 64; ++lane)
                        for (int j = 0; j < 8; ++j, ++dst) {
                            const int row = r0 + 16 * mt + (lane & 15), col = 32 * kb + 8 * (lane >> 4) + j;
                            *dst = src && row < rows ? to_bf16(src[(size_t)row * kW + col]) : 0;
                        }
    };
    for (int l = 0; l < 2 * nb; ++l) swizzle(&w[(size_t)l * kW * kW], W[1 + l], kW, 64);
    swizzle(&w[(size_t)2 * nb * kW * kW], W[L - 1], C, 32);

    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    m.cus = (uint32_t)cus;
    m.rw_bytes = (uint32_t)(w.size() * 2);
    if (e == hipSuccess) e = dev_alloc(&m.rin, win.size() * 4);
    if (e == hipSuccess) e = hipMemcpy(m.rin, win.data(), win.size() * 4, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = dev_alloc(&m.bias, bias.size() * 4);
    if (e == hipSuccess) e = hipMemcpy(m.bias, bias.data(), bias.size() * 4, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = dev_alloc(&m.rw, w.size() * 2);
    if (e == hipSuccess) e = hipMemcpy(m.rw, w.data(), w.size() * 2, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = dev_alloc(&m.ws, kWorkspace);
    if (e != hipSuccess) {
        model_free(m);
        return hip_fail(e, "residual model upload");
    }
    m.bytes = win.size() * 4 + bias.size() * 4 + w.size() * 2 + kWorkspace;
    m.loaded = 1;
    model_free(rs->model);
    rs->model = m;
    rs->version++;
    return TANG_OK;
}

hipError_t launch_resnet(const tang_ruleset_t* rs, const tang_header_t* d_hdr, size_t n,
                         uint32_t* cand, float* logits, uint16_t* cand16, hipStream_t s) {
    const ModelDev& m = rs->model;
    const size_t chunk = (size_t)1 << 30;
    for (size_t base = 0; base < n; base += chunk) {
        const uint32_t c = (uint32_t)std::min(chunk, n - base);
        auto tiles = [&](uint32_t headers) { return (c + headers - 1) / headers; };
        auto rounds = [&](uint32_t headers) { return (tiles(headers) + m.cus - 1) / m.cus; };
        auto go = [&](auto kern, uint32_t headers) {
            hipLaunchKernelGGL(kern, dim3(std::min(tiles(headers), m.cus)), dim3(512), 0, s,
                               reinterpret_cast<const uint4*>(d_hdr + base), c, m.rin, m.bias,
                               static_cast<const uint16_t*>(m.rw), m.rw_bytes, m.n_blocks, m.n_out, m.topk,
                               cand ? cand + base : nullptr,
                               logits ? logits + base * (size_t)m.n_out : nullptr,
                               cand16 ? cand16 + base * (size_t)m.topk : nullptr);
        };
        // Tiles of 96 headers or of 64, whichever takes less for the rounds of one tile per CU:
        // a round of 64 takes three quarters of one of 96 (6 blocks, 25 classes: 16,384 headers
        // 98 us in one round of 64, 127 in one of 96; 24,576 headers 180 in two of 64, 137 in
        // one of 96; 262,144 headers 1,414 against 1,344).
        if (3 * rounds(64) <= 4 * rounds(96)) go(k_res<4>, 64);
        else go(k_res<6>, 96);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace tang
