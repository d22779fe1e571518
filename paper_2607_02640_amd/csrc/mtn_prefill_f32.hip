// gfx950 chunk prefill over fp32 pools, D = 64 or 128.
//
// Method: Metronome (arXiv 2607.02640) §2 (a frame prefills its chunk, causal
// inside it and over the retained cache), §4.1 / App. A for what a query sees.
#include "mtn_kernels.h"
#include "mtn_device.h"

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

namespace mtn {
namespace {

// One workgroup of four waves per (sequence, pass of 64 query rows, kv head, key
// segment); a row is (token, group head), a wave holds a tile of 16.  Keys
// stream one 16-token block per stage through an LDS ring that all four waves
// fill by DMA and read, so a block is read once per 64 rows.
//   S^T[key][row] = K[key][:] . Qrot[row][:]      (A = K, B = Q^T)
//   O^T[d][row]  += V^T[d][key] . P^T[key][row]   (A = V^T, B = P^T)
// with the fp32 16x16x4 MFMA.  Its k index (lane / 16 = lg) stands for dim
// 16 c + 4 lg + e in product (c, e) of QK and for key 4 lg + e in product e of
// PV: a lane's operands are then whole 16-byte reads of a K row and of a V^T
// row, and the scores it receives (keys 4 lg .. 4 lg + 3 of row lane % 16) are
// its own PV operand.  Everything is fp32, as in the vector kernel.
//
// Bound by the chain of a stage: 64 products of 32 cycles per wave and block at
// D = 128, the barrier and the softmax between them, one wave per SIMD.  The
// vector kernel, one wave per chunk token and kv head, read the window once per
// token: 13 sessions of 5 .. 21 tokens over 900 keys, G = 4, D = 128, 88.2 us
// per layer; this kernel 36.2 and 4.7 of merge at 3 segments (36.4 at 7, with
// two workgroups per CU).
constexpr int kF32Waves = 4;
constexpr int kF32Rows = 16 * kF32Waves;
constexpr int kF32Stages = 4;  // ring depth in blocks: two workgroups per CU at D = 128

struct F32Args {
    AttnArgs a;
    const int32_t *items;
};

__device__ __forceinline__ f32x4_t mfma_f32(float a, float b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <int D, int G>
__global__ __launch_bounds__(64 * kF32Waves) void k_prefill_f32(F32Args pa) {
    constexpr int ROW = D * 4;            // bytes of a key row
    constexpr int TILE = kBlock * ROW;    // ... of a K (or V^T) tile
    constexpr int BLK = 2 * TILE;
    constexpr int NPW = BLK / 1024 / kF32Waves;  // DMA instructions per wave and stage
    constexpr int NC = D / 16;            // 16-wide slices of d
    constexpr int NS = kF32Stages;
    static_assert(NPW * (NS - 1) <= 63, "the DMA waits count at most 63");
    __shared__ __attribute__((aligned(16))) uint8_t ring[NS][BLK];
    const AttnArgs &a = pa.a;
    const PoolGeom &g = a.g;
    const uint32_t ns = (uint32_t)a.n_split;
    const uint32_t iu = blockIdx.x / ns;
    const uint32_t seg = blockIdx.x - iu * ns;
    const int item = (int)(iu / (uint32_t)g.hkv);
    const int kvh = (int)(iu - (uint32_t)item * (uint32_t)g.hkv);
    const int32_t *rec = pa.items + (int64_t)item * kPfItem;
    const int pass = scalar_ld(rec, 0);
    const int tok0 = scalar_ld(rec, 1);
    const int ntok = scalar_ld(rec, 2);
    const int sid = scalar_ld(rec, 3);
    const int pos0 = scalar_ld(rec, 4);
    const int row_t0 = scalar_ld(rec, 5);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ln16 = lane & 15, lg = lane >> 4;
    const int pass_row0 = pass * kF32Rows;
    const int pass_end = min(ntok * G, pass_row0 + kF32Rows);
    const int tq_min = pos0 + pass_row0 / G;
    const int tq_max = pos0 + (pass_end - 1) / G;

    // union of the visible sets of the pass's queries: sinks, then the ring
    // run [A, tq_max]
    const int sink_tokens = min(g.n_sink, tq_max + 1);
    const int n_sb = (sink_tokens + kBlock - 1) / kBlock;
    const int A = g.window < 0 ? 0 : max(g.n_sink, tq_min - g.window + 1);
    const int ring_n = max(0, tq_max - A + 1);
    const int first = g.window < 0 ? A : (A - g.n_sink) % g.ring;
    const int first_off = first % kBlock;
    const int rb_start = first / kBlock;
    const int ring_blocks = g.ring / kBlock;
    const int n_rb = ring_n > 0 ? (first_off + ring_n + kBlock - 1) / kBlock : 0;
    const int last_hi = ring_n > 0 ? (first_off + ring_n - 1) % kBlock + 1 : kBlock;
    const int ring_p0 = A - first_off;
    const int nvb = n_sb + n_rb;
    const int v0 = seg_begin(seg, ns, nvb), v1 = seg_begin(seg + 1, ns, nvb);
    const int nst = v1 - v0;

    // stage st (block v0 + st) into its ring slot; stages past the segment move
    // the zero page, so that every stage costs a wave the same NPW copies and
    // its waits are constant
    const int32_t *trow = g.table + (int64_t)sid * g.row_len;
    const uint8_t *base = g.kv + (int64_t)a.layer * g.layer_stride + (int64_t)kvh * g.head_stride;
    auto phys = [&](int st) {
        if (st >= nst) return -1;
        const int v = v0 + st;
        int rb = rb_start + v - n_sb;
        rb = rb >= ring_blocks ? rb - ring_blocks : rb;
        return scalar_ld(trow, v < n_sb ? v : g.n_sink_blocks + rb);
    };
    // The 16-byte chunk at LDS offset `off` of a slot: chunks of a K row are
    // permuted by the key, the four chunks of a V^T row by bits 2, 3 of d, so
    // the 16 lanes that read one chunk index take 16 columns of the banks.
    uint32_t dsrc[NPW];
#pragma unroll
    for (int m = 0; m < NPW; ++m) {
        const int off = (wv * NPW + m) * 1024 + lane * 16;
        if (off < TILE) {
            const int key = off / ROW, p = (off % ROW) >> 4;
            dsrc[m] = (uint32_t)(key * ROW + ((p ^ key) << 4));
        } else {
            const int r = off - TILE, d = r >> 6, p = (r >> 4) & 3;
            dsrc[m] = (uint32_t)(TILE + d * 64 + ((p ^ ((d >> 2) & 3)) << 4));
        }
    }
    const uint32_t ring0 = lds_addr(&ring[0][0]);
    auto issue = [&](int st, int ph) {
        const uint8_t *src = ph >= 0 ? base + (int64_t)ph * g.block_stride : a.zero_page;
        const uint32_t dst = ring0 + (uint32_t)((st % NS) * BLK + wv * NPW * 1024);
#pragma unroll
        for (int m = 0; m < NPW; ++m) dma16_s(dsrc[m], src, dst + m * 1024);
    };
#pragma unroll
    for (int st = 0; st < NS - 1; ++st) issue(st, phys(st));
    int nph = phys(NS - 1);

    // ---- this wave's query tile, rotated and scaled (log2 domain)
    const int r0 = pass_row0 + wv * 16 + ln16;
    const bool live = pass_row0 + wv * 16 < pass_end;
    const bool rv = r0 < pass_end;
    const int tj = rv ? r0 / G : 0, gh = rv ? r0 % G : 0;
    const int tq = pos0 + tj;
    const int hq0 = kvh * G;
    float q[NC][4];
    {
        const float *qh = (const float *)a.q + ((int64_t)(row_t0 + tj) * g.hq + hq0 + gh) * D;
        const float2 *rp = a.p.rope + (int64_t)(tok0 + tj) * (D / 2);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int d0 = 16 * c + 4 * lg;
            const float4 x = *(const float4 *)(qh + d0);
            const float4 y = *(const float4 *)(qh + (d0 ^ (D / 2)));
            const float4 c0 = *(const float4 *)(rp + (d0 & (D / 2 - 1)));
            const float4 c1 = *(const float4 *)(rp + (d0 & (D / 2 - 1)) + 2);
            const float sg = d0 < D / 2 ? -1.f : 1.f;
            const float xv[4] = {x.x, x.y, x.z, x.w}, yv[4] = {y.x, y.y, y.z, y.w};
            const float cs[4] = {c0.x, c0.z, c1.x, c1.z}, sn[4] = {c0.y, c0.w, c1.y, c1.w};
#pragma unroll
            for (int e = 0; e < 4; ++e)
                q[c][e] = rv ? fmaf(xv[e], cs[e], sg * yv[e] * sn[e]) * a.scale_log2 : 0.f;
        }
    }

    // per-lane LDS offsets: K chunks 4 c + lg of key ln16, V^T chunk lg of
    // row ln16 (+ 16 dt rows of 64 bytes)
    int koff[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) koff[c] = ln16 * ROW + (((4 * c + lg) ^ ln16) << 4);
    const int voff = TILE + ln16 * 64 + ((lg ^ ((ln16 >> 2) & 3)) << 4);

    // the row reference: starts at the lowest finite float, moves only when a
    // score exceeds it by more than 2^8 (probabilities stay <= 256)
    float m_ref, ls;
    // two sums per output, over the even and the odd keys: chains half as long
    // (error against 64 bits of 22 unsplit sessions over 1500 keys 7.2e-7 with
    // one, 5.3e-7 with two, the vector kernel's 5.2e-7; a frame of 13 sessions
    // 332.7 us with one, 333.0 with two)
    f32x4_t acc[NC], acc1[NC];
    auto reset = [&]() __attribute__((always_inline)) {
        m_ref = -3.402823466e38f;
        ls = 0.f;
#pragma unroll
        for (int dt = 0; dt < NC; ++dt) acc[dt] = acc1[dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    };
    reset();

    // Scores, softmax and PV of block st from its fragments.  APART: the PV
    // product is taken token by token (a token's G rows lie in one tile), V
    // zeroed past what each sees.
    auto block = [&](int st, const float4 (&kf)[NC], float4 (&vf)[NC], auto masked_c, auto apart_c)
                     __attribute__((always_inline)) {
        constexpr bool MASKED = decltype(masked_c)::value, APART = decltype(apart_c)::value;
        // four chains of D / 4 products, as long as the vector kernel's sums
        f32x4_t sq[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) sq[k] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < NC; c += 4) {
#pragma unroll
            for (int k = 0; k < 4; ++k) sq[k] = mfma_f32(kf[c + k].x, q[c + k][0], sq[k]);
#pragma unroll
            for (int k = 0; k < 4; ++k) sq[k] = mfma_f32(kf[c + k].y, q[c + k][1], sq[k]);
#pragma unroll
            for (int k = 0; k < 4; ++k) sq[k] = mfma_f32(kf[c + k].z, q[c + k][2], sq[k]);
#pragma unroll
            for (int k = 0; k < 4; ++k) sq[k] = mfma_f32(kf[c + k].w, q[c + k][3], sq[k]);
        }
        int vlo = 0, vhi = kBlock;  // the slots of the block that this lane's query sees
        float s[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) s[r] = (sq[0][r] + sq[1][r]) + (sq[2][r] + sq[3][r]);
        if constexpr (MASKED) {
            // [lo, hi): the slots that any query of the pass sees; V of others may
            // hold NaN
            const int v = v0 + st;
            int lo = 0, hi = kBlock;
            if (v < n_sb) {
                hi = min(kBlock, sink_tokens - v * kBlock);
                vhi = min(hi, tq + 1 - v * kBlock);
            } else {
                const int u = v - n_sb, p0 = ring_p0 + u * kBlock;
                lo = u == 0 ? first_off : 0;
                hi = u == n_rb - 1 ? last_hi : kBlock;
                vlo = g.window < 0 ? lo : max(lo, tq - g.window + 1 - p0);
                vhi = min(hi, tq + 1 - p0);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int key = 4 * lg + r;
                s[r] = key >= vlo && key < vhi ? s[r] : -INFINITY;
            }
            const int k0 = 4 * lg;
#pragma unroll
            for (int dt = 0; dt < NC; ++dt) {
                vf[dt].x = k0 >= lo && k0 < hi ? vf[dt].x : 0.f;
                vf[dt].y = k0 + 1 >= lo && k0 + 1 < hi ? vf[dt].y : 0.f;
                vf[dt].z = k0 + 2 >= lo && k0 + 2 < hi ? vf[dt].z : 0.f;
                vf[dt].w = k0 + 3 >= lo && k0 + 3 < hi ? vf[dt].w : 0.f;
            }
        }
        const float m4 = vmax3(vmax3(s[0], s[1], s[2]), s[3], s[0]);
        if (__builtin_amdgcn_ballot_w64(m4 > m_ref + 8.f)) {
            const float mx = rows_max(m4);
            const bool up = mx > m_ref + 8.f;
            const float mnew = up ? mx : m_ref;
            const float alpha = up ? __builtin_amdgcn_exp2f(m_ref - mnew) : 1.f;
            m_ref = mnew;
            ls *= alpha;
#pragma unroll
            for (int dt = 0; dt < NC; ++dt) {
                acc[dt] *= alpha;
                acc1[dt] *= alpha;
            }
        }
        float p[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) p[r] = __builtin_amdgcn_exp2f(s[r] - m_ref);
        ls += (p[0] + p[1]) + (p[2] + p[3]);
        if constexpr (APART) {
#pragma nounroll
            for (int t0 = 0; t0 < 16; t0 += G) {
                const int tlo = __builtin_amdgcn_readlane(vlo, t0);
                const int thi = __builtin_amdgcn_readlane(vhi, t0);
                const bool mine = ln16 >= t0 && ln16 < t0 + G;
#pragma unroll
                for (int dt = 0; dt < NC; ++dt) {
                    const float vw[4] = {vf[dt].x, vf[dt].y, vf[dt].z, vf[dt].w};
                    f32x4_t t[2] = {acc[dt], acc1[dt]};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int key = 4 * lg + e;
                        t[e & 1] = mfma_f32(key >= tlo && key < thi ? vw[e] : 0.f, p[e], t[e & 1]);
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        acc[dt][r] = mine ? t[0][r] : acc[dt][r];
                        acc1[dt][r] = mine ? t[1][r] : acc1[dt][r];
                    }
                }
            }
            return;
        }
#pragma unroll
        for (int dt = 0; dt < NC; ++dt) acc[dt] = mfma_f32(vf[dt].x, p[0], acc[dt]);
#pragma unroll
        for (int dt = 0; dt < NC; ++dt) acc1[dt] = mfma_f32(vf[dt].y, p[1], acc1[dt]);
#pragma unroll
        for (int dt = 0; dt < NC; ++dt) acc[dt] = mfma_f32(vf[dt].z, p[2], acc[dt]);
#pragma unroll
        for (int dt = 0; dt < NC; ++dt) acc1[dt] = mfma_f32(vf[dt].w, p[3], acc1[dt]);
    };
    auto step = [&](int st, auto masked_c) __attribute__((always_inline)) {
        // this wave's share of the stage has landed; the barrier covers the
        // other shares and frees the slot last read at st - 1
        vm_wait<NPW * (NS - 2)>();
        __syncthreads();
        issue(st + NS - 1, nph);
        nph = phys(st + NS);
        if (!live) return;
        const uint8_t *sm = &ring[st % NS][0];
        float4 kf[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) kf[c] = *(const float4 *)(sm + koff[c]);
        float4 vf[NC];
#pragma unroll
        for (int dt = 0; dt < NC; ++dt) vf[dt] = *(const float4 *)(sm + voff + dt * 1024);
        block(st, kf, vf, masked_c, std::false_type{});
    };
    // ring blocks that every row sees whole, as stages of the segment
    int full_lo = first_off == 0 ? 0 : 1;
    if (g.window >= 0) full_lo = max(full_lo, (max(0, tq_max - g.window + 1 - ring_p0) + kBlock - 1) / kBlock);
    const int lim = tq_min - (kBlock - 1) - ring_p0;  // 16 u <= lim
    const int full_hi = min(lim < 0 ? 0 : lim / kBlock + 1, last_hi == kBlock ? n_rb : n_rb - 1);
    const int st_a = max(0, min(nst, n_sb + full_lo - v0));
    const int st_b = max(st_a, min(nst, n_sb + full_hi - v0));
    {
        int st = 0;
        for (; st < st_a; ++st) step(st, std::true_type{});
        for (; st < st_b; ++st) step(st, std::false_type{});
        for (; st < nst; ++st) step(st, std::true_type{});
    }
    vm_wait<0>();  // no DMA may land in LDS after the workgroup has ended

    if (!live) return;
    // A key that some row of the tile sees and another does not has probability 0
    // in the second one's column of the PV product, and 0 * Inf is NaN.  A tile
    // that ends with a non-finite sum is therefore computed once more, block by
    // block from memory with each token's V apart: the same sums for every other
    // row.  A finite tile pays for the test alone (D / 4 instructions).
    float m[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int dt = 0; dt < NC; ++dt)
#pragma unroll
        for (int r = 0; r < 4; ++r) m[r] = vmaxabs3(acc[dt][r], acc1[dt][r], m[r]);
    if (__builtin_amdgcn_ballot_w64(!(vmaxabs3(m[0], m[1], vmaxabs3(m[2], m[3], 0.f)) < INFINITY))) {
        reset();
#pragma nounroll
        for (int st = 0; st < nst; ++st) {
            const uint8_t *src = base + (int64_t)phys(st) * g.block_stride;
            float4 kf[NC], vf[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) kf[c] = ((const float4 *)(src + ln16 * ROW))[4 * c + lg];
#pragma unroll
            for (int dt = 0; dt < NC; ++dt)
                vf[dt] = ((const float4 *)(src + TILE + (16 * dt + ln16) * 64))[lg];
            block(st, kf, vf, std::true_type{}, std::true_type{});
        }
    }
    const float l = rows_sum(ls);  // every lane of the wave takes part
    if (!rv) return;
#pragma unroll
    for (int dt = 0; dt < NC; ++dt) acc[dt] += acc1[dt];
    if (ns > 1) {  // the segment's partial row (one that sees nothing of it: sum 0)
        const int64_t u = ((int64_t)(tok0 + tj) * g.hq + hq0 + gh) * ns + seg;
#pragma unroll
        for (int dt = 0; dt < NC; ++dt)
            *(f32x4_t *)(a.part + u * D + 16 * dt + 4 * lg) = acc[dt];
        if (lg == 0)
            *(float2 *)(a.part + (int64_t)a.p.n_tok * g.hq * ns * D + 2 * u) = make_float2(m_ref, l);
        return;
    }
    const int64_t oh = (int64_t)(row_t0 + tj) * g.hq + hq0 + gh;
    const float inv = 1.f / l;
#pragma unroll
    for (int dt = 0; dt < NC; ++dt)
        *(f32x4_t *)((float *)a.out + oh * D + 16 * dt + 4 * lg) = acc[dt] * inv;
    if (a.lse && lg == 0) a.lse[oh] = row_lse(m_ref, l);
}

template <int D>
void launch_d(int G, dim3 grid, hipStream_t s, const F32Args &pa) {
    const dim3 block(64 * kF32Waves);
    switch (G) {
        case 1: hipLaunchKernelGGL((k_prefill_f32<D, 1>), grid, block, 0, s, pa); break;
        case 2: hipLaunchKernelGGL((k_prefill_f32<D, 2>), grid, block, 0, s, pa); break;
        case 4: hipLaunchKernelGGL((k_prefill_f32<D, 4>), grid, block, 0, s, pa); break;
        default: hipLaunchKernelGGL((k_prefill_f32<D, 8>), grid, block, 0, s, pa); break;
    }
}

}  // namespace

int prefill_f32_rows_per_pass() { return kF32Rows; }

hipError_t launch_prefill_f32(const AttnArgs &a, const int32_t *items, int32_t n_items,
                              hipStream_t s) {
    const int G = a.g.hq / a.g.hkv;
    if (!prefill_mfma_supported(0, a.g.d, G) || n_items <= 0 || !items || !a.zero_page ||
        a.k_new || a.n_split < 1 || a.n_split > kMaxSplit || ((uintptr_t)items & 31) != 0)
        return hipErrorInvalidValue;
    const int64_t wgs = (int64_t)n_items * a.g.hkv * a.n_split;
    if (wgs > INT32_MAX) return hipErrorInvalidValue;
    const F32Args pa{a, items};
    if (a.g.d == 128)
        launch_d<128>(G, dim3((unsigned)wgs), s, pa);
    else
        launch_d<64>(G, dim3((unsigned)wgs), s, pa);
    return hipGetLastError();
}

}  // namespace mtn
