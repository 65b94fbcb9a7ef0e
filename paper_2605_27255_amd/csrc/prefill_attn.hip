// Causal grouped-query flash attention for a chunk of prompt positions.
//
// Both products take fp16 operands (32x32x16 MFMAs): the query, rounded once
// by the QKV GEMM's epilogue, and the probabilities carry 11 significant bits
// (against 8 for bf16), and K and V, stored as bf16, are widened to fp16
// exactly for every value in fp16's normal range (|x| in [2^-14, 65504];
// smaller values keep 2^-24 absolute precision; larger ones would overflow, a
// limit of the prefill only).  The widened K and V of one layer live in a
// scratch copy of the cache (kh, vh): the QKV epilogue writes the chunk's own
// positions and k_widen_kv the earlier ones, so that a stage moves from
// memory into LDS with no conversion.
//
// One workgroup of four waves per (sequence, KV group, group of up to four
// query heads, 32-query block), two workgroups per CU, which share no barrier
// and so overlap one's softmax with the other's MFMAs.  A wave computes one
// head: scores transposed, S^T[key][query] = K Q^T, a lane holding one query
// (l % 32) and half the keys, so that the row maximum takes one exchange
// between the halves and the row sum one at the very end; the probabilities,
// keys 8 q + 4 h .. + 3 of a 32-key tile in accumulator group q, are already
// the B operand of O^T += V^T P^T in the V tile's slot order (vslot): slot
// group h holds the keys of q = 0 and 2, slot group 2 + h those of 1 and 3.
// What bounds it: per 64-key stage and wave 32 MFMAs (about 1030 cycles of its
// SIMD's matrix core) against about 1000 cycles of softmax arithmetic (32
// exponentials a lane at a quarter of the rate) and 32 KB of LDS reads (at 128
// bytes a cycle, eight waves: as long as the MFMAs of a SIMD's two waves).
// 4096 queries over up to 32768 keys, 8 KV groups of four heads (mean over the
// chunks of a 65536-token prompt): 1481 us before (eight waves behind one
// barrier, 16x16x32 MFMAs, K and V widened by each workgroup), 1010 us now
// (1.06 PFLOP/s).  One V buffer and three workgroups per CU: 1030 us.
#include "device_common.h"
#include "kernels.h"

namespace pipo {

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;

__device__ __forceinline__ f32x16 mfma32_f16(u32x4 a, u32x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0,
                                                  0);
}
// The other half's value (lanes l and l ^ 32 hold one query).
__device__ __forceinline__ float half_max(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

constexpr int kAQ = 32;         // queries per workgroup
constexpr int kAK = 64;         // keys per LDS stage

template <int D>
__global__ __launch_bounds__(256, 2) void k_attn_prefill(AttnPrefillParams p) {
    constexpr int NC = D / 32, ND = D / 32;
    constexpr int KV = kAK * D / 512;            // 1 KB pieces of a stage's K (and of its V)
    static_assert(2 * 2 * KV <= 64, "M0 holds a 16-bit LDS offset");
    __shared__ __align__(16) uint16_t lds[2][2 * KV * 512];   // [buffer][K tiles, V blocks]

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j = lane & 31, h = lane >> 5;
    const int qpg = p.n_q / p.n_kv;
    const int nhg = (qpg + 3) / 4;               // head groups per KV group
    const int nqb = (p.g.clen + kAQ - 1) / kAQ;
    const int pairs = p.g.B * p.n_kv * nhg;
    // Late query blocks see more keys and go first; where every workgroup is
    // resident at once (two per CU), the second half goes the other way round,
    // so that a CU holds a long and a short one.
    const int at = (int)blockIdx.x / pairs, rest = (int)blockIdx.x - at * pairs;
    const int half_q = (nqb + 1) >> 1;
    const int qblk = pairs * nqb <= 512 && at >= half_q ? at - half_q : nqb - 1 - at;
    const int hg = rest % nhg, bk = rest / nhg;
    const int b = bk / p.n_kv, kvh = bk - b * p.n_kv;
    const int hig = hg * 4 + wave;               // head index inside the KV group
    const bool active = hig < qpg;
    const int head = kvh * qpg + (active ? hig : 0);
    const int q0 = qblk * kAQ;                   // chunk-local first query
    const int qpos0 = p.g.c0 + q0;               // ... its absolute position
    const float scale = 1.4426950408889634f / sqrtf((float)D);
    // a ragged batch: a block wholly past this sequence's last position holds
    // only PAD rows, whose outputs nothing reads
    if (p.g.ntok && qpos0 >= seq_positions(p.g, b)) return;

    // the stages: K tiles (16 keys x 32 dims) and V blocks (16 dims x 32 keys
    // in operand order) of 64 keys are contiguous in kh and vh
    const int64_t base = (int64_t)b * p.kv_bstride + (int64_t)kvh * p.lmax_pad * D;
    const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) uint16_t *)&lds[0][0];
    const uint32_t lane16 = lane * 16;
    const int nstage = (qpos0 + kAQ + kAK - 1) / kAK;        // keys [0, qpos0 + 32) may be visible
    auto issue = [&](int st, int buf) {
        const int64_t off = base + (int64_t)min(st, nstage - 1) * kAK * D + wave * (KV / 4) * 512;
        const uint32_t dst = lds0 + (buf * 2 * KV + wave * (KV / 4)) * 1024;
#pragma unroll
        for (int u = 0; u < KV / 4; ++u) {
            load_to_lds(p.kh + off + u * 512, dst + u * 1024, lane16);
            load_to_lds(p.vh + off + u * 512, dst + (KV + u) * 1024, lane16);
        }
    };
    // This lane's query row in fp16, dims 32 c + 16 s + 8 h ..  Rows past the
    // chunk, and past a shorter prompt's positions, hold what an earlier call
    // left: they take zeros, whose scores never move a running maximum, so that
    // they have no say in the rescaling of the rows beside them.
    u32x4 qb[NC][2];
    {
        const int nrow = p.g.ntok ? min(p.g.clen, seq_positions(p.g, b) - p.g.c0) : p.g.clen;
        const bool own = q0 + j < nrow;
        const uint16_t *q = p.q + (((int64_t)b * p.n_q + head) * p.g.mpad + min(q0 + j, nrow - 1)) * D + 8 * h;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const u32x4 v = *(const u32x4 *)(q + 32 * c + 16 * s);
                qb[c][s] = own ? v : u32x4{0u, 0u, 0u, 0u};
            }
    }
    issue(0, 0);

    f32x16 o[ND];
#pragma unroll
    for (int t = 0; t < ND; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[t][v] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;        // l_run: this half's keys only

    // this lane's piece of a 32-row operand from two 1 KB tiles `step` apart
    auto frag = [&](const uint16_t *t, int step, int s) {
        return *(const u32x4 *)(t + ((lane >> 4) & 1) * step + ((2 * s + h) * 16 + (lane & 15)) * 8);
    };
    for (int st = 0; st < nstage; ++st) {
        // this wave's share of stage st has landed; the barrier: the others'
        // too, and every wave has read the buffer the next stage overwrites
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        issue(st + 1, (st + 1) & 1);             // (past the end: the last stage again, not read)
        if (!active) continue;
        const uint16_t *ks = lds[st & 1], *vs = ks + KV * 512;
        f32x16 sc[2];
#pragma unroll
        for (int v = 0; v < 16; ++v) sc[0][v] = sc[1][v] = 0.f;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int t = 0; t < 2; ++t)      // keys 32 t .. : K tiles (2 t, c) and (2 t + 1, c)
                    sc[t] = mfma32_f16(frag(ks + (2 * t * NC + c) * 512, NC * 512, s), qb[c][s], sc[t]);
        const int kb0 = st * kAK;
        if (kb0 + kAK - 1 > qpos0) {             // some key lies past some query: the causal mask
            const int lim = qpos0 + j - kb0 - 4 * h;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (32 * t + 8 * (v >> 2) + (v & 3) > lim) sc[t][v] = -INFINITY;
        }
        float mx = -INFINITY;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) mx = fmaxf(mx, sc[t][v]);
        mx = half_max(mx);
        // The running max moves only when some query's grows by more than 2^8
        // (in exp2 units), so the accumulators are rarely rescaled and every
        // exponent stays at most 256; o / l is the same quotient.  (A query
        // sees key 0 in the first stage, so the max is finite from then on.)
        const float m_cand = fmaxf(m_run, mx * scale);
        if (__any(m_cand > m_run + 8.0f)) {
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_cand);
            l_run *= alpha;
#pragma unroll
            for (int t = 0; t < ND; ++t) o[t] *= alpha;
            m_run = m_cand;
        }
        // probabilities, their sum and P^T in fp16
        u32x4 ph[2][2];
        float ps[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float e = __builtin_amdgcn_exp2f(fmaf(sc[t][v], scale, -m_run));
                sc[t][v] = e;
                ps[v & 3] += e;
            }
#pragma unroll
            for (int s = 0; s < 2; ++s)          // slot group 2 s + h: accumulator groups s and 2 + s
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int v = 4 * (s + 2 * (i >> 1)) + 2 * (i & 1);
                    ph[t][s][i] = pack_f16x2(sc[t][v], sc[t][v + 1]);
                }
        }
        l_run += (ps[0] + ps[1]) + (ps[2] + ps[3]);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int dt = 0; dt < ND; ++dt)  // dims 32 dt .. of the 32-key tile t
                    o[dt] = mfma32_f16(frag(vs + (t * (D / 16) + 2 * dt) * 512, 512, s), ph[t][s], o[dt]);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no load to LDS outlives the workgroup
    const int i = q0 + j;
    l_run += __shfl_xor(l_run, 32);
    // (a ragged batch: rows past this sequence's positions are another's)
    if (!active || i >= p.g.clen || (p.g.ntok && p.g.c0 + i >= seq_positions(p.g, b))) return;
    const float inv = 1.0f / l_run;
    const int qd = p.n_q * D;
    const int64_t m = row_of(p.g, b, i);
#pragma unroll
    for (int t = 0; t < ND; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t hi[4], lo[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) split_bf(o[t][4 * q + e] * inv, hi[e], lo[e]);
            const int64_t at2 = tiled_index(m, head * D + 32 * t + 8 * q + 4 * h, qd);
            *(u32x2 *)(p.out_hi + at2) = u32x2{hi[0] | (hi[1] << 16), hi[2] | (hi[3] << 16)};
            *(u32x2 *)(p.out_lo + at2) = u32x2{lo[0] | (lo[1] << 16), lo[2] | (lo[3] << 16)};
        }
}

// Positions [0, c0) of one layer's cache into kh and vh (16-byte pieces; a V
// piece that also holds later positions repeats what the QKV epilogue wrote).
template <int D>
__global__ __launch_bounds__(256) void k_widen_kv(AttnPrefillParams p) {
    const int bk = blockIdx.y, b = bk / p.n_kv, kvh = bk - b * p.n_kv;
    int n = p.g.c0;
    if (p.g.ntok && p.g.c0 >= seq_positions(p.g, b)) return;   // no query of this chunk reads them
    const int64_t base = (int64_t)b * p.kv_bstride + (int64_t)kvh * p.lmax_pad * D;
    const int64_t pieces = (int64_t)((n + 31) / 32) * 32 * D / 8;
    for (int64_t i = blockIdx.x * 256ll + threadIdx.x; i < pieces; i += gridDim.x * 256ll) {
        const u32x4 k = *(const u32x4 *)(p.kc + base + i * 8);
        // piece (dim block, slot group g, dim j) of vh from dim 16 block + j of vc
        const int64_t blk = i >> 6;
        const int l = (int)(i & 63);
        const u32x4 v = *(const u32x4 *)(p.vc + base + blk * 512 + (l & 15) * 32 + (l >> 4) * 8);
        u32x4 ko, vo;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            ko[e] = pack_f16x2(bf_lo(k[e]), bf_hi(k[e]));
            vo[e] = pack_f16x2(bf_lo(v[e]), bf_hi(v[e]));
        }
        *(u32x4 *)(p.kh + base + i * 8) = ko;
        *(u32x4 *)(p.vh + base + i * 8) = vo;
    }
}

void launch_attn_prefill(const AttnPrefillParams &p, hipStream_t s) {
    const int qpg = p.n_q / p.n_kv;
    const int nhg = (qpg + 3) / 4;
    const int nqb = (p.g.clen + kAQ - 1) / kAQ;
    const int grid = p.g.B * p.n_kv * nhg * nqb;
    if (p.g.c0 > 0) {
        const int64_t pieces = (int64_t)((p.g.c0 + 31) / 32) * 32 * p.d / 8;
        const dim3 wg((unsigned)((pieces + 1023) / 1024), p.g.B * p.n_kv);
        if (p.d == 128) hipLaunchKernelGGL(k_widen_kv<128>, wg, dim3(256), 0, s, p);
        else hipLaunchKernelGGL(k_widen_kv<64>, wg, dim3(256), 0, s, p);
    }
    if (p.d == 128) hipLaunchKernelGGL(k_attn_prefill<128>, dim3(grid), dim3(256), 0, s, p);
    else hipLaunchKernelGGL(k_attn_prefill<64>, dim3(grid), dim3(256), 0, s, p);
}

}  // namespace pipo
