// The prefill's MFMA GEMM  C^T[N][M] = W[N][K] X[M][K]^T  with fused epilogues.
// W and X are tiled (16x32 tiles of 1 KB, device_common.h); X is a bf16 pair
// hi + lo (two products per weight) or exact in bf16 (one).
#include "device_common.h"
#include "kernels.h"

namespace pipo {

typedef __attribute__((ext_vector_type(16))) float f32x16;

__device__ __forceinline__ f32x16 mfma32(u32x4 a, u32x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                   0, 0);
}
__device__ __forceinline__ float silu_p(float u) { return u / (1.0f + __expf(-u)); }

// ---- fused epilogue of one 16-row strip ------------------------------------
// Lane (token l % 32, half h = l / 32) of a 32x32 accumulator holds rows
// 4 h .. 4 h + 3 (a) and 8 + 4 h .. (c) of the strip for token m.  The row
// permutations put what an epilogue pairs (gate and up, a RoPE pair) eight
// rows apart, so both halves of a pair are in one lane.
template <int EPI>
__device__ __forceinline__ void gemm_epi(const GemmParams &p, f32x4 a, f32x4 c, int strip, int m) {
    const int h = (threadIdx.x >> 5) & 1;
    if (strip >= (p.N >> 4) || m >= p.M) return;
    int b, i, pos;
    if (p.dpos) {   // a decode step: one row per sequence
        if (m >= p.rows) return;
        b = m;
        i = 0;
        pos = EPI == EPI_QKV ? p.dpos[m] : 0;
    } else {
        row_seq(p.g, m, b, i);
        pos = p.g.c0 + i;
        // rows that pad a sequence to 32 hold nothing; the cache keeps finite
        // values at positions no prompt has reached
        if (i >= p.g.clen || (p.g.ntok && pos >= seq_positions(p.g, b))) return;
    }
    const int row0 = strip * 16 + 4 * h;
    if (EPI == EPI_STORE) {
        if (p.bias) {
            a += *(const f32x4 *)(p.bias + row0);
            c += *(const f32x4 *)(p.bias + row0 + 8);
        }
        float *o = p.out + (int64_t)m * p.N + row0;
        *(f32x4 *)o = a;
        *(f32x4 *)(o + 8) = c;
    } else if (EPI == EPI_RESID) {
        float *o = p.out + (int64_t)m * p.N + row0;
        a += *(const f32x4 *)o;
        c += *(const f32x4 *)(o + 8);
        *(f32x4 *)o = a;
        *(f32x4 *)(o + 8) = c;
        if (p.ss_out) {
            float sq = (a[0] * a[0] + a[1] * a[1]) + (a[2] * a[2] + a[3] * a[3]) + (c[0] * c[0] + c[1] * c[1]) +
                       (c[2] * c[2] + c[3] * c[3]);
            sq += __shfl_xor(sq, 32);   // the strip's other eight rows (the same token: both lanes are here)
            if (h == 0) p.ss_out[(int64_t)m * (p.N >> 4) + strip] = sq;
        }
        if (p.xn_hi) {
            const f32x4 ga = *(const f32x4 *)(p.gain + row0), gc = *(const f32x4 *)(p.gain + row0 + 8);
            const float f[8] = {a[0] * ga[0], a[1] * ga[1], a[2] * ga[2], a[3] * ga[3],
                                c[0] * gc[0], c[1] * gc[1], c[2] * gc[2], c[3] * gc[3]};
            u32x4 hi, lo;
            split8(f, hi, lo);
            const int64_t at = tiled_index(m, row0, p.N);          // row0 + 8: the next 16 lanes' pieces
            *(u32x2 *)(p.xn_hi + at) = u32x2{hi[0], hi[1]};
            *(u32x2 *)(p.xn_lo + at) = u32x2{lo[0], lo[1]};
            *(u32x2 *)(p.xn_hi + at + 128) = u32x2{hi[2], hi[3]};
            *(u32x2 *)(p.xn_lo + at + 128) = u32x2{lo[2], lo[3]};
        }
    } else if (EPI == EPI_SILU) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const f32x4 v = q ? c : a;
            uint32_t hi[4], lo[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) split_bf(silu_p(v[e]), hi[e], lo[e]);
            const int64_t at = tiled_index(m, row0 + 8 * q, p.N);
            *(u32x2 *)(p.act_hi + at) = u32x2{hi[0] | (hi[1] << 16), hi[2] | (hi[3] << 16)};
            *(u32x2 *)(p.act_lo + at) = u32x2{lo[0] | (lo[1] << 16), lo[2] | (lo[3] << 16)};
        }
    } else if (EPI == EPI_SWIGLU) {
        uint32_t hi[4], lo[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) split_bf(silu_p(a[e]) * c[e], hi[e], lo[e]);
        const int64_t at = tiled_index(m, strip * 8 + 4 * h, p.N >> 1);
        *(u32x2 *)(p.act_hi + at) = u32x2{hi[0] | (hi[1] << 16), hi[2] | (hi[3] << 16)};
        *(u32x2 *)(p.act_lo + at) = u32x2{lo[0] | (lo[1] << 16), lo[2] | (lo[3] << 16)};
    } else if (EPI == EPI_QKV) {
        const int d = p.d, hs = d >> 4;
        const int qs = p.n_q * hs, ks = p.n_kv * hs;
        const int gs = strip + p.strip0;            // strip of the whole QKV matrix
        if (gs < qs + ks) {
            const bool isq = gs < qs;
            const int sidx = isq ? gs : gs - qs;
            const int head = sidx / hs, t = sidx - head * hs;
            const int jr = 8 * t + 4 * h;           // dims jr .. (a) and d/2 + jr .. (c)
            const f32x4 cs = *(const f32x4 *)(p.rope_cos + (int64_t)pos * (d >> 1) + jr);
            const f32x4 sn = *(const f32x4 *)(p.rope_sin + (int64_t)pos * (d >> 1) + jr);
            float r[2][4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                r[0][e] = a[e] * cs[e] - c[e] * sn[e];
                r[1][e] = c[e] * cs[e] + a[e] * sn[e];
            }
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int dim0 = q ? (d >> 1) + jr : jr;
                if (isq && p.qf) {
                    *(f32x4 *)(p.qf + ((int64_t)m * p.n_q + head) * d + dim0) = f32x4{r[q][0], r[q][1], r[q][2], r[q][3]};
                } else if (isq) {   // the query in fp16, as the prefill attention takes it
                    const int64_t at = (((int64_t)b * p.n_q + head) * p.g.mpad + i) * d + dim0;
                    *(u32x2 *)(p.q + at) = u32x2{pack_f16x2(r[q][0], r[q][1]), pack_f16x2(r[q][2], r[q][3])};
                } else {     // the key, stored in bf16 (the cache's format), and widened for the prefill attention
                    const u32x2 w = u32x2{pack_bf2(r[q][0], r[q][1]), pack_bf2(r[q][2], r[q][3])};
                    const int64_t at = (int64_t)b * p.kv_bstride + (int64_t)head * p.lmax_pad * d + tiled_index(pos, dim0, d);
                    *(u32x2 *)(p.kc + at) = w;
                    if (p.kh)
                        *(u32x2 *)(p.kh + at) =
                            u32x2{pack_f16x2(bf_lo(w[0]), bf_hi(w[0])), pack_f16x2(bf_lo(w[1]), bf_hi(w[1]))};
                }
            }
        } else {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const f32x4 v = q ? c : a;
                const int r0 = (gs - qs - ks) * 16 + 4 * h + 8 * q;
                const int kvh = r0 / d, dim = r0 - kvh * d;
                const int64_t tile = (int64_t)b * p.kv_bstride + (int64_t)(kvh * (p.lmax_pad >> 5) + (pos >> 5)) * d * 32;
                const int slot = vslot(pos & 31);
                uint16_t *dst = p.vc + tile + dim * 32 + slot;
                // widened: 16-dim blocks in operand order (slot group, dim, slot)
                uint16_t *wide = p.vh ? p.vh + tile + (dim >> 4) * 512 + ((slot >> 3) * 16 + (dim & 15)) * 8 + (slot & 7) : nullptr;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t w = f2bf(v[e]);
                    dst[e * 32] = (uint16_t)w;
                    if (wide) wide[e * 8] = __builtin_bit_cast(uint16_t, (_Float16)bf2f(w));
                }
            }
        }
    }
}

// A decode step's RMSNorm scale of row m from its sum-of-squares parts (hidden /
// 16 of them, an even number): lane (m, half h) adds its half of them in order,
// then the halves.
template <int EPI>
__device__ __forceinline__ float norm_scale(const GemmParams &p, int m) {
    if (!(EPI == EPI_QKV || EPI == EPI_SWIGLU) || !p.ss_in) return 1.f;
    const int h = (threadIdx.x >> 5) & 1, half = p.nss >> 1;
    const float *q = p.ss_in + (int64_t)min(m, p.rows - 1) * p.nss + h * half;
    float s = 0.f;
    if ((p.nss & 7) == 0) {      // 16-byte pieces
#pragma unroll 10
        for (int i = 0; i < half; i += 4) {
            const f32x4 v = *(const f32x4 *)(q + i);
            s += (v[0] + v[1]) + (v[2] + v[3]);
        }
    } else {
#pragma unroll 8
        for (int i = 0; i < half; ++i) s += q[i];
    }
    s += __shfl_xor(s, 32);
    return rsqrtf(s / (float)p.K + p.eps);
}

// WR (weight rows) x WT (tokens) = four waves, each of NR x NT 32x32
// accumulators.  Both operands' 1 KB tiles of one 32-wide k step go from
// memory into an LDS stage (S stages, loads straight to LDS, S - 1 steps
// ahead of their use), so every byte is requested once per workgroup: what
// bounds the GEMM next to the matrix cores is the traffic from L2, which this
// access pattern moves at about 13 TB/s.  32x32x16 MFMAs take their operands
// from the 16x32 tiles as they are: lane l's row is l % 32 (two tiles), its 8
// k-values those of the tile's lane group 2 s + l / 32 for half s.
// The hi plane's MFMAs run over all accumulators before the lo plane's, so
// dependent MFMAs are NR NT apart.
// Work units: the first `full` tiles whole, the rest cut into p.ksplit
// k-ranges of nearly equal length, whose accumulators go to p.part as they
// are (64 lanes x 4 floats contiguous); k_gemm_fin adds the ranges in order.
// Workgroups are placed per XCD (workgroup i runs on XCD i % 8): each XCD
// takes a contiguous run of tiles in grouped order (kGroup weight tiles by
// every token tile), so those resident on one XCD share weight and token
// tiles in its L2.
constexpr int kGroup = 8;

template <int NR_, int NT_, int WR_, int WT_, int S_, int MINW_>
struct GemmTile {
    static constexpr int NR = NR_, NT = NT_, WR = WR_, WT = WT_, S = S_, MINW = MINW_;
    static constexpr int ROWS = 32 * NR * WR, TOKS = 32 * NT * WT;
    static constexpr int BLOCKS = NR * WR * NT * WT;           // 32x32 blocks
    static_assert(WR * WT == 4, "four waves");
};

__device__ __forceinline__ void tile_of(int u, int nbn, int nbm, int &bn, int &bm) {
    const int gsz = kGroup * nbm;
    const int grp = u / gsz, r = u - grp * gsz;
    const int first = grp * kGroup;
    const int gs = min(kGroup, nbn - first);
    bn = first + r % gs;
    bm = r / gs;
}

template <int EPI, bool HASLO, class TL>
__global__ __launch_bounds__(256, TL::MINW) void k_gemm(GemmParams p) {
    constexpr int NR = TL::NR, NT = TL::NT, WT = TL::WT, S = TL::S;
    constexpr int NP = HASLO ? 2 : 1;
    constexpr int RS = TL::ROWS / 16, TS = TL::TOKS / 16;     // 16-row strips, 16-token strips of the tile
    constexpr int ST = RS + NP * TS;                          // 1 KB tiles per stage: W strips, X hi, X lo
    constexpr int SC = ST / 4;                                // ... per wave
    static_assert(ST % 4 == 0, "stage tiles split evenly over the waves");
    static_assert(S * ST <= 64, "M0 holds a 16-bit LDS offset");
    extern __shared__ __align__(16) uint16_t lds[];           // [S][ST][512]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nbn = (p.N + TL::ROWS - 1) / TL::ROWS, nbm = (p.M + TL::TOKS - 1) / TL::TOKS;
    const int T = nbn * nbm, full = p.full, parts = (T - full) * p.ksplit;
    const int gfull = 8 * ((full + 7) / 8);                   // workgroups of the whole tiles
    const bool part = (int)blockIdx.x >= gfull;
    const int id = part ? (int)blockIdx.x - gfull : (int)blockIdx.x, units = part ? parts : full;
    const int u = (id & 7) * ((units + 7) / 8) + (id >> 3);
    if (u >= units) return;
    const int range = part ? u / (T - full) : 0, pt = part ? u - range * (T - full) : 0;
    int bn, bm;
    tile_of(part ? full + pt : u, nbn, nbm, bn, bm);
    const int KT = p.K >> 5;
    const int kt0 = part ? (int)((int64_t)range * KT / p.ksplit) : 0;
    const int kt1 = part ? (int)((int64_t)(range + 1) * KT / p.ksplit) : KT;
    const int NS = p.N >> 4, MS = p.M >> 4;
    const int wr = wave / WT, wt = wave % WT;

    // stage tiles of this wave: t = wave + 4 r (padding strips read strip 0,
    // masked in the epilogue)
    const uint16_t *src[SC];
#pragma unroll
    for (int r = 0; r < SC; ++r) {
        const int t = wave + 4 * r;
        int strip = t < RS ? bn * RS + t : bm * TS + (t - RS) % TS;
        strip = strip < (t < RS ? NS : MS) ? strip : 0;
        src[r] = (t < RS ? p.W : (NP == 1 || t < RS + TS) ? p.X : p.Xlo) + ((int64_t)strip * KT + kt0) * 512;
    }
    const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) uint16_t *)lds + wave * 1024;
    const uint32_t lane16 = lane * 16;
    // k tiles past the end re-read the last one (into a stage nothing reads)
    auto issue = [&](int it, int stage) {
        const int64_t at = (int64_t)min(it, kt1 - kt0 - 1) * 512;
#pragma unroll
        for (int r = 0; r < SC; ++r) load_to_lds(src[r] + at, lds0 + (stage * ST + 4 * r) * 1024, lane16);
    };

    f32x16 acc[NR][NT];
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    // this lane's piece of a fragment's half 0 (strip (lane >> 4) & 1 of the two)
    const int within = ((lane >> 4) & 1) * 512 + (((lane >> 5) << 4) + (lane & 15)) * 8;
    auto mma = [&](int stage) {
        const uint16_t *L = lds + stage * ST * 512 + within;
        const uint16_t *LW = L + wr * 2 * NR * 512, *LX = L + (RS + wt * 2 * NT) * 512;
        // (all of the step's operands requested before its first MFMA)
        u32x4 w[2][NR], bh[2][NT], bl[2][NT];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
            for (int j = 0; j < NT; ++j) bh[s][j] = *(const u32x4 *)(LX + 2 * j * 512 + s * 256);
#pragma unroll
            for (int i = 0; i < NR; ++i) w[s][i] = *(const u32x4 *)(LW + 2 * i * 512 + s * 256);
            if (HASLO) {
#pragma unroll
                for (int j = 0; j < NT; ++j) bl[s][j] = *(const u32x4 *)(LX + (TS + 2 * j) * 512 + s * 256);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
            for (int i = 0; i < NR; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[i][j] = mfma32(w[s][i], bh[s][j], acc[i][j]);
            if (HASLO) {
#pragma unroll
                for (int i = 0; i < NR; ++i)
#pragma unroll
                    for (int j = 0; j < NT; ++j) acc[i][j] = mfma32(w[s][i], bl[s][j], acc[i][j]);
            }
        }
    };

    const int n = kt1 - kt0;
#pragma unroll
    for (int st = 0; st < S - 1; ++st) issue(st, st);
    // step it: wait for its stage (this wave's share; the barrier for the
    // others', and for every wave to have read the stage the new loads
    // overwrite), request step it + S - 1, multiply
    int st = 0;
    for (int it = 0; it < n; ++it) {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"((S - 2) * SC) : "memory");
        issue(it + S - 1, st == 0 ? S - 1 : st - 1);
        mma(st);
        st = st == S - 1 ? 0 : st + 1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no load to LDS outlives the workgroup

    const int rb0 = wr * NR, tb0 = wt * NT;
    float sc[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j)
        sc[j] = part ? 1.f : norm_scale<EPI>(p, bm * TL::TOKS + (tb0 + j) * 32 + (lane & 31));
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            if (part) {
                float *o = p.part + (((int64_t)range * (T - full) + pt) * TL::BLOCKS + (rb0 + i) * (NT * WT) + tb0 + j) *
                                        1024 + lane * 4;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *(f32x4 *)(o + q * 256) =
                        f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
            } else {
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    gemm_epi<EPI>(p,
                                  f32x4{acc[i][j][8 * t], acc[i][j][8 * t + 1], acc[i][j][8 * t + 2], acc[i][j][8 * t + 3]} *
                                      sc[j],
                                  f32x4{acc[i][j][8 * t + 4], acc[i][j][8 * t + 5], acc[i][j][8 * t + 6],
                                        acc[i][j][8 * t + 7]} * sc[j],
                                  bn * RS + 2 * (rb0 + i) + t, bm * TL::TOKS + (tb0 + j) * 32 + (lane & 31));
            }
        }
}

// The k-ranges' sums in range order, then the fused epilogue: one wave per
// 16-row strip and 32 tokens of the split tiles.
template <int EPI, class TL>
__global__ __launch_bounds__(128) void k_gemm_fin(GemmParams p) {
    const int lane = threadIdx.x & 63, t = threadIdx.x >> 6;
    const int nbn = (p.N + TL::ROWS - 1) / TL::ROWS, nbm = (p.M + TL::TOKS - 1) / TL::TOKS;
    const int pt = blockIdx.x / TL::BLOCKS, blk = blockIdx.x - pt * TL::BLOCKS;
    constexpr int TB = TL::NT * TL::WT;
    const int rb = blk / TB, tb = blk - rb * TB;
    int bn, bm;
    tile_of(p.full + pt, nbn, nbm, bn, bm);
    const int strip = bn * (TL::ROWS / 16) + 2 * rb + t, m0 = bm * TL::TOKS + tb * 32;
    if (strip >= (p.N >> 4) || m0 >= p.M) return;
    const float *src = p.part + (int64_t)blockIdx.x * 1024 + 512 * t + lane * 4;
    const int64_t stride = (int64_t)gridDim.x * 1024;
    f32x4 a = f32x4{0.f, 0.f, 0.f, 0.f}, c = a;
    for (int r0 = 0; r0 < p.ksplit; r0 += 8) {
        f32x4 v[8][2];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const float *s = src + min(r0 + k, p.ksplit - 1) * stride;
            v[k][0] = *(const f32x4 *)s;
            v[k][1] = *(const f32x4 *)(s + 256);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (r0 + k < p.ksplit) {
                a += v[k][0];
                c += v[k][1];
            }
    }
    const float sc = norm_scale<EPI>(p, m0 + (lane & 31));
    gemm_epi<EPI>(p, a * sc, c * sc, strip, m0 + (lane & 31));
}

// `full` tiles whole, the others in ksplit ranges
template <int EPI, bool HASLO, class TL>
static void launch_tile(const GemmParams &p, hipStream_t s) {
    const int tiles = ((p.N + TL::ROWS - 1) / TL::ROWS) * ((p.M + TL::TOKS - 1) / TL::TOKS);
    const int rest = tiles - p.full;
    const int grid = 8 * ((p.full + 7) / 8) + 8 * ((rest * p.ksplit + 7) / 8);
    const size_t lds = (size_t)TL::S * (TL::ROWS + (HASLO ? 2 : 1) * TL::TOKS) / 16 * 1024;
    hipLaunchKernelGGL((k_gemm<EPI, HASLO, TL>), dim3(grid), dim3(256), lds, s, p);
    if (rest > 0) hipLaunchKernelGGL((k_gemm_fin<EPI, TL>), dim3(rest * TL::BLOCKS), dim3(128), 0, s, p);
}

// ---- tile shape and split --------------------------------------------------
using TileL = GemmTile<4, 2, 2, 2, 2, 2>;   // 256 x 128, 64 KB of LDS, two workgroups per CU
using TileM = GemmTile<2, 2, 2, 2, 2, 3>;   // 128 x 128, 48 KB, three
using TileS = GemmTile<2, 1, 2, 2, 4, 2>;   // 128 x 64, 64 KB (four stages)
using TileT = GemmTile<1, 1, 4, 1, 4, 4>;   // 128 x 32, 48 KB (four stages)

// The shape and split with the shortest estimated time.  A CU runs the tiles
// it is given at a measured cost per 32-wide k step and tile (us; a quarter
// more while it holds one workgroup only): whole rounds of 256 tiles plus the
// rest, cut into ksplit ranges over the CUs, plus the finishing launch and the
// traffic of the partial sums.  Measured inside whole prefills on MI355X (us,
// finishing launch included; the 16x16x32 kernel with W straight to registers
// that this one replaced -> the choice here):
//   rows x K, tokens            before     now
//   19456 x 2560, 4096          625        610 (256 x 128, the last half round in two ranges)
//    6144 x 2560, 4096          239        223 (256 x 128)
//    2560 x 9728, 4096          324        341 (256 x 128, the last quarter round in four)
//    2560 x 4096, 4096          147        163 (the same)
//    2560 x 9728, 2048          191        190 (256 x 128 in three ranges)
//    2560 x 4096, 2048           89         92 (128 x 64, the last half round in two)
//    2560 x 9728, 1024          150        117 (128 x 64, the last quarter round in four)
//   19456 x 2560, 128            53         41 (128 x 64, 48 tiles past a round in five)
//    2560 x 9728, 128           162         25 (128 x 64 in six)
//   19456 x 2560, 64             53         34 (128 x 64)
//   19456 x 2560, 32             51         27 (128 x 32 in three)
// At 4096 tokens the matrices run at 1.06-1.34 PFLOP/s (hi and lo plane counted);
// a large library product reaches 1.32 on this card.
struct GemmPlan {
    int shape, full, ksplit;
};
static GemmPlan gemm_plan(const GemmParams &p) {
    struct Shape { int rows, toks; double us; };
    static const Shape shapes[4] = {{256, 128, 0.78}, {128, 128, 0.48}, {128, 64, 0.25}, {128, 32, 0.21}};
    constexpr int kCU = 256, kMinTiles = 16;      // k tiles a range keeps at least
    constexpr double kPartBytesPerUs = 4.5e6;
    const double fin_us = p.ss_in ? 9.0 : 5.0;    // (with the RMSNorm scale to form)
    const int KT = p.K >> 5;
    GemmPlan best{1, 0, 1};
    double tbest = 1e30;
    for (int sh = 0; sh < 4; ++sh) {
        if (sh == 3 && !p.Xlo) continue;
        const Shape &c = shapes[sh];
        const int64_t tiles = (int64_t)((p.N + c.rows - 1) / c.rows) * ((p.M + c.toks - 1) / c.toks);
        const double us = p.Xlo ? c.us : 0.55 * c.us;
        for (int R = 1; R <= 16 && (R == 1 || KT / R >= kMinTiles); ++R) {
            const int64_t full = R == 1 ? tiles : tiles / kCU * kCU, rest = tiles - full;
            if (R > 1 && (!rest || rest * R * c.rows * c.toks > p.part_cap)) continue;
            const int64_t units = rest * R;
            double steps = (double)((full + kCU - 1) / kCU) * KT;
            // (split units next to whole tiles do not spread over the CUs quite evenly)
            if (R > 1) steps += (full ? 1.3 : 1.0) * ((units + kCU - 1) / kCU) * ((KT + R - 1) / R);
            if (full + units <= kCU) steps *= 1.25;
            const double t = steps * us + (R > 1 ? fin_us + 8.0 * units * c.rows * c.toks / kPartBytesPerUs : 0.0);
            if (t < tbest) tbest = t, best = GemmPlan{sh, (int)full, R};
        }
    }
    return best;
}

template <int EPI, bool HASLO>
static void launch_gemm_epi(GemmParams p, hipStream_t s) {
    const GemmPlan pl = gemm_plan(p);
    p.full = pl.full;
    p.ksplit = pl.ksplit;
    switch (pl.shape) {
        case 0: launch_tile<EPI, HASLO, TileL>(p, s); break;
        case 1: launch_tile<EPI, HASLO, TileM>(p, s); break;
        case 2: launch_tile<EPI, HASLO, TileS>(p, s); break;
        default:
            if constexpr (HASLO) launch_tile<EPI, HASLO, TileT>(p, s);
    }
}

void launch_gemm(const GemmParams &p, hipStream_t s) {
    if (!p.Xlo) {   // the gathered embedding pairs are exact in bf16
        if (p.epi == EPI_SILU) launch_gemm_epi<EPI_SILU, false>(p, s);
        else launch_gemm_epi<EPI_STORE, false>(p, s);
        return;
    }
    switch (p.epi) {
        case EPI_STORE: launch_gemm_epi<EPI_STORE, true>(p, s); break;
        case EPI_RESID: launch_gemm_epi<EPI_RESID, true>(p, s); break;
        case EPI_SWIGLU: launch_gemm_epi<EPI_SWIGLU, true>(p, s); break;
        default: launch_gemm_epi<EPI_QKV, true>(p, s); break;
    }
}

}  // namespace pipo
