// Compressed-prompt prefill: the pair step batched over a chunk of latent
// positions of every sequence.  Activations that feed an MFMA GEMM are kept
// in the 16x32 tiled bf16 layout, as two planes hi and lo (x ~= hi + lo,
// about 16 significant bits), so that both GEMM operands move as contiguous
// 1 KB tiles straight into LDS.
#include "device_common.h"
#include "kernels.h"

namespace pipo {

// ---- rows of a ragged chunk (one wave; lane b: sequence b, up to 64) -------
__global__ __launch_bounds__(64) void k_row_map(PrefillGeom g, int32_t *row0, uint32_t *blk) {
    const int b = threadIdx.x;
    const int n = b < g.B ? min(max(seq_positions(g, b) - g.c0, 0), g.clen) : 0;
    const int nb = (n + 31) >> 5;
    int end = nb;
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(end, d);
        if (b >= d) end += y;
    }
    if (b < g.B) row0[b] = (end - nb) * 32;
    for (int k = 0; k < nb; ++k) blk[end - nb + k] = row_block(b, k);
}

void launch_row_map(const PrefillGeom &g, int32_t *row0, uint32_t *blk, hipStream_t s) {
    hipLaunchKernelGGL(k_row_map, dim3(1), dim3(64), 0, s, g, row0, blk);
}

// ---- pair gather: X_in[m] = [E[a]; E[b]] for latent c0 + i of sequence b ----
__global__ void k_gather_pairs(const int32_t *tokens, const uint16_t *embed, int H, int V, int pad_id,
                               PrefillGeom g, uint16_t *xin) {
    const int cpr = (2 * H) >> 3;
    const int64_t total = (int64_t)g.M * cpr;
    for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * blockDim.x) {
        const int m = (int)(idx / cpr);
        const int k = (int)(idx - (int64_t)m * cpr) << 3;
        int b, i;
        row_seq(g, m, b, i);
        int row = pad_id;
        if (i < g.clen) {   // rows past a sequence's prompt (ragged batch) hold (PAD, PAD)
            const int t = 2 * (g.c0 + i) + (k < H ? 0 : 1);
            row = t < seq_tokens(g, b) ? clamp_id(tokens[(int64_t)b * g.n_tok + t], V) : pad_id;
        }
        const u32x4 v = *(const u32x4 *)(embed + tiled_index(row, k < H ? k : k - H, H));
        *(u32x4 *)(xin + tiled_index(m, k, 2 * H)) = v;
    }
}

void launch_gather_pairs(const int32_t *tokens, const uint16_t *embed, int H, int V, int pad_id,
                         const PrefillGeom &g, uint16_t *xin, hipStream_t s) {
    const int64_t total = (int64_t)g.M * ((2 * H) >> 3);
    int grid = (int)((total + 255) / 256);
    grid = grid > 65536 ? 65536 : grid;
    hipLaunchKernelGGL(k_gather_pairs, dim3(grid), dim3(256), 0, s, tokens, embed, H, V, pad_id, g, xin);
}

// ---- MLP compressor's skip path: x[m] = E[a] + E[b] for latent c0 + i -------
__global__ void k_gather_pair_sum(const int32_t *tokens, const uint16_t *embed, int H, int V, int pad_id,
                                  PrefillGeom g, float *x) {
    const int cpr = H >> 3;
    const int64_t total = (int64_t)g.M * cpr;
    for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * blockDim.x) {
        const int m = (int)(idx / cpr);
        const int k = (int)(idx - (int64_t)m * cpr) << 3;
        int b, i;
        row_seq(g, m, b, i);
        int ra = pad_id, rb = pad_id;
        if (i < g.clen) {
            const int t = 2 * (g.c0 + i), nb = seq_tokens(g, b);
            ra = t < nb ? clamp_id(tokens[(int64_t)b * g.n_tok + t], V) : pad_id;
            rb = t + 1 < nb ? clamp_id(tokens[(int64_t)b * g.n_tok + t + 1], V) : pad_id;
        }
        const u32x4 va = *(const u32x4 *)(embed + tiled_index(ra, k, H));
        const u32x4 vb = *(const u32x4 *)(embed + tiled_index(rb, k, H));
        float4 *dst = (float4 *)(x + (int64_t)m * H + k);
        dst[0] = make_float4(bf_lo(va[0]) + bf_lo(vb[0]), bf_hi(va[0]) + bf_hi(vb[0]),
                             bf_lo(va[1]) + bf_lo(vb[1]), bf_hi(va[1]) + bf_hi(vb[1]));
        dst[1] = make_float4(bf_lo(va[2]) + bf_lo(vb[2]), bf_hi(va[2]) + bf_hi(vb[2]),
                             bf_lo(va[3]) + bf_lo(vb[3]), bf_hi(va[3]) + bf_hi(vb[3]));
    }
}

void launch_gather_pair_sum(const int32_t *tokens, const uint16_t *embed, int H, int V, int pad_id,
                            const PrefillGeom &g, float *x, hipStream_t s) {
    const int64_t total = (int64_t)g.M * (H >> 3);
    int grid = (int)((total + 255) / 256);
    grid = grid > 65536 ? 65536 : grid;
    hipLaunchKernelGGL(k_gather_pair_sum, dim3(grid), dim3(256), 0, s, tokens, embed, H, V, pad_id, g, x);
}

// ---- MTP layer inputs of the prompt's latents (one wave per row) -----------
// Row (b, i) = [RMSNorm(h_b; g_mh); RMSNorm(E[t]; g_me)] with t the prompt token
// after latent c0 + i's pair (PAD where there is none: the last latent, whose
// row is recomputed with the selected token once it is known), written as
// tiled hi / lo planes of width 2H.
__global__ __launch_bounds__(256) void k_mtp_rows(const float *xb, const int32_t *tokens, const uint16_t *embed,
                                                  const float *gh, const float *ge, int H, int V, int pad_id,
                                                  float eps, PrefillGeom g, int M, uint16_t *xh, uint16_t *xl) {
    const int lane = threadIdx.x & 63;
    const int m = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (m >= M) return;
    int b, i;
    row_seq(g, m, b, i);
    const int t = 2 * (g.c0 + i) + 2;
    const int tok = (i < g.clen && t < seq_tokens(g, b)) ? clamp_id(tokens[(int64_t)b * g.n_tok + t], V) : pad_id;
    const float *xr = xb + (int64_t)m * H;
    float a = 0.f, e = 0.f;
    for (int k = lane * 8; k < H; k += 512) {
        const float4 x0 = *(const float4 *)(xr + k), x1 = *(const float4 *)(xr + k + 4);
        a += x0.x * x0.x + x0.y * x0.y + x0.z * x0.z + x0.w * x0.w + x1.x * x1.x + x1.y * x1.y + x1.z * x1.z +
             x1.w * x1.w;
        const u32x4 w = *(const u32x4 *)(embed + tiled_index(tok, k, H));
#pragma unroll
        for (int q = 0; q < 4; ++q) e += bf_lo(w[q]) * bf_lo(w[q]) + bf_hi(w[q]) * bf_hi(w[q]);
    }
    a = wave_sum(a);
    e = wave_sum(e);
    const float s1 = rsqrtf(a / (float)H + eps), s2 = rsqrtf(e / (float)H + eps);
    for (int k = lane * 8; k < H; k += 512) {
        const float4 x0 = *(const float4 *)(xr + k), x1 = *(const float4 *)(xr + k + 4);
        const float4 g0 = *(const float4 *)(gh + k), g1 = *(const float4 *)(gh + k + 4);
        const float f[8] = {x0.x * s1 * g0.x, x0.y * s1 * g0.y, x0.z * s1 * g0.z, x0.w * s1 * g0.w,
                            x1.x * s1 * g1.x, x1.y * s1 * g1.y, x1.z * s1 * g1.z, x1.w * s1 * g1.w};
        u32x4 hi, lo;
        split8(f, hi, lo);
        const int64_t at = tiled_index(m, k, 2 * H);
        *(u32x4 *)(xh + at) = hi;
        *(u32x4 *)(xl + at) = lo;
        const u32x4 w = *(const u32x4 *)(embed + tiled_index(tok, k, H));
        const float4 e0 = *(const float4 *)(ge + k), e1 = *(const float4 *)(ge + k + 4);
        const float fe[8] = {bf_lo(w[0]) * s2 * e0.x, bf_hi(w[0]) * s2 * e0.y, bf_lo(w[1]) * s2 * e0.z,
                             bf_hi(w[1]) * s2 * e0.w, bf_lo(w[2]) * s2 * e1.x, bf_hi(w[2]) * s2 * e1.y,
                             bf_lo(w[3]) * s2 * e1.z, bf_hi(w[3]) * s2 * e1.w};
        split8(fe, hi, lo);
        const int64_t at2 = tiled_index(m, H + k, 2 * H);
        *(u32x4 *)(xh + at2) = hi;
        *(u32x4 *)(xl + at2) = lo;
    }
}

void launch_mtp_rows(const float *xb, const int32_t *tokens, const uint16_t *embed, const float *gh, const float *ge,
                     int H, int V, int pad_id, float eps, const PrefillGeom &g, int M, uint16_t *xh, uint16_t *xl,
                     hipStream_t s) {
    hipLaunchKernelGGL(k_mtp_rows, dim3((M + 3) / 4), dim3(256), 0, s, xb, tokens, embed, gh, ge, H, V, pad_id, eps,
                       g, M, xh, xl);
}

// ---- regular decoding: the prompt's tokens one per position, x = E[t] -----
// Row (b, i) of the chunk holds token c0 + i of sequence b (rows past the
// chunk hold E[pad_id]); fp32 residual rows [M][H].
__global__ void k_gather_tokens(const int32_t *tokens, const uint16_t *embed, int H, int V, int pad_id,
                                PrefillGeom g, float *x) {
    const int cpr = H >> 3;
    const int64_t total = (int64_t)g.M * cpr;
    for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * blockDim.x) {
        const int m = (int)(idx / cpr);
        const int k = (int)(idx - (int64_t)m * cpr) << 3;
        int b, i;
        row_seq(g, m, b, i);
        const int t = g.c0 + i;
        const int row = (i < g.clen && t < seq_tokens(g, b)) ? clamp_id(tokens[(int64_t)b * g.n_tok + t], V) : pad_id;
        const u32x4 v = *(const u32x4 *)(embed + tiled_index(row, k, H));
        float4 *dst = (float4 *)(x + (int64_t)m * H + k);
        dst[0] = make_float4(bf_lo(v[0]), bf_hi(v[0]), bf_lo(v[1]), bf_hi(v[1]));
        dst[1] = make_float4(bf_lo(v[2]), bf_hi(v[2]), bf_lo(v[3]), bf_hi(v[3]));
    }
}

void launch_gather_tokens(const int32_t *tokens, const uint16_t *embed, int H, int V, int pad_id,
                          const PrefillGeom &g, float *x, hipStream_t s) {
    const int64_t total = (int64_t)g.M * (H >> 3);
    int grid = (int)((total + 255) / 256);
    grid = grid > 65536 ? 65536 : grid;
    hipLaunchKernelGGL(k_gather_tokens, dim3(grid), dim3(256), 0, s, tokens, embed, H, V, pad_id, g, x);
}

// ---- RMSNorm of fp32 rows into the tiled bf16 layout ----------------------
// One workgroup of sixteen waves per 16-row tile row: wave w first forms the
// sum of squares of row w (five 1 KB loads in flight), then writes every
// sixteenth 16x32 tile whole: lane l normalises row l mod 16, columns
// 8 (l / 16) .. + 7 of the tile, so each store instruction covers one
// contiguous 1 KB tile (full cache lines, no partial-line writes shared with
// other workgroups).  A small prompt has few tile rows, so the row's latency
// is what counts there.
__global__ __launch_bounds__(1024) void k_rmsnorm_tiled(const float *x, const float *gain, int H, float eps,
                                                        int M, uint16_t *xh, uint16_t *xl) {
    __shared__ float s_sc[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r0 = blockIdx.x * 16;
    if (r0 >= M) return;
    {
        const float *xr = x + (int64_t)min(r0 + wave, M - 1) * H;
        float a = 0.f;
#pragma unroll 5
        for (int k = lane * 4; k < H; k += 256) {
            const float4 v = *(const float4 *)(xr + k);
            a += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
        }
        a = wave_sum(a);
        if (lane == 0) s_sc[wave] = rsqrtf(a / (float)H + eps);
    }
    __syncthreads();
    const int j = lane & 15, c = lane >> 4;
    const float sc = s_sc[j];
    const float *xr = x + (int64_t)min(r0 + j, M - 1) * H;
    const int KT = H >> 5;
    uint16_t *th = xh + (int64_t)(r0 >> 4) * KT * 512 + lane * 8;
    uint16_t *tl = xl + (int64_t)(r0 >> 4) * KT * 512 + lane * 8;
#pragma unroll 2
    for (int kt = wave; kt < KT; kt += 16) {
        const int k = kt * 32 + c * 8;
        const float4 x0 = *(const float4 *)(xr + k), x1 = *(const float4 *)(xr + k + 4);
        const float4 g0 = *(const float4 *)(gain + k), g1 = *(const float4 *)(gain + k + 4);
        const float f[8] = {x0.x * sc * g0.x, x0.y * sc * g0.y, x0.z * sc * g0.z, x0.w * sc * g0.w,
                            x1.x * sc * g1.x, x1.y * sc * g1.y, x1.z * sc * g1.z, x1.w * sc * g1.w};
        u32x4 hi, lo;
        split8(f, hi, lo);
        *(u32x4 *)(th + (int64_t)kt * 512) = hi;
        *(u32x4 *)(tl + (int64_t)kt * 512) = lo;
    }
}

// Few rows: one wave per row, the row in registers between its sum and its
// stores, so one round trip to memory (16-byte pieces of the tiles; with
// sixteen rows a workgroup reads its 16-row tile alone through one CU).
// 128 rows of 2560: 10.9 us with the 16-row kernel, 5.7 us here.
constexpr int kRowPieces = 10;       // 512-column pieces of a row: up to 5120 columns
constexpr int kRowsSmall = 1024;
__global__ __launch_bounds__(256) void k_rmsnorm_rows(const float *x, const float *gain, int H, float eps, int M,
                                                      int rows, uint16_t *xh, uint16_t *xl) {
    const int lane = threadIdx.x & 63;
    const int m = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (m >= rows) return;
    const float *xr = x + (int64_t)min(m, M - 1) * H;
    float4 v[kRowPieces][2];
    float a = 0.f;
#pragma unroll
    for (int i = 0; i < kRowPieces; ++i) {
        const int k = i * 512 + lane * 8;
        const float4 *q = (const float4 *)(xr + (k < H ? k : 0));
        v[i][0] = q[0];
        v[i][1] = q[1];
    }
#pragma unroll
    for (int i = 0; i < kRowPieces; ++i) {
        const float4 p = v[i][0], q = v[i][1];
        const float t = p.x * p.x + p.y * p.y + p.z * p.z + p.w * p.w + q.x * q.x + q.y * q.y + q.z * q.z + q.w * q.w;
        a += i * 512 + lane * 8 < H ? t : 0.f;
    }
    const float sc = rsqrtf(wave_sum(a) / (float)H + eps);
#pragma unroll
    for (int i = 0; i < kRowPieces; ++i) {
        const int k = i * 512 + lane * 8;
        if (k >= H) break;
        const float4 g0 = *(const float4 *)(gain + k), g1 = *(const float4 *)(gain + k + 4);
        const float f[8] = {v[i][0].x * sc * g0.x, v[i][0].y * sc * g0.y, v[i][0].z * sc * g0.z, v[i][0].w * sc * g0.w,
                            v[i][1].x * sc * g1.x, v[i][1].y * sc * g1.y, v[i][1].z * sc * g1.z, v[i][1].w * sc * g1.w};
        u32x4 hi, lo;
        split8(f, hi, lo);
        const int64_t at = tiled_index(m, k, H);
        *(u32x4 *)(xh + at) = hi;
        *(u32x4 *)(xl + at) = lo;
    }
}

void launch_rmsnorm_tiled(const float *x, const float *gain, int H, float eps, int M, uint16_t *xh,
                          uint16_t *xl, hipStream_t s) {
    const int tiles = (M + 15) / 16;
    if (tiles * 16 <= kRowsSmall && H <= 512 * kRowPieces)
        hipLaunchKernelGGL(k_rmsnorm_rows, dim3(tiles * 4), dim3(256), 0, s, x, gain, H, eps, M, tiles * 16, xh, xl);
    else
        hipLaunchKernelGGL(k_rmsnorm_tiled, dim3(tiles), dim3(1024), 0, s, x, gain, H, eps, M, xh, xl);
}

// ---- last latent of each sequence into the decode residual buffer --------
// The last position's residual becomes the decode state x (with the
// sum-of-squares part of every 16-element strip, as the decode GEMVs read
// them); pos is set to that position, so the heads that follow run there and
// advance it, and the step counter restarts.
__global__ __launch_bounds__(256) void k_pick_last(const float *x, int H, PrefillGeom g, float *xdec,
                                                   float *ss, int32_t *pos, int32_t *step, int regular) {
    const int b = blockIdx.x;
    const int nb = seq_tokens(g, b);
    const int last = (regular ? nb : (nb + 1) / 2) - 1;   // the sequence's last position
    if (last < g.c0 || last >= g.c0 + g.clen) return;
    const float *xr = x + (int64_t)row_of(g, b, last - g.c0) * H;
    for (int k = threadIdx.x; k < H; k += 256) xdec[(int64_t)b * H + k] = xr[k];
    for (int st = threadIdx.x; st < (H >> 4); st += 256) {
        float a = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) a += xr[16 * st + i] * xr[16 * st + i];
        ss[(int64_t)b * (H >> 4) + st] = a;
    }
    if (threadIdx.x == 0) {
        pos[b] = last;
        step[b] = 0;
    }
}

void launch_pick_last(const float *x, int H, const PrefillGeom &g, float *xdec, float *ss, int32_t *pos,
                      int32_t *step, int regular, hipStream_t s) {
    hipLaunchKernelGGL(k_pick_last, dim3(g.B), dim3(256), 0, s, x, H, g, xdec, ss, pos, step, regular);
}

}  // namespace pipo
