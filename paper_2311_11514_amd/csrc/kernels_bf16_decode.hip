// Decode projections (up to 64 token rows): weight-streaming skinny GEMMs on the matrix cores with the
// whole sub-layer glue fused into their tails.  Two forms: decode_proj_kernel (one or two rows, and up to 32 where the
// operand is small: one kernel, complete dot products per block, no scratch buffers, no atomics) and, further down,
// decode_splitk_kernel + decode_finish_kernel (operand shared through LDS, contraction split over blocks);
// decode_single_kernel chooses.
//
// Main loop of decode_proj_kernel.  Each wave streams 1 KB weight tiles with one 128-bit load per lane (fully coalesced,
// non-temporal) and feeds them to v_mfma_f32_16x16x32_bf16 against a 16-token activation tile: 16 MFMA
// cycles per KB, a quarter of what unpacking bf16 on the vector ALU would cost, so the kernel stays
// HBM-bound up to 32 rows.  Activations arrive as hi + lo bf16 pairs (two MFMAs per tile, free here).
// A block owns one unit = UT 16-feature tiles over the WHOLE contraction; its waves interleave over the
// k-tiles and are summed through LDS in wave order (bit-reproducible).  Because a block holds complete
// dot products, the epilogue runs in registers on the 16x16 accumulator layout (lane = one token, four
// consecutive features):
//   QKV    : x rstd of the input rows, RoPE, q -> hi/lo rows, k / v -> KV cache.  The QKV weight tiles are
//            packed so that a tile holds 8 rotary pairs (features i and i + d/2), which lie 32 lanes apart.
//   RESID  : h += partial; (h * gain of the next norm) -> hi/lo operand of the next projection (dec_act_offset);
//            per-unit sum of squares of the new h, from which the next kernel derives rstd
//   SWIGLU : x rstd, silu(gate) * up -> hi/lo operand of the W2 projection (gate / up tiles interleaved)
//   RAW    : x rstd (if the input is a normalised stream), plain fp32 partial (validation surface)
//   BEST   : x rstd, the unit's largest value per row and its column (LM head: no logits leave the kernel)
// RMSNorm is thus never a kernel of its own in decode: y = rstd * ((h*g) . W), with rstd a per-row
// scalar applied after the contraction.
#include <algorithm>
#include <cstdlib>

#include "kernels.h"
#include "kvlayout.h"

namespace HX_NS {


// rstd of a token row from the per-unit sums of squares of the residual stream
__device__ inline void rstd_row(const DecodeEpi &e, int t, int lane, float *s_rstd) {
    float r = 1.0f;
    if (e.ssq_in) {
        float ss = 0.f;
        for (int i = lane; i < e.ssq_units; i += 64) ss += e.ssq_in[(size_t)t * e.ssq_units + i];
        ss = wave_sum(ss);
        r = 1.0f / sqrtf(ss / (float)e.norm_dim + e.eps);
    }
    if (lane == 0) s_rstd[t] = r;
}
// The same in two halves, so that the loads can be requested ahead of other memory traffic and summed later: the
// first RSTD_REGS * 64 units wait in registers (hidden sizes up to 8192), any further ones are fetched in the second half.
constexpr int RSTD_REGS = 8;
__device__ inline void rstd_request(const DecodeEpi &e, int t, int lane, float (&sv)[RSTD_REGS]) {
#pragma unroll
    for (int j = 0; j < RSTD_REGS; ++j) sv[j] = e.ssq_in[(size_t)t * e.ssq_units + min(lane + 64 * j, e.ssq_units - 1)];
}
__device__ inline void rstd_finish(const DecodeEpi &e, int t, int lane, const float (&sv)[RSTD_REGS], float *s_rstd) {
    float ss = 0.f;
#pragma unroll
    for (int j = 0; j < RSTD_REGS; ++j) ss += lane + 64 * j < e.ssq_units ? sv[j] : 0.f;      // lane's units ascending
    for (int i = lane + 64 * RSTD_REGS; i < e.ssq_units; i += 64) ss += e.ssq_in[(size_t)t * e.ssq_units + i];
    ss = wave_sum(ss);
    if (lane == 0) s_rstd[t] = 1.0f / sqrtf(ss / (float)e.norm_dim + e.eps);
}

__device__ inline void store_split4(const float x[4], h16_t *hi, h16_t *lo, size_t off) {
    uint2 o, ol;
    split_pack2(x[0], x[1], o.x, ol.x);
    split_pack2(x[2], x[3], o.y, ol.y);
    *reinterpret_cast<uint2 *>(hi + off) = o;
    *reinterpret_cast<uint2 *>(lo + off) = ol;
}
// 4 consecutive features k..k+3 of one of T tokens into a decode operand (hi and lo parts)
__device__ inline void store_act4(const float x[4], h16_t *xa, int token, int k, int k_tiles, int T) {
    uint2 o, ol;
    split_pack2(x[0], x[1], o.x, ol.x);
    split_pack2(x[2], x[3], o.y, ol.y);
    *reinterpret_cast<uint2 *>(xa + dec_act_offset(token, k, k_tiles, 0, T)) = o;
    *reinterpret_cast<uint2 *>(xa + dec_act_offset(token, k, k_tiles, 1, T)) = ol;
}

// What the register epilogue reads from memory, requested long before it is used (the finishing wave asks for it at
// kernel start, so the answers arrive behind the first weights instead of adding two memory round trips to the
// block's tail).  Rows beyond T re-read row T - 1, so that no request sits behind a branch.
//   QKV   : first the row's position, then (once it is known) the rotary table entries of this lane's four pairs
//   RESID : the residual stream and the next norm's gain at this lane's four columns
struct EpiPre {
    floatx4 a, b;
    int pos;
};
template <int MODE>
__device__ inline void epi_request_first(EpiPre &p, int unit, int b, int lane, int N, int T, const DecodeEpi &e) {
    const int token = min((lane & 15) + 16 * b, T - 1), g = lane >> 4;
    if (MODE == DEC_QKV) p.pos = e.row_pos[token];
    if (MODE == DEC_RESID) {
        const int n0 = unit * 16 + 4 * g;
        p.a = *reinterpret_cast<const floatx4 *>(e.h + (size_t)token * N + n0);
        if (!e.last_layer) p.b = *reinterpret_cast<const floatx4 *>(e.g_next + n0);
    }
}
template <int MODE>
__device__ inline void epi_request_second(EpiPre &p, int unit, int lane, const DecodeEpi &e) {
    if (MODE == DEC_QKV) {
        const int d = e.kg.d, half = d >> 1, tiles_per_head = d >> 4, g = lane >> 4;
        const int head = unit / tiles_per_head, tl = unit - head * tiles_per_head;
        if (head < e.hq_l + e.kg.hkv_l) {
            const int i0 = tl * 8 + 4 * (g & 1);
            p.a = *reinterpret_cast<const floatx4 *>(e.cos_tab + (size_t)p.pos * half + i0);
            p.b = *reinterpret_cast<const floatx4 *>(e.sin_tab + (size_t)p.pos * half + i0);
        }
    }
}

// Register epilogue of one unit (UT 16-feature tiles) and one 16-token tile, on complete dot products in the
// 16x16 accumulator layout: lane = (token j = lane % 16, row group g = lane / 16) holds rows 4g .. 4g+3 of each tile.
// Must be called by a whole wave (it shuffles across the row groups).
template <int MODE, int UT>
__device__ inline void decode_epilogue(const floatx4 (&v)[UT], int unit, int b, int lane, int N, int T, const DecodeEpi &e,
                                       const float *s_rstd, const EpiPre &pre) {
    const int token = (lane & 15) + 16 * b, g = lane >> 4;
    const bool valid = token < T;
    const float r = (MODE != DEC_RESID && valid) ? s_rstd[token] : 1.0f;

    if (MODE == DEC_RAW) {
#pragma unroll
        for (int u = 0; u < UT; ++u) {
            const int n0 = (unit * UT + u) * 16 + 4 * g;
            if (valid) *reinterpret_cast<floatx4 *>(e.raw_out + (size_t)token * N + n0) = v[u] * r;
        }
    } else if (MODE == DEC_BEST) {
        float bv = -INFINITY;
        int bi = 0x7fffffff;
#pragma unroll
        for (int u = 0; u < UT; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float x = v[u][j] * r;
                const int n = (unit * UT + u) * 16 + 4 * g + j;
                if (n < e.valid && (x > bv || (x == bv && n < bi))) { bv = x; bi = n; }
            }
#pragma unroll
        for (int o = 16; o <= 32; o <<= 1) {
            const float x = __shfl_xor(bv, o, 64);
            const int n = __shfl_xor(bi, o, 64);
            if (x > bv || (x == bv && n < bi)) { bv = x; bi = n; }
        }
        if (g == 0 && valid) {
            const size_t at = (size_t)token * (N / 16 / UT) + unit;
            e.best_val[at] = bv;
            e.best_id[at] = bi;
        }
    } else if (MODE == DEC_RESID) {
        const int n0 = unit * 16 + 4 * g;
        float ss = 0.f;
        if (valid) {
            const floatx4 h4 = pre.a;
            if (e.last_layer) {
                // stage output: the partial without residual, and the residual it belongs to
                uint2 po;
                po.x = pack_h16x2(v[0][0], v[0][1]);
                po.y = pack_h16x2(v[0][2], v[0][3]);
                *reinterpret_cast<uint2 *>(e.out_partial + (size_t)token * N + n0) = po;
                if (e.out_resid) {
                    uint2 ro;
                    ro.x = pack_h16x2(h4[0], h4[1]);
                    ro.y = pack_h16x2(h4[2], h4[3]);
                    *reinterpret_cast<uint2 *>(e.out_resid + (size_t)token * N + n0) = ro;
                }
            } else {
                const floatx4 hn = h4 + v[0];
                *reinterpret_cast<floatx4 *>(e.h + (size_t)token * N + n0) = hn;
                const floatx4 g4 = pre.b;
                const float x[4] = {hn[0] * g4[0], hn[1] * g4[1], hn[2] * g4[2], hn[3] * g4[3]};
                store_act4(x, e.hg, token, n0, N >> 5, T);
                ss = hn[0] * hn[0] + hn[1] * hn[1] + hn[2] * hn[2] + hn[3] * hn[3];
            }
        }
        if (!e.last_layer) {
            ss += __shfl_xor(ss, 16, 64);
            ss += __shfl_xor(ss, 32, 64);
            if (g == 0 && valid) e.ssq_out[(size_t)token * (N >> 4) + unit] = ss;
        }
    } else if (MODE == DEC_SWIGLU) {
        // unit = one gate tile (v[0]) and the matching up tile (v[1]): 16 features of u
        if (valid) {
            const int f0 = unit * 16 + 4 * g;
            float uu[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float aa = v[0][j] * r;
                uu[j] = aa / (1.0f + __expf(-aa)) * (v[UT - 1][j] * r);
            }
            store_act4(uu, e.u, token, f0, e.F_l >> 5, T);
        }
    } else {   // DEC_QKV
        const int d = e.kg.d, half = d >> 1, tiles_per_head = d >> 4;
        const int head = unit / tiles_per_head, tl = unit - head * tiles_per_head;
        floatx4 mine = v[0] * r, other;
#pragma unroll
        for (int j = 0; j < 4; ++j) other[j] = __shfl_xor(mine[j], 32, 64);
        const bool low = g < 2;                       // rows 0-7 of the tile: features i; rows 8-15: i + d/2
        const int i0 = tl * 8 + 4 * (g & 1);          // first rotary pair index held by this lane
        if (valid) {
            const int pos = pre.pos;
            float out[4];
            if (head < e.hq_l + e.kg.hkv_l) {
                const floatx4 c4 = pre.a, s4 = pre.b;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float lo = low ? mine[j] : other[j], hi = low ? other[j] : mine[j];
                    out[j] = low ? lo * c4[j] - hi * s4[j] : hi * c4[j] + lo * s4[j];
                }
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) out[j] = mine[j];
            }
            const int e0 = i0 + (low ? 0 : half);     // element index inside the head
            if (head < e.hq_l) {
                store_split4(out, e.q_hi, e.q_lo, ((size_t)token * e.hq_l + head) * d + e0);
            } else if (head < e.hq_l + e.kg.hkv_l) {
                const size_t slab = (size_t)token * e.kg.seq_stride + (size_t)(head - e.hq_l) * e.kg.smax * d;
                uint2 o;
                o.x = pack_h16x2(out[0], out[1]);
                o.y = pack_h16x2(out[2], out[3]);
                *reinterpret_cast<uint2 *>(e.kc + slab + kv_k_offset(pos, e0, d)) = o;
            } else {
                const size_t slab =
                    (size_t)token * e.kg.seq_stride + (size_t)(head - e.hq_l - e.kg.hkv_l) * e.kg.smax * d;
#pragma unroll
                for (int j = 0; j < 4; ++j) e.vc[slab + kv_v_offset(pos, e0 + j, d)] = f32_to_h16(out[j]);
            }
        }
    }
}

constexpr int kXldsMaxBytes = 64 * 1024;      // activation operand staged in LDS up to this size

// NP = 0: one or two rows, compact operand.  XLDS: the whole operand is staged once per block in LDS, so the main loop
// issues nothing but weight loads; otherwise each lane fetches its 16-byte pieces per k-tile (L2 hits).
// NP = 1, 2, 4: 3 to 8, 16, 32 rows, NP operand tiles per k-tile (dec_act_offset), each one contiguous 1 KB request.
// UT: feature tiles of a block: one unit of the epilogue (a gate and an up tile for SWIGLU), or two of them (unit_pairs).
template <int NP, int UT, int WAVES, int UNROLL, int MODE, bool XLDS, int XR>
__global__ __launch_bounds__(WAVES * 64) void decode_proj_kernel(const h16_t *__restrict__ Wp,
                                                                const h16_t *__restrict__ Xa, int N, int k_tiles,
                                                                int T, DecodeEpi e) {
    constexpr int NB = NP <= 2 ? 1 : NP / 2;       // 16-token result tiles
    constexpr int NX = NP == 0 ? 2 : NP;           // operand pieces per k-tile
    static_assert(!XLDS || NP == 0, "only the compact operand is staged");
    __shared__ floatx4 red[WAVES][UT * NB][64];
    __shared__ float s_rstd[32];
    extern __shared__ h16x8 xs[];          // XLDS: copy of Xa, [token][k_tile][plane][lane group]
    const int unit = blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;

    // QKV: the lo products have sums of their own, as in the split form (half as many roundings per sum)
    constexpr int LO = MODE == DEC_QKV && NP >= 2 ? 1 : 0;
    floatx4 acc[1 + LO][UT][NB];
#pragma unroll
    for (int u = 0; u < UT; ++u)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[0][u][b] = acc[LO][u][b] = floatx4{0.f, 0.f, 0.f, 0.f};

    const h16x8 *wp[UT];
#pragma unroll
    for (int u = 0; u < UT; ++u)
        wp[u] = reinterpret_cast<const h16x8 *>(Wp) + (size_t)(unit * UT + u) * 64 + lane;
    const size_t kstride = (size_t)(N >> 4) * 64;          // k-tile-major weights: one k-tile of all features
    // operand B.  Compact: lane (token j, group g) takes hi at xg[kt * 8] and lo at xg[kt * 8 + 4]; tiles: slot `lane` of tile
    // kt * NP + piece
    const bool xv = NP > 0 || (lane & 15) < T;
    const h16x8 *xg = NP > 0 ? reinterpret_cast<const h16x8 *>(Xa) + lane
                             : (XLDS ? xs : reinterpret_cast<const h16x8 *>(Xa)) + (size_t)(xv ? lane & 15 : 0) * k_tiles * 8 + (lane >> 4);
    const h16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
    // Wave w owns k-tiles w, w + WAVES, ...; it holds a ring of UNROLL of them per feature tile in registers.  The
    // first ring round is requested before anything else, so the weights are already on their way while the block
    // stages the activation operand and derives the rows' rstd.
    const int rounds = (k_tiles - wave + WAVES - 1) / WAVES / UNROLL;
    // request order = arrival order: the operand copy and the sums of squares (L2 hits) go out first and are
    // waited for first; the weights requested right behind them stay in flight meanwhile
    // (every request below is unconditional, out-of-range ones re-read a valid address: the compiler can only count
    // requests in flight exactly, and so wait for the oldest alone, when none of them sits behind a branch)
    EpiPre pre;
    // wave b finishes token tile b; the two feature tiles of a residual block are finished by waves of their own
    constexpr int FU = MODE == DEC_RESID || MODE == DEC_QKV ? 1 : MODE == DEC_SWIGLU ? 2 : UT, FG = UT / FU;
    const int fb = wave % NB, fu = wave / NB;
    const bool finisher = wave < NB * FG;
    if (finisher) epi_request_first<MODE>(pre, unit * FG + fu, fb, lane, N, T, e);
    h16x8 xr[XLDS ? XR : 1];
    const int n16 = T * k_tiles * 8;
    if (XLDS) {
#pragma unroll
        for (int j = 0; j < XR; ++j)
            xr[j] = reinterpret_cast<const h16x8 *>(Xa)[min((int)threadIdx.x + j * WAVES * 64, n16 - 1)];
    }
    float sv[RSTD_REGS], sv2[NP >= 2 ? RSTD_REGS : 1];
    const bool rstd_wave = MODE != DEC_RESID && wave < T && e.ssq_in != nullptr;       // wave t derives rstd of row t (and t + WAVES)
    const bool rstd_wave2 = NP >= 2 && rstd_wave && wave + WAVES < T;
    if (rstd_wave) rstd_request(e, wave, lane, sv);
    if constexpr (NP >= 2) {
        if (rstd_wave2) rstd_request(e, wave + WAVES, lane, sv2);
    }
    // ring slot = the weight tiles of one k-tile and, when the operand is not staged in LDS, its hi / lo pieces too
    // (requested together, so that no wait for an operand piece ever drains the weight requests behind it)
    h16x8 a[UNROLL][UT], xq[XLDS ? 1 : UNROLL][NX];
    auto request = [&](int i, int kt) {
        if (!XLDS) {
#pragma unroll
            // unconditional (see above): lanes past the last row re-read row 0 and feed output columns nobody stores
            for (int q = 0; q < NX; ++q) xq[i][q] = NP > 0 ? xg[((size_t)kt * NX + q) * 64] : xg[kt * 8 + 4 * q];
        }
#pragma unroll
        for (int u = 0; u < UT; ++u) a[i][u] = __builtin_nontemporal_load(wp[u] + (size_t)kt * kstride);
    };
#pragma unroll
    for (int i = 0; i < UNROLL; ++i) request(i, min(wave + i * WAVES, k_tiles - 1));
    if (finisher) epi_request_second<MODE>(pre, unit * FG + fu, lane, e);
    if (XLDS) {
#pragma unroll
        for (int j = 0; j < XR; ++j) {
            const int idx = threadIdx.x + j * WAVES * 64;
            if (idx < n16) xs[idx] = xr[j];
        }
    }
    if (rstd_wave) rstd_finish(e, wave, lane, sv, s_rstd);
    if constexpr (NP >= 2) {
        if (rstd_wave2) rstd_finish(e, wave + WAVES, lane, sv2, s_rstd);
    }
    if (MODE != DEC_RESID)
        for (int t = wave + (rstd_wave2 ? 2 * WAVES : rstd_wave ? WAVES : 0); t < T; t += WAVES) rstd_row(e, t, lane, s_rstd);
    if (XLDS) __syncthreads();       // (s_rstd is read behind the barrier of the reduction below)

    // the k-tile held by ring slot i against the operand: lo, then hi (NP = 1: both in one tile)
    auto contract = [&](int i, int kt) {
        h16x8 x[NX];
#pragma unroll
        for (int q = 0; q < NX; ++q) x[q] = XLDS ? (xv ? xg[kt * 8 + 4 * q] : zero) : xq[i][q];
#pragma unroll
        for (int u = 0; u < UT; ++u)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                if (NX > 1) acc[LO][u][b] = hx_mfma16(a[i][u], x[NX > 1 ? 2 * b + 1 : 0], acc[LO][u][b]);
                acc[0][u][b] = hx_mfma16(a[i][u], x[2 * b], acc[0][u][b]);
            }
    };
    // steady state: slot i is consumed and at once refilled with the tile one ring round ahead, so UNROLL - 1
    // requests per feature tile stay in flight all the time
    for (int rd = 1; rd < rounds; ++rd) {
#pragma unroll
        for (int i = 0; i < UNROLL; ++i) {
            const int kt = wave + ((rd - 1) * UNROLL + i) * WAVES;
            contract(i, kt);
            request(i, kt + UNROLL * WAVES);
            if (!XLDS) __builtin_amdgcn_sched_barrier(0);       // keep each refill right behind its slot's use
        }
    }
    // The last full round is refilled as well, with the wave's remaining (fewer than UNROLL) k-tiles, so that those are
    // in flight while the round is consumed instead of being fetched one by one behind it; slots past the last k-tile
    // re-read it (unconditional requests, see above) and are not used.  With no full round at all the first ring round,
    // requested at kernel start, already is this remainder.
    const int kt_rem = wave + rounds * UNROLL * WAVES;       // the wave's first k-tile beyond its full rounds
    if (rounds > 0) {
        if (kt_rem < k_tiles) {       // (uniform over the wave; a wave without remainder issues no request it does not use)
#pragma unroll
            for (int i = 0; i < UNROLL; ++i) {
                contract(i, wave + ((rounds - 1) * UNROLL + i) * WAVES);
                request(i, min(kt_rem + i * WAVES, k_tiles - 1));
                if (!XLDS) __builtin_amdgcn_sched_barrier(0);
            }
        } else {
#pragma unroll
            for (int i = 0; i < UNROLL; ++i) contract(i, wave + ((rounds - 1) * UNROLL + i) * WAVES);
        }
    }
#pragma unroll
    for (int i = 0; i < UNROLL; ++i) {
        const int kt = kt_rem + i * WAVES;       // uniform over the wave
        if (kt < k_tiles) contract(i, kt);
    }

#pragma unroll
    for (int u = 0; u < UT; ++u)
#pragma unroll
        for (int b = 0; b < NB; ++b) red[wave][u * NB + b][lane] = LO ? acc[0][u][b] + acc[LO][u][b] : acc[0][u][b];
    __syncthreads();
    if (!finisher) return;

    floatx4 v[FU];
#pragma unroll
    for (int u = 0; u < FU; ++u) {
        const int at = (fu * FU + u) * NB + fb;
        v[u] = red[0][at][lane];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) v[u] += red[w][at][lane];
        if (NP == 1) {          // token columns 8 .. 15 hold the lo parts of tokens 0 .. 7
#pragma unroll
            for (int r = 0; r < 4; ++r) v[u][r] += __shfl_xor(v[u][r], 8, 64);
        }
    }
    decode_epilogue<MODE, FU>(v, unit * FG + fu, fb, lane, N, T, e, s_rstd, pre);
}

// -------------------------------------------------------------------------------------------------
// Batched decode (3 <= T <= 64 rows).  With more than a couple of rows the activation operand outweighs the
// weights a block streams (32 rows of hi + lo pairs are 4 KB per k-tile against 1 KB of weights per 16 features).  Here the
// eight waves of a block own eight neighbouring feature tiles and walk the SAME k-tiles, so the block stages each
// chunk of k-tiles of the operand once in LDS (global -> registers -> LDS, double-buffered, whole 1 KB fragment tiles) and all
// waves read it from there; a k-tile's weights for the block are one contiguous 8 KB run.  To still fill the chip the
// contraction is split over blockIdx.y; the fp32 partial sums go to a scratch buffer [split][token][feature] and
// decode_finish_kernel adds them in split order (bit-reproducible) and runs the same register epilogue as the
// single-kernel path.  Bound by HBM up to 32 rows (W1/W3 of the full-width 70B layer: 939 MB in 157 us), beyond by the LDS
// reads: a wave reads NP KB for every KB of weights.  Chunks of 4 k-tiles instead of 8 beyond 32 rows (the LM head: up to 64
// rows per pass) keep two blocks on a CU, one covering the other's barriers: 48 rows of the 8192 x 32000 head 113 -> 108 us,
// two passes of 32 rows 195.
// -------------------------------------------------------------------------------------------------
// k-tiles per chunk: 16 .. 64 KB of operand in the two LDS buffers, so that two blocks fit a CU at any number of rows
constexpr int sk_chunk(int np) { return np <= 4 ? 8 : 4; }

// NP: operand tiles per k-tile (dec_act_tiles), 1 .. 8 for 3 .. 64 rows
// MODE (DEC_SWIGLU, DEC_BEST; UT feature tiles per unit): one split, the block finishes its own units -- the waves of a unit of two tiles meet through
// LDS -- and no partial sums or finishing launch are needed; else -1: partial sums, and the rows' rstd on the side.
template <int NP, int MODE, int UT>
__global__ __launch_bounds__(512) void decode_splitk_kernel(const h16_t *__restrict__ Wp, const h16_t *__restrict__ Xa,
                                                           int n_tiles, int k_tiles, int T,
                                                           float *__restrict__ part, float *__restrict__ rstd_out, DecodeEpi e) {
    constexpr int NB = NP == 1 ? 1 : NP / 2, CH = sk_chunk(NP), RW = NP;       // RW rows per wave for rstd
    constexpr bool OWN = MODE >= 0;
    __shared__ float s_rstd[OWN ? 64 : 1];
    const float *ssq_in = e.ssq_in;
    const int ssq_units = e.ssq_units, norm_dim = e.norm_dim;
    const float eps = e.eps;
    constexpr int XT = CH * NP / 8;                    // operand tiles of a chunk each wave copies
    extern __shared__ h16x8 sk_lds[];                  // [2][CH][NP][64]
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, j = lane & 15, g = lane >> 4;
    const int tile = blockIdx.x * 8 + wave;
    const bool tile_ok = tile < n_tiles;
    // the chunks of the contraction are dealt out evenly over the splits (blockIdx.y)
    const int chunks = (k_tiles + CH - 1) / CH;
    const int kt0 = (int)((long)blockIdx.y * chunks / gridDim.y) * CH;
    const int kt1 = min(k_tiles, (int)((long)(blockIdx.y + 1) * chunks / gridDim.y) * CH);
    const int n_chunks = (kt1 - kt0 + CH - 1) / CH;
    const int N = n_tiles * 16;

    // a chunk's operand tiles are contiguous; this wave copies tiles wave, wave + 8, ... (past the end: the last one, unused)
    auto load_x = [&](int c, h16x8(&x)[XT]) {
#pragma unroll
        for (int i = 0; i < XT; ++i)
            x[i] = reinterpret_cast<const h16x8 *>(Xa)[(size_t)min((kt0 + c * CH) * NP + wave + 8 * i, k_tiles * NP - 1) * 64 + lane];
    };
    auto store_x = [&](int c, const h16x8(&x)[XT]) {
        h16x8 *buf = sk_lds + ((c & 1) * CH * NP + wave) * 64 + lane;
#pragma unroll
        for (int i = 0; i < XT; ++i) buf[i * 8 * 64] = x[i];
    };
    // this wave's weight tile for the k-tiles of chunk c
    const h16x8 *wsrc = reinterpret_cast<const h16x8 *>(Wp) + (size_t)min(tile, n_tiles - 1) * 64 + lane;
    const size_t kstride = (size_t)n_tiles * 64;
    const h16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
    auto load_w = [&](int c, h16x8(&w)[CH]) {
        const int kc = kt0 + c * CH;
#pragma unroll
        for (int i = 0; i < CH; ++i)
            w[i] = (c < n_chunks && kc + i < kt1) ? __builtin_nontemporal_load(wsrc + (size_t)(kc + i) * kstride) : zero;
    };

    // On the side: the rows' rstd for the finishing kernel, each row by one wave of one block of the launch (the
    // sums of squares are requested now and added up after the main loop, when they have long arrived).
    const int n_blocks = gridDim.x * gridDim.y, bid = blockIdx.y * gridDim.x + blockIdx.x;
    const int rstd_row = bid + wave * n_blocks;
    const bool rstd_mine = !OWN && rstd_out != nullptr && rstd_row < T;
    float sv[RSTD_REGS], so[OWN ? RW : 1][RSTD_REGS];
    if constexpr (OWN) {          // every row's, by every block: requested ahead of the weights (rows past the last re-read it)
        if (ssq_in != nullptr) {
#pragma unroll
            for (int r = 0; r < RW; ++r) rstd_request(e, min(wave + 8 * r, T - 1), lane, so[r]);
        }
    }
    if (rstd_mine && ssq_in != nullptr) {
#pragma unroll
        for (int q = 0; q < RSTD_REGS; ++q) sv[q] = ssq_in[(size_t)rstd_row * ssq_units + min(lane + 64 * q, ssq_units - 1)];
    }

    // the hi and the lo products are summed apart and added at the end: half as many roundings per sum
    floatx4 acc[NB], acl[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = acl[b] = floatx4{0.f, 0.f, 0.f, 0.f};
    h16x8 xr[XT], wc[CH], wn[CH];
    load_x(0, xr);
    load_w(0, wc);
    if constexpr (OWN) {
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const int t = wave + 8 * r;
            if (t >= T) continue;
            if (ssq_in != nullptr) rstd_finish(e, t, lane, so[r], s_rstd);
            else if (lane == 0) s_rstd[t] = 1.0f;
        }
    }
    store_x(0, xr);
    load_x(1, xr);
    for (int c = 0; c < n_chunks; ++c) {
        // chunk c is complete in LDS for every wave, and nobody reads the other buffer (chunk c - 1) any more;
        // a bare s_barrier: __syncthreads() would also drain the weight loads in flight
        __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));
        asm volatile("s_barrier" ::: "memory");
        store_x(c + 1, xr);
        load_x(c + 2, xr);
        load_w(c + 1, wn);
        const h16x8 *buf = sk_lds + (c & 1) * CH * NP * 64 + lane;
        const int nk = min(CH, kt1 - (kt0 + c * CH));
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            if (i < nk) {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    if (NP > 1) acl[b] = hx_mfma16(wc[i], buf[(i * NP + 2 * b + 1) * 64], acl[b]);
                    acc[b] = hx_mfma16(wc[i], buf[(i * NP + 2 * b) * 64], acc[b]);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < CH; ++i) wc[i] = wn[i];
    }
    if (rstd_mine) {
        float r = 1.0f;
        if (ssq_in != nullptr) {
            float ss = 0.f;
#pragma unroll
            for (int q = 0; q < RSTD_REGS; ++q) ss += lane + 64 * q < ssq_units ? sv[q] : 0.f;
            for (int i = lane + 64 * RSTD_REGS; i < ssq_units; i += 64) ss += ssq_in[(size_t)rstd_row * ssq_units + i];
            ss = wave_sum(ss);
            r = 1.0f / sqrtf(ss / (float)norm_dim + eps);
        }
        if (lane == 0) rstd_out[rstd_row] = r;
    }
    if (!OWN && rstd_out != nullptr)   // a launch of fewer than T / 8 blocks: the rows not dealt out above
        for (int row = rstd_row + 8 * n_blocks; row < T; row += 8 * n_blocks) {
            float r = 1.0f;
            if (ssq_in != nullptr) {
                float ss = 0.f;
                for (int i = lane; i < ssq_units; i += 64) ss += ssq_in[(size_t)row * ssq_units + i];
                ss = wave_sum(ss);
                r = 1.0f / sqrtf(ss / (float)norm_dim + eps);
            }
            if (lane == 0) rstd_out[row] = r;
        }
    if (!OWN && !tile_ok) return;
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] += acl[b];
    if (NP == 1) {          // token columns 8 .. 15 hold the lo parts of tokens 0 .. 7
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[0][r] += __shfl_xor(acc[0][r], 8, 64);
    }
    if constexpr (OWN) {
        const EpiPre pre{};
        if constexpr (UT == 1) {
            if (!tile_ok) return;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const floatx4 v[1] = {acc[b]};
                decode_epilogue<MODE, 1>(v, tile, b, lane, N, T, e, s_rstd, pre);
            }
        } else {             // a unit's even wave finishes its even token tiles, the odd one the others
            floatx4 *ex = reinterpret_cast<floatx4 *>(sk_lds);
            __syncthreads();                 // nobody reads the operand any more
#pragma unroll
            for (int b = 0; b < NB; ++b)
                if ((b ^ wave) & 1) ex[(wave * NB + b) * 64 + lane] = acc[b];
            __syncthreads();
            if (!tile_ok) return;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                if ((b ^ wave) & 1) continue;
                const floatx4 other = ex[((wave ^ 1) * NB + b) * 64 + lane];
                const floatx4 v[2] = {wave & 1 ? other : acc[b], wave & 1 ? acc[b] : other};
                decode_epilogue<MODE, 2>(v, tile >> 1, b, lane, N, T, e, s_rstd, pre);
            }
        }
        return;
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int token = j + 16 * b;
        if (token < T)
            *reinterpret_cast<floatx4 *>(part + ((size_t)blockIdx.y * T + token) * N + tile * 16 + 4 * g) = acc[b];
    }
}

// Sums the split partials in split order and runs the register epilogue; one wave per (unit, 16-token tile).
// rstd[T]: the rows' reciprocal rms, left by the split kernel of the same projection.
template <int MODE, int UT>
__global__ __launch_bounds__(256) void decode_finish_kernel(const float *__restrict__ part, int splits, int N, int T,
                                                           int n_units, DecodeEpi e, const float *__restrict__ rstd) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int nbt = (T + 15) >> 4;
    const int idx = blockIdx.x * 4 + wave;
    if (idx >= n_units * nbt) return;
    const int unit = idx / nbt, b = idx - unit * nbt;
    const int token = (lane & 15) + 16 * b, g = lane >> 4;
    EpiPre pre;
    epi_request_first<MODE>(pre, unit, b, lane, N, T, e);
    epi_request_second<MODE>(pre, unit, lane, e);
    floatx4 v[UT];
#pragma unroll
    for (int u = 0; u < UT; ++u) {
        v[u] = floatx4{0.f, 0.f, 0.f, 0.f};
        if (token < T)
#pragma unroll 4
            for (int ks = 0; ks < splits; ++ks)
                v[u] += *reinterpret_cast<const floatx4 *>(part + ((size_t)ks * T + token) * N + (unit * UT + u) * 16 + 4 * g);
    }
    decode_epilogue<MODE, UT>(v, unit, b, lane, N, T, e, rstd, pre);
}

namespace {

template <int NP, int UT, int UNR, int MODE, bool XLDS, int XR>
void launch_one(const h16_t *Wp, const h16_t *Xa, int N, int k_tiles, int T, const DecodeEpi &e, hipStream_t s) {
    constexpr int WAVES = 8;
    auto kern = decode_proj_kernel<NP, UT, WAVES, UNR, MODE, XLDS, XR>;
    size_t dyn = 0;
    if (XLDS) {
        dyn = (size_t)T * k_tiles * 8 * sizeof(h16x8);
        static bool raised = false;       // static + dynamic LDS may exceed the default 64 KB per block
        if (!raised) {
            (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                      kXldsMaxBytes);
            raised = true;
        }
    }
    hipLaunchKernelGGL(kern, dim3(N / 16 / UT), dim3(WAVES * 64), dyn, s, Wp, Xa, N, k_tiles, T, e);
}

template <int UT, int MODE>
void launch_mode(const h16_t *Wp, const h16_t *Xa, int N, int k_tiles, int T, const DecodeEpi &e, hipStream_t s) {
    // a contraction of at most 32 k-tiles gives a wave 4 of them: a ring of 4 requests nothing it does not use.  The LM head beyond 16
    // rows takes it at any length: 106 registers for 186, so that a CU holds two blocks (32 rows of 512 / 1024 x 16000 31.3 / 34.2 ->
    // 19.7 / 22.0 us, of 1536 / 2048 x 8000 22.6 / 23.8 -> 18.6 / 20.1, of 4096 x 4000 20.9 -> 20.8).
    constexpr int RING = 8 / UT, SHORT = UT == 1 && (MODE == DEC_RESID || MODE == DEC_BEST) ? 4 : RING;
#define HX_ONE(NP)                                                                                              \
    do {                                                                                                        \
        constexpr int LONG = MODE == DEC_BEST && (NP) == 4 ? SHORT : RING;                                      \
        if (k_tiles <= 32) launch_one<NP, UT, SHORT, MODE, false, 1>(Wp, Xa, N, k_tiles, T, e, s);              \
        else launch_one<NP, UT, LONG, MODE, false, 1>(Wp, Xa, N, k_tiles, T, e, s);                             \
    } while (0)
    constexpr int NPM = UT == 4 ? 2 : 4;          // (blocks of four feature tiles take 16 rows at most: unit_pairs)
    if (T > 16) HX_ONE(NPM);
    else if (T > 8) HX_ONE(2);
    else if (T > 2) HX_ONE(1);
    // One or two rows.  With W_O, W2 and W1/W3 each wave fetches its operand pieces through its request ring instead of the
    // block staging the operand in LDS behind a barrier (measured: W_O 17.9 -> 16.6 us and W2 44.0 -> 43.4 at one row, W1/W3
    // 81.0 -> 77.9 at two rows and unchanged at one).  The QKV projection keeps the staged operand -- XR 16-byte pieces per
    // thread (512 threads), 4 up to 32 KB, 8 up to 64 KB: through the ring it loses 3.5 us.
    else if constexpr (MODE == DEC_RESID || MODE == DEC_SWIGLU) HX_ONE(0);
    else {
        const size_t xbytes = (size_t)T * k_tiles * 8 * sizeof(h16x8);
        if (xbytes > (size_t)kXldsMaxBytes) HX_ONE(0);
        else if (xbytes <= (size_t)kXldsMaxBytes / 2) launch_one<0, UT, 8 / UT, MODE, true, 4>(Wp, Xa, N, k_tiles, T, e, s);
        else launch_one<0, UT, 8 / UT, MODE, true, 8>(Wp, Xa, N, k_tiles, T, e, s);
    }
#undef HX_ONE
}
}  // namespace

namespace {
template <int NP, int MODE, int UT>
void launch_splitk_main(dim3 grid, const h16_t *Wp, const h16_t *Xa, int n_tiles, int k_tiles, int T, float *part, const DecodeEpi &e,
                        float *rstd, hipStream_t s) {
    const size_t lds = (size_t)2 * sk_chunk(NP) * NP * 64 * sizeof(h16x8);
    if constexpr (MODE == DEC_BEST || (MODE == DEC_SWIGLU && NP <= 4)) {           // (more than 32 rows: the head)
        if (grid.y == 1) {
            auto kern = decode_splitk_kernel<NP, MODE, UT>;
            static bool raised = false;       // static + dynamic LDS exceed the default 64 KB per block at four and eight operand tiles
            if (!raised) {
                (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
                raised = true;
            }
            hipLaunchKernelGGL(kern, grid, dim3(512), lds, s, Wp, Xa, n_tiles, k_tiles, T, nullptr, nullptr, e);
            return;
        }
    }
    hipLaunchKernelGGL((decode_splitk_kernel<NP, -1, 1>), grid, dim3(512), lds, s, Wp, Xa, n_tiles, k_tiles, T, part, rstd, e);
}

// Number of splits of the split form.  Two blocks fit a CU (registers, 64 KB of LDS), 512 on the chip.  The number (at most 8, or 16 for a matrix of
// fewer than 64 feature groups: the finishing kernel walks them one after the other; partials within the scratch)
// minimises rounds of blocks x chunks per block, in units of one chunk per block (512 blocks x 64 KB: about 5.6 us), plus the
// partial sums' way through memory and back (about 5 TB/s: a wide matrix with a short contraction is not split into
// eight to save half a round); on a tie the fewer splits win.
int splitk_splits(int N, int k_tiles, int T, size_t scratch_floats) {
    const int groups = (N / 16 + 7) / 8, np = dec_act_tiles(T), chunks = (k_tiles + sk_chunk(np) - 1) / sk_chunk(np);
    const int cap = groups * 8 < 512 ? 16 : 8;      // a narrow matrix (TP8 QKV: 10 groups) fills more of the chip with 16
    int splits = 1;
    long best = -1;
    for (int c = 1; c <= std::min(cap, chunks); ++c) {
        if (c > 1 && (size_t)c * T * N > scratch_floats - DEC_SCRATCH_RSTD) break;
        const long traffic = c > 1 ? (long)((double)c * T * N * 8.0 / 5e6 / 5.6 * 16.0) : 0;
        const long cost = (long)((groups * c + 511) / 512) * ((chunks + c - 1) / c) * 16 + c + traffic;
        if (best < 0 || cost < best) { best = cost; splits = c; }
    }
    return splits;
}

template <int MODE, int UT>
void launch_splitk(const h16_t *Wp, const h16_t *Xa, int N, int k_tiles, int T, const DecodeEpi &e, float *scratch,
                   size_t scratch_floats, int splits, hipStream_t s, hipEvent_t mid, QkvTail *tail = nullptr) {
    const int n_tiles = N / 16, groups = (n_tiles + 7) / 8, np = dec_act_tiles(T);
    float *rstd = scratch + scratch_floats - DEC_SCRATCH_RSTD;      // the tail of the scratch carries the rows' rstd
    const dim3 grid(groups, splits);
    switch (np) {
        case 1: launch_splitk_main<1, MODE, UT>(grid, Wp, Xa, n_tiles, k_tiles, T, scratch, e, rstd, s); break;
        case 2: launch_splitk_main<2, MODE, UT>(grid, Wp, Xa, n_tiles, k_tiles, T, scratch, e, rstd, s); break;
        case 4: launch_splitk_main<4, MODE, UT>(grid, Wp, Xa, n_tiles, k_tiles, T, scratch, e, rstd, s); break;
        case 6: launch_splitk_main<6, MODE, UT>(grid, Wp, Xa, n_tiles, k_tiles, T, scratch, e, rstd, s); break;
        default: launch_splitk_main<8, MODE, UT>(grid, Wp, Xa, n_tiles, k_tiles, T, scratch, e, rstd, s); break;
    }
    if (mid) (void)hipEventRecord(mid, s);
    // One split: the kernel has finished its units (W1/W3 of the full-width 70B layer, 448 groups, at 4 / 16 / 32 rows: whole calls of four steps 1218 /
    // 1255 / 1547 -> 1208 / 1244 / 1513 us; the 4096 x 50304 head at 24 rows 93.0 -> 88.2).  A second split saves less than its launch costs only
    // where one leaves CUs empty: forced to one, the 250 groups of the 8192 x 32000 head at 48 rows take 124.6 us instead of 111.
    if ((MODE == DEC_BEST || (MODE == DEC_SWIGLU && np <= 4)) && splits == 1) return;
    if constexpr (MODE == DEC_QKV) {          // the decode attention finishes the projection
        *tail = QkvTail{scratch, splits, T, N, rstd, e.cos_tab, e.sin_tab};
    } else {
        const int n_units = n_tiles / UT, nbt = (T + 15) / 16;
        hipLaunchKernelGGL((decode_finish_kernel<MODE, UT>), dim3((n_units * nbt + 3) / 4), dim3(256), 0, s, scratch, splits, N, T,
                           n_units, e, rstd);
    }
}
}  // namespace

namespace {
// two feature tiles per unit of the LM head from 1024 tiles on: 2 KB of weights per wave and k-tile stream a few percent faster
bool best_pairs(int N) { return (N / 16) % 2 == 0 && N / 32 >= 512; }

// Single kernel: one unit (16 result features) per block, or two?  Two halve what the blocks read of the operand and the number
// of blocks; what decides is how evenly the blocks go over the 256 CUs -- with n units the fullest CU has ceil(n / 256) units, or
// 2 ceil(n / 512) in pairs -- how long a contraction a block walks (see decode_single_kernel: one CU's load path, not HBM, sets the
// pace of a block) and, on a long stream of weights, the requests in flight.  The lines stand where measurements on both sides put them.
//   RESID, one or two rows: pairs for n = 256 .. 511 (5120 wide, two ranks, at one row 74.4 -> 66.1 us per layer, 6144 wide 82.7 ->
//          76.9, 6144 x 16384 150.2 -> 142.1); n = 512: +0 .. +0.3, +4 for the 224 MiB of TP2's W2; beyond: -0.7 .. +1.1.
//   RESID, 3 rows on, weights up to 120 MiB (128 MiB: +0 .. +2), k = k-tiles, at 3 .. 8 / 9 .. 16 / 17 .. 32 rows (one, two or four
//          operand tiles), the best other form -> two, us per projection:
//          n = 256  one unit is as good from 9 rows on; up to 8 rows k = 192 16.6 -> 15.8, 320 23.5 -> 23.0, 448 29.1 -> 30.3
//          n = 288  k = 144 17.0 -> 13.9 / 18.6 -> 16.4 / 20.7 -> 20.2;  272 21.1 -> 21.4 / 23.4 -> 26.4 / 26.2 -> 33.4
//          n = 320  k = 160 17.7 -> 14.8 / 19.6 -> 17.8 / 21.8 -> 21.6;  256 22.4 -> 20.9 / 24.4 -> 25.0 / 27.0 -> 31.6
//          n = 384  k = 192 20.2 -> 17.5 / 23.1 -> 20.5 / 25.3 -> 26.0;  312 28.4 -> 25.1 / 29.8 -> 30.2 / 32.4 -> 39.2
//          n = 448  k = 176 20.1 -> 19.0 / 23.3 -> 20.9 / 25.5 -> 25.5;  272 27.8 -> 26.7 / 28.9 -> 29.0 / 31.8 -> 35.9
//          n = 512  k = 224 26.9 -> 25.7 / 28.8 -> 27.9 / 31.7 -> 31.4
//          n = 416  k = 208 at 17 / 30 rows 25.6 -> 28.5 / 28.3 -> 29.2
//          hence k up to n, 3 n / 4, 3 n / 8 (n / 2 at 512: every CU has one block).  Two blocks of pairs on the fullest CU, n = 513 .. 1024:
//          n = 576  k = 36 11.0 -> 10.7 / 12.8 -> 11.7 / 18.9 -> 15.0;  144 at 3 rows 21.4 -> 25.0;  200 31.4 -> 32.7 / 28.9 -> 37.4 / 34.3 -> 48.1
//          n = 704  k = 44 13.5 -> 12.0 / 14.3 -> 13.7 / 20.4 -> 17.0;  160 26.9 -> 26.0 / 27.9 -> 30.1 / 33.2 -> 39.7
//          n = 768  k = 48 14.5 -> 12.5 / 15.2 -> 14.4 / 22.4 -> 17.9;  160 29.6 -> 26.7 / 29.1 -> 30.7 / 34.1 -> 39.9
//          n = 896  k = 56 15.4 -> 13.7 / 19.0 -> 15.5 / 23.0 -> 19.8;  128 26.0 -> 23.1 / 27.6 -> 26.5 / 33.2 -> 34.7
//          n = 1024 k = 64 17.1 -> 14.8 / 21.3 -> 16.7 / 25.1 -> 21.7;  120 27.8 -> 23.3 / 28.8 -> 26.6 / 33.9 -> 34.9
//          hence k up to n / 8, n / 8, n / 16 where pairs are the more uneven (n up to 768), beyond that any, any, n / 8.
//   QKV    up to 8 rows, n = 288 / 320 / 384: 7168 wide 109.1 -> 106.1 us per layer, TP2 155.1 -> 152.9, 3072 wide at 1 / 8 rows 51.3 /
//          55.9 -> 50.1 / 53.4, 4096 wide at 8 rows 83.8 -> 82.1; n = 160, 192, 480, 640: +0.6 .. +4.4.
//   W1/W3  (a unit is a gate and an up tile) up to 16 rows, n = 288 / 352 / 432 / 448 / 512: 2048 wide at 1 / 8 / 16 rows 35.4 / 36.9 /
//          42.8 -> 34.4 / 35.6 / 40.6 us per layer, TP4 at 8 / 16 rows 91.6 / 99.8 -> 89.5 / 95.1 (16: the split contraction before), 5120
//          wide at 16 rows 95.0 -> 89.9; one and two rows gain below 384 and lose 0.4 .. 0.8 at 432, 448; up to 8 rows at n = 800 (4096
//          wide at 1 / 3 / 8 rows 85.8 / 91.8 / 93.4 -> 83.7 / 88.9 / 91.0) and 864 / 896 (TP2 152.9 / 155.5 / 157.7 -> 150.9 / 154.4 /
//          155.6; 3 and 8: split before).  n = 928, 960, 1024: +0.2 .. +1.3 at one row, -2.6 .. +0.8 at 3 and 8: not taken.
//          n = 224, 640, 704, 1280 (more units on the fullest CU): +1.5 .. +7.  A long contraction is split instead (n = 280, k = 320 at
//          8 / 16 rows 37.5 -> 38.6 / 39.0 -> 45.3, n = 288, k = 288 at 15 rows 36.5 -> 41.1): k up to n, 3 n / 4.
bool unit_pairs(int mode, int N, int k_tiles, int T) {
    const int n = N / 16 / (mode == DEC_SWIGLU ? 2 : 1), np = dec_act_tiles(T);
    if (n % 2 != 0) return false;
    switch (mode) {
        case DEC_BEST: return best_pairs(N);
        case DEC_RESID:
            if (T <= 2) return n >= 256 && n < 512;
            if (n < 256 || n > 1024 || (size_t)N * k_tiles * 64 > (size_t)120 << 20) return false;
            if (n == 256 && T > 8) return false;
            if (n <= 512) return 8 * k_tiles <= n * (np == 1 ? 8 : np == 2 ? 6 : n == 512 ? 4 : 3);
            if (n <= 768) return (np <= 2 ? 8 : 16) * k_tiles <= n;
            return np <= 2 || 8 * k_tiles <= n;
        case DEC_QKV: return n > 256 && n <= 384 && T <= 8;
        case DEC_SWIGLU:
            if (n > 768 && n <= 896) return T <= 8;
            if (n <= 256 || n > 512) return false;
            return T <= 2 ? n <= 384 : T <= 8 ? k_tiles <= n : T <= 16 && 4 * k_tiles <= 3 * n;
    }
    return false;
}

// One kernel with complete dot products per block, or a contraction split over blocks and a finishing pass?  One or two
// rows: always one kernel.  More: the single kernel saves the partial sums and the second launch (4 .. 5 us), and pays with
// the operand, which every block reads for itself from L2 where the split kernel's eight feature tiles share it through LDS, and
// with blocks that walk the whole contraction: a block takes about 5 us plus 0.024 + 0.012 x operand tiles per k-tile (twice
// that where the fullest CU has two), however few blocks there are.
//   * Operand reads, blocks x k-tiles x operand tiles x 1 KB (single minus split, us per projection, one unit per block):
//     W1/W3  8 rows:  58 MB -2.9 (TP8 of the 70B shape), 92 -6.4 (4096-wide layer), 117 -2.2 (TP4), 235 +2.4 (TP2), 470 +9.5
//           16 rows:  46 -2.9 (2048-wide), 117 -1.3 (TP8), 235 +3.0 (TP4)
//     W2     8 rows:  23 -4.1 (2048-wide), 59 -2.0 (TP8), 117 0.0 (TP4), 235 +1.7    16 rows: 46 -3.3, 117 -0.9, 185 +1.4, 235 +3.7
//     W_O    8 rows:  17 -3.5, 33 -2.3, 134 -0.8    16 rows: 34 -2.8, 134 -0.2, 268 +3.8    32 rows: 67 -3.2, 134 -2.7, 268 +2.0
//     The line is 128 MiB; blocks of two units halve the reads (TP4's W1/W3 at 16 rows 99.8 -> 95.1 us per layer).
//   * W_O and W2 with 257 .. 1024 units, but for 512, are one kernel exactly where pairs are: lone units fill the CUs unevenly
//     and lose to the split contraction wherever pairs do (n = 288, k = 400 at 3 rows: one unit 36.6, two 29.1, split 27.0).
//   * Few blocks (fewer than 192): the contraction a block may walk grows with their number.  Split -> single at 3 .. 8 / 16 / 32 rows:
//     W2     n =  64, k = 88 11.1 -> 8.5 / 11.7 -> 9.5 / 12.7 -> 12.2;  176 13.0 -> 10.9 / 13.7 -> 13.3 / 14.9 -> 17.5;  352 15.6 -> 16.8 / 16.4
//            -> 21.7 / 18.1 -> 29.9
//            n = 128, k = 128 12.3 -> 9.5 / 13.1 -> 11.2 / 15.3 -> 14.4;  256 16.5 -> 14.1 / 17.6 -> 17.5 / 20.0 -> 23.4;  352 17.6 -> 18.1 /
//            18.6 -> 22.7 / 21.1 -> 31.2
//     W1/W3  n =  44, k = 128 12.7 -> 11.9 / 14.1 -> 13.7 / 15.3 -> 20.0;  256 14.9 -> 18.5 / 16.3 -> 22.2 / 17.8 -> 34.1
//            n =  88, k = 128 14.7 -> 12.3 / 16.7 -> 14.0 / 19.4 -> 20.0;  256 18.4 -> 19.8 / 21.0 -> 22.9 / 24.7 -> 34.6
//            n = 176, k = 128 17.0 -> 13.5 / 18.8 -> 15.7 / 21.9 -> 20.9
//     (W2 at 19 rows, n = 160, k = 132: 14.9 -> 16.0.)  k x (weight + operand tiles) up to 384 + 3 n, beyond 16 rows 320 + 2 n (W1/W3 300 + 3 n).
//     From 192 units on the operand line is the tighter one, except for one operand tile of a long stream (n = 256: 80 MB 23.2 ->
//     23.5, 112 MB 29.1 -> 30.3).
//   * W1/W3 in lone units: the last round of 256 has to be filled.  Split -> single at 3 .. 8 rows n = 540 48.6 -> 50.3, 560 43.2 -> 44.1, 600
//     40.9 -> 43.2, 640 44.5 -> 46.3 (k = 192) and 27.1 -> 25.5 (96), but 512 28.0 -> 23.9, 704 24.3 -> 19.6; at 19 .. 32 rows n = 264 20.4 -> 23.3, 300 16.6 -> 17.6, 352 21.7 ->
//     22.2, but 512 24.2 -> 23.5.
//   * LM head beyond 16 rows in pairs: one block on a CU (148 registers), four rounds of them with little to do each where the contraction is
//     short.  Whole call at 32 rows, split -> single: 512 x 32000 22.7 -> 28.1 us, 1024 x 32000 27.7 -> 31.8, 1024 x 50304 34.4 -> 34.7.
//   * The QKV projection has no finishing launch to save (the attention sums its partials):
//           8 rows:  42 -0.9 (TP4), 50 -0.6, 84 +3.5 (TP2)    16 rows: 25 -1.0, 84 +1.5
//     56 MiB, and at least 128 blocks (TP8 of the 70B shape has 80: +0.9 .. +4.7) or a contraction so short that one block walks it in the
//     time the partial sums take: without them the attention's blocks begin with the context at once.  Whole layers of shards,
//     split -> single, n units, k k-tiles, at 3 / 7 / 12 / 20 / 32 rows:
//           n = 12, k =  16 24.8 -> 23.1 / 25.4 -> 23.4 / 25.5 -> 23.6 / 29.6 -> 28.7 / 30.3 -> 29.7 us
//           n = 24, k =  64 28.7 -> 26.8 / 28.8 -> 27.0 / 30.2 -> 28.7 / 33.7 -> 34.1 / 35.2 -> 36.7
//           n = 40, k = 128 35.1 -> 34.6 / 35.7 -> 34.9 / 37.3 -> 38.1 / 44.5 -> 47.7 / 46.4 -> 51.9
//           n = 48, k =  16 27.5 -> 25.4 / 27.8 -> 25.6 / 29.2 -> 27.4 / 32.7 -> 31.9 / 33.9 -> 33.8
//           n = 96, k =  32 30.4 -> 27.6 / 30.6 -> 28.3 / 32.2 -> 30.7 / 38.1 -> 37.2 / 39.3 -> 39.6
//           n = 96, k =  64 32.8 -> 31.0 / 33.4 -> 31.2 / 35.3 -> 34.0 / 41.3 -> 41.6 / 43.2 -> 44.2
//           n = 96, k = 128 41.1 -> 40.0 / 41.5 -> 40.1 / 44.9 -> 44.6 / 52.5 -> 55.1 / 56.0 -> 60.0  (n = 48 at 12 rows 38.8 -> 39.2)
//           n = 80, k = 256 55.3 -> 56.5 / 56.2 -> 57.3 / 61.5 -> 65.6
//     So up to 128, 64 and 16 k-tiles at one, two and four operand tiles, whatever the number of units (12 to 96 measured).  The sums are
//     as good either way: chains of k / 8 tiles and eight waves' sums in the one, of a chunk's eight tiles and k / 8 splits in the
//     other, the lo products with sums of their own in both.
bool decode_single_kernel(int mode, int N, int k_tiles, int T) {
    if (T <= 2) return true;
    if (T > 32) return false;
    if (k_tiles < 8) return true;              // not one chunk of the split kernel
    const int tiles = mode == DEC_SWIGLU ? 2 : 1, units = N / 16 / tiles, pair = unit_pairs(mode, N, k_tiles, T) ? 2 : 1, np = dec_act_tiles(T);
    const size_t operand = (size_t)(units / pair) * k_tiles * np << 10;
    if (mode == DEC_QKV)
        return units < 128 ? k_tiles <= (np == 1 ? 128 : np == 2 ? 64 : 16) : operand * pair <= (size_t)56 << 20;
    if (mode == DEC_RESID && units > 256 && units <= 1024 && units != 512) return pair == 2;
    if (mode == DEC_RESID && pair == 2) return true;
    if (units < 192) return k_tiles * (tiles + np) <= (np < 4 ? 384 + 3 * units : mode == DEC_SWIGLU ? 300 + 3 * units : 320 + 2 * units);
    if (mode == DEC_SWIGLU && pair == 1 && units > 256 && 20 * units < 17 * 256 * ((units + 255) / 256)) return false;
    if (mode == DEC_BEST && pair == 2 && np == 4 && k_tiles <= 32) return false;
    if (mode == DEC_RESID && units <= 256 && (size_t)N * k_tiles * 64 > (size_t)80 << 20) return false;
    return operand <= (size_t)128 << 20;
}
}  // namespace

int decode_best_units(int N) { return best_pairs(N) ? N / 32 : N / 16; }

int decode_splits(int mode, int N, int K, int T, size_t scratch_floats) {
    if (decode_single_kernel(mode, N, K / 32, T) || scratch_floats < (size_t)T * N + DEC_SCRATCH_RSTD) return 0;
    return splitk_splits(N, K / 32, T, scratch_floats);
}

void launch_decode_proj(const h16_t *Wp, const h16_t *Xa, int N, int K, int T, const DecodeEpi &e, float *scratch,
                        size_t scratch_floats, hipStream_t s, hipEvent_t mid) {
    const int k_tiles = K / 32, splits = scratch != nullptr && e.mode != DEC_QKV ? decode_splits(e.mode, N, K, T, scratch_floats) : 0;
    if (splits > 0) {
#define HX_SPLITK(MODE, UT) launch_splitk<MODE, UT>(Wp, Xa, N, k_tiles, T, e, scratch, scratch_floats, splits, s, mid)
        switch (e.mode) {
            case DEC_RAW: HX_SPLITK(DEC_RAW, 1); break;
            case DEC_RESID: HX_SPLITK(DEC_RESID, 1); break;
            case DEC_SWIGLU: HX_SPLITK(DEC_SWIGLU, 2); break;
            case DEC_BEST:
                if (best_pairs(N)) HX_SPLITK(DEC_BEST, 2);
                else HX_SPLITK(DEC_BEST, 1);
                break;
        }
#undef HX_SPLITK
        return;
    }
    const bool pair = unit_pairs(e.mode, N, k_tiles, T);
    switch (e.mode) {
#define HX_UNITS(MODE, U)                                                          \
    case MODE:                                                                     \
        if (pair) launch_mode<2 * U, MODE>(Wp, Xa, N, k_tiles, T, e, s);           \
        else launch_mode<U, MODE>(Wp, Xa, N, k_tiles, T, e, s);                    \
        break;
        case DEC_RAW: launch_mode<1, DEC_RAW>(Wp, Xa, N, k_tiles, T, e, s); break;
        HX_UNITS(DEC_QKV, 1)
        HX_UNITS(DEC_RESID, 1)
        HX_UNITS(DEC_SWIGLU, 2)
        HX_UNITS(DEC_BEST, 1)
#undef HX_UNITS
    }
    if (mid) (void)hipEventRecord(mid, s);
}

void launch_decode_qkv(const h16_t *Wp, const h16_t *Xa, int N, int K, int T, const DecodeEpi &e, float *scratch,
                       size_t scratch_floats, QkvTail *tail, hipStream_t s) {
    *tail = QkvTail{nullptr, 0, T, N, nullptr, e.cos_tab, e.sin_tab};
    const int k_tiles = K / 32;
    const int splits = e.mode == DEC_QKV && scratch != nullptr ? decode_splits(e.mode, N, K, T, scratch_floats) : 0;
    if (splits > 0)
        launch_splitk<DEC_QKV, 1>(Wp, Xa, N, k_tiles, T, e, scratch, scratch_floats, splits, s, nullptr, tail);
    else
        launch_decode_proj(Wp, Xa, N, K, T, e, scratch, scratch_floats, s, nullptr);
}

// -------------------------------------------------------------------------------------------------
// Per-step prologue: stage input rows (bf16, or fp32 for the validation surface) -> fp32 residual
// stream, (x * gain) hi/lo operand of the first projection, per-unit sums of squares (one unit = 16
// columns, as written by the RESID epilogue).  Block 0 also publishes each row's position (the
// sequence's committed length) and, when asked, advances the lengths.
// grid = H / 128 blocks of 512 threads; thread = (token, 4-column group).
// -------------------------------------------------------------------------------------------------
template <bool IN_H16>
__global__ __launch_bounds__(512) void decode_prologue_kernel(const void *__restrict__ in, const void *__restrict__ in2,
                                                             float *__restrict__ h_out,
                                                             const float *__restrict__ g, h16_t *__restrict__ hg,
                                                             float *__restrict__ ssq_out,
                                                             int T, int H, int32_t *lens, int32_t *row_pos,
                                                             int advance) {
    if (blockIdx.x == 0 && lens != nullptr && threadIdx.x < T) {
        const int l = lens[threadIdx.x];
        row_pos[threadIdx.x] = l;
        if (advance) lens[threadIdx.x] = l + 1;
    }
    // 32 column quads per block (128 columns), 16 tokens per pass
    const int quad = threadIdx.x & 31, tsub = threadIdx.x >> 5;
    const int col = blockIdx.x * 128 + quad * 4;
    for (int t = tsub; t < T; t += 16) {
        float ss = 0.f;
        if (col < H) {
            float x[4];
            if (IN_H16) {
                uint2 raw = *reinterpret_cast<const uint2 *>(reinterpret_cast<const h16_t *>(in) + (size_t)t * H + col);
                h16x2_to_f32(raw.x, x[0], x[1]);
                h16x2_to_f32(raw.y, x[2], x[3]);
                if (in2) {      // second addend (e.g. a stage's partial on top of its residual stream)
                    raw = *reinterpret_cast<const uint2 *>(reinterpret_cast<const h16_t *>(in2) + (size_t)t * H + col);
                    float y0, y1, y2, y3;
                    h16x2_to_f32(raw.x, y0, y1);
                    h16x2_to_f32(raw.y, y2, y3);
                    x[0] += y0; x[1] += y1; x[2] += y2; x[3] += y3;
                }
            } else {
                const floatx4 a = *reinterpret_cast<const floatx4 *>(reinterpret_cast<const float *>(in) + (size_t)t * H + col);
                x[0] = a[0]; x[1] = a[1]; x[2] = a[2]; x[3] = a[3];
                if (in2) {
                    const floatx4 c = *reinterpret_cast<const floatx4 *>(reinterpret_cast<const float *>(in2) + (size_t)t * H + col);
                    x[0] += c[0]; x[1] += c[1]; x[2] += c[2]; x[3] += c[3];
                }
            }
            if (h_out) *reinterpret_cast<floatx4 *>(h_out + (size_t)t * H + col) = floatx4{x[0], x[1], x[2], x[3]};
            const floatx4 g4 = *reinterpret_cast<const floatx4 *>(g + col);
            const float y[4] = {x[0] * g4[0], x[1] * g4[1], x[2] * g4[2], x[3] * g4[3]};
            store_act4(y, hg, t, col, H >> 5, T);
            ss = x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + x[3] * x[3];
        }
        // the 4 quads of one 16-column unit are 4 consecutive lanes
        ss += __shfl_xor(ss, 1, 64);
        ss += __shfl_xor(ss, 2, 64);
        if ((quad & 3) == 0 && col < H) ssq_out[(size_t)t * (H >> 4) + (col >> 4)] = ss;
    }
}

void launch_decode_prologue(const void *in, const void *in2, int in_is_h16, float *h_out, const float *g, h16_t *hg,
                            float *ssq_out, int T, int H, int32_t *lens, int32_t *row_pos, int advance, hipStream_t s) {
    const int blocks = (H + 127) / 128;
    if (in_is_h16)
        hipLaunchKernelGGL(decode_prologue_kernel<true>, dim3(blocks), dim3(512), 0, s, in, in2, h_out, g, hg, ssq_out, T, H,
                           lens, row_pos, advance);
    else
        hipLaunchKernelGGL(decode_prologue_kernel<false>, dim3(blocks), dim3(512), 0, s, in, in2, h_out, g, hg, ssq_out, T, H,
                           lens, row_pos, advance);
}

}  // namespace HX_NS
