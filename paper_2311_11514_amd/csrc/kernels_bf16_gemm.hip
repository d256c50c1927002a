// Prefill projection: LDS-staged MFMA GEMM, D^T[n][t] = sum_k Wp[n][k] * Xp[t][k].
//
// A block is a WM x WT grid of waves; each wave owns FM x FT tiles of 32 features x 32 tokens computed with
// v_mfma_f32_32x32x16_bf16 (measured on this chip: 89 % of the datasheet rate from registers against 64 % for
// the 16x16x32 form, which is issue-limited).  The large configurations cover 256 x 256 per block: 8 waves of
// 128 x 64 (two waves per SIMD, 128 accumulator registers each) or 4 waves of 128 x 128 (256 accumulators).
// Operands stay in the 16 x 32 fragment tiles shared with the decode kernels (see common.h): global -> LDS
// is a straight copy, and a 32x32x16 operand is gathered from two neighbouring 16-row tiles with per-lane
// LDS addresses (every 16 lanes read 256 contiguous bytes: conflict-free).  Both MFMA inputs use the
// same gather, so the k-order inside a tile cancels.
// Weights are k-tile-major, so the weight tiles of a block's k-step are one contiguous run of HBM.
//
// blockIdx.x is remapped so that each XCD (blocks are dealt round-robin to the 8 XCDs) works on a
// contiguous range of tiles, token-block fastest: tiles resident on one XCD share weight panels in
// that XCD's L2.
#include <atomic>
#include <type_traits>

#include "kernels.h"
#include "kvlayout.h"

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;

namespace HX_NS {


// ---- epilogue, in registers.  32 x 32 result: lane l holds token column l % 32 and, per register quad q,
// features 8 q + 4 (l / 32) .. + 3 of the 32-feature block, i.e. of the 16-row tile q / 2 its rows
// (q % 2) * 8 + 4 (l / 32) .. + 3.  Rotary pairs (tile rows r, r + 8) and gate / up pairs (tiles 2m, 2m + 1)
// therefore sit in the same lane, in quads q and q ^ 1 respectively q and q + 2: no cross-lane traffic.
// acc_of(i, j): the wave's result tile (i, j) of its FM x FT tiles of block (bm, bt), wave (wm, wt), each asked for once
// (the two-phase loop converts its 16 x 16 results tile by tile on demand); rstd_of(t): 1 / rms of the block's token column t.
// pre (RESID, FM = FT = 1; else nullptr): residual and next gain per quad, requested by the caller ahead of its sums.
struct ResidPre {
    floatx4 h[4], g[4];
};
// token column `token`, features n0 .. n0 + 31 of a lane's 32 x 32 tile; entries outside the matrix re-read valid ones
__device__ __forceinline__ void resid_request(ResidPre &p, int token, int n0, int hl, int N, int T, const GemmEpi &e) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int n = min(n0 + 8 * q, N - 8) + 4 * hl;
        p.h[q] = *reinterpret_cast<const floatx4 *>(e.h + h_tile_offset(min(token, T - 1), n, N));
        if (!e.last_layer) p.g[q] = *reinterpret_cast<const floatx4 *>(e.g_next + n);
    }
}
template <int FM, int FT, int WM, int NTOK, int MODE, typename AccF, typename RstdF>
__device__ __forceinline__ void gemm_epilogue(AccF acc_of, int bm, int bt, int wm, int tl0, int lane, int N,
                                              int n_tiles, int T, const GemmEpi &e, RstdF rstd_of,
                                              float *ssq_lds = nullptr, const ResidPre *pre = nullptr) {
    constexpr int TA = 2 * FM * WM;
    const int hl = lane >> 5;
    if (MODE == DEC_RESID) {
        // Residual read-modify-write.  Walks the wave tile one 32-feature block (i) at a time and fetches the
        // residual values of block i + 1 before the stores of block i: the stream is loaded and stored through
        // the same pointer, so the compiler would not move a load above a store by itself, and with one or
        // two waves per SIMD nothing else hides the latency.
        float ssq[FT];
        int token[FT];
#pragma unroll
        for (int j = 0; j < FT; ++j) {
            ssq[j] = 0.f;
            token[j] = bt * NTOK + tl0 + 32 * j + (lane & 31);
        }
        // a step of the walk: JC of the wave's FT token blocks (all of them, or one where they are many: registers)
        constexpr int JC = FT > 2 ? 1 : FT, STEPS = FM * FT / JC;
        floatx4 hv[2][JC][4];
        auto load_h = [&](floatx4(&dst)[JC][4], int step) {
            const int i = step / (FT / JC), j0 = step % (FT / JC) * JC;
#pragma unroll
            for (int j = 0; j < JC; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int n = (bm * TA + (wm * FM + i) * 2) * 16 + 8 * q + 4 * hl;
                    dst[j][q] = (token[j0 + j] < T && n < N)
                                    ? *reinterpret_cast<const floatx4 *>(e.h + h_tile_offset(token[j0 + j], n, N))
                                    : floatx4{0.f, 0.f, 0.f, 0.f};
                }
        };
        if (pre == nullptr) {
            load_h(hv[0], 0);
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) hv[0][0][q] = pre->h[q];
        }
        floatx4 gv[4];
#pragma unroll
        for (int step = 0; step < STEPS; ++step) {
            const int i = step / (FT / JC), j0 = step % (FT / JC) * JC;
            if (j0 == 0) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int n = (bm * TA + (wm * FM + i) * 2) * 16 + 8 * q + 4 * hl;
                    if (pre != nullptr) gv[q] = pre->g[q];
                    else gv[q] = (n < N && !e.last_layer) ? *reinterpret_cast<const floatx4 *>(e.g_next + n)
                                                     : floatx4{0.f, 0.f, 0.f, 0.f};
                }
            }
            if (step + 1 < STEPS) load_h(hv[(step + 1) & 1], step + 1);
#pragma unroll
            for (int jj = 0; jj < JC; ++jj) {
                const int j = j0 + jj;
                const floatx16 c = acc_of(i, j);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int n = (bm * TA + (wm * FM + i) * 2) * 16 + 8 * q + 4 * hl;
                    if (token[j] >= T || n >= N) continue;
                    const floatx4 h4 = hv[step & 1][jj][q];
                    const floatx4 v = {c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]};
                    if (e.last_layer) {
                        uint2 po;
                        po.x = pack_h16x2(v[0], v[1]);
                        po.y = pack_h16x2(v[2], v[3]);
                        *reinterpret_cast<uint2 *>(e.out_partial + (size_t)token[j] * N + n) = po;
                        if (e.out_resid) {
                            uint2 ro;
                            ro.x = pack_h16x2(h4[0], h4[1]);
                            ro.y = pack_h16x2(h4[2], h4[3]);
                            *reinterpret_cast<uint2 *>(e.out_resid + (size_t)token[j] * N + n) = ro;
                        }
                    } else {
                        const floatx4 hn = h4 + v;
                        *reinterpret_cast<floatx4 *>(e.h + h_tile_offset(token[j], n, N)) = hn;
                        const floatx4 g4 = gv[q];
                        uint2 o;
                        o.x = pack_h16x2(hn[0] * g4[0], hn[1] * g4[1]);
                        o.y = pack_h16x2(hn[2] * g4[2], hn[3] * g4[3]);
                        *reinterpret_cast<uint2 *>(e.hg + frag_offset(token[j], n, N >> 5)) = o;
                        ssq[j] += hn[0] * hn[0] + hn[1] * hn[1] + hn[2] * hn[2] + hn[3] * hn[3];
                    }
                }
            }
        }
        if (!e.last_layer) {
            // sum of squares of each token over the 128 features of one partial: the two lane halves hold disjoint rows
            constexpr int WP = GEMM_SSQ_COLS / (32 * FM);           // waves that share a partial
            static_assert(MODE != DEC_RESID || (WP * 32 * FM == GEMM_SSQ_COLS && WM % WP == 0), "whole waves per partial, whole partials per block");
            if constexpr (32 * FM == GEMM_SSQ_COLS) {
                const int grp = (bm * TA + wm * FM * 2) * 16 / GEMM_SSQ_COLS;
#pragma unroll
                for (int j = 0; j < FT; ++j) {
                    const float tot = ssq[j] + __shfl_xor(ssq[j], 32, 64);
                    if (hl == 0 && token[j] < T) e.ssq_out[(size_t)grp * T + token[j]] = tot;
                }
            } else {
                // WP neighbouring waves hold a partial's features between them: summed through LDS in wave order
#pragma unroll
                for (int j = 0; j < FT; ++j) {
                    const float tot = ssq[j] + __shfl_xor(ssq[j], 32, 64);
                    if (hl == 0) ssq_lds[wm * NTOK + tl0 + 32 * j + (lane & 31)] = tot;
                }
                __syncthreads();
                if (wm % WP == 0) {
                    const int grp = (bm * WM + wm) / WP;
#pragma unroll
                    for (int j = 0; j < FT; ++j) {
                        float tot = 0.f;
#pragma unroll
                        for (int w = 0; w < WP; ++w) tot += ssq_lds[(wm + w) * NTOK + tl0 + 32 * j + (lane & 31)];
                        if (hl == 0 && token[j] < T && grp * GEMM_SSQ_COLS < N) e.ssq_out[(size_t)grp * T + token[j]] = tot;
                    }
                }
            }
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < FT; ++j) {
        const int tl = tl0 + 32 * j + (lane & 31);             // token column inside the block tile
        const int token = bt * NTOK + tl;
        const bool tv = token < T;
        const float r = e.ssq_in != nullptr ? rstd_of(tl) : 1.0f;
        int seq = 0, pos = 0;
        if (MODE == DEC_QKV && tv) { seq = e.rm.row_seq[token]; pos = e.rm.row_pos[token]; }
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const int t16 = bm * TA + (wm * FM + i) * 2;        // first 16-row tile of this 32-feature block
            const floatx16 c = acc_of(i, j);
            if (MODE == DEC_RAW) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int n = t16 * 16 + 8 * q + 4 * hl;
                    if (tv && n < N)
                        *reinterpret_cast<floatx4 *>(e.raw_out + (size_t)token * N + n) =
                            floatx4{c[4 * q] * r, c[4 * q + 1] * r, c[4 * q + 2] * r, c[4 * q + 3] * r};
                }
            } else if (MODE == DEC_SWIGLU) {
                // tile t16 = gate, t16 + 1 = up (interleaved packing): quads 0, 1 against quads 2, 3
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int f = (t16 >> 1) * 16 + 8 * q + 4 * hl;
                    if (!tv || f >= e.F_l) continue;
                    float u[4];
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const float aa = c[4 * q + x] * r;
                        u[x] = aa / (1.0f + __expf(-aa)) * (c[4 * (q + 2) + x] * r);
                    }
                    uint2 o;
                    o.x = pack_h16x2(u[0], u[1]);
                    o.y = pack_h16x2(u[2], u[3]);
                    *reinterpret_cast<uint2 *>(e.u + frag_offset(token, f, e.F_l >> 5)) = o;
                }
            } else {   // DEC_QKV: each 16-row tile holds 8 rotary pairs (rows r, r + 8)
                const int d = e.kg.d, half = d >> 1, tph = d >> 4;
#pragma unroll
                for (int m = 0; m < 2; ++m) {              // the two 16-row tiles of this block
                    const int tile = t16 + m;
                    if (!tv || tile >= n_tiles) continue;
                    const int head = tile / tph, tl16 = tile - head * tph;
                    const int i0 = tl16 * 8 + 4 * hl;            // first rotary pair index of this lane
                    float lo[4], hi[4];
#pragma unroll
                    for (int x = 0; x < 4; ++x) { lo[x] = c[4 * (2 * m) + x] * r; hi[x] = c[4 * (2 * m + 1) + x] * r; }
                    if (head < e.hq_l + e.kg.hkv_l) {
                        const floatx4 c4 = *reinterpret_cast<const floatx4 *>(e.cos_tab + (size_t)pos * half + i0);
                        const floatx4 s4 = *reinterpret_cast<const floatx4 *>(e.sin_tab + (size_t)pos * half + i0);
#pragma unroll
                        for (int x = 0; x < 4; ++x) {
                            const float a = lo[x], b = hi[x];
                            lo[x] = a * c4[x] - b * s4[x];
                            hi[x] = b * c4[x] + a * s4[x];
                        }
                    }
                    uint2 plo, phi;
                    plo.x = pack_h16x2(lo[0], lo[1]); plo.y = pack_h16x2(lo[2], lo[3]);
                    phi.x = pack_h16x2(hi[0], hi[1]); phi.y = pack_h16x2(hi[2], hi[3]);
                    if (head < e.hq_l) {
                        const int qkt = (e.hq_l * d) >> 5;
                        *reinterpret_cast<uint2 *>(e.q + frag_offset(token, head * d + i0, qkt)) = plo;
                        *reinterpret_cast<uint2 *>(e.q + frag_offset(token, head * d + i0 + half, qkt)) = phi;
                    } else if (head < e.hq_l + e.kg.hkv_l) {
                        const size_t slab = (size_t)seq * e.kg.seq_stride + (size_t)(head - e.hq_l) * e.kg.smax * d;
                        *reinterpret_cast<uint2 *>(e.kc + slab + kv_k_offset(pos, i0, d)) = plo;
                        *reinterpret_cast<uint2 *>(e.kc + slab + kv_k_offset(pos, i0 + half, d)) = phi;
                    } else {
                        const size_t slab =
                            (size_t)seq * e.kg.seq_stride + (size_t)(head - e.hq_l - e.kg.hkv_l) * e.kg.smax * d;
#pragma unroll
                        for (int x = 0; x < 4; ++x) {
                            e.vc[slab + kv_v_offset(pos, i0 + x, d)] = f32_to_h16(lo[x]);
                            e.vc[slab + kv_v_offset(pos, i0 + half + x, d)] = f32_to_h16(hi[x]);
                        }
                    }
                }
            }
        }
    }
}

// Partial sums of a split contraction: [split][32-feature block][32-token block][quad][lane][4], a 4 KB piece per result
// tile in the order it sits in the registers (1 KB per store), whatever kernel and tile shape wrote it; blocks that hold
// nothing but padding are not stored.  nb feature blocks from the launch's first one, tb token blocks.
struct PartGeom {
    int nb, tb;
};
__host__ __device__ inline PartGeom part_geom(int n_tiles, int t_tiles, int nb32_first, int nb32_count) {
    const int all = (n_tiles + 1) / 2 - nb32_first;
    return PartGeom{all < nb32_count ? all : nb32_count, (t_tiles + 1) / 2};
}
__host__ __device__ inline size_t part_offset(const PartGeom &g, int split, int nb, int tb) {
    return (((size_t)split * g.nb + nb) * g.tb + tb) * 1024;
}
__device__ __forceinline__ void part_store(float *dst, const floatx16 &c, int lane) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
        *reinterpret_cast<floatx4 *>(dst + q * 256 + lane * 4) = floatx4{c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]};
}

// The same for a block of the same launch: past the caches of the die (common.h, device-scope accesses)
__device__ __forceinline__ void part_store_dev(float *dst, const floatx16 &c, int lane) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const floatx4 v = {c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]};
        asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" : : "v"(dst + q * 256 + lane * 4), "v"(v) : "memory");
    }
}
__device__ __forceinline__ void part_load_dev(const float *src, floatx4 (&v)[4], int lane) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        union { uint64_t u[2]; floatx4 f; } r;
        const uint64_t *p = reinterpret_cast<const uint64_t *>(src + q * 256 + lane * 4);
        r.u[0] = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        r.u[1] = __hip_atomic_load(p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        v[q] = r.f;
    }
}

// Linear tile id -> (feature block bm, token block bt).  Ids are dealt out patch by patch: a patch is pm_h feature
// blocks x pt_w token blocks (lower / narrower at the edges), patches run along the token blocks first, and inside a
// patch the feature block varies fastest.  pm_h = 1, pt_w = t_blocks is the plain row-major order.
__device__ __forceinline__ void gemm_tile_of_id(int id, int n_blocks, int t_blocks, int pm_h, int pt_w, int &bm, int &bt) {
    const int row = pm_h * t_blocks;                       // tiles of a full patch row
    const int pm = id / row, rem = id - pm * row;
    const int hm = min(pm_h, n_blocks - pm * pm_h);        // height of this patch row (the last one may be lower)
    const int pt = rem / (hm * pt_w), rem2 = rem - pt * hm * pt_w;
    bm = pm * pm_h + rem2 % hm;
    bt = pt * pt_w + rem2 / hm;
}

// Operand tiles travel HBM -> LDS with direct-to-LDS loads (no registers in between): a wave copies one
// 1 KB fragment tile per instruction, lane l's 16 bytes landing at tile base + 16 l.  S stages of the k-loop
// are resident; the wait before a step only covers that step's loads (vmcnt counts the rest).
//
// Block = WM x WT waves; each wave owns FM x FT tiles of 32 features x 32 tokens, so the block tile is
// (32 FM WM) features x (32 FT WT) tokens.
//
// PP = true (8 waves, two per SIMD): the two waves of a SIMD run the k-loop half a step out of phase.  Every wave
// alternates a MEMORY phase (all operand fragments of one 32-deep k-step from LDS into registers, its share of the
// direct-to-LDS loads of a later stage) and a COMPUTE phase (the k-step's MFMAs back to back, nothing else in the
// stream), each closed by a workgroup barrier; waves 4..7 pass one extra barrier before their loop, waves 0..3 one
// after it.  So while one wave of a SIMD waits for LDS data, for its loads or at a barrier, the other one is inside
// its MFMA run: the barriers and waits that idle the matrix core in the lock-stepped loop below fall into the
// shadow of the other wave's MFMAs.
//
// ABL (measurement only; results are garbage, every access stays in bounds and every barrier is kept): the same kernel
// with one activity of its k-loop taken out, to price that activity on a power-limited chip.  1: no direct-to-LDS
// loads inside the loop (the MFMAs run on the stages the prologue fetched); 2: the loads are issued but every k-step
// re-reads the block's first k-step (cache hits, no new bytes from HBM); 3: the operand fragments are read from LDS
// for the first k-step only.
template <int FM, int FT, int WM, int WT, int S, int MODE, bool PP = false, int ABL = 0>
__global__ __launch_bounds__(64 * WM * WT) void gemm_mfma_kernel(const h16_t *__restrict__ Wp,
                                                                 const h16_t *__restrict__ Xp, int N, int k_tiles,
                                                                 int n_tiles, int t_tiles, int T, int n_blocks,
                                                                 int t_blocks, GemmEpi e, float *__restrict__ part,
                                                                 int pm_h, int pt_w, int nb0) {
    constexpr int NW = WM * WT, NT = 64 * NW;
    constexpr int TA = 2 * FM * WM, TB = 2 * FT * WT;   // 16-row operand tiles per block and k-step
    constexpr int LA = TA / NW, LB = TB / NW;         // direct-to-LDS loads per wave and stage, per operand
    constexpr int LPT = LA + LB;
    constexpr int STAGE = (TA + TB) * 64;            // h16x8 elements per stage
    constexpr int NTOK = TB * 16;                    // token columns of the block tile
    static_assert(TA % NW == 0 && TB % NW == 0, "operand tiles must divide evenly over the waves");
    extern __shared__ h16x8 smem[];                 // [S][TA + TB][64], then NT floats
    float *ssq_s = reinterpret_cast<float *>(smem + (size_t)S * STAGE);
    // XCD-aware remap of the linear block id
    const int total = n_blocks * t_blocks;
    int id = blockIdx.x;
    const int per_xcd = (total + 7) / 8;
    id = (id & 7) * per_xcd + (id >> 3);
    if (id >= total) return;                     // only when total is not a multiple of 8
    // Consecutive ids (the blocks one XCD runs at the same time) form a patch of pm_h feature blocks x pt_w token
    // blocks: per k-step the patch fetches (pm_h + pt_w) operand slices into that XCD's L2 for pm_h x pt_w tiles.
    int bm, bt;
    gemm_tile_of_id(id, n_blocks, t_blocks, pm_h, pt_w, bm, bt);
    bm += nb0;               // the launch covers feature blocks nb0 .. nb0 + n_blocks - 1 of the matrix
    // the wave index is made provably uniform: tile addresses and LDS destinations then stay in scalar registers
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int wm = wave % WM, wt = wave / WM;
    // split contraction (few token tiles, see launch_cfg): blockIdx.y takes k-steps [k0, k0 + k_len) and leaves its
    // fp32 result tiles in `part`; gemm_finish_kernel adds the splits up and runs the epilogue
    const int k0 = (int)((long)blockIdx.y * k_tiles / gridDim.y);
    const int k_len = (int)((long)(blockIdx.y + 1) * k_tiles / gridDim.y) - k0;

    // The sums of squares of the block's token columns from the producer's partials, once per block while the pipeline fills:
    // NT / NTOK threads per token, each with its share of the partials in one round of requests (one thread per token
    // and 16 at a time was four round trips, about 3 us of a block's start); 1 / rms follows in the epilogue.
    constexpr int SSP = NT / NTOK;
    static_assert(SSP >= 1 && NT % NTOK == 0, "whole threads per token");
    auto sum_squares = [&]() {
        if (MODE == DEC_RESID || e.ssq_in == nullptr || part != nullptr) return;
        const int groups = e.norm_dim / GEMM_SSQ_COLS, tok = (int)threadIdx.x % NTOK, token = min(bt * NTOK + tok, T - 1);
        float ss = 0.f;
#pragma unroll 32
        for (int gI = threadIdx.x / NTOK; gI < groups; gI += SSP) ss += e.ssq_in[(size_t)gI * T + token];
        ssq_s[threadIdx.x] = ss;
    };
    auto rstd_of = [&](int tl) {
        float ss = ssq_s[tl];
#pragma unroll
        for (int w = 1; w < SSP; ++w) ss += ssq_s[w * NTOK + tl];
        return 1.0f / sqrtf(ss / (float)e.norm_dim + e.eps);
    };

    // result tile (i, j) of this wave to the partial sums of this split
    const PartGeom pg = part_geom(n_tiles, t_tiles, nb0 * FM * WM, n_blocks * FM * WM);
    auto store_part = [&](int i, int j, const floatx16 &c) {
        const int nb = (bm - nb0) * FM * WM + wm * FM + i, tb = (bt * WT + wt) * FT + j;
        if (nb < pg.nb && tb < pg.tb) part_store(part + part_offset(pg, blockIdx.y, nb, tb), c, lane);
    };

    floatx16 acc[FM][FT];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    const h16x8 *A = reinterpret_cast<const h16x8 *>(Wp);
    const h16x8 *B = reinterpret_cast<const h16x8 *>(Xp);
    // this wave copies tiles wave, wave + NW, ... of both operands; out-of-range tiles are clamped to the last
    // valid tile (their products are never stored) so that every wave issues LPT loads per stage.  Tile bases
    // are uniform (scalar registers); the lane adds its 16-byte slot as a 32-bit offset.
    const h16x8 *asrc[LA], *bsrc[LB];
#pragma unroll
    for (int i = 0; i < LA; ++i) asrc[i] = A + (size_t)min(bm * TA + wave + NW * i, n_tiles - 1) * 64 + (size_t)k0 * n_tiles * 64;
#pragma unroll
    for (int i = 0; i < LB; ++i) bsrc[i] = B + ((size_t)min(bt * TB + wave + NW * i, t_tiles - 1) * k_tiles + k0) * 64;
    const size_t astep = (size_t)n_tiles * 64;       // k-tile-major weights
    // One direct-to-LDS load: index x < LA is a weight tile, the rest are activation tiles.  k-steps past
    // the end are clamped to the last one (they land in a buffer nobody reads any more), so that every
    // k-step issues exactly LPT loads and the loop body stays one basic block.
    // One direct-to-LDS load of a 1 KB tile: index x < LA is a weight tile, the rest are activation tiles.
    // k-steps past the end are clamped to the last one (they land in a buffer nobody reads any more), so that
    // every k-step issues exactly LPT loads and the loop body stays one basic block.  The load is written in
    // its scalar-base form (tile address in scalar registers, the lane's 16-byte slot as the 32-bit vector
    // offset, LDS destination in M0: hx_load_lds16), which the compiler does not select for this instruction by itself: it
    // would spend a 64-bit vector add per load inside the MFMA stream.  vmcnt is drained before the epilogue issues
    // ordinary loads.
    const unsigned lane_bytes = (unsigned)lane * 16u;
    auto issue_one = [&](int kt, int x) {
        const int kc = ABL == 2 ? 0 : min(kt, k_len - 1);
        h16x8 *st = smem + (size_t)(kt % S) * STAGE;
        const h16x8 *src = x < LA ? asrc[x] + kc * astep : bsrc[x - LA] + (size_t)kc * 64;
        h16x8 *dst = x < LA ? st + (wave + NW * x) * 64 : st + (TA + wave + NW * (x - LA)) * 64;
        hx_load_lds16(hx_lds_addr(dst), lane_bytes, src);
    };
    // 32x32x16 operand for k-half kh of a pair of 16-row tiles: lane l takes row l % 32, k-group 2 kh + l / 32
    const int frag = ((lane & 31) >> 4) * 64 + (lane & 15) + 16 * (lane >> 5);
    // Software pipeline.  (1) The operand registers of one 16-deep half step are fetched from LDS while the
    // MFMAs of the previous half step run.  (2) The barrier sits in the MIDDLE of a k-step: it publishes stage
    // kt + 1, whose first half is then fetched under the second half of stage kt, and frees the buffer of
    // stage kt - 1.  (3) The loads of stage kt + S - 1 into that buffer are spread over one whole step, half
    // behind the barrier of step kt and half in front of the barrier of step kt + 1, one load every few MFMAs.
    if constexpr (PP) {
        static_assert(NW == 8 && S >= 3, "ping-pong: two waves per SIMD");
        const int grp = wave >> 2;                 // waves w and w + 4 share a SIMD
#pragma unroll
        for (int p2 = 0; p2 < S - 1; ++p2)
#pragma unroll
            for (int x = 0; x < LPT; ++x) issue_one(p2, x);
        sum_squares();
        HX_WAIT_VM((S - 2) * LPT);                 // stage 0 has landed (this wave's share of it)
        HX_LDS_BARRIER();                          // ... and everybody's
        if (grp == 1) asm volatile("s_barrier" ::: "memory");       // half a step behind waves 0..3 from here on
        // The MFMAs of this loop are v_mfma_f32_16x16x32_bf16 on the fragment tiles as they lie in LDS (one 128-bit read per
        // 16-row tile and k-step, lane l reads entry l): on operands whose bits toggle the chip is power-limited, and this
        // form sustains about 12 % more flops than 32x32x16 at the same socket power (register-only probe,
        // profiles/hbm_mfma_calibration.txt).  Same LDS traffic and MFMA cycles per k-step as the 32x32x16 form: 12 reads,
        // 32 x 16 cycles.  a16[i][j] = features 16 i .. + 15 of the wave tile x tokens 16 j .. + 15; lane l holds token
        // l % 16 and features 4 (l / 16) .. + 3.
        floatx4 a16[2 * FM][2 * FT];
#pragma unroll
        for (int i = 0; i < 2 * FM; ++i)
#pragma unroll
            for (int j = 0; j < 2 * FT; ++j) a16[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
        h16x8 pa[2 * FM], pb[2 * FT];
        for (int kt = 0; kt < k_len; ++kt) {
            // memory phase: the whole k-step's operands, then this wave's loads of stage kt + S - 1 into the buffer
            // of stage kt - 1, which both halves of the block have finished reading (barriers below)
            const h16x8 *sa = smem + (size_t)(kt % S) * STAGE + (wm * FM * 2) * 64 + lane;
            const h16x8 *sb = smem + (size_t)(kt % S) * STAGE + (TA + wt * FT * 2) * 64 + lane;
            if (ABL != 3 || kt == 0) {
#pragma unroll
                for (int x = 0; x < 2 * FT; ++x) pb[x] = sb[x * 64];
#pragma unroll
                for (int x = 0; x < 2 * FM; ++x) pa[x] = sa[x * 64];
            }
            if (ABL != 1) {
#pragma unroll
                for (int x = 0; x < LPT; ++x) issue_one(kt + S - 1, x);
            }
            __builtin_amdgcn_sched_barrier(0);
            HX_WAIT_VM(ABL == 1 ? 0 : (S - 2) * LPT);      // this wave's loads of stage kt + 1 have landed
            HX_LDS_BARRIER();                      // operands in registers; barrier
            __builtin_amdgcn_sched_barrier(0);
            // compute phase
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int i = 0; i < 2 * FM; ++i)
#pragma unroll
                for (int j = 0; j < 2 * FT; ++j)
                    a16[i][j] = hx_mfma16(pa[i], pb[j], a16[i][j]);
            __builtin_amdgcn_s_setprio(0);
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_barrier" ::: "memory");
        }
        if (grp == 0) asm volatile("s_barrier" ::: "memory");       // the barrier waves 4..7 passed ahead of their loop
        HX_WAIT_VM(0);
        // Into the register layout of a 32 x 32 MFMA result, which the epilogues are written for: lane L holds token
        // L % 32 and, in register 4 q + r, feature 8 q + 4 (L / 32) + r of the 32 x 32 block.  That value sits in the
        // 16 x 16 tile (q / 2, (L % 32) / 16) of the block, register r, lane 16 (2 (q % 2) + L / 32) + L % 16.  Converted
        // tile by tile when the epilogue asks for it, so that the two layouts never hold the whole wave tile at once.
        auto acc_of = [&](int i, int j) {
            floatx16 c;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int src = 16 * (2 * (q & 1) + (lane >> 5)) + (lane & 15);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float v0 = __shfl(a16[2 * i + (q >> 1)][2 * j][r], src, 64);
                    const float v1 = __shfl(a16[2 * i + (q >> 1)][2 * j + 1][r], src, 64);
                    c[4 * q + r] = (lane & 16) ? v1 : v0;
                }
            }
            return c;
        };
        if (part != nullptr) {
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FT; ++j) store_part(i, j, acc_of(i, j));
            return;
        }
        gemm_epilogue<FM, FT, WM, NTOK, MODE>(acc_of, bm, bt, wm, wt * FT * 32, lane, N, n_tiles, T, e, rstd_of);
        return;
    }
    constexpr int H1 = (LPT + 1) / 2, H2 = LPT / 2;  // loads issued behind / in front of the barrier
    constexpr int HL = H1;
    // MFMA slots of a half step: the first FM + FT also carry an LDS fetch; the loads go behind them when
    // there is room, else they are spread over all slots
    constexpr int FREE = FM * FT - (FM + FT);
    constexpr int LOAD0 = FREE >= HL ? FM + FT : 0;
    constexpr int GAP = FREE >= HL ? FREE / HL : ((FM * FT) / HL > 0 ? (FM * FT) / HL : 1);
    static_assert(S >= 3, "the pipeline needs three stages");
#pragma unroll
    for (int p = 0; p < S - 2; ++p)
#pragma unroll
        for (int x = 0; x < LPT; ++x) issue_one(p, x);
#pragma unroll
    for (int x = 0; x < H1; ++x) issue_one(S - 2, x);
    sum_squares();
    h16x8 fa0[FM], fb0[FT], fa1[FM], fb1[FT];
    // x-th operand fetch of a half step: the FT token operands first, then the FM feature operands
    auto fetch_one = [&](h16x8(&fa)[FM], h16x8(&fb)[FT], int kt, int kh, int x) {
        const h16x8 *sa = smem + (size_t)(kt % S) * STAGE + (wm * FM * 2) * 64 + frag + kh * 32;
        const h16x8 *sb = smem + (size_t)(kt % S) * STAGE + (TA + wt * FT * 2) * 64 + frag + kh * 32;
        if (x < FT) fb[x] = sb[x * 128];
        else fa[x - FT] = sa[(x - FT) * 128];
    };
    auto fetch = [&](h16x8(&fa)[FM], h16x8(&fb)[FT], int kt, int kh) {
#pragma unroll
        for (int x = 0; x < FM + FT; ++x) fetch_one(fa, fb, kt, kh, x);
    };
    static_assert(PP || FM + FT <= FM * FT, "one operand fetch per MFMA slot");
    HX_WAIT_VM((S - 3) * LPT + H1);
    HX_LDS_BARRIER();
    fetch(fa0, fb0, 0, 0);
    HX_WAIT_LGKM0();
    // The memory pipeline of a CU accepts one wave-wide 1 KB load every ~26 cycles and hardly queues: waves
    // that issue their loads at the same point of the (lock-stepped) MFMA stream block each other for tens of
    // cycles with the matrix core idle.  Each wave therefore runs a copy of the loop whose loads sit OFF
    // MFMAs later than its neighbour's, which gives the CU one load per MFMA slot.
    auto k_loop = [&](auto off_c) {
        constexpr int OFF = decltype(off_c)::value;
    for (int kt = 0; kt < k_len; ++kt) {
        // one slot = one MFMA, at most one LDS fetch for the NEXT half step and at most one global load; the
        // slots are fenced so that the order below is the order in the instruction stream
#pragma unroll
        for (int m = 0; m < FM * FT; ++m) {
            acc[m / FT][m % FT] = hx_mfma32(fa0[m / FT], fb0[m % FT], acc[m / FT][m % FT]);
            if (m < FM + FT) fetch_one(fa1, fb1, kt, 1, m);
            if (m >= LOAD0 && (m - LOAD0) % GAP == OFF && (m - LOAD0) / GAP < H2) issue_one(kt + S - 2, H1 + (m - LOAD0) / GAP);
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_sched_barrier(0);
        HX_WAIT_VM((S - 3) * LPT);      // stage kt + 1 has landed; later stages stay in flight
        HX_LDS_BARRIER();
#pragma unroll
        for (int m = 0; m < FM * FT; ++m) {
            acc[m / FT][m % FT] = hx_mfma32(fa1[m / FT], fb1[m % FT], acc[m / FT][m % FT]);
            if (m < FM + FT) fetch_one(fa0, fb0, kt + 1, 0, m);
            if (m >= LOAD0 && (m - LOAD0) % GAP == OFF && (m - LOAD0) / GAP < H1) issue_one(kt + S - 1, (m - LOAD0) / GAP);
            __builtin_amdgcn_sched_barrier(0);
        }
        // the fetch of the next half step has had FM FT MFMAs to complete: waiting here, instead of where
        // the compiler would place it (behind the next fetch), costs nothing and keeps that fetch covered
        __builtin_amdgcn_sched_barrier(0);
        HX_WAIT_LGKM0();
    }
    };
    {
        const int off = (wave * GAP) / NW;
        if (GAP > 3 && off == 3) k_loop(std::integral_constant<int, (GAP > 3 ? 3 : 0)>{});
        else if (GAP > 2 && off == 2) k_loop(std::integral_constant<int, (GAP > 2 ? 2 : 0)>{});
        else if (GAP > 1 && off == 1) k_loop(std::integral_constant<int, (GAP > 1 ? 1 : 0)>{});
        else k_loop(std::integral_constant<int, 0>{});
    }
    HX_WAIT_VM(0);
    if (part != nullptr) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FT; ++j) store_part(i, j, acc[i][j]);
        return;
    }
    gemm_epilogue<FM, FT, WM, NTOK, MODE>([&](int i, int j) { return acc[i][j]; }, bm, bt, wm, wt * FT * 32, lane, N, n_tiles, T, e, rstd_of);
}

// -------------------------------------------------------------------------------------------------
// 256 features x 32 (TA32 + TB32) tokens per block: the two-phase loop above with wave tiles of 64 features x 32 TA32 tokens (waves 0 .. 3)
// and x 32 TB32 tokens (waves 4 .. 7).  The two waves of a SIMD are one of either kind and take turns on the matrix core, so the kinds need
// not be equal: 7 x 32 tokens are 4 + 3, and a k-step is 512 + 384 cycles of MFMAs.  One prompt of 430 rows pays for 448 in it instead of
// 512.  Bound like the 256-wide tiles by the power limit when the chip is full (that prompt's W1/W3 on a TP2 shard, 224 tiles either
// way: 1.65 GHz, 416 -> 403 us per layer) and by LDS traffic, 11 or 10 reads of 1 KB per wave and k-step instead of 12.  Waves 0 .. 3 load the weights, waves
// 4 .. 7 the activations.  Every result is one chain over the block's k-steps, as in those tiles: the same bits before the epilogue.
// -------------------------------------------------------------------------------------------------
template <int TA32, int TB32, int MODE>
__global__ __launch_bounds__(512) void gemm_cols_kernel(const h16_t *__restrict__ Wp, const h16_t *__restrict__ Xp, int N, int k_tiles,
                                                        int n_tiles, int t_tiles, int T, int n_blocks, int t_blocks, GemmEpi e,
                                                        float *__restrict__ part) {
    constexpr int S = 4, WA = 16, TT = 2 * (TA32 + TB32), STAGE = (WA + TT) * 64, NTOK = 16 * TT;
    extern __shared__ h16x8 smem[];                 // [S][WA + TT][64], then 1024 floats
    float *ssq_s = reinterpret_cast<float *>(smem + (size_t)S * STAGE);
    const int total = n_blocks * t_blocks;
    int id = blockIdx.x;
    const int per_xcd = (total + 7) / 8;
    id = (id & 7) * per_xcd + (id >> 3);
    if (id >= total) return;                     // only when total is not a multiple of 8
    int bm, bt;
    gemm_tile_of_id(id, n_blocks, t_blocks, 4, min(8, t_blocks), bm, bt);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int k0 = (int)((long)blockIdx.y * k_tiles / gridDim.y);
    const int k_len = (int)((long)(blockIdx.y + 1) * k_tiles / gridDim.y) - k0;
    auto sum_squares = [&]() {
        if (MODE == DEC_RESID || e.ssq_in == nullptr || part != nullptr) return;
        const int groups = e.norm_dim / GEMM_SSQ_COLS, tok = tid & 255, token = min(bt * NTOK + tok, T - 1);
        float ss = 0.f;
#pragma unroll 32
        for (int gI = tid >> 8; gI < groups; gI += 2) ss += e.ssq_in[(size_t)gI * T + token];
        ssq_s[tid] = ss;
    };
    auto rstd_of = [&](int tl) { return 1.0f / sqrtf((ssq_s[tl] + ssq_s[256 + tl]) / (float)e.norm_dim + e.eps); };
    const PartGeom pg = part_geom(n_tiles, t_tiles, 0, n_blocks * 8);

    auto group = [&](auto grp_c) {
        constexpr int GRP = decltype(grp_c)::value, FT = GRP == 0 ? TA32 : TB32;
        // waves 0 .. 3 copy the weight tiles of a k-step, waves 4 .. 7 the activation tiles (the last ones may be copied twice); tiles
        // outside the matrix are clamped to its last ones, k-steps past the end to the last one
        constexpr int LPT = GRP == 0 ? WA / 4 : (TT + 3) / 4;
        const int wm = wave & 3;
        const h16x8 *src[LPT];
        unsigned dst[LPT];
#pragma unroll
        for (int x = 0; x < LPT; ++x) {
            const int i = wm + 4 * x, j = min(i, TT - 1);
            src[x] = GRP == 0 ? reinterpret_cast<const h16x8 *>(Wp) + ((size_t)k0 * n_tiles + min(bm * WA + i, n_tiles - 1)) * 64
                              : reinterpret_cast<const h16x8 *>(Xp) + ((size_t)min(bt * TT + j, t_tiles - 1) * k_tiles + k0) * 64;
            dst[x] = hx_lds_addr(smem + (GRP == 0 ? i : WA + j) * 64);
        }
        const size_t step = GRP == 0 ? (size_t)n_tiles * 64 : 64;
        const unsigned lane_bytes = (unsigned)lane * 16u;
        auto issue = [&](int kt) {
            const int kc = min(kt, k_len - 1);
            const unsigned st = (unsigned)(kt % S) * (STAGE * 16u);
#pragma unroll
            for (int x = 0; x < LPT; ++x) hx_load_lds16(dst[x] + st, lane_bytes, src[x] + kc * step);
        };
#pragma unroll
        for (int p2 = 0; p2 < S - 1; ++p2) issue(p2);
        sum_squares();
        HX_WAIT_VM((S - 2) * LPT);
        HX_LDS_BARRIER();
        if (GRP == 1) asm volatile("s_barrier" ::: "memory");       // half a step behind waves 0 .. 3 from here on
        floatx4 a16[4][2 * FT];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2 * FT; ++j) a16[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
        h16x8 pa[4], pb[2 * FT];
        for (int kt = 0; kt < k_len; ++kt) {
            const h16x8 *sa = smem + (size_t)(kt % S) * STAGE + wm * 4 * 64 + lane;
            const h16x8 *sb = smem + (size_t)(kt % S) * STAGE + (WA + GRP * 2 * TA32) * 64 + lane;
#pragma unroll
            for (int x = 0; x < 2 * FT; ++x) pb[x] = sb[x * 64];
#pragma unroll
            for (int x = 0; x < 4; ++x) pa[x] = sa[x * 64];
            issue(kt + S - 1);
            __builtin_amdgcn_sched_barrier(0);
            HX_WAIT_VM((S - 2) * LPT);
            HX_LDS_BARRIER();
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 2 * FT; ++j) a16[i][j] = hx_mfma16(pa[i], pb[j], a16[i][j]);
            __builtin_amdgcn_s_setprio(0);
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_barrier" ::: "memory");
        }
        if (GRP == 0) asm volatile("s_barrier" ::: "memory");       // the barrier waves 4 .. 7 passed ahead of their loop
        HX_WAIT_VM(0);
        auto acc_of = [&](int i, int j) {           // into the register layout of a 32 x 32 result, as in gemm_mfma_kernel
            floatx16 c;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int from = 16 * (2 * (q & 1) + (lane >> 5)) + (lane & 15);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float v0 = __shfl(a16[2 * i + (q >> 1)][2 * j][r], from, 64);
                    const float v1 = __shfl(a16[2 * i + (q >> 1)][2 * j + 1][r], from, 64);
                    c[4 * q + r] = (lane & 16) ? v1 : v0;
                }
            }
            return c;
        };
        if (part != nullptr) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < FT; ++j) {
                    const int nb = bm * 8 + wm * 2 + i, tb = bt * (TA32 + TB32) + GRP * TA32 + j;
                    const floatx16 c = acc_of(i, j);
                    if (nb < pg.nb && tb < pg.tb) part_store(part + part_offset(pg, blockIdx.y, nb, tb), c, lane);
                }
            return;
        }
        gemm_epilogue<2, FT, 4, NTOK, MODE>(acc_of, bm, bt, wm, GRP * TA32 * 32, lane, N, n_tiles, T, e, rstd_of, ssq_s);
    };
    if (wave < 4) group(std::integral_constant<int, 0>{});
    else group(std::integral_constant<int, 1>{});
}

// Second pass of a split contraction.  A block of 4 waves finishes 128 features x 32 tokens, a wave one 32 x 32 result tile:
// it adds the tile up over the splits, in split order, and runs the epilogue (the residual epilogue's sum of squares over
// the 128 features goes through LDS).  The partial sums come from blocks all over the chip, so every read is a trip to the
// memory-side cache: what bounds this pass is how many of those are in flight, hence small tiles (as many waves as there
// are 4 KB pieces) and four splits requested at a time.  Measured against one block per GEMM tile walking the splits one
// after the other: W2 of a TP2 70B shard at 430 rows (64 tiles x 4 splits) 24.5 -> 20 us, W_O 16.4 -> 12, W_O of a 2048-wide
// layer at 1131 rows (72 x 3) 13.0 -> 10.2, TP4 QKV at 2048 rows (80 x 3) 24.2 -> 14.9, at 117 rows (8 splits) 7.7 -> 6.1.
template <int MODE>
__global__ __launch_bounds__(256) void gemm_finish_kernel(const float *__restrict__ part, int splits, int N, int n_tiles, int T,
                                                          PartGeom pg, int fb0, GemmEpi e) {
    __shared__ float rstd_s[32], ssum[8][32];
    __shared__ float ssq_lds[MODE == DEC_RESID ? 4 * 32 : 1];
    const int fb = blockIdx.x / pg.tb, bt = blockIdx.x - fb * pg.tb;        // 128-feature block of the launch, 32-token block
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int nb = fb * 4 + wave;
    const bool mine = nb < pg.nb;                                            // the last block's waves may lie beyond the matrix
    const bool norm = MODE != DEC_RESID && e.ssq_in != nullptr;
    // eight threads per token share its sums of squares
    float ss = 0.f;
    if (norm) {
        const int groups = e.norm_dim / GEMM_SSQ_COLS, token = min(bt * 32 + (tid & 31), T - 1);
#pragma unroll 8
        for (int gI = tid >> 5; gI < groups; gI += 8) ss += e.ssq_in[(size_t)gI * T + token];
    }
    // residual and gain are here with the first sums (kernel trace, W2 of a TP4 70B shard: 117 rows 6.8 -> 6.0 us, 90 rows 5.8 -> 5.2)
    ResidPre pre;
    floatx16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    auto add = [&](int z0, auto count, bool first) {
        constexpr int C = decltype(count)::value;
        floatx4 v[C][4];
#pragma unroll
        for (int z = 0; z < C; ++z)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                v[z][q] = *reinterpret_cast<const floatx4 *>(part + part_offset(pg, z0 + z, nb, bt) + q * 256 + lane * 4);
        if (MODE == DEC_RESID && first) resid_request(pre, bt * 32 + (lane & 31), ((fb0 + fb) * 4 + wave) * 32, lane >> 5, N, T, e);
#pragma unroll
        for (int z = 0; z < C; ++z)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int x = 0; x < 4; ++x) acc[4 * q + x] += v[z][q][x];
    };
    if (mine) {
        // the first one to four splits, whatever their number is modulo four, then four at a time
        int z = (splits - 1) % 4 + 1;
        if (z == 4) add(0, std::integral_constant<int, 4>{}, true);
        else if (z == 3) add(0, std::integral_constant<int, 3>{}, true);
        else if (z == 2) add(0, std::integral_constant<int, 2>{}, true);
        else add(0, std::integral_constant<int, 1>{}, true);
        for (; z < splits; z += 4) add(z, std::integral_constant<int, 4>{}, false);
    }
    if (norm) {
        ssum[tid >> 5][tid & 31] = ss;
        __syncthreads();
        if (tid < 32) {
            float tot = ssum[0][tid];
#pragma unroll
            for (int w = 1; w < 8; ++w) tot += ssum[w][tid];
            rstd_s[tid] = 1.0f / sqrtf(tot / (float)e.norm_dim + e.eps);
        }
        __syncthreads();
    }
    gemm_epilogue<1, 1, 4, 32, MODE>([&](int, int) { return acc; }, fb0 + fb, bt, wave, 0, lane, N, n_tiles, T, e, [&](int tl) { return rstd_s[tl]; },
                                    ssq_lds, MODE == DEC_RESID ? &pre : nullptr);
}

// the finishing launch of a split contraction over feature blocks (of 32) nb32_first .. + nb32_count - 1
template <int MODE>
static void launch_finish(const float *part, int splits, int N, int n_tiles, int t_tiles, int T, int nb32_first, int nb32_count,
                          const GemmEpi &e, hipStream_t s) {
    const PartGeom pg = part_geom(n_tiles, t_tiles, nb32_first, nb32_count);
    hipLaunchKernelGGL(gemm_finish_kernel<MODE>, dim3((pg.nb + 3) / 4 * pg.tb), dim3(256), 0, s, part, splits, N, n_tiles, T, pg,
                       nb32_first / 4, e);
}

// -------------------------------------------------------------------------------------------------
// Skinny form for up to 128 tokens (a short prompt): the launch is bound by streaming the weights, not by the matrix
// cores, so it is built like the decode projections.  A group of 4 waves owns 128 features x 32 NT tokens, a wave 32
// features; the weights never touch LDS: a lane requests the 16 bytes of the two 16-row tiles that the
// 32x32x16 operand wants from it (two 512-byte runs per request), RING k-steps ahead, in a register ring that is
// refilled slot by slot.  The activations of a k-step (2 NT KB, L2 hits) are shared by the group's waves through LDS,
// global -> registers (same ring) -> LDS one k-step before use.  The contraction is split over blockIdx.y; result
// tiles go to `part`.  NT follows the prompt: what a launch pays for tokens beside its weights (operand reads, LDS, MFMAs) is
// paid for 32-token blocks that exist (a TP4 layer of the 70B shape at 20 / 50 / 90 rows 142 / 145 / 153 -> 117 / 132 / 144 us).
// (Meeting at a barrier once per chunk of 4 k-steps, with the next chunk's weights requested at its start instead of slot by
// slot, is slower: W1/W3 of a TP4 70B shard at 117 rows 51 -> 59 us.)
// KG = 2: a block of 8 waves = two groups of 4, each group walking one half of the block's share of the contraction
// in step with the other (one barrier serves both) and the second group's results added to the first's through LDS
// before anything is stored: as many waves and k-steps per wave as two blocks of 4 on two splits, half the partial sums.
// -------------------------------------------------------------------------------------------------
// OWN (W1/W3): no finishing launch.  With one split a block holds the whole contraction.  With two, the block that arrives last adds the
// other's partial sums to its own and finishes the tile: nobody waits for anybody, the sums go past the dies' caches and are added in
// split order, so the results are the finishing kernel's whoever was last.  The arrivals are only ever counted up, two a launch, and an
// odd one is the last: even launches that overlap, which a caller must not have, leave nothing behind for the next.
struct SkinnyOwn {
    const float *ssq_in;       // as in GemmEpi
    int norm_dim, T, F_l;
    float eps;
    h16_t *u;
    unsigned *arrived;         // two splits: per block of features, even between launches
};
template <int KG, int NT, bool OWN>
__global__ __launch_bounds__(256 * KG) void gemm_skinny_kernel(const h16_t *__restrict__ Wp, const h16_t *__restrict__ Xp, int k_tiles,
                                                              int n_tiles, int t_tiles, float *part, int T_rows, SkinnyOwn e) {
    constexpr int RING = NT <= 2 ? 8 : 6, XT = 2 * NT, XW = (XT + 3) / 4;      // 16-token tiles of the block, and per wave
    constexpr int XBUF = 2 * XT * 64, RED = 4 * NT * 16 * 64 / 4;       // LDS in h16x8: staging per group; sums of a group
    __shared__ h16x8 smem[KG == 2 && RED > KG * XBUF ? RED : KG * XBUF];
    const int id = blockIdx.x;                       // 128-feature block
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int kg = wave >> 2, w4 = wave & 3;         // k-group, wave inside the group (32 features each)
    const int b0 = (int)((long)blockIdx.y * k_tiles / gridDim.y);
    const int b_len = (int)((long)(blockIdx.y + 1) * k_tiles / gridDim.y) - b0;       // the block's k-steps ...
    const int g0 = (int)((long)kg * b_len / KG);
    const int k0 = b0 + g0, k_len = (int)((long)(kg + 1) * b_len / KG) - g0;          // ... and this group's
    const int steps = (b_len + KG - 1) / KG;         // k-steps every wave of the block walks (the longer group's)

    // weights: lane l of k-half kh takes slot (l % 16) + 16 (l / 32) + 32 kh of tile t16 + (l % 32) / 16
    const int t16 = min(id * 8 + w4 * 2 + ((lane & 31) >> 4), n_tiles - 1);
    const h16x8 *wsrc = reinterpret_cast<const h16x8 *>(Wp) + ((size_t)k0 * n_tiles + t16) * 64 + (lane & 15) + 16 * (lane >> 5);
    const size_t wstep = (size_t)n_tiles * 64;
    // activations: wave w of a group copies token tiles w and w + 4 of each k-step (clamped to the last valid tile)
    const h16x8 *xsrc[XW];
#pragma unroll
    for (int i = 0; i < XW; ++i)
        xsrc[i] = reinterpret_cast<const h16x8 *>(Xp) + ((size_t)min(w4 + 4 * i, t_tiles - 1) * k_tiles + k0) * 64 + lane;
    h16x8 *xs = smem + kg * XBUF;
    const int frag = ((lane & 31) >> 4) * 64 + (lane & 15) + 16 * (lane >> 5);

    floatx16 acc[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;

    // Ring slot = one k-step: the wave's two weight operands and its pieces of the activations.  Every request is
    // unconditional (k-steps past the end re-read the last one, an L2 hit, unused), so the compiler counts requests in
    // flight exactly; because loads return in order, a piece of the activations must not be requested later than the
    // weights it is used with, or the wait for it would drain the weight requests behind which it sits.
    h16x8 a[RING][2], xq[RING][XW];
    auto request = [&](int slot, int kt) {
        const int kc = min(kt, k_len - 1);
#pragma unroll
        for (int i = 0; i < XW; ++i) xq[slot][i] = xsrc[i][(size_t)kc * 64];
        const h16x8 *src = wsrc + (size_t)kc * wstep;
        a[slot][0] = __builtin_nontemporal_load(src);
        a[slot][1] = __builtin_nontemporal_load(src + 32);
    };
    auto store_x = [&](int slot, int kt) {
#pragma unroll
        for (int i = 0; i < XW; ++i)
            if (w4 + 4 * i < XT) xs[((kt & 1) * XT + w4 + 4 * i) * 64 + lane] = xq[slot][i];
    };
    auto step = [&](int slot, int kt) {
        if (KG > 1 && kt >= k_len) return;          // the shorter group's last k-step (uniform over the wave)
        const h16x8 *sb = xs + (kt & 1) * XT * 64 + frag;
#pragma unroll
        for (int kh = 0; kh < 2; ++kh)
#pragma unroll
            for (int j = 0; j < NT; ++j)
                acc[j] = hx_mfma32(a[slot][kh], sb[j * 128 + kh * 32], acc[j]);
    };
#pragma unroll
    for (int i = 0; i < RING; ++i) request(i, i);
    store_x(0, 0);
    const int rounds = steps / RING;
    for (int rd = 0; rd < rounds; ++rd) {
#pragma unroll
        for (int i = 0; i < RING; ++i) {
            const int kt = rd * RING + i;
            // k-step kt is complete in LDS; the other buffer (k-step kt - 1) is free; a bare s_barrier behind the LDS
            // stores only: __syncthreads() would also drain the requests in flight
            HX_LDS_BARRIER();
            store_x((i + 1) % RING, kt + 1);
            step(i, kt);
            request(i, kt + RING);
        }
    }
    // fewer than RING k-steps left: k-step rounds * RING + i already sits in slot i
#pragma unroll
    for (int i = 0; i < RING; ++i) {
        const int kt = rounds * RING + i;
        if (kt < steps) {                 // uniform over the block
            HX_LDS_BARRIER();
            store_x((i + 1) % RING, kt + 1);
            step(i, kt);
        }
    }
    // From here on a wave has 32 features and the token blocks j0 .. j0 + FTW - 1 (those from NT on do not exist): all of them, or with two
    // groups one half each, whose sums over both groups meet through the staging buffers -- group 0 + group 1, in that order, every time.
    constexpr int FTW = KG == 2 ? (NT + 1) / 2 : NT;
    const int j0 = kg * FTW;
    floatx16 sum[FTW];
    if constexpr (KG == 2) {
        float *red = reinterpret_cast<float *>(smem);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < NT; ++j)
            if ((j < FTW) == (kg == 1)) {
#pragma unroll
                for (int r = 0; r < 16; ++r) red[((w4 * NT + j) * 16 + r) * 64 + lane] = acc[j][r];
            }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < FTW; ++j) {
            const bool there = j0 + j < NT;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float mine = kg == 0 ? acc[j][r] : FTW + j < NT ? acc[FTW + j < NT ? FTW + j : 0][r] : 0.f;
                sum[j][r] = there ? mine + red[((w4 * NT + j0 + j) * 16 + r) * 64 + lane] : 0.f;
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < FTW; ++j) sum[j] = acc[j];
    }
    const PartGeom pg = part_geom(n_tiles, t_tiles, 0, gridDim.x * 4);
    const int nb = id * 4 + w4, split = blockIdx.y, splits = gridDim.y;
    if constexpr (!OWN) {
        if (T_rows > 0) {                    // row-major sums [split][row][feature] for a consumer that works on whole rows
            const int n0 = nb * 32 + 4 * (lane >> 5), N = n_tiles * 16;
#pragma unroll
            for (int j = 0; j < FTW; ++j) {
                const int row = 32 * (j0 + j) + (lane & 31);
                if (row >= T_rows) continue;
                float *dst = part + ((size_t)split * T_rows + row) * N;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (n0 + 8 * q < N)
                        *reinterpret_cast<floatx4 *>(dst + n0 + 8 * q) = floatx4{sum[j][4 * q], sum[j][4 * q + 1], sum[j][4 * q + 2], sum[j][4 * q + 3]};
            }
            return;
        }
#pragma unroll
        for (int j = 0; j < FTW; ++j)
            if (nb < pg.nb && j0 + j < pg.tb) part_store(part + part_offset(pg, split, nb, j0 + j), sum[j], lane);
    } else {
        constexpr int NTP = 32 * KG * FTW, SH = 256 * KG / NTP;        // token columns of the block's waves
        __shared__ float s_ss[8][NTP];
        __shared__ int s_last;
        if (splits > 1) {
#pragma unroll
            for (int j = 0; j < FTW; ++j)
                if (nb < pg.nb && j0 + j < pg.tb) part_store_dev(part + part_offset(pg, split, nb, j0 + j), sum[j], lane);
        }
        if (e.ssq_in != nullptr) {          // the rows' sums of squares, in the finishing kernel's eight shares, while the stores are on their way
            const int groups = e.norm_dim / GEMM_SSQ_COLS, tok = tid % NTP, token = min(tok, e.T - 1);
            for (int sh = tid / NTP; sh < 8 && tid < SH * NTP; sh += SH) {
                float ss = 0.f;
#pragma unroll 8
                for (int gI = sh; gI < groups; gI += 8) ss += e.ssq_in[(size_t)gI * e.T + token];
                s_ss[sh][tok] = ss;
            }
        }
        if (splits > 1) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // this wave's stores have reached memory ...
            __syncthreads();                                      // ... and every other wave's of the block,
            if (tid == 0) {                                       // before the block counts itself
                s_last = __hip_atomic_fetch_add(&e.arrived[id], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 1u;
            }
            __syncthreads();
            if (!s_last) return;
#pragma unroll
            for (int j = 0; j < FTW; ++j) {
                if (nb >= pg.nb || j0 + j >= pg.tb) continue;
                floatx4 v[4];
                floatx16 tot;
#pragma unroll
                for (int r = 0; r < 16; ++r) tot[r] = 0.f;
                for (int z = 0; z < splits; ++z) {                // in split order
                    if (z != split) part_load_dev(part + part_offset(pg, z, nb, j0 + j), v, lane);
#pragma unroll
                    for (int r = 0; r < 16; ++r) tot[r] += z == split ? sum[j][r] : v[r >> 2][r & 3];
                }
                sum[j] = tot;
            }
        } else {
            __syncthreads();
        }
        auto rstd_of = [&](int tl) {
            float ss = s_ss[0][tl];
#pragma unroll
            for (int w = 1; w < 8; ++w) ss += s_ss[w][tl];
            return 1.0f / sqrtf(ss / (float)e.norm_dim + e.eps);
        };
        GemmEpi g;
        g.ssq_in = e.ssq_in;
        g.u = e.u;
        g.F_l = e.F_l;
        gemm_epilogue<1, FTW, 4, NTP, DEC_SWIGLU>([&](int, int j) { return sum[j]; }, id, 0, w4, 32 * j0, lane, n_tiles * 16, n_tiles, e.T, g, rstd_of);
    }
}

// -------------------------------------------------------------------------------------------------
// 128 features x 128 tokens per block and the whole contraction in it, no partial sums and no finishing pass: for launches that larger
// tiles would leave with few blocks and a split contraction, for short contractions and for short prompts on wide matrices (takes_panel).
// Eight waves of 64 x 64, four on the even and four on the odd k-steps, which takes a third off what 64 x 32 wave tiles read from LDS;
// their sums meet through LDS at the end.  A stage holds two k-steps (32 KB, four stages).  A wave's operands of the next stage are read
// under the MFMAs of this one, so that at its one barrier a stage's buffer is already in registers everywhere and free to be loaded again.
// A k-step is 256 cycles of MFMAs and 256 of LDS reads (32 KB), with 16 KB written to LDS by the loads beside them; it takes 0.14 .. 0.2 us
// (340 .. 480 cycles at 2.4 GHz) on cached operands and 0.16 .. 0.25 in earnest: cache misses cost the difference.
// -------------------------------------------------------------------------------------------------
template <int MODE>
__global__ __launch_bounds__(512) void gemm_panel_kernel(const h16_t *__restrict__ Wp, const h16_t *__restrict__ Xp, int N, int k_tiles,
                                                         int n_tiles, int t_tiles, int T, int n_blocks, int t_blocks, GemmEpi e) {
    constexpr int S = 4, STEP = 16 * 64, STAGE = 2 * STEP;        // h16x8: a k-step holds 8 weight, then 8 activation tiles
    constexpr int NTOK = 128, SSP = 512 / NTOK;
    extern __shared__ h16x8 smem[];                               // [S][2][16][64], then 512 floats
    float *ssq_s = reinterpret_cast<float *>(smem + S * STAGE);
    const int total = n_blocks * t_blocks, per_xcd = (total + 7) / 8, id = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || id >= total) return;
    int bm, bt;
    gemm_tile_of_id(id, n_blocks, t_blocks, 4, min(8, t_blocks), bm, bt);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int grp = wave >> 2, wm = wave & 1, wt = (wave >> 1) & 1;
    const int stages = (k_tiles + 1) >> 1;

    // the sums of squares of the block's token columns, four threads per token (gemm_mfma_kernel)
    if (MODE != DEC_RESID && e.ssq_in != nullptr) {
        const int groups = e.norm_dim / GEMM_SSQ_COLS, token = min(bt * NTOK + tid % NTOK, T - 1);
        float ss = 0.f;
#pragma unroll 16
        for (int gI = tid / NTOK; gI < groups; gI += SSP) ss += e.ssq_in[(size_t)gI * T + token];
        ssq_s[tid] = ss;
        HX_WAIT_VM(0);
    }
    auto rstd_of = [&](int tl) {
        float ss = ssq_s[tl];
#pragma unroll
        for (int w = 1; w < SSP; ++w) ss += ssq_s[w * NTOK + tl];
        return 1.0f / sqrtf(ss / (float)e.norm_dim + e.eps);
    };

    // Wave w copies weight tile w and activation tile w of both k-steps of a stage; k-steps past the end re-read the last one (the odd one of
    // an odd contraction is not multiplied, later stages are not read).
    const h16x8 *asrc = reinterpret_cast<const h16x8 *>(Wp) + (size_t)min(bm * 8 + wave, n_tiles - 1) * 64;
    const h16x8 *bsrc = reinterpret_cast<const h16x8 *>(Xp) + (size_t)min(bt * 8 + wave, t_tiles - 1) * k_tiles * 64;
    const size_t astep = (size_t)n_tiles * 64;
    const unsigned lane_bytes = (unsigned)lane * 16u;
    const unsigned lds0 = hx_lds_addr(smem) + wave * 1024u;
    auto issue = [&](int stage, int x) {            // x: 0, 1 weights, 2, 3 activations of the even and the odd k-step
        const int kt = min(2 * stage + (x & 1), k_tiles - 1);
        const h16x8 *src = x < 2 ? asrc + kt * astep : bsrc + (size_t)kt * 64;
        const unsigned lds = lds0 + (unsigned)(stage % S) * (STAGE * 16u) + (x & 1) * (STEP * 16u) + (x < 2 ? 0u : 8192u);
        hx_load_lds16(lds, lane_bytes, src);
    };
    struct Ops { h16x8 a[4], b[4]; } f0, f1;
    auto fetch = [&](Ops &o, int stage, int x) {    // operand x: four activation tiles, then four weight tiles
        const h16x8 *st = smem + (stage % S) * STAGE + grp * STEP + lane;
        if (x < 4) o.b[x] = st[(8 + wt * 4 + x) * 64];
        else o.a[x - 4] = st[(wm * 4 + x - 4) * 64];
    };
    floatx4 acc0[4][4], acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int p = 0; p < S; ++p)
#pragma unroll
        for (int x = 0; x < 4; ++x) issue(p, x);
    HX_WAIT_VM((S - 1) * 4);
    asm volatile("s_barrier" ::: "memory");
#pragma unroll
    for (int x = 0; x < 8; ++x) fetch(f0, 0, x);
    auto step = [&](int u, Ops &now, Ops &next, bool mult, floatx4 (&acc)[4][4]) {
        HX_WAIT_VM((S - 2) * 4);                     // this wave's loads of stage u + 1 have landed
        HX_LDS_BARRIER();                            // ... and everybody's; stage u is in registers everywhere
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            if (mult) acc[m >> 2][m & 3] = hx_mfma16(now.a[m >> 2], now.b[m & 3], acc[m >> 2][m & 3]);
            if (m % 2 == 0) fetch(next, u + 1, m / 2);
            if (m % 4 == 1) issue(u + S, m / 4);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // From 48 k-tiles on each half of the stages is summed up by itself, so that a chain of additions is a quarter of the contraction, no
    // longer than the splits' that this kernel replaces (16 k-tiles and more).  With one chain per wave group the fp32 sums were up to
    // 1.37 times as far from 64 bits as those (2048 x 2048 at 600 rows 1.53e-7 -> 2.08e-7, now 1.53e-7).  It costs 64 registers and 0.2 us.
    const int full = k_tiles >> 1;                   // stages with two k-steps
    const bool quarters = k_tiles >= 48;
    int u = 0;
    if (quarters) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc0[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
        for (; u + 4 <= full - u; u += 2) {
            step(u, f0, f1, true, acc0);
            step(u + 1, f1, f0, true, acc0);
        }
    }
    for (; u + 2 <= full; u += 2) {
        step(u, f0, f1, true, acc);
        step(u + 1, f1, f0, true, acc);
    }
    if (u < full) {
        step(u, f0, f1, true, acc);
        if (u + 1 < stages) step(u + 1, f1, f0, grp == 0, acc);
    } else if (u < stages) {
        step(u, f0, f1, grp == 0, acc);
    }
    if (quarters) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] += acc0[i][j];
    }
    HX_WAIT_VM(0);
    HX_LDS_BARRIER();

    // The two halves of the contraction meet: waves 0..3 finish the first 32 of a wave tile's 64 token columns, waves 4..7 the others.
    floatx4 *red = reinterpret_cast<floatx4 *>(smem);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            floatx4 v = acc[i][j];
            const floatx4 w = acc[i][2 + j];
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = grp == 0 ? w[r] : v[r];
            red[((wave * 4 + i) * 2 + j) * 64 + lane] = v;
        }
    HX_LDS_BARRIER();
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const floatx4 o = red[(((wave ^ 4) * 4 + i) * 2 + j) * 64 + lane];
            floatx4 v = acc[i][j];
            const floatx4 w = acc[i][2 + j];
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = (grp == 0 ? v[r] : w[r]) + o[r];
            acc[i][j] = v;
        }
    // into the register layout of a 32 x 32 result, as in gemm_mfma_kernel
    auto acc_of = [&](int i, int) {
        floatx16 c;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int src = 16 * (2 * (q & 1) + (lane >> 5)) + (lane & 15);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float v0 = __shfl(acc[2 * i + (q >> 1)][0][r], src, 64);
                const float v1 = __shfl(acc[2 * i + (q >> 1)][1][r], src, 64);
                c[4 * q + r] = (lane & 16) ? v1 : v0;
            }
        }
        return c;
    };
    gemm_epilogue<2, 1, 2, NTOK, MODE>(acc_of, bm, bt, wm, (2 * wt + grp) * 32, lane, N, n_tiles, T, e, rstd_of, ssq_s);
}

// Which launches: one round of 128 x 128 tiles on the 256 CUs, and a contraction of k k-tiles that is short for the number of tiles.
// The alternative has tiles of twice or four times the size, with the contraction split over the CUs that leaves idle: it pays for
// its partial sums and a second launch whatever the contraction's length, and walks it faster.  It also pays for token rows up
// to a multiple of 256 (residual projections: 128), this kernel for those up to a multiple of 16.
// The lines follow what whole calls of 16 widths at 60 row counts take with this kernel and with the other, one projection changed
// at a time and the rest left to this rule (us per projection, this kernel - the other; both in turn in one process.  A kernel trace
// will not do: it puts 2 us and more between the two launches of a split contraction, and favours this kernel by that):
//   tiles   k     rows: difference
//    44-64  48    400 / 600 rows of 1536 -3 / -2;  but k = 64: 200 / 384 rows of 2048 +1.9 / +3.1
//    96     64    272 / 330 / 384 rows -1.5 / -0.9 / +0.4;  but k = 96: 200 / 470 rows +4.1 / +4.6
//   112     88    1792 rows (14 token blocks that share the weights) -3.9;  but 128, k = 112: 256 rows (2 of them) +6.8
//   144     96    272 / 330 / 384 rows -1.5 / -0.9 / +3.3
//   160    108    400 / 464 / 470 / 512 rows -3.3 / -1.2 / +0.2 / +1.9;  but k = 128: 600 / 640 rows +2.0 / +3.9
//   192    256    330 / 464 / 470 / 512 rows -8.4 / -1.8 / +0.2 / +5.8;  k = 176: 1500 rows -2.5;  but k = 256: 1024 rows +4.7
//   256    224    400 / 470 / 512 rows -9.5 / -1.3 / 0;  but k = 256: 512 rows +7.5, k = 448: 400 rows +7
// Every line also leaves out what would add up longer chains (48 and more k-tiles: quarters) than the split contraction does.
// "padded": at least a twentieth of the token blocks' rows do not exist.  600 rows of 640 win, 384 of 384 and 512 of 512 lose.
// Without the residual the other's tiles are 256 tokens wide, and beyond 128 k-tiles it depends on how full the last of them is:
// 224 tiles, k = 256 at 174 / 184 / 200 rows over a multiple of 256 -1.7 / +0.4 / +1.0, 240 tiles at 192 / 208 / 256 -6.9 / -1.2 / +0.1,
// 216, k = 160 at 184 / 208 / 256 -1.6 / +0.6 / +1.6.
// Up to 128 rows the alternative is the skinny kernel with a finishing pass of its own; it needs 32 k-tiles.  Below, this kernel is
// 2 to 7 us shorter than 128 x 128 tiles of four waves at every size.  From there on there have to be enough blocks -- W1/W3 of 88
// tiles, k = 64 at 33 / 64 / 96 / 128 rows -2.0 / -2.0 / -4.6 / -6.9, 216, k = 160 -1.1 / -0.3 / -3.2 / -3.5, but 44, k = 32 +0.9 / +0.6 / 0 / -1.4,
// 128, k = 96 +0.5 / +1.9 / +0.8 / +1.7 -- or the prompt has to be nearly 128 rows (64, k = 48 +0.3 / +0.7 / -0.7 / -2.9) and the skinny kernel
// must not fill the chip, as it does at 128, k = 96.  profiles/prefill_tile_choice.txt has every figure.
static bool takes_panel(bool resid, int n_tiles, int t_tiles, int k_tiles, int T) {
    const int token_blocks = (t_tiles + 7) / 8, tiles = ((n_tiles + 7) / 8) * token_blocks;
    if (t_tiles <= 8) {
        if (k_tiles < 32) return true;
        if (resid || t_tiles <= 2 || tiles > 256) return false;
        const int skinny = tiles * std::min({8, 512 / tiles, k_tiles / 16}) / 2;          // its blocks of eight waves (launch_skinny)
        if (t_tiles > 6 && skinny <= 224) return 3 * tiles >= 4 * k_tiles;
        return tiles >= 64 && k_tiles <= 160 && 20 * tiles >= 27 * k_tiles;
    }
    if (tiles > 256) return false;
    const bool padded = 20 * t_tiles <= 19 * 8 * token_blocks;
    if (tiles <= 128) return k_tiles <= std::max(48, token_blocks >= 9 ? 4 + 3 * tiles / 4 : padded ? 28 + tiles / 2 : tiles / 2);
    if (tiles < 180) return k_tiles <= (padded || tiles >= 168 ? tiles - 36 : tiles - 80);
    if (resid) return k_tiles <= (padded ? 256 : tiles - 16);
    return k_tiles <= 128 || (tiles >= 216 && k_tiles <= 256 && (T - 1) % 256 < (k_tiles <= 192 || tiles >= 232 ? 210 : 176));
}

template <int MODE>
static void launch_panel(const h16_t *Wp, const h16_t *Xp, int N, int k_tiles, int n_tiles, int t_tiles, int T, const GemmEpi &e, hipStream_t s) {
    const int nb = (n_tiles + 7) / 8, tb = (t_tiles + 7) / 8;
    const size_t dyn = (size_t)4 * 32 * 1024 + 512 * sizeof(float);
    auto kern = gemm_panel_kernel<MODE>;
    static bool raised = false;
    if (!raised) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn);
        raised = true;
    }
    hipLaunchKernelGGL(kern, dim3((nb * tb + 7) / 8 * 8), dim3(512), dyn, s, Wp, Xp, N, k_tiles, n_tiles, t_tiles, T, nb, tb, e);
}

// Few tiles, each walking the whole contraction, leave most of the chip idle, and the weights arrive at a fraction of the HBM rate:
// the contraction is then split over blockIdx.y (at most 8 ways, at least 16 k-steps each, partials within the scratch) until the chip
// holds as many blocks as it can (`resident`).
static int tile_splits(long total, int resident, int k_tiles, const PartGeom &pg, const float *part, size_t part_floats) {
    if (part == nullptr || 2 * total > resident || k_tiles < 32) return 1;
    int splits = (int)std::max<long>(1, std::min<long>({8, resident / total, k_tiles / 16}));
    while (splits > 1 && part_offset(pg, splits, 0, 0) > part_floats) --splits;
    return splits;
}

template <int FM, int FT, int WM, int WT, int S, int MODE, bool PP = false, int ABL = 0>
static void launch_cfg(const h16_t *Wp, const h16_t *Xp, int N, int k_tiles, int n_tiles, int t_tiles, int T,
                       const GemmEpi &e, float *part, size_t part_floats, hipStream_t s, int nb0 = 0, int nb_count = -1) {
    constexpr int TA = 2 * FM * WM, TB = 2 * FT * WT;
    // feature blocks nb0 .. nb0 + nb_count - 1 of the matrix (all of them by default)
    const int n_blocks = nb_count >= 0 ? nb_count : (n_tiles + TA - 1) / TA, t_blocks = (t_tiles + TB - 1) / TB;
    const int total = n_blocks * t_blocks;
    const int grid = (total + 7) / 8 * 8;
    auto kern = gemm_mfma_kernel<FM, FT, WM, WT, S, MODE, PP, ABL>;
    const int pm_h = 4, pt_w = 8;         // patch of tiles one XCD works on at a time: 4 feature blocks x 8 token blocks
    const size_t dyn = (size_t)S * (TA + TB) * 64 * sizeof(h16x8) + (size_t)64 * WM * WT * sizeof(float);
    static bool raised = false;           // more than the default 64 KB of LDS per block
    if (!raised) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)dyn);
        raised = true;
    }
    // (by default these are launches of more than 128 rows that takes_panel leaves)
    const PartGeom pg = part_geom(n_tiles, t_tiles, nb0 * FM * WM, n_blocks * FM * WM);
    const int resident = dyn <= 72 * 1024 ? 512 : 256;       // blocks the chip holds at once (LDS: two per CU or one)
    const int splits = tile_splits(total, resident, k_tiles, pg, part, part_floats);
    hipLaunchKernelGGL(kern, dim3(grid, splits), dim3(64 * WM * WT), dyn, s, Wp, Xp, N, k_tiles, n_tiles, t_tiles, T,
                       n_blocks, t_blocks, e, splits > 1 ? part : nullptr, pm_h, std::min(pt_w, t_blocks), nb0);
    if (splits > 1) launch_finish<MODE>(part, splits, N, n_tiles, t_tiles, T, nb0 * FM * WM, n_blocks * FM * WM, e, s);
}

// splits of a launch of 256 features x tt16 token tiles; at most one block per CU of a die (tiles are dealt to the dies in turn)
static int cols_splits(int tt16, int n_tiles, int t_tiles, int k_tiles, const float *part, size_t part_floats) {
    const int n_blocks = (n_tiles + 15) / 16, total = n_blocks * ((t_tiles + tt16 - 1) / tt16);
    const int splits = tile_splits(total, 256, k_tiles, part_geom(n_tiles, t_tiles, 0, n_blocks * 8), part, part_floats);
    return std::min(splits, std::max(1, 32 / ((total + 7) / 8)));
}

template <int TA32, int TB32, int MODE>
static void launch_cols(const h16_t *Wp, const h16_t *Xp, int N, int k_tiles, int n_tiles, int t_tiles, int T, const GemmEpi &e, float *part,
                        size_t part_floats, hipStream_t s) {
    constexpr int TT = 2 * (TA32 + TB32);
    const int n_blocks = (n_tiles + 15) / 16, t_blocks = (t_tiles + TT - 1) / TT, total = n_blocks * t_blocks;
    const size_t dyn = (size_t)4 * (16 + TT) * 1024 + 1024 * sizeof(float);
    auto kern = gemm_cols_kernel<TA32, TB32, MODE>;
    static bool raised = false;
    if (!raised) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn);
        raised = true;
    }
    const int splits = cols_splits(TT, n_tiles, t_tiles, k_tiles, part, part_floats);
    hipLaunchKernelGGL(kern, dim3((total + 7) / 8 * 8, splits), dim3(512), dyn, s, Wp, Xp, N, k_tiles, n_tiles, t_tiles, T, n_blocks, t_blocks, e,
                       splits > 1 ? part : nullptr);
    if (splits > 1) launch_finish<MODE>(part, splits, N, n_tiles, t_tiles, T, 0, n_blocks * 8, e, s);
}

// tile configuration forced for every GEMM launch of the process (0 = choose by shape); a measurement and test hook
static std::atomic<int> g_force_tile{0};
bool set_gemm_tile(int code) {
    for (int ok : {0, 160, 192, 224, 44, 48, 84, 88, 94, 49, 98, 72, 128, 198, 194, 184, 1198, 2198, 3198})
        if (code == ok) { g_force_tile.store(code, std::memory_order_relaxed); return true; }
    return false;
}

// Estimated time in microseconds of one projection with block tiles of tm features x tt tokens (both multiples of 16),
// `step_us` per 32-deep k-step of a block; constants fitted to this chip (TP4-shaped projections at 128 .. 2048 rows):
//   * a block walks its k-steps and pays a fixed 11 us (pipeline fill, epilogue; 15 more when the epilogue is the
//     residual read-modify-write); the chip holds 256 such blocks at once (their LDS fills a CU), and a launch takes
//     whole rounds of them;
//   * launch_cfg splits the contraction when the tiles fill less than half of the chip: the partial sums are written
//     (about 5 TB/s) and a finishing pass reads them back (about 2.5 TB/s) behind a second launch.
static double gemm_estimate_us(int tm, int tt, double step_us, int n_tiles, int t_tiles, int k_tiles, bool resid, bool can_split) {
    const int resident = 256;
    const long total = (long)((n_tiles * 16 + tm - 1) / tm) * ((t_tiles * 16 + tt - 1) / tt);
    int splits = 1;
    if (can_split && 2 * total <= resident && k_tiles >= 32)
        splits = (int)std::max<long>(1, std::min<long>({8, resident / total, k_tiles / 16}));
    const long rounds = (total * splits + resident - 1) / resident;
    const double ksteps = (double)((k_tiles + splits - 1) / splits);
    double us = rounds * (ksteps * step_us + 11.0 + (resid && splits == 1 ? 15.0 : 0.0));
    if (splits > 1) {
        const double part_mb = (double)splits * total * tm * tt * 4.0 / 1e6;
        us += part_mb / 5.0 + 8.0 + part_mb / 2.5 + (resid ? 15.0 : 0.0);
    }
    return us;
}

// Time of one projection with tm x tt tiles in `splits`, for the choice between tiles of 160, 192 and 224 tokens and the ones of 256 (or
// 128) that the estimate above has picked.  Fitted to whole calls of one prompt of 140 .. 5000 rows on layers of the 70B shape (one to
// eight ranks) and of 1024 .. 5120 columns, each projection's tiles changed alone (5300 differences).  A k-step of a 256 x 256 block
// takes 0.65 us when every CU has one and 0.40 when few have, most of it in proportion to the tile: beyond that the power limit sets the
// clock.  Blocks are dealt to the eight dies in turn and 32 CUs each: 84 tiles in three splits are 33 blocks on seven of them, two rounds.
static double tile_us(int mode, int tm, int tt, int splits, int n_tiles, int t_tiles, int k_tiles) {
    const int total = (int)((long)((n_tiles * 16 + tm - 1) / tm) * ((t_tiles * 16 + tt - 1) / tt));
    const long blocks = (long)((total + 7) / 8) * 8 * splits, full = blocks / 256, rem = blocks % 256;
    const double area = tm * tt / 65536.0, ks = (double)k_tiles / splits;
    double us = full * (ks * (0.155 + 0.49 * area) + 5.7);
    if (rem > 0) us += ks * (0.155 + area * (0.24 + 0.25 * rem / 256.0)) + 5.7;
    // what the epilogue adds: the residual stream's values, scattered cache rows
    if (splits == 1) return us + (mode == DEC_RESID ? 3.4 * area * (full + (rem > 0)) : mode == DEC_QKV ? 10.0 * blocks / 256.0 : 0.0);
    return us + splits * (double)n_tiles * t_tiles * 1024.0 / 1e6 * 0.40;          // MB of partial sums, written and read
}

// one 128-token tile, at least 32 k-tiles: skinny kernel + finishing pass; returns false when it does not apply
template <int MODE>
static bool launch_skinny(const h16_t *Wp, const h16_t *Xp, int N, int k_tiles, int n_tiles, int t_tiles, int T,
                          const GemmEpi &e, float *part, size_t part_floats, hipStream_t s, QkvTail *tail = nullptr) {
    if (part == nullptr || t_tiles > 8 || k_tiles < 32) return false;
    const int n_blocks = (n_tiles + 7) / 8;
    const PartGeom pg = part_geom(n_tiles, t_tiles, 0, n_blocks * 4);
    // two blocks fit a CU (registers): about 512 blocks in flight, at most 8 splits of at least 16 k-steps
    int splits = std::max(1, std::min({8, 512 / n_blocks, k_tiles / 16}));
    while (splits > 1 && part_offset(pg, splits, 0, 0) > part_floats) --splits;
    if (part_offset(pg, splits, 0, 0) > part_floats) return false;
    // An even number of splits over enough blocks runs as half as many splits of 8-wave blocks, the pairs of splits summed
    // inside the block: half the partial sums written, and read by the finishing pass.  Measured on the TP4 shard of the
    // 70B shape at 128 rows: W1/W3 (112 blocks x 4 -> x 2) 64.8 -> 59.4 us, W2 (64 x 8 -> x 4) 43.0 -> 38.5, 158.9 -> 149.8 us
    // per layer; with fewer than 160 blocks left the CUs that stay empty cost more (W_O 64 x 4 -> x 2: 22.1 -> 25.9,
    // QKV 20 x 8 -> x 4: 25.6 -> 32.4), and 8-wave blocks at an unchanged number of splits gain nothing there either.
    const bool pair = splits % 2 == 0 && n_blocks * (splits / 2) >= 160;
    if (pair) splits /= 2;
    // W1/W3 finishes its own tiles up to two splits: a finishing launch is 8 to 10 us of a call.  Whole calls: TP1 (one split) 90 / 33 rows 398 / 351
    // -> 377 / 339 us, 50 decoding sequences 1402 -> 1332; TP2 (one) 60 rows 410 -> 399; TP4 (two; of three layers and of eight steps, least of three processes
    // each) 40 / 60 / 90 / 117 rows 372 / 384 / 424 / 450 -> 363 / 373 / 416 / 445, 40 / 60 / 120 sequences 2710 / 2826 / 3428 -> 2631 / 2749 / 3385, 90 ragged ones
    // 3354 -> 3281.  With four splits (W_O, W2) and eight (QKV) the last blocks, a quarter and less of the CUs, take 2.5 and 10 us longer than the launch.
    const bool own = MODE == DEC_SWIGLU && splits <= 2 && tail == nullptr && (splits == 1 || e.arrived != nullptr);
    const SkinnyOwn oe{e.ssq_in, e.norm_dim, T, e.F_l, e.eps, e.u, e.arrived};
    auto run = [&](auto kern, int kg) {
        hipLaunchKernelGGL(kern, dim3(n_blocks, splits), dim3(256 * kg), 0, s, Wp, Xp, k_tiles, n_tiles, t_tiles, part, tail != nullptr ? T : 0, oe);
    };
#define HX_SK(KG, NT)                                                                   \
    do {                                                                                \
        if constexpr (MODE == DEC_SWIGLU) {                                             \
            if (own) { run(gemm_skinny_kernel<KG, NT, true>, KG); break; }              \
        }                                                                               \
        run(gemm_skinny_kernel<KG, NT, false>, KG);                                     \
    } while (0)
    switch ((t_tiles + 1) / 2) {
        case 1: if (pair) HX_SK(2, 1); else HX_SK(1, 1); break;
        case 2: if (pair) HX_SK(2, 2); else HX_SK(1, 2); break;
        case 3: if (pair) HX_SK(2, 3); else HX_SK(1, 3); break;
        default: if (pair) HX_SK(2, 4); else HX_SK(1, 4); break;
    }
#undef HX_SK
    if (own) return true;
    if (tail != nullptr) *tail = QkvTail{part, splits, T, N, nullptr, e.cos_tab, e.sin_tab, e.ssq_in, e.norm_dim, e.eps};
    else launch_finish<MODE>(part, splits, N, n_tiles, t_tiles, T, 0, n_blocks * 4, e, s);
    return true;
}

// Tiles of 256 features x 160, 192 or 224 tokens (gemm_cols_kernel) in place of `cfg`, 198 (nA > 0: in two launches) or 194?  Rows are
// then paid for up to fewer than 256, and the number of tiles fits the CUs more often.  Whole calls of one prompt: TP1 shard of the 70B
// shape (one layer) at 285 / 437 / 604 rows 714 / 757 / 1102 -> 606 / 732 / 1004 us, TP2 (two) at 328 / 430 / 600 792 / 855 / 1239 -> 710 / 812 /
// 1194, TP4 (three) at 274 / 570 / 737 667 / 1046 / 1135 -> 643 / 931 / 1054, 3072-wide (three) at 312 / 449 / 1087 569 / 579 / 1026 -> 496 / 546 / 944.
// At 470 .. 512, 900 .. 1024 and 2048 rows 256 is the better tile (TP2's W1/W3 at 470 rows +112 us in tiles of 224, +85 in 192) and stays.
//   * At least 4 us and 2 % by the estimate, whose error is of that size; up to 256 rows nothing is that much better.
//   * No chain of additions gets longer: at least as many splits as the launch had (two launches: its second one).
template <int MODE>
static int token_tile(int cfg, int nA, int n_tiles, int t_tiles, int k_tiles, const float *part, size_t part_floats) {
    constexpr bool resid = MODE == DEC_RESID;
    const int tm = cfg == 198 || resid ? 256 : 128, tt = cfg == 198 || !resid ? 256 : 128;
    const int n = n_tiles - 16 * nA, blocks = (n * 16 + tm - 1) / tm;
    const int now = tile_splits((long)blocks * ((t_tiles * 16 + tt - 1) / tt), 256, k_tiles, part_geom(n, t_tiles, 0, blocks * (tm / 32)), part, part_floats);
    double best = tile_us(MODE, tm, tt, now, n, t_tiles, k_tiles);
    if (nA > 0) best += tile_us(MODE, tm, tt, 1, 16 * nA, t_tiles, k_tiles);
    best = 0.98 * best - 4.0;
    for (int t : {160, 192, 224}) {
        const int sp = cols_splits(t / 16, n_tiles, t_tiles, k_tiles, part, part_floats);
        if (sp < now) continue;
        const double us = tile_us(MODE, 256, t, sp, n_tiles, t_tiles, k_tiles);
        if (us < best) { best = us; cfg = t; }
    }
    return cfg;
}

template <int MODE>
static void launch_mode(const h16_t *Wp, const h16_t *Xp, int N, int K, int T, const GemmEpi &e, float *part,
                        size_t part_floats, hipStream_t s) {
    const int k_tiles = K / 32, n_tiles = N / 16, t_tiles = (T + 15) / 16;
    const int force = g_force_tile.load(std::memory_order_relaxed);
    // 198 = 256 x 256 on 8 waves with the two waves of a SIMD half a k-step out of phase; the smaller tile, on the same
    // loop, is 128 x 256 (194), or 256 x 128 (184) for the residual epilogue.  Which one: the shorter of two estimates
    // (gemm_estimate_us), i.e. rounds of blocks over the chip x a block's time, plus what a split contraction costs in
    // partial sums.
    const bool resid = MODE == DEC_RESID;
    const double t198 = gemm_estimate_us(256, 256, 0.55, n_tiles, t_tiles, k_tiles, resid, part != nullptr);
    const double tsml = gemm_estimate_us(resid ? 256 : 128, resid ? 128 : 256, 0.37, n_tiles, t_tiles, k_tiles, resid, part != nullptr);
    int cfg = t198 <= tsml ? 198 : 194;
    if (force) cfg = force;
    if (cfg == 128 || (!force && takes_panel(resid, n_tiles, t_tiles, k_tiles, T))) {
        launch_panel<MODE>(Wp, Xp, N, k_tiles, n_tiles, t_tiles, T, e, s);
        return;
    }
    // A launch of `total` 256 x 256 tiles, a few more than a multiple of the 256 that the chip holds, would run its last round nearly
    // empty (1280 rows x 14336 features: 280 tiles, two rounds for 1.09 rounds of work).  Then the feature blocks whose tiles fill
    // whole rounds go first (nA of them), and the few that remain follow as a launch of their own, which launch_cfg splits along the
    // contraction so that it fills the chip as well.
    const int nb = (n_tiles + 15) / 16, tb = (t_tiles + 15) / 16, total = nb * tb, rem = total % 256;
    int nA = (total - rem) / tb;
    if (force || cfg != 198 || total <= 256 || rem == 0 || rem > 128 || part == nullptr || k_tiles < 32 || nA < 1 || nA >= nb ||
        gemm_estimate_us(256, 256, 0.55, nA * 16, t_tiles, k_tiles, resid, true) +
                gemm_estimate_us(256, 256, 0.55, (nb - nA) * 16, t_tiles, k_tiles, resid, true) >= t198)
        nA = 0;
    if (!force && t_tiles > 16) cfg = token_tile<MODE>(cfg, nA, n_tiles, t_tiles, k_tiles, part, part_floats);
#define HX_COLS(A, B) launch_cols<A, B, MODE>(Wp, Xp, N, k_tiles, n_tiles, t_tiles, T, e, part, part_floats, s)
    if (cfg == 224) { HX_COLS(4, 3); return; }
    if (cfg == 192) { HX_COLS(3, 3); return; }
    if (cfg == 160) { HX_COLS(3, 2); return; }
#undef HX_COLS
    // the RESID epilogue emits one sum-of-squares partial per wave: its 32 FM features must be 128
    if (MODE == DEC_RESID && cfg != 88 && cfg != 84 && cfg != 184 && cfg != 98 && cfg % 1000 != 198) cfg = cfg == 72 ? 198 : (cfg == 194 ? 184 : 84);
    if (!force && t_tiles <= 8 && launch_skinny<MODE>(Wp, Xp, N, k_tiles, n_tiles, t_tiles, T, e, part, part_floats, s)) return;
#define HX_G(FM, FT, WM, WT, S) launch_cfg<FM, FT, WM, WT, S, MODE>(Wp, Xp, N, k_tiles, n_tiles, t_tiles, T, e, part, part_floats, s)
    if (cfg == 88) HX_G(4, 4, 2, 2, 4);
    else if (cfg == 98) HX_G(4, 2, 2, 4, 4);
    else if (cfg == 198) {
        if (nA > 0) {
            launch_cfg<4, 2, 2, 4, 4, MODE, true>(Wp, Xp, N, k_tiles, n_tiles, t_tiles, T, e, part, part_floats, s, 0, nA);
            launch_cfg<4, 2, 2, 4, 4, MODE, true>(Wp, Xp, N, k_tiles, n_tiles, t_tiles, T, e, part, part_floats, s, nA, nb - nA);
        } else {
            launch_cfg<4, 2, 2, 4, 4, MODE, true>(Wp, Xp, N, k_tiles, n_tiles, t_tiles, T, e, part, part_floats, s);
        }
    }
    else if (cfg == 1198) launch_cfg<4, 2, 2, 4, 4, MODE, true, 1>(Wp, Xp, N, k_tiles, n_tiles, t_tiles, T, e, part, part_floats, s);
    else if (cfg == 2198) launch_cfg<4, 2, 2, 4, 4, MODE, true, 2>(Wp, Xp, N, k_tiles, n_tiles, t_tiles, T, e, part, part_floats, s);
    else if (cfg == 3198) launch_cfg<4, 2, 2, 4, 4, MODE, true, 3>(Wp, Xp, N, k_tiles, n_tiles, t_tiles, T, e, part, part_floats, s);
    else if (cfg == 194) { if constexpr (MODE != DEC_RESID) launch_cfg<2, 2, 2, 4, 4, MODE, true>(Wp, Xp, N, k_tiles, n_tiles, t_tiles, T, e, part, part_floats, s); }
    else if (cfg == 184) launch_cfg<4, 1, 2, 4, 4, MODE, true>(Wp, Xp, N, k_tiles, n_tiles, t_tiles, T, e, part, part_floats, s);
    else if (cfg == 94) { if constexpr (MODE != DEC_RESID) HX_G(2, 2, 2, 4, 4); }
    else if (cfg == 49) { if constexpr (MODE != DEC_RESID) HX_G(2, 2, 4, 2, 4); }
    else if (cfg == 84) HX_G(4, 2, 2, 2, 4);
    else if (cfg == 72) { if constexpr (MODE != DEC_RESID) HX_G(7, 2, 2, 2, 4); }
    else if (cfg == 48) {
        if constexpr (MODE != DEC_RESID) HX_G(2, 4, 2, 2, 4);
    } else {
        if constexpr (MODE != DEC_RESID) HX_G(2, 2, 2, 2, 4);
    }
#undef HX_G
}

void launch_gemm_mfma(const h16_t *Wp, const h16_t *Xp, int N, int K, int T, const GemmEpi &e, float *part,
                      size_t part_floats, hipStream_t s) {
    switch (e.mode) {
        case DEC_RAW: launch_mode<DEC_RAW>(Wp, Xp, N, K, T, e, part, part_floats, s); break;
        case DEC_QKV: launch_mode<DEC_QKV>(Wp, Xp, N, K, T, e, part, part_floats, s); break;
        case DEC_RESID: launch_mode<DEC_RESID>(Wp, Xp, N, K, T, e, part, part_floats, s); break;
        case DEC_SWIGLU: launch_mode<DEC_SWIGLU>(Wp, Xp, N, K, T, e, part, part_floats, s); break;
    }
}

// A row's finishing pass -- its heads' sums over the splits, rotary embedding, cache append -- is a few KB that the attention
// block of the same (sequence, kv head) reads while its first K / V tiles are on their way: one launch and one trip of q
// through memory less.  It lengthens every block by about 3 us, so it is left to the attention only up to two blocks per CU (at
// head dim 64 both run at once, at 128 one after the other: 176 registers).  Measured per layer at 33 / 64 / 100 / 128 rows, 600 positions, without -> with: TP8 shard of
// the 70B shape 90.6 / 92.7 / 108.4 / 111.7 -> 86.2 / 89.8 / 106.1 / 109.8 us, TP4 119.4 / 123.5 / 144.4 / 152.2 -> 115.0 /
// 120.6 / 141.6 / 149.3; 8 kv heads of a 4096-wide model 126.5 / 143.5 / 185.5 / 197.5 -> 124.2 / 142.5 / 189.6 / 199.8, of a
// 2048-wide one 69.5 / 77.5 / 98.6 / 104.3 -> 68.5 / 76.8 / 102.9 / 107.3 (64-wide heads, since then two blocks on a CU: at 40 / 60 rows
// 68.2 / 72.6 -> 64.8 / 69.3): beyond 512 blocks it loses.
void launch_gemm_qkv_rows(const h16_t *Wp, const h16_t *Xp, int N, int K, int T, const GemmEpi &e, float *part,
                          size_t part_floats, QkvTail *tail, hipStream_t s) {
    *tail = QkvTail{};
    if (T * e.kg.hkv_l <= 512 && e.ssq_in != nullptr && g_force_tile.load(std::memory_order_relaxed) == 0 &&
        launch_skinny<DEC_QKV>(Wp, Xp, N, K / 32, N / 16, (T + 15) / 16, T, e, part, part_floats, s, tail))
        return;
    launch_gemm_mfma(Wp, Xp, N, K, T, e, part, part_floats, s);
}

// -------------------------------------------------------------------------------------------------
// Prefill prologue: stage input rows (bf16, or fp32 for the validation surface) -> fp32 residual stream in its
// tiled order, (x * gain) in fragment tiles, sums of squares per 128-column group.  A block owns 32 tokens x 128 columns, each
// of its four waves one 32 x 32 block of them in the lane layout of the MFMA result (lane = token % 32 + 32 * half, four
// consecutive features per lane and quad): every store of the residual stream is one contiguous 1 KB, every store of the
// operand two runs of 256 B, and the 64-byte row pieces it reads are fetched once.  Bound by memory on long batches, by the
// round trip on short ones: a wave has all its requests out at once (one wave per 128 columns went through them in turn:
// 117 rows of 8192 9.7 -> 4.9 us, 2048 rows 38.4 -> 32.3).
// lens != NULL (one new row per sequence): the first block publishes the rows' sequences and positions from the committed
// lengths and, when asked, advances the lengths.
// -------------------------------------------------------------------------------------------------
template <bool IN_H16>
__global__ __launch_bounds__(256) void prefill_prologue_kernel(const void *__restrict__ in, float *__restrict__ h_out,
                                                              const float *__restrict__ g, h16_t *__restrict__ hg,
                                                              float *__restrict__ ssq_out, int T, int H, int32_t *lens,
                                                              int32_t *row_seq, int32_t *row_pos, int advance) {
    __shared__ float s_ss[4][32];
    if (lens != nullptr && blockIdx.x == 0 && blockIdx.y == 0)
        for (int t = threadIdx.x; t < T; t += 256) {
            const int l = lens[t];
            row_seq[t] = t;
            row_pos[t] = l;
            if (advance) lens[t] = l + 1;
        }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int token = blockIdx.x * 32 + (lane & 31), hl = lane >> 5;
    const int n0 = blockIdx.y * GEMM_SSQ_COLS + wave * 32 + 4 * hl;
    const bool tv = token < T;
    float x[4][4];
    float4 g4[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const size_t at = (size_t)min(token, T - 1) * H + n0 + 8 * q;
        if (IN_H16) {
            const uint2 raw = *reinterpret_cast<const uint2 *>(reinterpret_cast<const h16_t *>(in) + at);
            h16x2_to_f32(raw.x, x[q][0], x[q][1]);
            h16x2_to_f32(raw.y, x[q][2], x[q][3]);
        } else {
            const float4 v = *reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(in) + at);
            x[q][0] = v.x; x[q][1] = v.y; x[q][2] = v.z; x[q][3] = v.w;
        }
        g4[q] = *reinterpret_cast<const float4 *>(g + n0 + 8 * q);
    }
    float ss = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int n = n0 + 8 * q;
        if (tv) {
            if (h_out) *reinterpret_cast<float4 *>(h_out + h_tile_offset(token, n, H)) = make_float4(x[q][0], x[q][1], x[q][2], x[q][3]);
            uint2 o;
            o.x = pack_h16x2(x[q][0] * g4[q].x, x[q][1] * g4[q].y);
            o.y = pack_h16x2(x[q][2] * g4[q].z, x[q][3] * g4[q].w);
            *reinterpret_cast<uint2 *>(hg + frag_offset(token, n, H >> 5)) = o;
        }
        ss += x[q][0] * x[q][0] + x[q][1] * x[q][1] + x[q][2] * x[q][2] + x[q][3] * x[q][3];
    }
    ss += __shfl_xor(ss, 32, 64);
    if (hl == 0) s_ss[wave][lane] = ss;
    __syncthreads();
    if (threadIdx.x < 32 && tv)
        ssq_out[(size_t)blockIdx.y * T + token] = s_ss[0][lane] + s_ss[1][lane] + s_ss[2][lane] + s_ss[3][lane];
}

void launch_prefill_prologue(const void *in, int in_is_h16, float *h_out, const float *g, h16_t *hg, float *ssq_out,
                             int T, int H, int32_t *lens, int32_t *row_seq, int32_t *row_pos, int advance, hipStream_t s) {
    if (T <= 0) return;
    const dim3 grid((T + 31) / 32, H / GEMM_SSQ_COLS);
    if (in_is_h16)
        hipLaunchKernelGGL(prefill_prologue_kernel<true>, grid, dim3(256), 0, s, in, h_out, g, hg, ssq_out, T, H, lens, row_seq, row_pos, advance);
    else
        hipLaunchKernelGGL(prefill_prologue_kernel<false>, grid, dim3(256), 0, s, in, h_out, g, hg, ssq_out, T, H, lens, row_seq, row_pos, advance);
}

// tiled residual stream -> row-major fp32 (debug taps)
__global__ void untile_h_kernel(const float *__restrict__ h_tiled, float *__restrict__ out, int T, int H) {
    const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
    if (i >= (int64_t)T * H) return;
    const int t = (int)(i / H), n = (int)(i % H);
    *reinterpret_cast<float4 *>(out + i) = *reinterpret_cast<const float4 *>(h_tiled + h_tile_offset(t, n, H));
}
void launch_untile_h(const float *h_tiled, float *out, int T, int H, hipStream_t s) {
    const int64_t n4 = (int64_t)T * H / 4;
    if (n4 <= 0) return;
    hipLaunchKernelGGL(untile_h_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s, h_tiled, out, T, H);
}

}  // namespace HX_NS
