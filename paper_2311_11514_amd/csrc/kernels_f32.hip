// fp32 stage path: plain row-major layouts, every product on the fp32 matrix instructions (each multiply-add is an fp32
// fused multiply-add, so operands, products and sums keep full precision).
//   * up to 32 rows: f32_stream_kernel -- a block streams the weights of 16 or 32 output columns over the whole
//     contraction and finishes them in registers (norm, residual, SwiGLU): five launches per layer in a decode step;
//   * more rows: f32_tile_kernel -- 64 x 128 tiles through LDS, their k-steps dealt out evenly over the CUs;
//   * attention: f32_attn_kernel -- 16 query columns (rows of one head, or the heads of one kv group) against the cache.
// Weight rows are padded with zeros to a multiple of 32 and matrix widths to a multiple of 16 (stage.hip), so no loop here
// has a ragged end in either direction.
#include <algorithm>

#include "kernels.h"

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
typedef float floatx2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ floatx4 f32_mfma16(float a, float b, floatx4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ floatx16 f32_mfma32(float a, float b, floatx16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ float f32_silu_mul(float a, float b) { return a / (1.0f + expf(-a)) * b; }

__global__ __launch_bounds__(256) void f32_rmsnorm_kernel(const float *__restrict__ in, const float *__restrict__ g,
                                                         float *__restrict__ out, int H, float eps) {
    __shared__ float red[4];
    constexpr int R = 4;                       // 16-byte pieces a thread keeps: rows of up to 4096 are read once
    const size_t row = (size_t)blockIdx.x * H;
    floatx4 x[R], gv[R];
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int c = min(4 * ((int)threadIdx.x + 256 * i), H - 4);
        x[i] = *reinterpret_cast<const floatx4 *>(in + row + c);
        gv[i] = *reinterpret_cast<const floatx4 *>(g + c);
    }
#pragma unroll
    for (int i = 0; i < R; ++i)
        if (4 * ((int)threadIdx.x + 256 * i) < H) ss += x[i][0] * x[i][0] + x[i][1] * x[i][1] + x[i][2] * x[i][2] + x[i][3] * x[i][3];
    for (int c = threadIdx.x + 1024 * R; c < H; c += 256) ss += in[row + c] * in[row + c];
    ss = block_sum_256(ss, red);
    const float rstd = 1.0f / sqrtf(ss / (float)H + eps);
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int c = 4 * ((int)threadIdx.x + 256 * i);
        if (c < H) *reinterpret_cast<floatx4 *>(out + row + c) = x[i] * rstd * gv[i];
    }
    for (int c = threadIdx.x + 1024 * R; c < H; c += 256) out[row + c] = in[row + c] * rstd * g[c];
}
void f32_launch_rmsnorm(const float *in, const float *g, float *out, int T, int H, float eps, hipStream_t s) {
    if (T <= 0) return;
    hipLaunchKernelGGL(f32_rmsnorm_kernel, dim3(T), dim3(256), 0, s, in, g, out, H, eps);
}

// -------------------------------------------------------------------------------------------------
// T <= 32 rows.  A block of 8 waves owns 16 V output columns (for SwiGLU: 16 V gate columns and the 16 V up columns that
// belong to them) over the whole contraction; the waves interleave over chunks of 16 weight rows and are summed through
// LDS in wave order.  v_mfma_f32_16x16x4_f32: operand A = 16 columns x 4 weight rows, B = 16 token rows x 4.  Which column
// is which row of A, and which weight row which k-slot, is free as long as A and B (and the epilogue) agree:
//   * lane l loads V neighbouring columns V (l % 16) .. of weight row 16 c + 4 (l / 16) + x in one request (four rows of
//     64 V bytes), one register of it per MFMA: column n0 + V i + j is row i of MFMA j;
//   * the lane's token row contributes x[t][16 c + 4 (l / 16) + 0 .. 3] in one 16-byte request, one value per x.
// 32 MFMA cycles per 256 bytes of weights and wave leave the kernel bound by memory up to two token tiles, and by latency
// (launch, one round trip, the reduction) on small matrices; the ring of four chunks covers a contraction of 512 at once.
// RMSNorm costs nothing extra: the block reads every element of its rows anyway, so it sums their squares on the way,
// multiplies by the gain at the operand and by 1 / rms after the contraction.
// V = 2 (128-byte pieces) where that leaves 128 blocks or more, else V = 1: twice the blocks.
// Measured, tiny stage (hidden 512, TP2): a projection of one row 55 -> 4 us (before: a vector-ALU tile kernel, 12 .. 22
// blocks walking the contraction 16 rows at a time), a decode step of two layers with its head 28 -> 12 launches, prefill of
// 32 rows and eight such steps 5030 -> 615 us.
// -------------------------------------------------------------------------------------------------
template <int MODE, int NB, int V, bool NORM, bool ADD>
__global__ __launch_bounds__(512) void f32_stream_kernel(F32Proj p) {
    constexpr int W = 8, U = 4, NM = MODE == F32_SWIGLU ? 2 : 1;
    static_assert(NM * V * NB <= 4, "32 KB of LDS for the sums over the waves");
    typedef float vec __attribute__((ext_vector_type(V == 1 ? 2 : V)));       // V = 1 uses element 0
    __shared__ floatx4 red[W][NM * V * NB][64];
    __shared__ float s_ss[W][NB * 16];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    const int n0 = blockIdx.x * 16 * V;
    const int col = min(n0 + V * i, p.cols - V);           // columns past the last one re-read it and are not stored
    const int chunks = p.Kp >> 4;
    const bool finisher = wave < NB;

    // the finishing wave of token tile `wave` asks for the residual now, so that it does not wait for it at the end
    floatx4 res[V];
    if (MODE == F32_RESID && finisher) {
#pragma unroll
        for (int q = 0; q < V; ++q)
            res[q] = *reinterpret_cast<const floatx4 *>(p.resid + (size_t)min(i + 16 * wave, p.T - 1) * p.N + min(n0 + 4 * V * g + 4 * q, p.cols - 4));
    }
    const float *xr[NB], *x2r[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const size_t row = (size_t)min(i + 16 * b, p.T - 1) * p.K;
        xr[b] = p.x + row;
        x2r[b] = ADD ? p.x2 + row : nullptr;
    }
    vec wv[U][NM][4];
    floatx4 xv[U][NB], x2v[U][ADD ? NB : 1], gv[U];
    auto request = [&](int u, int c) {
        const int k = 16 * c + 4 * g, kx = min(k, p.K - 4);          // K is a multiple of 4; weight rows K .. Kp - 1 are zero
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            xv[u][b] = *reinterpret_cast<const floatx4 *>(xr[b] + kx);
            if (ADD) x2v[u][b] = *reinterpret_cast<const floatx4 *>(x2r[b] + kx);
        }
        if (NORM) gv[u] = *reinterpret_cast<const floatx4 *>(p.g + kx);
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const float *src = p.w + (size_t)(k + x) * p.N + (m ? p.cols : 0) + col;
                if constexpr (V == 1) wv[u][m][x][0] = *src;
                else wv[u][m][x] = *reinterpret_cast<const vec *>(src);
            }
    };
    floatx4 acc[NM][V][NB];
    float ss[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        ss[b] = 0.f;
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int j = 0; j < V; ++j) acc[m][j][b] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    auto contract = [&](int u, int c) {
        const bool in = 16 * c + 4 * g < p.K;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            floatx4 x = xv[u][b];
            if (ADD) x += x2v[u][b];
            if (!in) x = floatx4{0.f, 0.f, 0.f, 0.f};
            if (NORM) {
                ss[b] += x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + x[3] * x[3];
                x *= gv[u];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int m = 0; m < NM; ++m)
#pragma unroll
                    for (int j = 0; j < V; ++j) acc[m][j][b] = f32_mfma16(wv[u][m][q][j], x[q], acc[m][j][b]);
        }
    };
#pragma unroll
    for (int u = 0; u < U; ++u) request(u, min(wave + u * W, chunks - 1));
    for (int c0 = wave; c0 < chunks; c0 += U * W)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = c0 + u * W;
            if (c < chunks) {                                        // uniform over the wave
                contract(u, c);
                request(u, min(c + U * W, chunks - 1));
            }
        }
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
        for (int j = 0; j < V; ++j)
#pragma unroll
            for (int b = 0; b < NB; ++b) red[wave][(m * V + j) * NB + b][lane] = acc[m][j][b];
    if (NORM) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            ss[b] += __shfl_xor(ss[b], 16, 64);
            ss[b] += __shfl_xor(ss[b], 32, 64);
            if (g == 0) s_ss[wave][b * 16 + i] = ss[b];
        }
    }
    __syncthreads();
    // every attention of the call has read the lengths: the step that was asked to advance them does so here
    if (p.lens != nullptr && blockIdx.x == 0 && (int)threadIdx.x < p.T) p.lens[threadIdx.x] += 1;
    if (!finisher) return;
    const int b = wave, t = i + 16 * b;
    floatx4 v[NM][V];
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
        for (int j = 0; j < V; ++j) {
            v[m][j] = red[0][(m * V + j) * NB + b][lane];
#pragma unroll
            for (int w = 1; w < W; ++w) v[m][j] += red[w][(m * V + j) * NB + b][lane];
        }
    if (NORM) {
        float tot = s_ss[0][t];
#pragma unroll
        for (int w = 1; w < W; ++w) tot += s_ss[w][t];
        const float r = 1.0f / sqrtf(tot / (float)p.K + p.eps);
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int j = 0; j < V; ++j) v[m][j] *= r;
    }
    if (t >= p.T) return;
    // lane: columns n0 + 4 V g .. + 4 V - 1, column 4 q + r of them in register (4 q + r) / V of v[(4 q + r) % V]
#pragma unroll
    for (int q = 0; q < V; ++q) {
        const int n = n0 + 4 * V * g + 4 * q;
        if (n >= p.cols) continue;
        floatx4 o;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float a = v[0][(4 * q + r) % V][(4 * q + r) / V];
            o[r] = MODE == F32_SWIGLU ? f32_silu_mul(a, v[NM - 1][(4 * q + r) % V][(4 * q + r) / V]) : a;
        }
        if (MODE == F32_RESID && p.resid_out == nullptr) {           // the stage's last projection: partial and residual apart
            *reinterpret_cast<floatx4 *>(p.out + (size_t)t * p.cols + n) = o;
            if (p.out_resid) *reinterpret_cast<floatx4 *>(p.out_resid + (size_t)t * p.cols + n) = res[q];
        } else if (MODE == F32_RESID) {
            *reinterpret_cast<floatx4 *>(p.resid_out + (size_t)t * p.cols + n) = res[q] + o;
        } else {
            *reinterpret_cast<floatx4 *>(p.out + (size_t)t * p.cols + n) = o;
        }
    }
}

// What leaves a tile or the sum of the splits: four consecutive columns n .. n + 3 of row t (for SwiGLU: a = gate, b = up)
// h: the residual at the same place (F32_RESID)
template <int MODE>
__device__ __forceinline__ void f32_finish4(const F32Proj &p, int t, int n, floatx4 a, floatx4 b, floatx4 h) {
    const size_t o = (size_t)t * p.cols + n;
    if (MODE == F32_SWIGLU) {
#pragma unroll
        for (int r = 0; r < 4; ++r) a[r] = f32_silu_mul(a[r], b[r]);
        *reinterpret_cast<floatx4 *>(p.out + o) = a;
    } else if (MODE == F32_RESID) {
        if (p.resid_out) {
            *reinterpret_cast<floatx4 *>(p.resid_out + o) = h + a;
        } else {
            *reinterpret_cast<floatx4 *>(p.out + o) = a;
            if (p.out_resid) *reinterpret_cast<floatx4 *>(p.out_resid + o) = h;
        }
    } else {
        *reinterpret_cast<floatx4 *>(p.out + o) = a;
    }
}

// -------------------------------------------------------------------------------------------------
// T > 32 rows: tiles of 64 rows x 128 columns (SwiGLU: 64 gate columns and their 64 up columns), one block of 8 waves per CU,
// a wave 32 rows x 32 columns on v_mfma_f32_32x32x2_f32 (operand A = columns, so that a lane ends up with neighbouring
// columns of one row).  A 32-deep k-step is 32 MFMAs of 64 cycles on every SIMD: bound by the matrix cores, as long as
//   * operands come in time: direct-to-LDS loads, four stages resident, three k-steps ahead of their use (with one step ahead, in
//     registers, memory latency showed in every step);
//   * LDS latency and barriers stay behind MFMAs: the operands of 8 rows are fetched while the 8 rows before them are multiplied,
//     and the step's one barrier sits in its middle, so that the next step's first operands are fetched before this one ends;
//   * every CU has about the same number of k-steps: the blocks are persistent.  The columns of tiles that fill whole rounds of
//     256 are walked as whole tiles; of the columns that are left, every token block's k-steps are dealt out evenly to as many
//     blocks -- partial sums, which f32_tile_finish_kernel adds up.  792 tiles as blocks of their own gave the fullest CU
//     four tiles where 3.1 is the average.
// All rows of a launch see a column's contraction cut at the same places, so that equal prompts and sequences have equal results
// wherever in the batch they sit.
// The stages run on over tile boundaries.  Measured, two layers of a 2048-wide stage at 572 rows (three prompts), whole call
// 1154 -> 948 us (under the profiler W1/W3 223 us, 118 TFLOP/s of the 154 a large library product reaches); 36 random layers of 256 to
// 4096 columns at 35 .. 1500 rows 1 .. 18 % less, 10 % on average.  Six stages, or a barrier every other step, change nothing.
// -------------------------------------------------------------------------------------------------
constexpr int F32_BT = 64, F32_BN = 128, F32_BK = 32, F32_ST = 4, F32_CUS = 256;
// An accumulator's sum joins the tile's after so many k-steps (256 instructions one behind the other): without it whole tiles and long
// shares had sums up to 1.2 times as far from 64 bits as a contraction split for the whole launch (2048 x 5632 at 572 / 1033 rows
// 6.0e-7 / 7.8e-7 -> 6.4e-7 / 9.2e-7, with it 3.9e-7 at either); the time is the same.
constexpr int F32_RUN = 32;
constexpr int F32_SLOT = F32_BT * F32_BN;                 // floats of one tile's partial sums
static_assert(kF32PartFloats == (size_t)2 * F32_CUS * F32_SLOT, "two pieces per block");

// What the blocks of a launch walk, see above.  Tiles are numbered token block fastest: tile = column * gy + token block.
struct F32Walk {
    int gy, ksteps;
    int whole, rounds;         // tiles 0 .. whole - 1 are whole ones; block w takes w, w + workers, ... (at most `rounds` of them)
    int cols, sharers;         // the columns behind them are dealt out: each token block's to `sharers` blocks, cols <= sharers
    int workers;               // blocks of the launch
};
// First k-step, counted over the dealt-out columns, of a token block's sharer i.  It does not depend on the token block, so that a
// column's contraction is cut at the same places for every row.  (sharers x cols x ksteps fits 31 bits: f32_proj_mode)
__device__ inline int f32_share(const F32Walk &k, int i) {
    return (int)((unsigned)min(i, k.sharers) * (unsigned)(k.cols * k.ksteps) / (unsigned)k.sharers);
}

// A wave's 32 x 32 result: lane l holds row l % 32 and, in register 4 q + r, column 8 q + 4 (l / 32) + r of the wave's columns (SwiGLU:
// quads 0, 1 are 16 gate columns, quads 2, 3 the up columns that belong to them)
template <int MODE>
__device__ __forceinline__ void f32_tile_store(const F32Proj &p, int bn, int bt, int wave, int lane, const floatx16 &c) {
    const int t = bt + 32 * (wave & 1) + (lane & 31), hl = lane >> 5, wn = wave >> 1;
    if (t >= p.T) return;
    constexpr int Q = MODE == F32_SWIGLU ? 2 : 4;
    floatx4 h[Q];
    if (MODE == F32_RESID) {
#pragma unroll
        for (int q = 0; q < Q; ++q)
            h[q] = *reinterpret_cast<const floatx4 *>(p.resid + (size_t)t * p.cols + min(bn + 32 * wn + 8 * q + 4 * hl, p.cols - 4));
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int n = bn + (MODE == F32_SWIGLU ? 16 : 32) * wn + 8 * q + 4 * hl;
        if (n >= p.cols) continue;
        const floatx4 a = {c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]};
        const int u = MODE == F32_SWIGLU ? 4 * (q + 2) : 0;
        f32_finish4<MODE>(p, t, n, a, floatx4{c[u], c[u + 1], c[u + 2], c[u + 3]}, h[q]);
    }
}

template <int MODE>
__global__ __launch_bounds__(512) void f32_tile_kernel(F32Proj p, F32Walk k, float *__restrict__ part) {
    constexpr bool GLU = MODE == F32_SWIGLU;
    constexpr int SW = F32_BK * F32_BN, STAGE = SW + F32_BT * F32_BK;          // floats: weight rows, then token rows
    __shared__ __align__(16) float smem[F32_ST * STAGE];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, hl = lane >> 5;
    // consecutive tiles on one die: they share weight columns (blocks are dealt to the eight dies in turn)
    const int w = (blockIdx.x & 7) * (k.workers >> 3) + (blockIdx.x >> 3);

    // This block's pieces: up to two ranges of k-steps of dealt-out tiles, then whole tiles (the last ones end everywhere at once).
    // All of this is uniform: said to the compiler, which divides in vector registers, so that the loop counts in scalar ones.
    int whole = 0;
    while (whole < k.rounds && w + whole * k.workers < k.whole) ++whole;
    int u0 = 0, u1 = 0, c0 = 0, first = 0;            // shared k-steps u0 .. u1 - 1, from column c0 on; its tile
    if (w < k.sharers * k.gy) {                       // (divisions a launch of whole tiles has no use for)
        const int i = __builtin_amdgcn_readfirstlane(w / k.gy);
        u0 = __builtin_amdgcn_readfirstlane(f32_share(k, i));
        u1 = __builtin_amdgcn_readfirstlane(f32_share(k, i + 1));
        c0 = __builtin_amdgcn_readfirstlane(u0 / k.ksteps);
        first = k.whole + c0 * k.gy + w - i * k.gy;
    }
    const int cut = min(u1, (c0 + 1) * k.ksteps);
    const int ranges = __builtin_amdgcn_readfirstlane((u1 > u0 ? 1 : 0) + (u1 > cut ? 1 : 0));
    const int n_pieces = ranges + whole, steps = whole * k.ksteps + u1 - u0;
    if (steps == 0) return;                           // the whole block leaves
    struct Piece { int tile, lo, hi; };
    auto piece = [&](int i) {
        if (i >= ranges) return Piece{w + (i - ranges) * k.workers, 0, k.ksteps};
        if (i == 0) return Piece{first, u0 - c0 * k.ksteps, cut - c0 * k.ksteps};
        return Piece{first + k.gy, 0, u1 - cut};
    };
    const int bnw = GLU ? F32_BN / 2 : F32_BN;

    // Loads: a wave copies weight rows 2 wave, 2 wave + 1 and those + 16 (512 bytes each) and token rows 8 wave .. + 7 (128 bytes each) of
    // every k-step; a lane's 16 bytes land at its slot of the 1 KB piece.  Which column it fetches spreads the later reads over the
    // banks: weight rows 4 .. 7 of every eight swap neighbouring 32-column blocks, a token row's 16-byte pieces are XORed
    // with the row.
    int li = 0, lleft = 0;                            // piece of the next load, k-steps left of it
    const float *wsrc = p.w, *xsrc = p.x;
    unsigned woff = 0, xoff = 0;
    const size_t wstep = (size_t)F32_BK * p.N, whalf = (size_t)16 * p.N;
    auto load_tile = [&]() {
        const Piece q = piece(li);
        const int col = __builtin_amdgcn_readfirstlane(q.tile / k.gy), bn = col * bnw, bt = (q.tile - col * k.gy) * F32_BT;
        lleft = __builtin_amdgcn_readfirstlane(q.hi - q.lo);
        const int c = (4 * l32) ^ ((wave & 2) ? 32 : 0);
        const int n = GLU ? min(bn + 16 * (c >> 5) + (c & 15), p.cols - 4) + ((c & 16) ? p.cols : 0) : min(bn + c, p.cols - 4);
        woff = ((unsigned)hl * (unsigned)p.N + (unsigned)n) * 4u;
        const int row = 8 * wave + (lane >> 3), t = min(bt + row, p.T - 1) - bt;
        xoff = ((unsigned)t * (unsigned)p.K + 4u * ((lane & 7) ^ (row & 7))) * 4u;
        xsrc = p.x + (size_t)bt * p.K + q.lo * F32_BK;
        wsrc = p.w + (size_t)(q.lo * F32_BK + 2 * wave) * p.N;
    };
    // the x-th of the three loads of a k-step into stage buffer `buf` (floats from the start of LDS)
    const unsigned lds0 = hx_lds_addr(smem) + wave * 1024u;
    auto issue = [&](int buf, int x) {
        const unsigned lds = lds0 + 4u * buf + (x == 0 ? 0u : x == 1 ? 8192u : 4u * SW);
        const float *src = x == 0 ? wsrc : x == 1 ? wsrc + whalf : xsrc;
        hx_load_lds16(lds, x < 2 ? woff : xoff, src);
    };
    size_t wadv = wstep;
    int xadv = F32_BK;
    auto advance = [&]() {       // past the last piece the last k-step is loaded again, into a stage nobody reads
        wsrc += wadv;
        xsrc += xadv;
        lleft = __builtin_amdgcn_readfirstlane(lleft - 1);
        if (lleft == 0) {
            ++li;
            if (li < n_pieces) {
                load_tile();
            } else {
                wsrc -= wadv;
                xsrc -= xadv;
                wadv = 0;
                xadv = 0;
                lleft = 0x7fffffff;
            }
        }
    };

    // operands of the 8-row group s of a stage; k-slot hl of MFMA x = row 8 s + 4 hl + x
    floatx4 x4[2];
    float wv[2][4];
    const unsigned xrow = (32 * (wave & 1) + l32) * F32_BK + 4 * (hl ^ (l32 & 7));
    const unsigned wcol = 4 * hl * F32_BN + 32 * ((wave >> 1) ^ hl) + l32;
    auto fetch = [&](int buf, int s) {
        const float *st = smem + buf;
        x4[s & 1] = *reinterpret_cast<const floatx4 *>(st + SW + (xrow ^ (8 * s)));
#pragma unroll
        for (int x = 0; x < 4; ++x) wv[s & 1][x] = st[wcol + (8 * s + x) * F32_BN];
    };
    floatx16 acc[2];
    auto mfma = [&](int s, int x) { acc[x & 1] = f32_mfma32(wv[s & 1][x], x4[s & 1][x], acc[x & 1]); };
    auto multiply = [&](int s) {
#pragma unroll
        for (int x = 0; x < 4; ++x) mfma(s, x);
        __builtin_amdgcn_sched_barrier(0);
    };
    floatx16 sum;                                     // what leaves acc after F32_RUN k-steps, or at a piece's end
    auto gather = [&]() {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            sum[r] += acc[0][r] + acc[1][r];
            acc[0][r] = acc[1][r] = 0.f;
        }
    };
    load_tile();
#pragma unroll
    for (int i = 0; i < F32_ST - 1; ++i) {
#pragma unroll
        for (int x = 0; x < 3; ++x) issue(i * STAGE, x);
        advance();
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) sum[r] = acc[0][r] = acc[1][r] = 0.f;
    HX_WAIT_VM((F32_ST - 2) * 3);
    asm volatile("s_barrier" ::: "memory");
    fetch(0, 0);
    int ci = 0, buf = 0, lbuf = (F32_ST - 1) * STAGE;
    Piece now = piece(0);
    int left = now.hi - now.lo, run = min(left, F32_RUN);          // k-steps to the end of the piece, and until acc is gathered
    // The order below is held by scheduling barriers.  Nothing but the two waits stands between the barrier and the next MFMA: what the step
    // computes for its loads is done ahead of it, the loads go between the MFMAs behind it.
    for (int u = 0; u < steps; ++u) {
        const int nbuf = buf + STAGE == F32_ST * STAGE ? 0 : buf + STAGE;
        fetch(buf, 1);
        __builtin_amdgcn_sched_barrier(0);
        multiply(0);
        fetch(buf, 2);
        __builtin_amdgcn_sched_barrier(0);
        multiply(1);
        HX_WAIT_VM((F32_ST - 3) * 3);          // this wave's loads of step u + 1 have landed ...
        HX_LDS_BARRIER();                       // ... and everybody's; nobody reads step u - 1 any more
        fetch(buf, 3);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            mfma(2, x);
            if (x < 3) issue(lbuf, x);
            __builtin_amdgcn_sched_barrier(0);
        }
        fetch(nbuf, 0);
        __builtin_amdgcn_sched_barrier(0);
        multiply(3);
        advance();
        lbuf = buf;
        buf = nbuf;
        if (--run == 0) {
            gather();
            left -= F32_RUN;
            if (left <= 0) {
                if (now.hi - now.lo == k.ksteps) {
                    f32_tile_store<MODE>(p, now.tile / k.gy * bnw, now.tile % k.gy * F32_BT, wave, lane, sum);
                } else {
                    float *dst = part + (size_t)(2 * w + ci) * F32_SLOT + wave * 1024 + lane * 4;
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        *reinterpret_cast<floatx4 *>(dst + q * 256) = floatx4{sum[4 * q], sum[4 * q + 1], sum[4 * q + 2], sum[4 * q + 3]};
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) sum[r] = 0.f;
                // (loads and stores complete in the order of their issue: with results still in flight the waits above only wait for more)
                now = piece(++ci);
                left = now.hi - now.lo;
            }
            run = min(left, F32_RUN);
        }
    }
    HX_WAIT_VM(0);
}

// The dealt-out tiles: adds a tile's pieces up in the order of the contraction.  One wave per 32 x 8 results (SwiGLU: 32 x 8 gate and
// the up columns that belong to them), eight pieces requested at a time: round trips to the memory-side cache bound it.
template <int MODE>
__global__ __launch_bounds__(256) void f32_tile_finish_kernel(F32Proj p, F32Walk k, const float *__restrict__ part) {
    constexpr bool GLU = MODE == F32_SWIGLU;
    constexpr int Q = GLU ? 2 : 4;                              // waves per 32 x 32
    const int lane = threadIdx.x & 63, idx = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t = idx / (8 * Q), wave = idx / Q % 8, q = idx % Q, col = t / k.gy, bt = t - col * k.gy;
    // the token block's sharers whose shares meet k-steps col * ksteps .. (col + 1) * ksteps - 1
    const int s0 = col * k.ksteps, s1 = s0 + k.ksteps;
    int i0 = col * k.sharers / k.cols;
    while (i0 > 0 && f32_share(k, i0) > s0) --i0;
    while (f32_share(k, i0 + 1) <= s0) ++i0;
    int i1 = i0;                                                // the last of them
    while (f32_share(k, i1 + 1) < s1) ++i1;
    if (f32_share(k, i0) <= s0 && i1 == i0) return;             // one block had all of it and has finished it
    const int row = bt * F32_BT + 32 * (wave & 1) + (lane & 31);
    const int n = (k.whole / k.gy + col) * (GLU ? F32_BN / 2 : F32_BN) + (GLU ? 16 : 32) * (wave >> 1) + 8 * q + 4 * (lane >> 5);
    // sharer i is block i * gy + bt; only the first one's piece can be its second one
    const size_t at0 = (size_t)2 * (i0 * k.gy + bt) * F32_SLOT + wave * 1024 + q * 256 + lane * 4, step = (size_t)2 * k.gy * F32_SLOT;
    const float *src = part + at0 + (f32_share(k, i0) / k.ksteps < col ? F32_SLOT : 0);
    const float *next = part + at0 + step;
    floatx4 a = {0.f, 0.f, 0.f, 0.f}, b = a, h = a;
    const bool inside = row < p.T && n < p.cols;
    if (MODE == F32_RESID && inside) h = *reinterpret_cast<const floatx4 *>(p.resid + (size_t)row * p.cols + n);
    for (int i = i0; i <= i1; i += 8) {
        floatx4 va[8], vb[GLU ? 8 : 1];
#pragma unroll
        for (int z = 0; z < 8; ++z) {
            const int iz = min(i + z, i1);
            const float *at = iz == i0 ? src : next + (size_t)(iz - i0 - 1) * step;
            va[z] = *reinterpret_cast<const floatx4 *>(at);
            if constexpr (GLU) vb[z] = *reinterpret_cast<const floatx4 *>(at + 512);
        }
#pragma unroll
        for (int z = 0; z < 8; ++z)
            if (i + z <= i1) {
                a += va[z];
                if constexpr (GLU) b += vb[z];
            }
    }
    if (inside) f32_finish4<MODE>(p, row, n, a, b, h);
}

namespace {
template <int MODE, int NB, int V>
void f32_stream_flags(const F32Proj &p, hipStream_t s) {
    const dim3 grid((p.cols + 16 * V - 1) / (16 * V));
    if constexpr (MODE != F32_RESID) {
        if (p.g != nullptr) {
            if constexpr (MODE == F32_PLAIN) {
                if (p.x2 != nullptr) { hipLaunchKernelGGL((f32_stream_kernel<MODE, NB, V, true, true>), grid, dim3(512), 0, s, p); return; }
            }
            hipLaunchKernelGGL((f32_stream_kernel<MODE, NB, V, true, false>), grid, dim3(512), 0, s, p);
            return;
        }
    }
    if constexpr (MODE != F32_SWIGLU) hipLaunchKernelGGL((f32_stream_kernel<MODE, NB, V, false, false>), grid, dim3(512), 0, s, p);
}

template <int MODE>
void f32_proj_mode(const F32Proj &p, float *n_buf, float *part, hipStream_t s) {
    if (p.T <= 32) {
        constexpr int NM = MODE == F32_SWIGLU ? 2 : 1;
        const bool wide = p.cols / 32 >= 128;
        if (p.T <= 16) {
            if (wide) f32_stream_flags<MODE, 1, 2>(p, s);
            else f32_stream_flags<MODE, 1, 1>(p, s);
        } else {
            if (wide && NM == 1) f32_stream_flags<MODE, 2, 3 - NM>(p, s);
            else f32_stream_flags<MODE, 2, 1>(p, s);
        }
        return;
    }
    F32Proj t = p;
    if (p.g != nullptr) {            // (no caller adds a second operand or advances lengths here)
        f32_launch_rmsnorm(p.x, p.g, n_buf, p.T, p.K, p.eps, s);
        t.x = n_buf;
    }
    const int bn = MODE == F32_SWIGLU ? F32_BN / 2 : F32_BN;
    F32Walk k;
    k.gy = (p.T + F32_BT - 1) / F32_BT;
    k.ksteps = p.Kp / F32_BK;
    // Whole tiles only: the fullest CU has ceil(tiles / 256) of them, a k-step is 0.95 us.  Dealing out the k-steps of the columns that
    // whole rounds leave over evens that out and costs the partial sums' way through memory (written and read, about 4 TB/s) and a
    // second launch, for which 3 us are charged: with 6, 9 or 12 two layers of 512 columns at 130 rows take 7, 15 and 27 % longer, at
    // 1000 rows 7 %, 1024 columns at 572 rows 0, 4 and 11 %, 2048 at 100 rows 0, 0 and 8 %, wider and longer ones the same.  It has to gain
    // 1.5 us by this account: contractions of 8 k-steps stay whole.
    const int cols = (p.cols + bn - 1) / bn, tiles = cols * k.gy, full = tiles / F32_CUS;
    const double step = 0.95;
    k.whole = tiles;
    k.rounds = (tiles + F32_CUS - 1) / F32_CUS;
    k.workers = std::min(F32_CUS, (tiles + 7) / 8 * 8);
    k.cols = k.sharers = 0;
    const int left = cols - (int)((long)F32_CUS * full / k.gy);
    // blocks that share a token block's: at least 4 k-steps each, and no share is longer than a tile
    const int most = (int)std::min<long>(F32_CUS / k.gy, (long)left * k.ksteps / 4);
    if (left > 0 && part != nullptr && most >= std::max(2, left) && (long)left * k.ksteps < (1l << 23)) {
        const double part_us = (most + left) * k.gy * (double)F32_SLOT * 8.0 / 4e6;
        const double us = step * (full * k.ksteps + ((double)left * k.ksteps + most - 1) / most) + 3.0 + part_us;
        if (us + 1.5 < step * k.rounds * k.ksteps) {
            k.whole = (cols - left) * k.gy;
            k.rounds = full;
            k.workers = full > 0 ? F32_CUS : (most * k.gy + 7) / 8 * 8;
            k.cols = left;
            k.sharers = most;
        }
    }
    hipLaunchKernelGGL((f32_tile_kernel<MODE>), dim3(k.workers), dim3(512), 0, s, t, k, part);
    const int finish = (MODE == F32_SWIGLU ? 4 : 8) * k.cols * k.gy;
    if (finish > 0) hipLaunchKernelGGL((f32_tile_finish_kernel<MODE>), dim3(finish), dim3(256), 0, s, t, k, part);
}
}  // namespace

void f32_launch_proj(int mode, const F32Proj &p, float *n_buf, float *part, hipStream_t s) {
    if (p.T <= 0 || p.cols <= 0) return;
    switch (mode) {
        case F32_PLAIN: f32_proj_mode<F32_PLAIN>(p, n_buf, part, s); break;
        case F32_RESID: f32_proj_mode<F32_RESID>(p, n_buf, part, s); break;
        case F32_SWIGLU: f32_proj_mode<F32_SWIGLU>(p, n_buf, part, s); break;
    }
}

// cache layout per layer: [seq][hkv_l][smax][d]
__global__ void f32_rope_append_kernel(const float *__restrict__ qkv, int hq_l, int hkv_l, int d, int smax, RowMap rm,
                                       const float *__restrict__ cos_tab, const float *__restrict__ sin_tab,
                                       float *__restrict__ q_out, float *__restrict__ kc, float *__restrict__ vc) {
    const int t = blockIdx.x, head = blockIdx.y, i = threadIdx.x, half = d >> 1;
    const int N = (hq_l + 2 * hkv_l) * d;
    float lo = qkv[(size_t)t * N + head * d + i], hi = qkv[(size_t)t * N + head * d + i + half];
    const int seq = rm.row_seq[t], pos = rm.row_pos[t];
    if (head < hq_l + hkv_l) {
        const float c = cos_tab[(size_t)pos * half + i], sn = sin_tab[(size_t)pos * half + i];
        const float rlo = lo * c - hi * sn, rhi = hi * c + lo * sn;
        lo = rlo; hi = rhi;
    }
    float *dst;
    if (head < hq_l) dst = q_out + ((size_t)t * hq_l + head) * d;
    else if (head < hq_l + hkv_l) dst = kc + (((size_t)seq * hkv_l + (head - hq_l)) * smax + pos) * d;
    else dst = vc + (((size_t)seq * hkv_l + (head - hq_l - hkv_l)) * smax + pos) * d;
    dst[i] = lo;
    dst[i + half] = hi;
}
void f32_launch_rope_append(const float *qkv, int T, int hq_l, int hkv_l, int d, int smax, RowMap rm,
                            const float *cos_tab, const float *sin_tab, float *q_out, float *kc, float *vc,
                            hipStream_t s) {
    if (T <= 0) return;
    hipLaunchKernelGGL(f32_rope_append_kernel, dim3(T, hq_l + 2 * hkv_l), dim3(d / 2), 0, s, qkv, hq_l, hkv_l, d, smax,
                       rm, cos_tab, sin_tab, q_out, kc, vc);
}

// -------------------------------------------------------------------------------------------------
// Attention over the cache for 16 query columns that share a kv head, W waves per block; a wave takes every W-th tile of 16
// positions, and the waves' (m, l, o) are merged through LDS in wave order.  v_mfma_f32_16x16x4_f32 throughout:
//   S^T (positions x columns) = K . Q^T: lane l loads 16 bytes of position l % 16's key per 16 head elements, k-slot l / 16;
//   in the result a lane owns column l % 16 and positions 4 (l / 16) + r, which is exactly operand B of
//   O^T (head elements x columns) = V^T . P^T for the MFMA that takes positions 4 (l / 16) + r: P never leaves its registers,
//   and V is read in 16-byte pieces of its rows (head element 64 h + 4 i + e is row i of MFMA (h, e)).
// DECODE: one new row per sequence; the columns are the G heads of kv head c.  The block first rotates its heads and its
// new key, appends key and value to the cache (nobody else reads them in this launch) and keeps q in LDS.
// Otherwise: 16 consecutive new rows of one head, whose keys and values f32_rope_append_kernel has put into the cache.
// A masked position has weight 0, but 0 x inf would still poison the sum: a tile that is masked for some column and holds a
// value that is not finite is multiplied out element by element, over the positions each column may see.
// -------------------------------------------------------------------------------------------------
template <int D, int W, bool DECODE>
__global__ __launch_bounds__(64 * W) void f32_attn_kernel(const float *__restrict__ q, float *kc, float *vc, int hq_l, int hkv_l,
                                                         int smax, const int32_t *__restrict__ pos0, const int32_t *__restrict__ cu_rows,
                                                         const int32_t *__restrict__ items, const float *__restrict__ cos_tab,
                                                         const float *__restrict__ sin_tab, float *__restrict__ o) {
    constexpr int KT = D / 16, VH = D / 64, HALF = D / 2, QS = D + 4;
    __shared__ __align__(16) float s_q[DECODE ? 16 : 1][QS];
    __shared__ float s_m[W][16], s_l[W][16];
    __shared__ __align__(16) float s_o[W][16][D];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    const int G = hq_l / hkv_l;
    int seq, c, head = 0, first_pos, n_col, row0 = 0;        // column j: position first_pos + (DECODE ? 0 : j), j < n_col
    if (DECODE) {
        c = blockIdx.x % hkv_l;
        seq = blockIdx.x / hkv_l;
        first_pos = pos0[seq];
        n_col = G;
    } else {
        const int tile = blockIdx.x / hq_l;                   // an item is 128 rows of a sequence: eight tiles
        head = blockIdx.x % hq_l;
        c = head / G;
        seq = items[2 * (tile >> 3)];
        const int r0 = items[2 * (tile >> 3) + 1] * 128 + (tile & 7) * 16;
        const int n_new = cu_rows[seq + 1] - cu_rows[seq];
        if (r0 >= n_new) return;                              // the whole block leaves
        n_col = min(16, n_new - r0);
        first_pos = pos0[seq] + r0;
        row0 = cu_rows[seq] + r0;
    }
    float *K = kc + ((size_t)seq * hkv_l + c) * smax * D, *V = vc + ((size_t)seq * hkv_l + c) * smax * D;
    const int last_pos = first_pos + (DECODE ? 0 : n_col - 1);
    const int my_pos = DECODE ? first_pos : min(first_pos + i, last_pos);
    if constexpr (DECODE) {
        const float *row = q + (size_t)seq * (hq_l + 2 * hkv_l) * D;          // raw projection of the new row
        for (int idx = threadIdx.x; idx < (G + 2) * HALF; idx += 64 * W) {
            const int hh = idx / HALF, e = idx - hh * HALF;
            const float *src = row + (size_t)(hh < G ? c * G + hh : (hh == G ? hq_l + c : hq_l + hkv_l + c)) * D;
            float lo = src[e], hi = src[e + HALF];
            if (hh <= G) {
                const float cs = cos_tab[(size_t)first_pos * HALF + e], sn = sin_tab[(size_t)first_pos * HALF + e];
                const float rlo = lo * cs - hi * sn, rhi = hi * cs + lo * sn;
                lo = rlo; hi = rhi;
            }
            float *dst = hh < G ? s_q[hh] : (hh == G ? K : V) + (size_t)first_pos * D;
            dst[e] = lo;
            dst[e + HALF] = hi;
        }
        __syncthreads();           // q in LDS; the new key and value visible to the block's loads
    }
    floatx4 qf[KT];
#pragma unroll
    for (int k = 0; k < KT; ++k) {
        const int j = min(i, n_col - 1);                      // columns past the last one repeat it and are not stored
        if constexpr (DECODE) qf[k] = *reinterpret_cast<const floatx4 *>(&s_q[j][16 * k + 4 * g]);
        else qf[k] = *reinterpret_cast<const floatx4 *>(q + ((size_t)(row0 + j) * hq_l + head) * D + 16 * k + 4 * g);
    }
    const float scale = 1.0f / sqrtf((float)D);
    floatx4 oacc[VH][4];
#pragma unroll
    for (int h = 0; h < VH; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e) oacc[h][e] = floatx4{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, lsum = 0.f;
    for (int t = wave; t <= last_pos >> 4; t += W) {
        floatx4 kf[KT], vf[4][VH];
#pragma unroll
        for (int k = 0; k < KT; ++k) kf[k] = *reinterpret_cast<const floatx4 *>(K + (size_t)min(16 * t + i, last_pos) * D + 16 * k + 4 * g);
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int h = 0; h < VH; ++h)
                vf[x][h] = *reinterpret_cast<const floatx4 *>(V + (size_t)min(16 * t + 4 * g + x, last_pos) * D + 64 * h + 4 * i);
        floatx4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < KT; ++k)
#pragma unroll
            for (int x = 0; x < 4; ++x) s = f32_mfma16(kf[k][x], qf[k][x], s);
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            s[r] = 16 * t + 4 * g + r <= my_pos ? s[r] * scale : -INFINITY;
            mx = fmaxf(mx, s[r]);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float m_new = fmaxf(m, mx);
        const float base = m_new == -INFINITY ? 0.f : m_new;      // a column that has seen no position yet: weights 0, no NaN
        const float alpha = expf(m - base);
        m = m_new;
        float ps = 0.f, pr[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            pr[r] = expf(s[r] - base);
            ps += pr[r];
        }
        lsum = lsum * alpha + ps;
#pragma unroll
        for (int h = 0; h < VH; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) oacc[h][e] *= alpha;
        bool odd = false;
        if (16 * t + 15 > first_pos) {                            // masked for some column
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int h = 0; h < VH; ++h)
#pragma unroll
                    for (int e = 0; e < 4; ++e) odd = odd || !(fabsf(vf[x][h][e]) < INFINITY);
        }
        if (__builtin_amdgcn_ballot_w64(odd) == 0) {
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int h = 0; h < VH; ++h)
#pragma unroll
                    for (int e = 0; e < 4; ++e) oacc[h][e] = f32_mfma16(vf[x][h][e], pr[x], oacc[h][e]);
        } else {
            for (int pp = 0; pp < 16; ++pp) {
                const int src = i + 16 * (pp >> 2);
                const float w0 = __shfl(pr[0], src, 64), w1 = __shfl(pr[1], src, 64), w2 = __shfl(pr[2], src, 64), w3 = __shfl(pr[3], src, 64);
                const float w = (pp & 3) == 0 ? w0 : (pp & 3) == 1 ? w1 : (pp & 3) == 2 ? w2 : w3;
                if (16 * t + pp > my_pos) continue;
#pragma unroll
                for (int h = 0; h < VH; ++h)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            oacc[h][e][r] = fmaf(w, V[(size_t)(16 * t + pp) * D + 64 * h + 4 * (4 * g + r) + e], oacc[h][e][r]);
            }
        }
    }
    lsum += __shfl_xor(lsum, 16, 64);
    lsum += __shfl_xor(lsum, 32, 64);
    if (g == 0) { s_m[wave][i] = m; s_l[wave][i] = lsum; }
    // register r of oacc[h][e]: head element 64 h + 4 (4 g + r) + e of column i
#pragma unroll
    for (int h = 0; h < VH; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            *reinterpret_cast<floatx4 *>(&s_o[wave][i][64 * h + 16 * g + 4 * r]) = floatx4{oacc[h][0][r], oacc[h][1][r], oacc[h][2][r], oacc[h][3][r]};
    __syncthreads();
    for (int idx = threadIdx.x * 4; idx < n_col * D; idx += 64 * W * 4) {
        const int j = idx / D, dd = idx % D;
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < W; ++w) M = fmaxf(M, s_m[w][j]);
        float L = 0.f;
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < W; ++w) {
            if (s_l[w][j] == 0.f) continue;                       // no position of this column (or all of them at weight 0)
            const float wt = expf(s_m[w][j] - M);
            L += s_l[w][j] * wt;
            acc += *reinterpret_cast<const floatx4 *>(&s_o[w][j][dd]) * wt;
        }
        const int64_t row = DECODE ? (int64_t)seq * hq_l + c * G + j : (int64_t)(row0 + j) * hq_l + head;
        *reinterpret_cast<floatx4 *>(o + row * D + dd) = acc / L;
    }
}
void f32_launch_attn_prefill(const float *q, float *kc, float *vc, int hq_l, int hkv_l, int d, int smax, const int32_t *pos0,
                             const int32_t *cu_rows, const int32_t *items, int n_items, float *o, hipStream_t s) {
    if (n_items <= 0) return;
    const dim3 grid((unsigned)n_items * 8u * (unsigned)hq_l);
    if (d == 128) hipLaunchKernelGGL((f32_attn_kernel<128, 4, false>), grid, dim3(256), 0, s, q, kc, vc, hq_l, hkv_l, smax, pos0, cu_rows, items, nullptr, nullptr, o);
    else hipLaunchKernelGGL((f32_attn_kernel<64, 4, false>), grid, dim3(256), 0, s, q, kc, vc, hq_l, hkv_l, smax, pos0, cu_rows, items, nullptr, nullptr, o);
}
void f32_launch_attn_decode(const float *qkv, float *kc, float *vc, int b, int hq_l, int hkv_l, int d, int smax, const int32_t *pos,
                            const float *cos_tab, const float *sin_tab, float *o, hipStream_t s) {
    if (b <= 0) return;
    const dim3 grid((unsigned)hkv_l * (unsigned)b);
    if (d == 128) hipLaunchKernelGGL((f32_attn_kernel<128, 4, true>), grid, dim3(256), 0, s, qkv, kc, vc, hq_l, hkv_l, smax, pos, nullptr, nullptr, cos_tab, sin_tab, o);
    else hipLaunchKernelGGL((f32_attn_kernel<64, 8, true>), grid, dim3(512), 0, s, qkv, kc, vc, hq_l, hkv_l, smax, pos, nullptr, nullptr, cos_tab, sin_tab, o);
}

// -------------------------------------------------------------------------------------------------
// A decode step's attention and W_O in one launch, for few sequences with short contexts on a narrow stage: every block computes
// the attention of all (sequence, kv head) pairs for itself -- at most four, two to eight waves each -- and goes on with 16 columns of W_O, whose
// weights it has requested before.  Bound by latency: the launch it saves and the trip of o through memory are longer than
// reading a few KB of keys and values 32 times from L2 (f32_attn_wo_fits; the tiny stage's 32-row prompt and eight steps with its head 600 ->
// 566 us, medians of eight processes).  The pairs' new keys and values are taken from LDS by every block, block 0 appends them to the cache.  W_O
// adds up in f32_stream_kernel's order.
// -------------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(512) void f32_attn_wo_kernel(const float *__restrict__ qkv, float *kc, float *vc, int hq_l, int hkv_l, int smax,
                                                         const int32_t *__restrict__ pos0, const float *__restrict__ cos_tab,
                                                         const float *__restrict__ sin_tab, F32Proj p) {
    constexpr int W = 8, KT = D / 16, VH = D / 64, HALF = D / 2, QS = D + 4, U = 4;
    extern __shared__ __align__(16) float lds[];
    __shared__ float s_m[W][16], s_l[W][16];
    __shared__ floatx4 red[W][64];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    const int G = hq_l / hkv_l, pairs = p.T * hkv_l, qw = hq_l * D;
    float *s_o = lds, *s_new = lds + W * 16 * D;          // [W][16][D]; [pairs][G + 2][QS]: rotated heads, new key and value; then o [T][qw]
    const int n0 = blockIdx.x * 16, col = n0 + i, chunks = p.Kp >> 4;
    float wv[U][4];
    auto request = [&](int u, int c) {
#pragma unroll
        for (int x = 0; x < 4; ++x) wv[u][x] = p.w[(size_t)(16 * c + 4 * g + x) * p.N + col];
    };
    floatx4 res = {0.f, 0.f, 0.f, 0.f};
    if (wave == 0) res = *reinterpret_cast<const floatx4 *>(p.resid + (size_t)min(i, p.T - 1) * p.N + n0 + 4 * g);
    for (int idx = threadIdx.x; idx < pairs * (G + 2) * HALF; idx += 64 * W) {
        const int row = idx / HALF, e = idx - row * HALF, pair = row / (G + 2), hh = row - pair * (G + 2), seq = pair / hkv_l, c = pair - seq * hkv_l;
        const float *src = qkv + ((size_t)seq * (hq_l + 2 * hkv_l) + (hh < G ? c * G + hh : (hh == G ? hq_l + c : hq_l + hkv_l + c))) * D;
        const int pos = pos0[seq];
        float lo = src[e], hi = src[e + HALF];
        if (hh <= G) {
            const float cs = cos_tab[(size_t)pos * HALF + e], sn = sin_tab[(size_t)pos * HALF + e];
            const float rlo = lo * cs - hi * sn, rhi = hi * cs + lo * sn;
            lo = rlo; hi = rhi;
        }
        s_new[row * QS + e] = lo;
        s_new[row * QS + e + HALF] = hi;
        if (hh >= G && blockIdx.x == 0) {
            float *dst = (hh == G ? kc : vc) + (((size_t)seq * hkv_l + c) * smax + pos) * D;
            dst[e] = lo;
            dst[e + HALF] = hi;
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) request(u, min(wave + u * W, chunks - 1));
    HX_LDS_BARRIER();                                      // (the weights stay in flight)
    const int parts = W / pairs, pair = wave / parts, part = wave - pair * parts;
    if (pair < pairs) {
        const int seq = pair / hkv_l, c = pair - seq * hkv_l, pos = pos0[seq], there = max(pos - 1, 0);
        const float *K = kc + ((size_t)seq * hkv_l + c) * smax * D, *V = vc + ((size_t)seq * hkv_l + c) * smax * D;
        const float *q = s_new + (pair * (G + 2) + min(i, G - 1)) * QS, *nk = s_new + (pair * (G + 2) + G) * QS, *nv = nk + QS;
        floatx4 qf[KT];
#pragma unroll
        for (int k = 0; k < KT; ++k) qf[k] = *reinterpret_cast<const floatx4 *>(q + 16 * k + 4 * g);
        const float scale = 1.0f / sqrtf((float)D);
        floatx4 oacc[VH][4];
#pragma unroll
        for (int h = 0; h < VH; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) oacc[h][e] = floatx4{0.f, 0.f, 0.f, 0.f};
        float m = -INFINITY, lsum = 0.f;
        for (int t = part; t <= pos >> 4; t += parts) {
            floatx4 kf[KT], vf[4][VH];
#pragma unroll
            for (int k = 0; k < KT; ++k) kf[k] = *reinterpret_cast<const floatx4 *>(K + (size_t)min(16 * t + i, there) * D + 16 * k + 4 * g);
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int h = 0; h < VH; ++h)
                    vf[x][h] = *reinterpret_cast<const floatx4 *>(V + (size_t)min(16 * t + 4 * g + x, there) * D + 64 * h + 4 * i);
            if (16 * t + 15 >= pos) {                      // the new row, which block 0 is writing; values behind it are 0, as their weights will be
#pragma unroll
                for (int k = 0; k < KT; ++k)
                    if (16 * t + i >= pos) kf[k] = *reinterpret_cast<const floatx4 *>(nk + 16 * k + 4 * g);
#pragma unroll
                for (int x = 0; x < 4; ++x)
#pragma unroll
                    for (int h = 0; h < VH; ++h)
                        if (16 * t + 4 * g + x >= pos)
                            vf[x][h] = 16 * t + 4 * g + x == pos ? *reinterpret_cast<const floatx4 *>(nv + 64 * h + 4 * i) : floatx4{0.f, 0.f, 0.f, 0.f};
            }
            floatx4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < KT; ++k)
#pragma unroll
                for (int x = 0; x < 4; ++x) s = f32_mfma16(kf[k][x], qf[k][x], s);
            float mx = -INFINITY;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[r] = 16 * t + 4 * g + r <= pos ? s[r] * scale : -INFINITY;
                mx = fmaxf(mx, s[r]);
            }
            mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            const float m_new = fmaxf(m, mx);
            const float base = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = expf(m - base);
            m = m_new;
            float ps = 0.f, pr[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                pr[r] = expf(s[r] - base);
                ps += pr[r];
            }
            lsum = lsum * alpha + ps;
#pragma unroll
            for (int h = 0; h < VH; ++h)
#pragma unroll
                for (int e = 0; e < 4; ++e) oacc[h][e] *= alpha;
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int h = 0; h < VH; ++h)
#pragma unroll
                    for (int e = 0; e < 4; ++e) oacc[h][e] = f32_mfma16(vf[x][h][e], pr[x], oacc[h][e]);
        }
        lsum += __shfl_xor(lsum, 16, 64);
        lsum += __shfl_xor(lsum, 32, 64);
        if (g == 0) { s_m[wave][i] = m; s_l[wave][i] = lsum; }
#pragma unroll
        for (int h = 0; h < VH; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                *reinterpret_cast<floatx4 *>(s_o + (wave * 16 + i) * D + 64 * h + 16 * g + 4 * r) = floatx4{oacc[h][0][r], oacc[h][1][r], oacc[h][2][r], oacc[h][3][r]};
    }
    HX_LDS_BARRIER();
    for (int idx = threadIdx.x * 4; idx < p.T * qw; idx += 64 * W * 4) {
        const int seq = idx / qw, head = (idx - seq * qw) / D, dd = idx % D, c = head / G, j = head - c * G, w0 = (seq * hkv_l + c) * parts;
        float M = -INFINITY;
        for (int w = w0; w < w0 + parts; ++w) M = fmaxf(M, s_m[w][j]);
        float L = 0.f;
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int w = w0; w < w0 + parts; ++w) {
            if (s_l[w][j] == 0.f) continue;
            const float wt = expf(s_m[w][j] - M);
            L += s_l[w][j] * wt;
            acc += *reinterpret_cast<const floatx4 *>(s_o + (w * 16 + j) * D + dd) * wt;
        }
        *reinterpret_cast<floatx4 *>(s_new + idx) = acc / L;
    }
    HX_LDS_BARRIER();
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int c0 = wave; c0 < chunks; c0 += U * W)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = c0 + u * W;
            if (c < chunks) {
                const floatx4 x = *reinterpret_cast<const floatx4 *>(s_new + min(i, p.T - 1) * qw + 16 * c + 4 * g);
#pragma unroll
                for (int q = 0; q < 4; ++q) acc = f32_mfma16(wv[u][q], x[q], acc);
                request(u, min(c + U * W, chunks - 1));
            }
        }
    red[wave][lane] = acc;
    __syncthreads();
    if (wave != 0) return;
    floatx4 v = red[0][lane];
#pragma unroll
    for (int w = 1; w < W; ++w) v += red[w][lane];
    if (i < p.T) *reinterpret_cast<floatx4 *>(p.resid_out + (size_t)i * p.cols + n0 + 4 * g) = res + v;
}
static size_t f32_attn_wo_lds(int T, int hq_l, int hkv_l, int d) {
    return (size_t)(8 * 16 * d + T * (hq_l + 2 * hkv_l) * (d + 4)) * sizeof(float);
}
// Few pairs (what every block stages), and about two tiles of 16 positions per wave at head dim 64, one at 128: a further one is 2 us of
// latency, which is what the fused launch saves.  Two layers and eight steps, us, apart -> fused:
//   head dim 64   4 pairs at 8 / 20 / 50 / 64 positions 396 / 398 / 400 / 401 -> 368 / 382 / 398 / 426, from 33 on (a prompt of 32, with the head) 600 ->
//                 566, 1024 columns at 20 / 50 628 / 637 -> 617 / 642; 3 pairs at 20 / 50 372 / 374 -> 358 / 378; 2 pairs at 60 / 110 / 250 461 / 469 / 501 ->
//                 448 / 453 / 519; 1 pair at 60 / 240 / 500 375 / 405 / 454 -> 354 / 386 / 439; 8 pairs at 20 458 -> 464
//   head dim 128  1 pair at 60 / 110 397 / 410 -> 373 / 392; 2 pairs at 30 / 56 651 / 658 -> 647 / 662, two sequences of one at 20 656 -> 673
// 2048 columns at 20 positions 1332 -> 1327.
bool f32_attn_wo_fits(int T, int hq_l, int hkv_l, int d, int cols, int positions) {
    const int pairs = T * hkv_l;
    if (pairs > 4 || hq_l / hkv_l > 16 || cols > 1024 || f32_attn_wo_lds(T, hq_l, hkv_l, d) > 128 * 1024) return false;
    if (d != 64) return pairs == 1 && positions <= 128;
    return positions <= (pairs <= 2 ? 256 / pairs : 48);
}
void f32_launch_attn_wo(const float *qkv, float *kc, float *vc, int hq_l, int hkv_l, int d, int smax, const int32_t *pos, const float *cos_tab,
                        const float *sin_tab, const F32Proj &p, hipStream_t s) {
    const dim3 grid(p.cols / 16);
    const size_t lds = f32_attn_wo_lds(p.T, hq_l, hkv_l, d);
    static bool raised = false;
    if (!raised) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(f32_attn_wo_kernel<64>), hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(f32_attn_wo_kernel<128>), hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);
        raised = true;
    }
    if (d == 128) hipLaunchKernelGGL(f32_attn_wo_kernel<128>, grid, dim3(512), lds, s, qkv, kc, vc, hq_l, hkv_l, smax, pos, cos_tab, sin_tab, p);
    else hipLaunchKernelGGL(f32_attn_wo_kernel<64>, grid, dim3(512), lds, s, qkv, kc, vc, hq_l, hkv_l, smax, pos, cos_tab, sin_tab, p);
}

// staging [n][hkv_l][d] <-> cache rows pos0.. of sequence seq
__global__ void f32_kv_copy_kernel(float *kc, float *vc, float *k, float *v, int hkv_l, int d, int smax, int seq,
                                   int pos0, int n, int to_cache) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)n * hkv_l * d) return;
    const int e = (int)(i % d), c = (int)((i / d) % hkv_l), p = pos0 + (int)(i / ((int64_t)d * hkv_l));
    const size_t o = (((size_t)seq * hkv_l + c) * smax + p) * d + e;
    if (to_cache) { kc[o] = k[i]; vc[o] = v[i]; } else { k[i] = kc[o]; v[i] = vc[o]; }
}
void f32_launch_kv_copy(float *kc, float *vc, float *k, float *v, int hkv_l, int d, int smax, int seq, int pos0,
                        int n, int to_cache, hipStream_t s) {
    int64_t tot = (int64_t)n * hkv_l * d;
    if (tot <= 0) return;
    hipLaunchKernelGGL(f32_kv_copy_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, kc, vc, k, v, hkv_l, d,
                       smax, seq, pos0, n, to_cache);
}
