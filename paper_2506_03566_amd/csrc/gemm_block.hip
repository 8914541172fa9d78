// Matrix product for many activation rows (a prompt's chunk):  Y[m][n] = sum_k X[m][k] W[n][k], M > 256, 16-bit types, with
// the operation that follows it in a Llama decoder layer in its epilogue.  The weights are the ones the streaming kernels use
// (packed in operand order of v_mfma_f32_16x16x32); here each is used for hundreds of rows and the matrix pipe is the bound.
//
// A workgroup owns a TM x TN tile and the whole K, or (EPI_PLAIN) a part of it whose sums go to a plane.  Both operands go from
// memory straight into LDS, one k-step of 32 per stage, NST stages in a ring: at k-step j a wave multiplies the fragments it
// read from LDS during j - 1, reads those of j + 1 and asks for a share of stage j + NST - 1, all three interleaved (a run of
// LDS-direct loads would stall the wave at issue while its SIMD has nothing to multiply), and there is one barrier per k-step.
// Against 256 rows per launch of gemm_tall_kernel (gate/up of the 8B shape: 16 x 69 us for 4096 rows, 870 TFLOP/s) 745 us (1291
// TFLOP/s), and the partial planes and their epilogue kernels are gone: a prompt of 8192 tokens through four layers and three
// specialists took 45.5 ms, now 24.0.  The product is formed transposed (weights as MFMA rows): a lane then holds four
// consecutive columns of one activation row, so the epilogues read and write 8 and 16 bytes at a time.
#include "device_utils.h"
#include <hip/hip_ext.h>

namespace poss {

typedef float  f32x4 __attribute__((ext_vector_type(4)));
typedef bf16_t bf16x8 __attribute__((ext_vector_type(8)));
typedef f16_t  f16x8 __attribute__((ext_vector_type(8)));

template <typename T> struct BlockMfma;
template <> struct BlockMfma<bf16_t> {
    static __device__ __forceinline__ f32x4 run(u32x4 a, u32x4 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
};
template <> struct BlockMfma<f16_t> {
    static __device__ __forceinline__ f32x4 run(u32x4 a, u32x4 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    }
};

template <typename T> struct __attribute__((aligned(8))) Quad { T v[4]; };

__device__ const u32x4 zero_piece = {0u, 0u, 0u, 0u};     // what a lane fetches where its k lies beyond K

struct BlockGeom {
    int M, N, K, ksteps_total;       // ksteps_total: of the packed matrix (padded K)
    int col0;                        // first column of the product (a multiple of 32): columns before it are not formed
    int ctiles;                      // 16-column tiles of the packed matrix
    int tiles_m, tiles_n, splits;    // splits > 1 (EPI_PLAIN): split s of K goes to plane s, [M][N], of part
    float *part;
};

template <int TM, int TN, int NST> constexpr int BLOCK_LDS_UNITS = NST * (TM + TN) / 16 * 64;   // 16 bytes each

// One workgroup's tile: number bid of the tiles of g.
template <typename T, int TM, int TN, int WM, int WN, int NST, int EPI>
__device__ __forceinline__ void gemm_block_body(u32x4 *__restrict__ xs, const int bid, const u32x4 *__restrict__ Wp, const T *__restrict__ X,
                                                int ldx, const BlockGeom &g, const EpiArgs &e) {
    typedef __attribute__((address_space(3))) void *LdsPtr;
    constexpr int WAVES = WM * WN, MTW = TM / (16 * WM), NTW = TN / (16 * WN);
    constexpr int XB = TM / 16, WB = TN / 16;                             // 1 KB operand blocks of a stage
    constexpr int XPW = XB / WAVES, WPW = WB / WAVES, LPS = XPW + WPW;    // loads of a wave per stage
    constexpr int STAGE_UNITS = (XB + WB) * 64;
    static_assert(XPW * WAVES == XB && WPW * WAVES == WB && NTW % 2 == 0 && NTW <= MTW && LPS <= MTW && NST >= 3, "tile shape");
    static_assert(NST * STAGE_UNITS == BLOCK_LDS_UNITS<TM, TN, NST>, "what the caller provides");
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int wm = wave % WM, wn = wave / WM;

    // Workgroup -> tile.  Consecutive ids go to the 8 XCDs in turn; an XCD is given a contiguous run of tiles, ordered so that
    // the ~32 it works on at a time are about 8 row tiles x 4 column tiles and share their operands in its L2.
    int id;
    {
        const int n = g.tiles_m * g.tiles_n, q = n >> 3, r = n & 7, x = bid & 7;
        id = x * q + (x < r ? x : r) + (bid >> 3);
    }
    constexpr int GM = 2048 / TM;
    const int grp = id / (GM * g.tiles_n), in_grp = id - grp * (GM * g.tiles_n);
    const int gm = min(GM, g.tiles_m - grp * GM);
    const int m0 = (grp * GM + in_grp % gm) * TM, ct0 = (g.col0 >> 4) + (in_grp / gm) * WB;

    // Activation block b = rows 16 b .. 16 b + 15 of the tile: four lanes per row, 16 bytes each; piece p of row r lies at
    // position p ^ (r / 2 % 4), so that an operand read (lane % 16 the row, lane / 16 the piece) meets every bank once.
    // Addresses are a scalar base that moves with k and 32 bits per lane (the operands are below 4 GiB: checked on the host).
    const int x_k = ((lane & 3) ^ ((lane >> 3) & 3)) * 8;
    unsigned x_off[XPW];
#pragma unroll
    for (int j = 0; j < XPW; ++j) {
        const int m = m0 + (wave + WAVES * j) * 16 + (lane >> 2);
        x_off[j] = ((unsigned)(m < g.M ? m : g.M - 1) * (unsigned)ldx + x_k) * (unsigned)sizeof(T);   // rows beyond M repeat the last row (never stored)
    }
    const unsigned w_off = lane * 16;
    const unsigned lds0 = (unsigned)(uintptr_t)(LdsPtr)&xs[0];
    const int n_full = g.K / GEMM_KSTEP;                  // k-steps that lie inside K as a whole
    const int n_pairs = ((g.K + GEMM_KSTEP - 1) / GEMM_KSTEP + 1) / 2;     // of k-steps; the packed weights are zero beyond K
    const int ks0 = EPI == EPI_PLAIN ? 2 * (int)((long long)blockIdx.y * n_pairs / g.splits) : 0;
    const int n_ks = EPI == EPI_PLAIN ? 2 * (int)((long long)(blockIdx.y + 1) * n_pairs / g.splits) - ks0 : 2 * n_pairs;
    auto issue_one = [&](int j, int ks_rel, int st) {     // load j (static) of this wave's share of k-step ks0 + ks_rel, into stage st
        const int ks = ks0 + ks_rel;
        const unsigned base = lds0 + (unsigned)(st * STAGE_UNITS * 16);
        if (j < XPW) {
            const unsigned off = x_off[j < XPW ? j : 0], dst = base + (unsigned)((wave + WAVES * j) * 1024);
            const T *src = X + ks * GEMM_KSTEP;
            if (ks < n_full) {
                lds_dma16_s(dst, src, off);
            } else {
                const char *p = reinterpret_cast<const char *>(src) + off;
                lds_dma16(dst, ks * GEMM_KSTEP + x_k < g.K ? static_cast<const void *>(p) : static_cast<const void *>(&zero_piece));
            }
        } else {
            const int i = j - XPW, ct = min(ct0 + wave + WAVES * i, g.ctiles - 1);   // columns beyond the matrix repeat the last tile (never stored)
            lds_dma16_s(base + (unsigned)((XB + wave + WAVES * i) * 1024),
                        Wp + (((size_t)(ct >> 1) * g.ksteps_total + ks) * GEMM_NT + (ct & 1)) * 64, w_off);
        }
    };

    f32x4 acc[NTW][MTW];
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt)
#pragma unroll
        for (int mt = 0; mt < MTW; ++mt) acc[nt][mt] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Stages beyond the last k-step are asked for too (of the last k-step again: valid memory, never read), so that every
    // step is the same straight line; the wait for them stands behind the epilogue.
#pragma unroll
    for (int s = 0; s < NST - 1; ++s)
#pragma unroll
        for (int j = 0; j < LPS; ++j) issue_one(j, min(s, n_ks - 1), s);
    dma_wait<(NST - 2) * LPS>();
    __syncthreads();

    const int x_rd = wm * MTW * 64 + (lane & 15) * 4 + ((lane >> 4) ^ ((lane >> 1) & 3));
    const int w_rd = (XB + wn * NTW) * 64 + lane;
    u32x4 xf[2][MTW], wf[2][NTW];
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt) wf[0][nt] = xs[w_rd + nt * 64];
#pragma unroll
    for (int mt = 0; mt < MTW; ++mt) xf[0][mt] = xs[x_rd + mt * 64];

    // k-step j: stage j + NST - 1 is asked for, into the buffer of stage j - 1 (every wave had its fragments of j - 1 before
    // the barrier below: it multiplied them in step j - 1); the fragments of step j + 1 are read.
    int st_next = 1, st_issue = NST - 1;                  // stage buffers of step j + 1 and of step j + NST - 1
    auto step = [&](int j, const u32x4 (&xc)[MTW], const u32x4 (&wc)[NTW], u32x4 (&xn)[MTW], u32x4 (&wn_)[NTW]) {
        dma_wait<(NST - 3) * LPS>();
        __syncthreads();
        const u32x4 *xr = &xs[st_next * STAGE_UNITS + x_rd], *wr = &xs[st_next * STAGE_UNITS + w_rd];
        const int ks = min(j + NST - 1, n_ks - 1);
#pragma unroll
        for (int mt = 0; mt < MTW; ++mt) {
            if (mt < LPS) issue_one(mt, ks, st_issue);
            if (mt < NTW) wn_[mt] = wr[mt * 64];
            xn[mt] = xr[mt * 64];
#pragma unroll
            for (int nt = 0; nt < NTW; ++nt) acc[nt][mt] = BlockMfma<T>::run(wc[nt], xc[mt], acc[nt][mt]);
            __builtin_amdgcn_sched_barrier(0);
        }
        st_next = st_next == NST - 1 ? 0 : st_next + 1;
        st_issue = st_issue == NST - 1 ? 0 : st_issue + 1;
    };
    for (int j = 0; j < n_ks; j += 2) {
        step(j, xf[0], wf[0], xf[1], wf[1]);
        step(j + 1, xf[1], wf[1], xf[0], wf[0]);
    }

    // D tile: lane -> activation row lane % 16, register r -> column 4 * (lane / 16) + r
    const int lg4 = (lane >> 4) * 4;
#pragma unroll
    for (int mt = 0; mt < MTW; ++mt) {
        const int m = m0 + (wm * MTW + mt) * 16 + (lane & 15);
        if (m >= g.M) continue;
        if constexpr (EPI == EPI_PLAIN) {
            float *plane = g.part + (size_t)blockIdx.y * g.M * g.N + (size_t)m * g.N;
#pragma unroll
            for (int nt = 0; nt < NTW; ++nt) {
                const int n = (ct0 + wn * NTW + nt) * 16 + lg4;
                if (n < g.N) *reinterpret_cast<f32x4 *>(plane + n) = acc[nt][mt];       // (N is a multiple of 8)
            }
        } else if constexpr (EPI == EPI_RESIDUAL) {
            const T *bias = static_cast<const T *>(e.bias);
#pragma unroll
            for (int nt = 0; nt < NTW; ++nt) {
                const int n = (ct0 + wn * NTW + nt) * 16 + lg4;
                if (n >= g.N) continue;                   // (N is a multiple of 8: four columns are inside or outside as a whole)
                f32x4 *dst = reinterpret_cast<f32x4 *>(e.h + (size_t)m * g.N + n);
                f32x4 add = f32x4{0.f, 0.f, 0.f, 0.f};
                if (e.residual) add = *dst;
                if (bias) {
                    const Quad<T> b = *reinterpret_cast<const Quad<T> *>(bias + n);
#pragma unroll
                    for (int r = 0; r < 4; ++r) add[r] += to_f(b.v[r]);
                }
                *dst = acc[nt][mt] + add;
            }
        } else if constexpr (EPI == EPI_SILU) {
            T *act = static_cast<T *>(e.act);
#pragma unroll
            for (int nt = 0; nt < NTW; nt += 2) {
                const int f = ((ct0 + wn * NTW + nt) >> 1) * 16 + lg4;
                if (f >= e.F) continue;                   // (F is a multiple of 8)
                Quad<T> o;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float gt = acc[nt][mt][r], up = acc[nt + 1][mt][r];
                    o.v[r] = mul_round<T>(gt / (1.0f + expf(-gt)), up);
                }
                *reinterpret_cast<Quad<T> *>(act + (size_t)m * e.F + f) = o;
            }
        } else {
            static_assert(EPI == EPI_ROPE_KV, "epilogues: rotary + cache writes, residual, SiLU");
            const int half = e.dh >> 1, tph = half >> 4, sl = e.slot[m];
            const int P = 1 << e.kv.page_shift, pg = e.kv.page_table[sl >> e.kv.page_shift], in_pg = sl & (P - 1);
#pragma unroll
            for (int nt = 0; nt < NTW; nt += 2) {
                const int tile = (ct0 + wn * NTW + nt) >> 1, gh = tile / tph, i = (tile % tph) * 16 + lg4;
                if (gh >= e.hq + 2 * e.hkv) continue;     // padding columns
                const f32x4 x1 = acc[nt][mt], x2 = acc[nt + 1][mt];
                if (gh >= e.hq + e.hkv) {
                    T *dst = static_cast<T *>(e.kv.vt) + ((size_t)(pg * e.hkv + gh - e.hq - e.hkv) * e.dh + i) * P + in_pg;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        dst[(size_t)r * P] = from_f<T>(x1[r]);
                        dst[(size_t)(r + half) * P] = from_f<T>(x2[r]);
                    }
                    continue;
                }
                Quad<T> o1, o2;
                const float2 *cs = e.cs + (size_t)m * half + i;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float a, b;
                    rope_pair(x1[r], x2[r], cs[r], a, b);
                    o1.v[r] = round_f<T>(a);
                    o2.v[r] = round_f<T>(b);
                }
                T *dst = gh < e.hq ? static_cast<T *>(e.q) + ((size_t)m * e.hq + gh) * e.dh + i
                                   : static_cast<T *>(e.kv.k) + ((size_t)(pg * e.hkv + gh - e.hq) * P + in_pg) * e.dh + i;
                *reinterpret_cast<Quad<T> *>(dst) = o1;
                *reinterpret_cast<Quad<T> *>(dst + half) = o2;
            }
        }
    }
    dma_wait<0>();                                        // the stages nobody reads: LDS must not be given back before they land
}

template <typename T, int TM, int TN, int WM, int WN, int NST, int EPI>
__global__ __launch_bounds__(WM * WN * 64, 2) void gemm_block_kernel(const u32x4 *__restrict__ Wp, const T *__restrict__ X, int ldx,
                                                                    BlockGeom g, EpiArgs e) {
    __shared__ __attribute__((aligned(1024))) u32x4 xs[BLOCK_LDS_UNITS<TM, TN, NST>];
    gemm_block_body<T, TM, TN, WM, WN, NST, EPI>(xs, blockIdx.x, Wp, X, ldx, g, e);
}

// Two tile shapes in one launch: whole rounds of 256 x 256 tiles (the columns of g), then 256 x 128 tiles for the columns that are
// left (those of rest), which the CUs take up as they become free.  A row's sums are the same either way.
template <typename T, int EPI>
__global__ __launch_bounds__(512, 2) void gemm_block_mixed_kernel(const u32x4 *__restrict__ Wp, const T *__restrict__ X, int ldx, BlockGeom g,
                                                                 BlockGeom rest, EpiArgs e) {
    __shared__ __attribute__((aligned(1024))) u32x4 xs[BLOCK_LDS_UNITS<256, 256, 5>];
    static_assert(BLOCK_LDS_UNITS<256, 256, 5> >= BLOCK_LDS_UNITS<256, 128, 6>, "both shapes fit");
    const int first = g.tiles_m * g.tiles_n;
    if ((int)blockIdx.x < first) gemm_block_body<T, 256, 256, 2, 4, 5, EPI>(xs, blockIdx.x, Wp, X, ldx, g, e);
    else gemm_block_body<T, 256, 128, 4, 2, 6, EPI>(xs, (int)blockIdx.x - first, Wp, X, ldx, rest, e);
}

// ------------------------------------------------------------------------------------------
// Tile shapes: 256 x 256 (eight waves of 128 x 64, five stages), 256 x 128 (eight of 64 x 64, six) and 128 x 128 (four waves, five
// stages, two workgroups per CU).  Measured (bf16, us and TFLOP/s):
//   M     N      K       256x256        256x128        128x128       (a library product of 8192^3 on this card: 1375)
//   4096  4096   4096    109 (1263)     131 (1050)     140  (984)    256 tiles of 256 x 256: one per CU
//   4096  28672  4096    745 (1291)     960 (1002)    1028  (936)
//   4096  6144   4096    197 (1044)     210  (984)     238  (868)    384 tiles: two rounds, the second half empty
//   1001  5120   5120    108  (487)      70  (748)      78  (674)
//   1001  4096   4096     86  (389)      57  (595)      42  (802)
//   512   28672  4096    113 (1062)     159  (755)     167  (719)
// The largest is bound by the matrix pipe (and the clock it can hold), the smaller ones by LDS: a wave of 64 x 64 reads 8 KB per
// sixteen MFMAs, 128 B/clk with two waves per SIMD.  The cost below is the measured time of a round of each shape, relative to
// one round of 256 x 256 (109 us at K = 4096): 256 x 128: 56 / 109 with the chip not full, 65 / 109 with it; 128 x 128: 40 / 109
// for up to one tile per CU, 68 / 109 for two.
static int block_tiles(int M, int cols, int tm, int tn) { return ((M + tm - 1) / tm) * ((cols + tn - 1) / tn); }
// Column tiles of 256 that fill whole rounds of the chip, with something left over: the fourth choice (gemm_block_mixed_kernel) is 256 x
// 256 tiles for these columns and 256 x 128 for the rest, where the last round would be less than about half full.  4096 x 6144 (K =
// 4096): 226 -> 195 us; a prompt through four layers, us, best single shape / so: 8B 1200 tokens 2757 / 2684, 3500 tokens 6607 / 6368,
// 8192 tokens 15690 / 15455; 13B 600 tokens 2640 / 2480, 4096 tokens 11920 / 11240.  With a few tiles left over there is little to gain
// (3000 tokens of 13B, 16 of 1296: 8030 / 8100), hence the 4 %: such a round has the chip's power to itself.
static int block_whole_rounds(int M, int cols) {
    const int rounds = block_tiles(M, cols, 256, 256) / 256, n = rounds * 256 / ((M + 255) / 256);
    return rounds > 0 && n * 256 < cols ? n : 0;
}
static int block_tile(int M, int cols, int *cost = nullptr) {
    const int t0 = block_tiles(M, cols, 256, 256), t1 = block_tiles(M, cols, 256, 128), t2 = block_tiles(M, cols, 128, 128), rest = t2 % 512;
    const auto rounds_1 = [](int t) { return t <= 256 ? 58 : (t + 255) / 256 * 65; };
    const int c0 = (t0 + 255) / 256 * 100, c1 = rounds_1(t1);
    const int c2 = t2 / 512 * 68 + (rest == 0 ? 0 : rest <= 256 ? 40 : 68);
    int tile = c0 <= c1 && c0 <= c2 ? 0 : c1 <= c2 ? 1 : 2, c = tile == 0 ? c0 : tile == 1 ? c1 : c2;
    if (const int whole = block_whole_rounds(M, cols)) {
        const int c3 = t0 / 256 * 100 + rounds_1(block_tiles(M, cols - whole * 256, 256, 128));
        // (a round of 256 x 256 tiles that is nearly empty takes 79)
        if (c3 * 1.04 < (tile == 0 ? c0 - 21 * (256 - t0 % 256) / 256 : c)) { tile = 3; c = c3; }
    }
    if (cost) *cost = c;
    return tile;
}

template <typename T, int EPI>
static void launch_block_e(BlockGeom g, const void *Wp, const void *X, int ldx, const EpiArgs &e, hipStream_t st,
                           hipEvent_t ev_start, hipEvent_t ev_stop) {
    const u32x4 *w = static_cast<const u32x4 *>(Wp);
    const T *x = static_cast<const T *>(X);
    const int cols = g.N - g.col0;
#define POSS_BLOCK(TM, TN, WM, WN, NST)                                                                                     \
    do {                                                                                                                    \
        g.tiles_m = (g.M + TM - 1) / TM; g.tiles_n = (cols + TN - 1) / TN;                                                   \
        dim3 grid(g.tiles_m * g.tiles_n, g.splits), block(WM * WN * 64);                                                    \
        if (ev_start && ev_stop)                                                                                            \
            hipExtLaunchKernelGGL((gemm_block_kernel<T, TM, TN, WM, WN, NST, EPI>), grid, block, 0, st, ev_start, ev_stop, 0, w, x, ldx, g, e); \
        else                                                                                                                \
            hipLaunchKernelGGL((gemm_block_kernel<T, TM, TN, WM, WN, NST, EPI>), grid, block, 0, st, w, x, ldx, g, e);      \
    } while (0)
    if constexpr (EPI == EPI_PLAIN) {
        POSS_BLOCK(256, 256, 2, 4, 5);                    // gemm_block_splits() counts on it
    } else {
        const int tile = block_tile(g.M, cols);
        if (tile == 3) {
            BlockGeom rest = g;
            g.tiles_m = rest.tiles_m = (g.M + 255) / 256;
            g.tiles_n = block_whole_rounds(g.M, cols);
            rest.col0 += g.tiles_n * 256;
            rest.tiles_n = (g.N - rest.col0 + 127) / 128;
            dim3 grid(g.tiles_m * (g.tiles_n + rest.tiles_n)), block(512);
            if (ev_start && ev_stop)
                hipExtLaunchKernelGGL((gemm_block_mixed_kernel<T, EPI>), grid, block, 0, st, ev_start, ev_stop, 0, w, x, ldx, g, rest, e);
            else
                hipLaunchKernelGGL((gemm_block_mixed_kernel<T, EPI>), grid, block, 0, st, w, x, ldx, g, rest, e);
        } else if (tile == 0) POSS_BLOCK(256, 256, 2, 4, 5);
        else if (tile == 1) POSS_BLOCK(256, 128, 4, 2, 6);
        else POSS_BLOCK(128, 128, 2, 2, 5);
    }
#undef POSS_BLOCK
}

// K splits of a product whose sums a kernel of its own adds up (the residual + norm epilogue): with few tiles for the chip
// 256 x 256 tiles over a part of K each are faster than small tiles over all of it, the planes included - in us, 109 for a round
// of K = 4096 and 3.5 TB/s for the planes' way out and back, against the same per-K time of the tile chosen without splits.  That
// time is of weights just touched.  A model's come from memory, and the small tiles, whose k-steps are short, feel it.  A product alone, us,
// repeated on one matrix / on matrices that no cache holds: 1001 x 5120 x 5120 by 160 tiles of 256 x 128 72 / 97, 2048 x 4096 x 4096 71 / 80,
// 1001 x 4096 x 4096 by 128 x 128 42 / 49; 256 x 256 the same either way.  Hence the factors, 0.9 where it is whole rounds of large tiles.
// In the trace of a request of 1001 tokens at the 13B shape: N = 5120, K = 5120 103 us and 7 for its norm, in three splits 61 + 25; K = 13824 and 10240
// 114 on average in three splits + 25 and 22 (over all of K 175, with an earlier build).  Prompt and catch-up through four layers, us, all at
// 0.9 / so: 8B 1500 tokens 3880 / 3539, 1700 4021 / 3859, 2048 4464 / 4256, 13B 1001 3696 / 3581, 1280 5129 / 4759, 1536 5421 / 5130; of 47 lengths
// from 513 to 2100 tokens none is slower by more than its runs differ (2 % at most, 3 at 900 of the 8B shape).  Error against 64 bits over 56
// requests whose splits are others, the ratio: logits 0.9998 +- 0.0004, features 0.9999 +- 0.0003.
int gemm_block_splits(int M, int N, int K, size_t part_floats) {
    int cost;
    const int tile = block_tile(M, N, &cost);
    const double per_k = 1.09 * K / 4096.0, t0 = block_tiles(M, N, 256, 256);
    double best = (tile == 1 ? 1.25 : tile == 2 ? 1.15 : 0.9) * cost * per_k;
    int S = 1;
    for (int s = 2; s <= 8 && K / s >= 1024 && (size_t)s * M * N <= part_floats; ++s) {
        const double rounds = (double)(((long long)t0 * s + 255) / 256);
        const double t = rounds * 100 * per_k / s + (double)M * N * 8 * s / 3.5e6;
        if (t < best) { best = t; S = s; }
    }
    return S;
}

template <typename T>
static void launch_block_t(const BlockGeom &g, const void *Wp, const void *X, int ldx, const EpiArgs &e, hipStream_t st,
                           hipEvent_t ev_start, hipEvent_t ev_stop) {
    switch (e.mode) {
        case EPI_ROPE_KV: launch_block_e<T, EPI_ROPE_KV>(g, Wp, X, ldx, e, st, ev_start, ev_stop); break;
        case EPI_RESIDUAL: launch_block_e<T, EPI_RESIDUAL>(g, Wp, X, ldx, e, st, ev_start, ev_stop); break;
        case EPI_PLAIN: launch_block_e<T, EPI_PLAIN>(g, Wp, X, ldx, e, st, ev_start, ev_stop); break;
        default: launch_block_e<T, EPI_SILU>(g, Wp, X, ldx, e, st, ev_start, ev_stop); break;
    }
}

bool launch_gemm_block(int dt, int M, int N, int K, int col0, const void *Wp, const void *X, int ldx, const EpiArgs &e, hipStream_t st,
                       hipEvent_t ev_start, hipEvent_t ev_stop, int splits, float *part) {
    if (!Wp || !X || M < 1 || N < 1 || K < 8 || K % 8 || col0 < 0 || col0 % 32 || col0 >= N || ldx < K || dt == DT_F32) return false;
    switch (e.mode) {
        case EPI_ROPE_KV:
            if (!e.cs || !e.slot || (col0 == 0 && !e.q) || (e.dh != 64 && e.dh != 128) || !e.kv.k || !e.kv.vt || !e.kv.page_table) return false;
            if (col0 != 0 && col0 != e.hq * e.dh) return false;           // all of it, or keys and values alone
            break;
        case EPI_RESIDUAL: if (!e.h || N % 8 || col0) return false; break;
        case EPI_SILU: if (!e.act || e.F % 8 || col0) return false; break;
        case EPI_PLAIN: if (!part || N % 8 || col0 || splits < 2 || splits > K / (2 * GEMM_KSTEP)) return false; break;
        default: return false;
    }
    const int Kpad = gemm_kpad(dt, K);
    if ((size_t)M * ldx * 2 > 0xffffffffull) return false;                // 32-bit lane offsets
    const BlockGeom g{M, N, K, Kpad / GEMM_KSTEP, col0, gemm_npad(N) / 16, 0, 0, e.mode == EPI_PLAIN ? splits : 1, part};
    if (dt == DT_BF16) launch_block_t<bf16_t>(g, Wp, X, ldx, e, st, ev_start, ev_stop); else launch_block_t<f16_t>(g, Wp, X, ldx, e, st, ev_start, ev_stop);
    return true;
}

}  // namespace poss
