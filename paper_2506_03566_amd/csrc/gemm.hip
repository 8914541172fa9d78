// Weight-streaming GEMM for M <= 256 activation rows:  Y[m][n] = sum_k X[m][k] W[n][k], with the
// operation that follows it in a Llama decoder layer fused into its epilogue.
//
// The round is bound by reading every weight once (the verify pass reads the whole target, each
// draft pass one specialist and the shared LM head; sections 3.3 and 6.2 of the paper discuss the
// cost of switching specialist parameters, which is exactly this stream).  Design:
//   * weights pre-packed in MFMA B-operand order: each lane issues 16-byte loads, a wave reads
//     GEMM_NT KiB contiguous per k-step straight into registers (no LDS hop for the big operand);
//   * a ring of PF k-steps of weight loads stays in flight per wave across LDS chunk boundaries;
//   * the (small, L2-resident) activation slice is staged in LDS in A-operand order, double
//     buffered, its global loads issued one chunk ahead so they are older than the weight loads
//     they overlap and never force the weight ring to drain;
//   * K is split across workgroups (as many splits as keep the launch at one workgroup per CU) into
//     partial planes; an epilogue kernel sums them in split order and applies the fused operation:
//     rotary embedding + KV-cache write (tile-parallel), or residual add followed by the RMSNorm
//     that feeds the next GEMM (one workgroup per row).  Bitwise repeatable, and a row's result
//     does not depend on how many rows the launch carries.  (Reducing inside the GEMM by the last
//     workgroup to arrive at a tile was measured 3.5x slower: agent-scope fences write back and
//     invalidate the per-XCD L2s.)
//   * the gate/up projection is not split: gate and up rows are interleaved so that one lane holds
//     both factors, and the kernel writes SiLU(gate) * up in the storage type itself;
//   * three kernels share the packed weights, the split rule and the order of every sum, so a row gets bit for bit
//     the same result from each: the stream kernel (up to 128 rows, bound by the weight stream), the tall kernel
//     (129..256 rows: several sequences in one stream, prefill; gate/up at 244 rows of the 8B shape: 65 us, 52 without loads from
//     memory, 42 without LDS operand reads as well, of which 31 are the MFMAs at the clock that they then hold, 2.1 GHz; the kernel
//     itself runs at 1.9, the matrix pipe busy 55 % of its workgroups' time) and the QKV kernels with the epilogue inside (few rows or
//     small matrices).
#include "attn_merge.h"

#include <hip/hip_ext.h>

#include <type_traits>

namespace poss {

typedef bf16_t bf16x8 __attribute__((ext_vector_type(8)));
typedef f16_t  f16x8 __attribute__((ext_vector_type(8)));

template <typename T> struct Mfma;
template <> struct Mfma<bf16_t> {
    static __device__ __forceinline__ f32x4 run(u32x4 a, u32x4 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
};
template <> struct Mfma<f16_t> {
    static __device__ __forceinline__ f32x4 run(u32x4 a, u32x4 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a),
                                                      __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    }
};

constexpr int KCS = GEMM_KCHUNK / GEMM_KSTEP;   // k-steps per LDS chunk (8)
// PF = weight k-steps in flight per wave (template parameter of the stream kernel): 4, or 8 for launches
// with fewer workgroups than CUs, where each CU has to keep more bytes in flight to fill the memory system.

// ------------------------------------------------------------------------------------------
// Epilogues of split products: the planes are added in split order, loads issued eight at a time.
constexpr int EPI_ROWS_PLAIN = 16;  // rows per workgroup of the plain epilogue,
constexpr int EPI_ROWS_PAIR = 4;    // of the rotary epilogue

__device__ __forceinline__ f32x4 sum_planes4(const float *part, size_t plane, int S, size_t idx) {
    f32x4 a = f32x4{0.f, 0.f, 0.f, 0.f};
    int s = 0;
    for (; s + 8 <= S; s += 8) {
        f32x4 v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = *reinterpret_cast<const f32x4 *>(part + (size_t)(s + j) * plane + idx);
#pragma unroll
        for (int j = 0; j < 8; ++j) a += v[j];
    }
    for (; s + 2 <= S; s += 2) {
        const f32x4 v0 = *reinterpret_cast<const f32x4 *>(part + (size_t)s * plane + idx);
        const f32x4 v1 = *reinterpret_cast<const f32x4 *>(part + (size_t)(s + 1) * plane + idx);
        a = (a + v0) + v1;
    }
    for (; s < S; ++s) a += *reinterpret_cast<const f32x4 *>(part + (size_t)s * plane + idx);
    return a;
}

// ------------------------------------------------------------------------------------------
// WPB waves per workgroup: 4 (one 128-column tile) or 8 (two tiles sharing one staged activation
// slice: halves the L2 traffic per weight byte; used where N alone fills the GPU).
// FUSE_SILU (K not split, gate/up interleaved per wave tile): the kernel applies SiLU(gate) * up to its
// accumulators and writes the activation act[M][F] itself; no partial plane, no epilogue kernel.
// HEAD (K not split, columns = vocabulary): the workgroup reduces its column tile per row in its own epilogue - the
// best (value, index) for greedy verification, or maximum, sum of exponentials and the k best for the drafter's
// log-softmax + top-k - so that no kernel has to read the logits back; they are written only on request.
struct HeadEpi { int mode, k, vocab; float *logits; int logits_rows; float *seg_out; float *pv; int *pi; };

// ---- epilogues on a finished output tile, shared by the stream kernel and the tall kernel --------------------------
// SiLU(gate) * up of a workgroup's rows x TW activation columns, collected in LDS (row stride TW + 8 elements: the four
// row groups of a wave hit different banks) and written out so that a row leaves as one contiguous piece in 16-byte
// stores instead of 16-column fragments of two bytes per lane.
template <typename T, int ROWS, int TW, int NTHREADS>
__device__ __forceinline__ void silu_tile_store(const T *tile, T *__restrict__ act, int M, int F, int f0, int tid) {
    constexpr int TWP = TW + 8, EPV = 16 / (int)sizeof(T), PPR = TW / EPV;   // elements per 16-byte store, pieces per row
    for (int p = tid; p < ROWS * PPR; p += NTHREADS) {
        const int m = p / PPR, f = f0 + (p % PPR) * EPV;
        if (m < M && f + EPV <= F)                       // F is a multiple of 8: a piece is inside or outside as a whole
            *reinterpret_cast<u32x4 *>(act + (size_t)m * F + f) = *reinterpret_cast<const u32x4 *>(tile + m * TWP + (p % PPR) * EPV);
    }
}

// The Head's reduction of a tile of logits in LDS, tile[row][TW] = columns [col0, col0 + TW): one half wave per row (NHW
// of them; the exchanges stay inside a half and in the vector ALU).  HEAD_ARGMAX: the best (value, index) of the row's segment;
// HEAD_TOPK: maximum, sum of exp(l - max) in a fixed order, and the k best, sorted.
// Every workgroup of a Head launch arrives here at the same time, so nothing streams meanwhile and what it costs is instructions
// (four waves to a SIMD).  The k best: the k-th largest of the 32 lanes' maxima is a lower bound of the k-th largest value, so
// the winners are among the values that reach it, a dozen, and those are ranked by counting.  10 rows of 256 columns, k = 10:
// 14.0 thousand cycles by k rounds of (argmax, remove), which remain for rows with more than HEAD_CAND values at the bound, 5.6
// thousand so; the argmax of 61 rows 7.0 -> 3.8 thousand (value first, then the lowest index that holds it).
constexpr int HEAD_CAND = 32;
template <int NVH>
__device__ __forceinline__ void head_topk_rounds(float (&v)[NVH], int hl, int col0, int k, float *rec) {
    float my_v = -INFINITY; int my_i = 0x7fffffff;
    for (int r = 0; r < k; ++r) {
        float wv = -INFINITY; int wi = 0x7fffffff;
#pragma unroll
        for (int j = 0; j < NVH; ++j)
            if (better(v[j], col0 + hl + 32 * j, wv, wi)) { wv = v[j]; wi = col0 + hl + 32 * j; }
        half_argmax(wv, wi);
        if (hl == r) { my_v = wv; my_i = wi; }
#pragma unroll
        for (int j = 0; j < NVH; ++j)
            if (col0 + hl + 32 * j == wi) v[j] = -INFINITY;   // indices are unique: removes exactly the winner
    }
    if (hl < k) {
        rec[2 + hl] = my_v;
        reinterpret_cast<int *>(rec)[2 + TOPK_MAXK + hl] = my_v > -INFINITY ? my_i : 0x7fffffff;
    }
}

// The tile's logits of the first logits_rows rows into the caller's array, a row's columns as one contiguous piece (as the accumulators hold
// them: 64 bytes of four rows per store: 61 rows x 32000 ids 53.3 us the product, 49.3 so; 244 rows 69.6, 67.3).
template <int TW, int NTHREADS>
__device__ __forceinline__ void head_tile_logits(const float *tile, int M, const HeadEpi &he, int col0, int tid) {
    const int rows = min(M, he.logits_rows);
    const bool quads = he.vocab % 4 == 0 && (reinterpret_cast<uintptr_t>(he.logits) & 15) == 0;      // (uniform)
    for (int p = tid; p < rows * (TW / 4); p += NTHREADS) {
        const int m = p / (TW / 4), c = p % (TW / 4) * 4, n = col0 + c;
        const f32x4 v = *reinterpret_cast<const f32x4 *>(tile + m * TW + c);
        float *dst = he.logits + (size_t)m * he.vocab + n;
        if (quads) {
            if (n < he.vocab) *reinterpret_cast<f32x4 *>(dst) = v;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (n + j < he.vocab) dst[j] = v[j];
        }
    }
}

template <int TW, int NHW>
__device__ __forceinline__ void head_tile_reduce(float *tile, int M, const HeadEpi &he, int seg, int n_seg, int tid) {
    constexpr int NVH = TW / 32;
    static_assert(TW >= 2 * HEAD_CAND + 32, "a row's candidates and its lanes' maxima take the place of its logits");
    const int hw = tid >> 5, hl = tid & 31, col0 = seg * TW;
    for (int row = hw; row < M; row += NHW) {
        float v[NVH], lane_max = -INFINITY;
#pragma unroll
        for (int j = 0; j < NVH; ++j) {                   // columns beyond the vocabulary: -inf, with indices above every real one
            const float x = tile[row * TW + hl + 32 * j];
            v[j] = col0 + hl + 32 * j < he.vocab ? x : -INFINITY;
            lane_max = fmaxf(lane_max, v[j]);
        }
        const float mx = half_max(lane_max);
        if (he.mode == HEAD_ARGMAX) {
            int bi = 0x7fffffff;                          // the lowest index that holds the maximum (none: a row of NaN)
#pragma unroll
            for (int j = NVH - 1; j >= 0; --j)
                if (v[j] == mx && col0 + hl + 32 * j < he.vocab) bi = col0 + hl + 32 * j;
            bi = half_min(bi);
            if (hl == 0) { he.pv[(size_t)row * n_seg + seg] = mx; he.pi[(size_t)row * n_seg + seg] = bi; }
            continue;
        }
        float se = 0.f;
#pragma unroll
        for (int j = 0; j < NVH; ++j) se += v[j] > -INFINITY ? expf(v[j] - mx) : 0.f;
        se = half_sum(se);
        float *rec = he.seg_out + ((size_t)row * n_seg + seg) * TOPK_REC;
        if (hl == 0) { rec[0] = mx; rec[1] = se; }
        float *cand_v = tile + row * TW, *maxima = cand_v + 2 * HEAD_CAND;
        int *cand_i = reinterpret_cast<int *>(cand_v + HEAD_CAND);
        wave_lds_sync();                                  // (the row has been read)
        maxima[hl] = lane_max;
        wave_lds_sync();
        int above = 0;                                    // lanes with a larger maximum
#pragma unroll
        for (int j = 0; j < 32; j += 4) {
            const f32x4 o = *reinterpret_cast<const f32x4 *>(maxima + j);
#pragma unroll
            for (int q = 0; q < 4; ++q) above += o[q] > lane_max;
        }
        const float thr = -half_max(above < he.k ? -lane_max : -INFINITY);   // (of equal maxima all count, k or more)
        int cnt = 0;
#pragma unroll
        for (int j = 0; j < NVH; ++j) {
            const bool in = v[j] > -INFINITY && v[j] >= thr;
            const unsigned who = (unsigned)(__ballot(in) >> (tid & 32));
            const int p = cnt + __popc(who & ((1u << hl) - 1u));
            if (in && p < HEAD_CAND) { cand_v[p] = v[j]; cand_i[p] = col0 + hl + 32 * j; }
            cnt += __popc(who);
        }
        wave_lds_sync();
        if (cnt > HEAD_CAND) {
            head_topk_rounds<NVH>(v, hl, col0, he.k, rec);
            continue;
        }
        const float cv = cand_v[hl]; const int ci = cand_i[hl];
        int rank = 0;
        for (int j = 0; j < cnt; j += 4) {
            const f32x4 ov = *reinterpret_cast<const f32x4 *>(cand_v + j);
            const u32x4 oi = *reinterpret_cast<const u32x4 *>(cand_i + j);
#pragma unroll
            for (int q = 0; q < 4; ++q) rank += j + q < cnt && better(ov[q], (int)oi[q], cv, ci);
        }
        if (hl < cnt && rank < he.k) {
            rec[2 + rank] = cv;
            reinterpret_cast<int *>(rec)[2 + TOPK_MAXK + rank] = ci;
        }
        if (hl >= cnt && hl < he.k) {                     // fewer than k values: no entry
            rec[2 + hl] = -INFINITY;
            reinterpret_cast<int *>(rec)[2 + TOPK_MAXK + hl] = 0x7fffffff;
        }
    }
}

__device__ __forceinline__ int xs_swizzle(int g) { return (0xea40 >> (4 * g)) & 15; }   // f(g) = 0, 4, 10, 14

template <typename T, int MT, int WPB, bool FUSE_SILU, int PF, bool HEAD = false>
__global__ __launch_bounds__(WPB * 64) void gemm_stream_kernel(
    const u32x4 *__restrict__ Wp, const T *__restrict__ X, int ldx, float *__restrict__ part,
    int M, int K, int Npad, int ksteps_total, T *__restrict__ act, int F, HeadEpi he) {
    static_assert(KCS % PF == 0, "ring index must be static");
    constexpr int XUNITS = KCS * MT * 64;                 // 16-byte units of one staged chunk
    // units per thread; where 64 * WPB does not divide the units the last threads stage the last unit again
    constexpr int XPT    = (XUNITS + WPB * 64 - 1) / (WPB * 64);
    __shared__ u32x4 xs[2][XUNITS];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    // split y of gridDim.y owns chunks [y * n / S, (y + 1) * n / S): sizes differ by at most one chunk
    const int n_chunks_total = ksteps_total / KCS;
    const int chunk0 = (int)blockIdx.y * n_chunks_total / (int)gridDim.y;
    const int chunk1 = ((int)blockIdx.y + 1) * n_chunks_total / (int)gridDim.y;
    const int ngroup = blockIdx.x * WPB + wave;
    const u32x4 *wp = Wp + ((size_t)ngroup * ksteps_total + (size_t)chunk0 * KCS) * (GEMM_NT * 64) + lane;

    // Global->LDS staging map: a wave instruction covers one A-operand block [k_step][m_tile] (64 units of 16
    // bytes): four consecutive lanes take the four 8-element groups of one row's k-step (64 contiguous bytes in
    // global memory), consecutive quads take consecutive rows.  In LDS the block is stored in operand order with the
    // row index swizzled by the k-group, unit g * 16 + (m ^ f(g)), f = {0, 4, 10, 14}: the four units a quad stores
    // (same row, g = 0..3) would otherwise lie 256 bytes apart, in the same banks; with f the 8 and the 16 lanes that
    // the LDS takes together always store to 8 and 16 different 16-byte columns, and a read (16 lanes of one g, all rows)
    // still covers one contiguous 256 bytes.
    // Loads are never predicated (a predicated load becomes a branch, and the compiler then waits
    // for every outstanding load at it): out-of-range units read a clamped, valid address and are
    // zeroed by a select.
    const T *x_src[XPT];
    int x_k[XPT], x_dst[XPT];
    bool x_row_ok[XPT];
#pragma unroll
    for (int i = 0; i < XPT; ++i) {
        const int u = min(tid + i * (WPB * 64), XUNITS - 1);
        const int blk = u >> 6, ln = u & 63;
        const int m = (blk % MT) * 16 + (ln >> 2), k8 = (blk / MT) * 4 + (ln & 3);
        x_row_ok[i] = m < M;
        x_src[i] = X + (size_t)(m < M ? m : M - 1) * ldx;
        x_k[i] = k8 * 8;
        x_dst[i] = blk * 64 + ((ln & 3) << 4) + ((ln >> 2) ^ xs_swizzle(ln & 3));
    }
    auto load_x = [&](int chunk, u32x4 (&xr)[XPT]) {
#pragma unroll
        for (int i = 0; i < XPT; ++i) {
            const int k = chunk * GEMM_KCHUNK + x_k[i];
            xr[i] = *reinterpret_cast<const u32x4 *>(x_src[i] + (k < K ? k : K - 8));
        }
    };
    auto store_x = [&](int chunk, int b, const u32x4 (&xr)[XPT]) {   // the select happens here, not at the load
#pragma unroll
        for (int i = 0; i < XPT; ++i) {
            const bool ok = x_row_ok[i] && chunk * GEMM_KCHUNK + x_k[i] < K;
            xs[b][x_dst[i]] = ok ? xr[i] : u32x4{0u, 0u, 0u, 0u};
        }
    };

    f32x4 acc[MT][GEMM_NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < GEMM_NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};

    u32x4 xr[XPT];
    load_x(chunk0, xr);
    u32x4 wr[PF][GEMM_NT];
#pragma unroll
    for (int p = 0; p < PF; ++p) {                   // a workgroup owns at least one chunk (KCS >= PF steps)
#pragma unroll
        for (int nt = 0; nt < GEMM_NT; ++nt) wr[p][nt] = __builtin_nontemporal_load(wp + nt * 64);
        wp += GEMM_NT * 64;
    }
    store_x(chunk0, 0, xr);
    __syncthreads();

    // One chunk of KCS k-steps.  MORE (another chunk follows) is a compile-time flag so that the
    // body is straight-line code: the weight ring is refilled PF steps ahead, across the chunk
    // boundary when MORE, and the next chunk's activations are requested before any of it.
    int buf = 0;
    const int lane_sw = (lane & 48) + ((lane & 15) ^ xs_swizzle(lane >> 4));   // this lane's A fragment inside a block
    auto chunk_body = [&](auto more_tag, int chunk) {
        constexpr bool MORE = decltype(more_tag)::value;
        if constexpr (MORE) load_x(chunk + 1, xr);
        __builtin_amdgcn_sched_barrier(0);           // keep these loads older than the weight loads below
        // A fragments of k-step i + 1 are requested from LDS before the MFMAs of k-step i are issued
        u32x4 a[2][MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) a[0][mt] = xs[buf][mt * 64 + lane_sw];
#pragma unroll
        for (int i = 0; i < KCS; ++i) {
            if (i + 1 < KCS) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) a[(i + 1) & 1][mt] = xs[buf][((i + 1) * MT + mt) * 64 + lane_sw];
            }
            // The MFMAs read the ring slot itself and the slot is refilled after them: with a copy taken first (so that
            // the refill could be issued ahead of the MFMAs) the compiler gathers the copies of all slots at the top of
            // the chunk and waits there for the whole ring, which empties the memory pipeline once per chunk.
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int nt = 0; nt < GEMM_NT; ++nt) acc[mt][nt] = Mfma<T>::run(a[i & 1][mt], wr[i % PF][nt], acc[mt][nt]);
            if (MORE || i + PF < KCS) {
#pragma unroll
                for (int nt = 0; nt < GEMM_NT; ++nt) wr[i % PF][nt] = __builtin_nontemporal_load(wp + nt * 64);
                wp += GEMM_NT * 64;
            }
            __builtin_amdgcn_sched_barrier(0);       // one k-step at a time: loads stay in ring order
        }
        if constexpr (MORE) {
            store_x(chunk + 1, buf ^ 1, xr);
            __syncthreads();
            buf ^= 1;
        }
    };
    for (int chunk = chunk0; chunk + 1 < chunk1; ++chunk) chunk_body(std::true_type{}, chunk);
    chunk_body(std::false_type{}, chunk1 - 1);

    // D tile: lane -> column n = lane % 16, register r -> row m = 4 * (lane / 16) + r
    if constexpr (FUSE_SILU) {
        static_assert(GEMM_NT == 2, "gate and up are the two column tiles of a wave");
        // The waves of the workgroup own WPB * 16 consecutive columns of act.  The tile is collected in LDS (the
        // staging memory, free after a barrier) so that a row leaves as one contiguous piece in 16-byte stores
        // instead of 16-column fragments written two bytes per lane.
        constexpr int TW = WPB * 16, TWP = TW + 8;       // padded row: the four row groups of a wave hit different banks
        static_assert((size_t)MT * 16 * TWP * sizeof(T) <= sizeof(xs), "the tile fits the staging memory");
        T *tile = reinterpret_cast<T *>(&xs[0][0]);
        __syncthreads();                                 // every wave has read its last operand fragments
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float g = acc[mt][0][r], up = acc[mt][1][r];
                tile[(mt * 16 + 4 * (lane >> 4) + r) * TWP + wave * 16 + (lane & 15)] = mul_round<T>(g / (1.0f + expf(-g)), up);
            }
        __syncthreads();
        silu_tile_store<T, MT * 16, TW, WPB * 64>(tile, act, M, F, blockIdx.x * TW, tid);
        return;
    }
    if constexpr (HEAD) {
        constexpr int TW = WPB * GEMM_NT * 16;           // columns of the workgroup's tile = one segment
        static_assert((size_t)MT * 16 * TW * sizeof(float) <= sizeof(xs), "the tile fits the staging memory");
        float *tile = reinterpret_cast<float *>(&xs[0][0]);
        __syncthreads();                                 // every wave has read its last operand fragments
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < GEMM_NT; ++nt)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    tile[(mt * 16 + 4 * (lane >> 4) + r) * TW + wave * (GEMM_NT * 16) + nt * 16 + (lane & 15)] = acc[mt][nt][r];
        __syncthreads();
        if (he.logits) {
            head_tile_logits<TW, WPB * 64>(tile, M, he, blockIdx.x * TW, tid);
            __syncthreads();                             // (the reduction works in the tile)
        }
        head_tile_reduce<TW, WPB * 2>(tile, M, he, blockIdx.x, gridDim.x, tid);
        return;
    }
    float *out = part + (size_t)blockIdx.y * (MT * 16) * Npad;
    const int n0 = ngroup * (GEMM_NT * 16) + (lane & 15);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < GEMM_NT; ++nt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = mt * 16 + 4 * (lane >> 4) + r;
                if (MT > 1 || m < M) out[(size_t)m * Npad + n0 + nt * 16] = acc[mt][nt][r];   // (rows beyond M are never read)
            }
}

// ------------------------------------------------------------------------------------------
// The output projection of up to 16 rows, whose attention splits every workgroup merges for itself: the heads its K split covers, all
// rows, into LDS in A-operand order, ahead of a loop that has no barrier.  Splits of K, order of the sums and planes are the
// streaming kernel's, the merge is attn_merge_kernel's: the same bits.  What it saves is a launch (4.8 us); what it costs is that the
// column tiles of a split repeat the merge (rows x K of the split x splits x 4 bytes a workgroup), which is why it is for few rows.
// us, product + merge / so: 13B, 1 row of 1024 keys (20 KB) 9.6 + 4.8 / 10.2, 8B, 10 rows of 512 keys (82 KB) 9.0 + 4.9 / 10.9: two of
// the five for 82 KB, hence the line at 96.  A thread's first quads are asked for ahead of the weights.
constexpr size_t MERGED_BYTES = (size_t)96 << 10;
template <typename T, int NR, int QB>                     // QB: quads of a thread at a time
__global__ __launch_bounds__(256) void gemm_merged_kernel(const u32x4 *__restrict__ Wp, AttnMerge src, float *__restrict__ part, int M, int K,
                                                          int Npad, int ksteps_total) {
    constexpr int PF = KCS;                               // weight k-steps in flight
    struct __attribute__((aligned(8))) Quad { T t[4]; };
    extern __shared__ __attribute__((aligned(16))) u32x4 xm[];          // [k-step of the split][64]
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int n_chunks_total = ksteps_total / KCS;
    const int ks0 = (int)blockIdx.y * n_chunks_total / (int)gridDim.y * KCS;
    const int n_ks = ((int)blockIdx.y + 1) * n_chunks_total / (int)gridDim.y * KCS - ks0;
    const int ngroup = blockIdx.x * 4 + wave, quads = n_ks * 8, G = src.hq / src.hkv;
    const size_t stride = (size_t)src.hkv * src.rho_pad;
    MergeQuad<NR> mq[QB];
    auto request = [&](int i0) {                          // quads i0 + tid, i0 + 256 + tid, ..: an index beyond the last re-reads it
#pragma unroll
        for (int j = 0; j < QB; ++j) {
            const int i = min(i0 + j * 256 + tid, M * quads - 1), m = i / quads, k = min(ks0 * GEMM_KSTEP + (i % quads) * 4, K - 4);
            const int qh = k / src.dh;
            const size_t row = (size_t)(qh / G) * src.rho_pad + m * G + qh % G;
            mq[j].load(src.o + row * src.dh + k % src.dh, src.ml + row * 2, stride, src.dh, src.n_splits);
        }
    };
    auto finish = [&](int i0) {
#pragma unroll
        for (int j = 0; j < QB; ++j) {
            const int i = i0 + j * 256 + tid, m = i / quads, kq = i % quads, ks = kq >> 3, g = (kq >> 1) & 3;
            if (i >= M * quads) continue;
            f32x4 num; float den;
            mq[j].merge(src.n_splits, num, den);
            const bool in = ks0 * GEMM_KSTEP + kq * 4 < K;               // (beyond K the weights are zero)
            Quad o;
#pragma unroll
            for (int r = 0; r < 4; ++r) o.t[r] = in ? from_f<T>(num[r] / den) : from_f<T>(0.f);
            *reinterpret_cast<Quad *>(reinterpret_cast<char *>(&xm[ks * 64 + g * 16 + (m ^ xs_swizzle(g))]) + (kq & 1) * 8) = o;
        }
    };
    request(0);
    __builtin_amdgcn_sched_barrier(0);                    // these loads ahead of the weights
    const u32x4 *wp = Wp + ((size_t)ngroup * ksteps_total + ks0) * (GEMM_NT * 64) + lane;
    u32x4 wr[PF][GEMM_NT];
#pragma unroll
    for (int p = 0; p < PF; ++p)
#pragma unroll
        for (int nt = 0; nt < GEMM_NT; ++nt) wr[p][nt] = __builtin_nontemporal_load(wp + (size_t)p * (GEMM_NT * 64) + nt * 64);
    __builtin_amdgcn_sched_barrier(0);
    finish(0);
    for (int i0 = QB * 256; i0 < M * quads; i0 += QB * 256) { request(i0); finish(i0); }
    __syncthreads();

    f32x4 acc[GEMM_NT];
#pragma unroll
    for (int nt = 0; nt < GEMM_NT; ++nt) acc[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int lane_sw = (lane & 48) + ((lane & 15) ^ xs_swizzle(lane >> 4));
    auto group = [&](auto more_tag, int g) {              // PF k-steps; the ring is refilled for the next PF
        constexpr bool MORE = decltype(more_tag)::value;
        u32x4 a[PF];
#pragma unroll
        for (int p = 0; p < PF; ++p) a[p] = xm[(g + p) * 64 + lane_sw];
#pragma unroll
        for (int p = 0; p < PF; ++p) {
#pragma unroll
            for (int nt = 0; nt < GEMM_NT; ++nt) acc[nt] = Mfma<T>::run(a[p], wr[p][nt], acc[nt]);
            if constexpr (MORE) {
#pragma unroll
                for (int nt = 0; nt < GEMM_NT; ++nt) wr[p][nt] = __builtin_nontemporal_load(wp + (size_t)(g + PF + p) * (GEMM_NT * 64) + nt * 64);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    for (int g = 0; g + PF < n_ks; g += PF) group(std::true_type{}, g);
    group(std::false_type{}, n_ks - PF);
    float *out = part + (size_t)blockIdx.y * 16 * Npad;
    const int n0 = ngroup * (GEMM_NT * 16) + (lane & 15);
#pragma unroll
    for (int nt = 0; nt < GEMM_NT; ++nt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = 4 * (lane >> 4) + r;
            if (m < M) out[(size_t)m * Npad + n0 + nt * 16] = acc[nt][r];
        }
}

// ------------------------------------------------------------------------------------------
// The same product for 129..256 rows (several sequences verified in one weight stream, prefill).  At that height a
// workgroup's 256 x 128 tile needs 16 KB of activations and 8 KB of weights per k-step and every workgroup re-reads the
// whole activation matrix.  Counters and timestamps of earlier versions of this kernel: with operands fetched by the
// waves that multiply (weights into registers, activations through registers into LDS) the matrix pipe was busy 29 % of
// the time, the waves waiting for loads 53 %, and 963 MB went through the L1s for 235 MB of weights, because the two
// waves that share a column group each fetched its weights; with both operands staged in LDS by LDS-direct loads, each
// fetched once, a wave still sat 450 - 1300 cycles of a 2600-cycle stage in the ISSUE of its six loads (the CU's vector
// memory pipe takes in about 64 bytes a cycle, and a wave issues in order: while it waits to issue a load it issues no
// MFMA), wherever in the stage the loads were put.  So the work is split by wave:
//   eight consumer waves, two per SIMD: wave (wm, wn) owns the rows [128 wm, 128 wm + 128) of the 32 columns wn of the
//       tile, reads its operand fragments from LDS and issues MFMAs, nothing else;
//   eight producer waves, two per SIMD, issue the loads, three stages of two k-steps (48 KB each) deep, and wait for
//       them (four of them were slower: a wave issues an LDS-direct load only every 100 - 250 cycles).
// Staging, by 16-byte LDS-direct loads (no staging registers, no masks):
//   activations: a stage holds 256 rows x 64 k, a row's 128 bytes (both k-steps) contiguous, its eight 16-byte units
//       xor-swizzled by a function of the row - eight consecutive lanes fetch one row's 128 bytes, a whole line of the
//       L2 (four lanes and 64 bytes, one k-step, made twice the requests), and an operand read (lane % 16 the row,
//       lane / 16 the k-group) runs at the full LDS rate;
//   weights: the packed layout is already the B-operand image, 1 KB per (k-step, column tile), copied as it is.  Matrices of
//       TALL_ONCE_BYTES and more with non-temporal loads: a workgroup's weights are its own, the activations are everyone's and
//       should stay in the L2.  Smaller ones fit the eight L2s (32 MB) beside the activations and are still in the caches when
//       the next pass comes.  Four sequences of 61 rows, four layers, us a pass, ordinary loads / non-temporal / by this rule:
//       8B shape (33 MB and more) 899 / 880 / 866, 2048 wide 536 / 532 / 525, 640 wide (5 MB and less, Head 41) 403 / 425 / 399.
// Rows >= M and k >= K are not zeroed: such a lane fetches a valid element of the matrix instead (row M - 1, k = 0);
// the rows are never read back and the packed weights are zero beyond K.
// Splits own whole groups of 8 k-steps as in the stream kernel and a wave adds its k-steps in ascending order, so a
// row's sums are bit for bit those of the stream kernel.
constexpr size_t TALL_ONCE_BYTES = (size_t)24 << 20;
constexpr int TALL_KCL = 2, TALL_NST = 3, TALL_THREADS = 1024;   // (row tiles per workgroup, MT: 16, or 12 for up to 192 rows)

// position of 16-byte unit u of row r (of a 16-row tile) inside the row's 128 bytes: u ^ tall_x_swizzle(r)
__device__ __forceinline__ int tall_x_swizzle(int r) { return (((r >> 1) & 1) << 2) | ((r >> 1) & 3); }

template <typename T, int MT, bool FUSE_SILU, bool HEAD>
__global__ __launch_bounds__(TALL_THREADS) void gemm_tall_kernel(
    const u32x4 *__restrict__ Wp, const T *__restrict__ X, int ldx, float *__restrict__ part,
    int M, int K, int Npad, int ksteps_total, int w_once, T *__restrict__ act, int F, HeadEpi he) {
    typedef __attribute__((address_space(3))) void *LdsPtr;
    constexpr int KCL = TALL_KCL, NST = TALL_NST, MTW = MT / 2;
    static_assert(KCS % KCL == 0, "a split's k-steps are whole stages");
    static_assert(KCL == 2 && GEMM_NT == 2 && (MT == 16 || MT == 12), "the schedules below are written for these");
    constexpr int XBLKS = KCL * MT, WBLKS = KCL * 4 * GEMM_NT;           // 1 KB blocks of a stage: activations, weights
    constexpr int XPP = XBLKS / 8;                                       // activation blocks per producer wave
    constexpr int STAGE_UNITS = (XBLKS + WBLKS) * 64;
    constexpr int LPS = (XBLKS + WBLKS) / 8;                             // loads of a producer wave per stage
    __shared__ __attribute__((aligned(1024))) u32x4 xs[NST * STAGE_UNITS];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const bool producer = wave >= 8;                      // wave-uniform
    const int wn = wave & 3, wm = (wave >> 2) & 1;
    const int n_chunks_total = ksteps_total / KCS;
    const int chunk0 = ((int)blockIdx.y * n_chunks_total / (int)gridDim.y) * (KCS / KCL);          // in stages
    const int chunk1 = (((int)blockIdx.y + 1) * n_chunks_total / (int)gridDim.y) * (KCS / KCL);
    const int ngroup = blockIdx.x * 4 + wn;

    f32x4 acc[MTW][GEMM_NT];
#pragma unroll
    for (int mt = 0; mt < MTW; ++mt)
#pragma unroll
        for (int nt = 0; nt < GEMM_NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};

    if (producer) {
        // Producer p = wave - 8 brings the blocks p, p + 8, p + 16 (, p + 24) of the stage's activations (block b = rows
        // 8 b .. 8 b + 7, eight lanes per row: the unit that belongs at the lane's position under the swizzle) and the two
        // column tiles of (k-step p / 4, column group p % 4).
        const int pw = wave - 8;
        const int f_row = lane >> 3;
        const T *x_row[XPP];
        int f_k[XPP];
#pragma unroll
        for (int j = 0; j < XPP; ++j) {
            const int m = (pw + 8 * j) * 8 + f_row;
            x_row[j] = X + (size_t)(m < M ? m : M - 1) * ldx;
            f_k[j] = ((lane & 7) ^ tall_x_swizzle(m & 15)) * 8;
        }
        const u32x4 *w_src = Wp + ((size_t)(blockIdx.x * 4 + (pw & 3)) * ksteps_total + (pw >> 2)) * (GEMM_NT * 64) + lane;
        const unsigned lds0 = (unsigned)(uintptr_t)(LdsPtr)&xs[0];
        auto fetch = [&](int chunk, int st) {             // stage st <- k-steps chunk KCL .. + KCL - 1
            const unsigned base = lds0 + (unsigned)(st * STAGE_UNITS * 16);
#pragma unroll
            for (int j = 0; j < XPP; ++j) {
                const int k = chunk * (KCL * GEMM_KSTEP) + f_k[j];
                lds_dma16(base + (unsigned)((pw + 8 * j) * 1024), x_row[j] + (k < K ? k : 0));
            }
#pragma unroll
            for (int nt = 0; nt < GEMM_NT; ++nt) {
                const unsigned dst = base + (unsigned)((XBLKS + ((pw >> 2) * 4 + (pw & 3)) * GEMM_NT + nt) * 1024);
                const u32x4 *src = w_src + (size_t)chunk * KCL * (GEMM_NT * 64) + nt * 64;
                if (w_once) lds_dma16_nt(dst, src); else lds_dma16(dst, src);      // (wave-uniform)
            }
        };
        static_assert(LPS == XPP + GEMM_NT && XBLKS == 8 * XPP, "the fetch above brings exactly one stage");
        fetch(chunk0, 0);
        if (chunk0 + 1 < chunk1) { fetch(chunk0 + 1, 1); dma_wait<LPS>(); } else dma_wait<0>();
        __syncthreads();
        int st = 0;
        for (int chunk = chunk0; chunk < chunk1; ++chunk) {
            // stage (st + 2) % 3 was read last in the iteration before this one: every wave is past that barrier;
            // the next stage has landed once only the loads just issued are outstanding
            if (chunk + 2 < chunk1) { fetch(chunk + 2, st == 0 ? 2 : st - 1); dma_wait<LPS>(); } else dma_wait<0>();
            __syncthreads();
            st = st == NST - 1 ? 0 : st + 1;
        }
    } else {
        // operand reads of this wave inside a stage, in 16-byte units
        const int a_row = (wm * MTW) * 128 + (lane & 15) * 8, a_swz = tall_x_swizzle(lane & 15), lg = lane >> 4;
        const int b_unit = XBLKS * 64 + wn * GEMM_NT * 64 + lane;
        __syncthreads();
        int st = 0;
        for (int chunk = chunk0; chunk < chunk1; ++chunk) {
            // The fragments of the stage's first k-step are asked for at once - the only LDS wait of the stage; those of the
            // second follow one by one behind the first k-step's MFMAs.  (The order is given to the scheduler as it stands:
            // left alone it puts every read next to its use and waits for it there.)
            const u32x4 *xa = &xs[st * STAGE_UNITS + a_row], *wb = &xs[st * STAGE_UNITS + b_unit];
            u32x4 w[KCL][GEMM_NT], a[KCL][MTW];
#pragma unroll
            for (int ks = 0; ks < KCL; ++ks) {
#pragma unroll
                for (int nt = 0; nt < GEMM_NT; ++nt) w[ks][nt] = wb[(ks * 4 * GEMM_NT + nt) * 64];
#pragma unroll
                for (int mt = 0; mt < MTW; ++mt) a[ks][mt] = xa[mt * 128 + ((ks * 4 + lg) ^ a_swz)];
            }
#pragma unroll
            for (int ks = 0; ks < KCL; ++ks)
#pragma unroll
                for (int mt = 0; mt < MTW; ++mt)
#pragma unroll
                    for (int nt = 0; nt < GEMM_NT; ++nt) acc[mt][nt] = Mfma<T>::run(a[ks][mt], w[ks][nt], acc[mt][nt]);
            constexpr int FR = GEMM_NT + MTW, MF = MTW * GEMM_NT;          // fragments and MFMAs of a k-step
            static_assert(MF >= FR && MF <= 2 * FR, "one or two MFMAs of the first k-step ahead of every read of the second");
            __builtin_amdgcn_sched_group_barrier(0x100, FR, 0);
#pragma unroll
            for (int i = 0; i < MF - FR; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
#pragma unroll
            for (int i = 0; i < 2 * FR - MF; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x008, MTW * GEMM_NT, 0);
            __syncthreads();
            st = st == NST - 1 ? 0 : st + 1;
        }
    }

    // D tile: lane -> column n = lane % 16, register r -> row m = 4 * (lane / 16) + r of row tile wm * MTW + mt.
    // (The producer waves take part in the barriers below and in nothing else.)
    const int row0 = wm * (MTW * 16) + 4 * (lane >> 4);
    if constexpr (FUSE_SILU) {
        constexpr int TW = 4 * 16, TWP = TW + 8;
        static_assert((size_t)MT * 16 * TWP * sizeof(T) <= sizeof(xs), "the tile fits the staging memory");
        T *tile = reinterpret_cast<T *>(&xs[0]);
        __syncthreads();                                 // every wave has read its last operand fragments
        if (!producer) {
#pragma unroll
            for (int mt = 0; mt < MTW; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float g = acc[mt][0][r], up = acc[mt][1][r];
                    tile[(row0 + mt * 16 + r) * TWP + wn * 16 + (lane & 15)] = mul_round<T>(g / (1.0f + expf(-g)), up);
                }
        }
        __syncthreads();
        if (!producer) silu_tile_store<T, MT * 16, TW, 512>(tile, act, M, F, blockIdx.x * TW, tid);
        return;
    }
    if constexpr (HEAD) {
        constexpr int TW = 4 * GEMM_NT * 16;
        static_assert((size_t)MT * 16 * TW * sizeof(float) <= sizeof(xs), "the tile fits the staging memory");
        float *tile = reinterpret_cast<float *>(&xs[0]);
        __syncthreads();
        if (!producer) {
#pragma unroll
            for (int mt = 0; mt < MTW; ++mt)
#pragma unroll
                for (int nt = 0; nt < GEMM_NT; ++nt)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        tile[(row0 + mt * 16 + r) * TW + wn * (GEMM_NT * 16) + nt * 16 + (lane & 15)] = acc[mt][nt][r];
        }
        __syncthreads();
        if (he.logits) {
            head_tile_logits<TW, TALL_THREADS>(tile, M, he, blockIdx.x * TW, tid);
            __syncthreads();                              // (the reduction works in the tile)
        }
        if (!producer) head_tile_reduce<TW, 16>(tile, M, he, blockIdx.x, gridDim.x, tid);
        return;
    }
    if (producer) return;
    float *out = part + (size_t)blockIdx.y * (MT * 16) * Npad;
    const int n0 = ngroup * (GEMM_NT * 16) + (lane & 15);
#pragma unroll
    for (int mt = 0; mt < MTW; ++mt)
#pragma unroll
        for (int nt = 0; nt < GEMM_NT; ++nt)
#pragma unroll
            for (int r = 0; r < 4; ++r) out[(size_t)(row0 + mt * 16 + r) * Npad + n0 + nt * 16] = acc[mt][nt][r];
}

// ------------------------------------------------------------------------------------------
// The QKV projection with its epilogue inside: K split INSIDE the workgroup.  One 32-column tile per workgroup; a pair of waves owns a
// K split - the very splits, and inside them the very order, of the streaming kernel.  Each brings half of the pair's operands into LDS
// by LDS-direct loads, two k-steps a stage, NST stages in a ring: activations in whole 128-byte lines under the swizzle of
// gemm_tall_kernel, weights as they are packed.  A pair's waves take half of the row tiles each (one row tile: of the columns).  The
// partial tiles meet in LDS and are added in split order, so the workgroup holds finished sums and applies the rotary embedding and
// writes queries, keys and values itself: no partial planes, no epilogue kernel.  The weight rows are packed so that the two 16-column
// tiles of a group are dims [16j, 16j+16) and [16j + dh/2, ..) of one head: a lane owns both members of a rotary pair.
// Bitwise repeatable; a row's result does not depend on the rows around it.
// Every workgroup reads every row over the whole K, so it is for few rows or small matrices (QKV_FUSED_BYTES below).
constexpr int QKV_MAX_SPLITS = 4;
constexpr int QKV_STAGE_BYTES(int mt) { return (2 * mt + 2 * GEMM_NT) * 1024; }   // of one wave
struct QkvEpi { const float2 *cs; const int32_t *slot; void *q; int hq, hkv, dh; RopeRanges rr; };

// What the epilogue needs of a lane's four rows (4 * (lane / 16) .. of row tile mt) besides their sums, for head gh and rotary pair i:
// asked for ahead of the partial tiles' exchange, whatever the rows turn out to be (row by row, behind the branches on what a row is,
// the same loads were a dependent trip to memory each).
struct QkvRows { float2 cs[4]; int slot[4], page[4]; };
__device__ __forceinline__ void qkv_rows(const QkvEpi &e, int gh, int i, int mt, int M, int lane, QkvRows &rows) {
    const int half = e.dh >> 1, m0 = mt * 16 + 4 * (lane >> 4);
    if (gh >= e.hq) {                                     // (workgroup-uniform)
#pragma unroll
        for (int r = 0; r < 4; ++r) rows.slot[r] = e.slot[min(m0 + r, M - 1)];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) rows.cs[r] = e.cs[min(m0 + r, M - 1) * half + i];
}
__device__ __forceinline__ void qkv_pages(const QkvEpi &e, int gh, QkvRows &rows) {   // of their slots; the slots have to be there
    if (gh >= e.hq) {
#pragma unroll
        for (int r = 0; r < 4; ++r)                       // (all ranges have one page table: ranges_ok)
            rows.page[r] = e.rr.kv[0].page_table[rows.slot[r] >> e.rr.kv[0].page_shift];
    }
}
// The finished sums x1, x2 of pair (i, i + dh / 2) of head gh for a lane's four rows, rotated and written.
template <typename T>
__device__ __forceinline__ void qkv_store(const QkvEpi &e, int gh, int i, int mt, int M, int lane, f32x4 x1, f32x4 x2, const QkvRows &rows) {
    const int half = e.dh >> 1;
    if (gh >= e.hq + 2 * e.hkv) return;                   // padding columns
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int m = mt * 16 + 4 * (lane >> 4) + r;
        float o1, o2;
        rope_pair(x1[r], x2[r], rows.cs[r], o1, o2);
        for (int qi = 0; qi < e.rr.n; ++qi) {             // (workgroup-uniform) the sequences that share this launch
            if (m < e.rr.r0[qi] || m >= e.rr.r1[qi] || m >= M) continue;
            const KVCache &kv = e.rr.kv[qi];
            if (gh < e.hq) {
                if (m >= e.rr.rows_q[qi]) continue;
                T *dst = static_cast<T *>(e.q) + ((size_t)m * e.hq + gh) * e.dh;
                dst[i] = round_f<T>(o1);
                dst[i + half] = round_f<T>(o2);
            } else if (gh < e.hq + e.hkv) {
                T *dst = static_cast<T *>(kv.k) + k_offset_in(kv, rows.page[r], rows.slot[r], gh - e.hq, e.hkv, e.dh);
                dst[i] = round_f<T>(o1);
                dst[i + half] = round_f<T>(o2);
            } else {
                T *dst = static_cast<T *>(kv.vt) + vt_offset_in(kv, rows.page[r], rows.slot[r], gh - e.hq - e.hkv, e.hkv, e.dh, i);
                dst[0] = from_f<T>(x1[r]);
                dst[(size_t)half << kv.page_shift] = from_f<T>(x2[r]);
            }
        }
    }
}
// The partial tiles of S splits, red[split][row tile, column tile][64], added in split order (as sum_planes4 adds planes), rotated and
// written.  D tile: lane -> column lane % 16, register r -> row 4 * (lane / 16) + r.  Wave w of n_waves finishes row tiles w, w + n_waves, ..,
// the first of them with the rows it has been given.
template <typename T, int MT>
__device__ __forceinline__ void qkv_epilogue(const f32x4 *red, int S, int gh, int i, int M, int wave, int n_waves, int lane, const QkvEpi &e, QkvRows &rows) {
    for (int mt = wave; mt < MT; mt += n_waves) {
        if (mt != wave) {
            qkv_rows(e, gh, i, mt, M, lane, rows);
            qkv_pages(e, gh, rows);
        }
        f32x4 x1 = f32x4{0.f, 0.f, 0.f, 0.f}, x2 = x1;
        for (int sp = 0; sp < S; ++sp) {
            x1 += red[(sp * (MT * GEMM_NT) + mt * GEMM_NT) * 64 + lane];
            x2 += red[(sp * (MT * GEMM_NT) + mt * GEMM_NT + 1) * 64 + lane];
        }
        qkv_store<T>(e, gh, i, mt, M, lane, x1, x2, rows);
    }
}

template <typename T, int MT, int NST>
__global__ __launch_bounds__(QKV_MAX_SPLITS * 128) void gemm_qkv_rope_kernel(const u32x4 *__restrict__ Wp, const T *__restrict__ X, int ldx,
                                                                             int M, int K, int ksteps_total, QkvEpi e) {
    typedef __attribute__((address_space(3))) void *LdsPtr;
    constexpr int NTILE = MT * GEMM_NT;
    constexpr int XBLKS = 2 * MT, BLKS = XBLKS + 2 * GEMM_NT;        // 1 KB blocks of a stage (two k-steps): activations, then weights
    constexpr int XPW = XBLKS / 2, LPW = BLKS / 2;                   // of which a wave of the pair loads half
    constexpr int MTW = MT > 1 ? MT / 2 : 1, NTW = MT > 1 ? GEMM_NT : 1;   // what it multiplies: half of the row tiles (one row tile: of the columns)
    static_assert(BLKS * 1024 == QKV_STAGE_BYTES(MT) && GEMM_NT == 2 && (MT == 1 || MT % 2 == 0) && KCS % 2 == 0, "two equal halves, whole stages");
    extern __shared__ __attribute__((aligned(1024))) u32x4 qlds[];   // [split][NST][BLKS * 64]; at the end [split][NTILE][64] partial tiles
    const int S = blockDim.x >> 7, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, tile = blockIdx.x;
    const int split = wave >> 1, p = wave & 1, lr = lane & 15, lg = lane >> 4;
    const int n_chunks = ksteps_total / KCS, k0 = split * n_chunks / S * KCS, n_st = ((split + 1) * n_chunks / S * KCS - k0) / 2;
    const int n_most = (n_chunks + S - 1) / S * (KCS / 2);           // stages of the longest split
    const u32x4 *w_src = Wp + ((size_t)tile * ksteps_total + k0) * (GEMM_NT * 64) + p * 64 + lane;
    const T *x_row[XPW];                                  // load j: rows 8 (2 j + p) + lane / 8, eight lanes per row
    int f_k[XPW];
#pragma unroll
    for (int j = 0; j < XPW; ++j) {
        const int m = (2 * j + p) * 8 + (lane >> 3);
        x_row[j] = X + (size_t)(m < M ? m : M - 1) * ldx;             // rows beyond M repeat the last (never stored)
        f_k[j] = k0 * GEMM_KSTEP + ((lane & 7) ^ tall_x_swizzle(m & 15)) * 8;
    }
    const unsigned lds0 = (unsigned)(uintptr_t)(LdsPtr)qlds + (unsigned)(split * NST * BLKS * 1024 + p * 1024);
    auto fetch = [&](int st) {
        const unsigned base = lds0 + (unsigned)((st % NST) * BLKS * 1024);
#pragma unroll
        for (int i = 0; i < 2; ++i) lds_dma16_nt(base + (XBLKS + 2 * i) * 1024, w_src + (size_t)(st * 2 + i) * (GEMM_NT * 64));
#pragma unroll
        for (int j = 0; j < XPW; ++j) {
            const int k = f_k[j] + st * (2 * GEMM_KSTEP);             // beyond K (the packed weights are zero there): the row's first elements
            lds_dma16(base + 2 * j * 1024, x_row[j] + (k < K ? k : 0));
        }
    };
    f32x4 acc[MTW][NTW];
#pragma unroll
    for (int mt = 0; mt < MTW; ++mt)
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int mt0 = MT > 1 ? p * MTW : 0, nt0 = MT > 1 ? 0 : p;
    const u32x4 *xb = qlds + split * NST * BLKS * 64 + mt0 * 128 + lr * 8, *wb = qlds + (split * NST * BLKS + XBLKS + nt0) * 64 + lane;
    const int swz = tall_x_swizzle(lr);
#pragma unroll
    for (int st = 0; st < NST - 1; ++st) if (st < n_st) fetch(st);
    for (int st = 0; st < n_most; ++st) {
        // the stage has landed once only the loads of the NST - 2 behind it are outstanding; behind the barrier its other half has,
        // too, and every wave has read the stage before it for the last time
        if (st + NST - 1 <= n_st) dma_wait<(NST - 2) * LPW>(); else dma_wait<0>();
        __syncthreads();
        if (st + NST - 1 < n_st) fetch(st + NST - 1);
        if (st < n_st) {                                  // (wave-uniform)
            const int at = (st % NST) * BLKS * 64;
            u32x4 a[2][MTW], w[2][NTW];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
                for (int nt = 0; nt < NTW; ++nt) w[ks][nt] = wb[at + (ks * GEMM_NT + nt) * 64];
#pragma unroll
                for (int mt = 0; mt < MTW; ++mt) a[ks][mt] = xb[at + mt * 128 + ((ks * 4 + lg) ^ swz)];
            }
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int mt = 0; mt < MTW; ++mt)
#pragma unroll
                    for (int nt = 0; nt < NTW; ++nt) acc[mt][nt] = Mfma<T>::run(a[ks][mt], w[ks][nt], acc[mt][nt]);
        }
    }
    const int tph = e.dh >> 5, gh = tile / tph, pi = (tile % tph) * 16 + (lane & 15);   // 32-column tiles per head; the lane's pair
    QkvRows rows;
    if (wave < MT) {
        qkv_rows(e, gh, pi, wave, M, lane, rows);
        qkv_pages(e, gh, rows);
    }
    __syncthreads();                                      // every wave is done with its stages
    f32x4 *red = reinterpret_cast<f32x4 *>(qlds);
#pragma unroll
    for (int mt = 0; mt < MTW; ++mt)
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt) red[(split * NTILE + (mt0 + mt) * GEMM_NT + nt0 + nt) * 64 + lane] = acc[mt][nt];
    __syncthreads();
    qkv_epilogue<T, MT>(red, S, gh, pi, M, wave, 2 * S, lane, e, rows);
}

// One row tile and four splits (plain decoding and the first drafting passes at the 8B shape): a wave's operands straight into
// registers, PF k-steps in flight (an A fragment of v_mfma 16x16x32 is 16 contiguous bytes of one activation row, and with K split
// among the waves no two of them want the same fragment): no LDS hop, no barrier in the loop.  4096 -> 6144, us with the boundary to
// the next launch, this kernel / the one above: 1 row 10.1 / 11.2, 10 rows 11.7 / 12.2; two row tiles of it, 20 rows 13.8 / 13.1,
// 31 rows 16.1 / 14.0 (64-byte pieces of the rows).  Other widths, passes of four layers, 1 and 8 rows: 2048 -> 3072 241 / 250 and 249 / 256,
// 2048 -> 6144 242 / 246 and 248 / 254, 6144 -> 8192 529 / 528 and 538 / 541; 16 rows within 1 %.
template <typename T, int PF>
__global__ __launch_bounds__(256) void gemm_qkv_row_kernel(const u32x4 *__restrict__ Wp, const T *__restrict__ X, int ldx,
                                                           int M, int K, int ksteps_total, QkvEpi e) {
    __shared__ f32x4 red[4 * GEMM_NT * 64];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, tile = blockIdx.x;
    const int w0 = wave * ksteps_total / 4, w1 = (wave + 1) * ksteps_total / 4, n_w = w1 - w0;
    const u32x4 *wp = Wp + ((size_t)tile * ksteps_total + w0) * (GEMM_NT * 64) + lane;      // this wave's first k-step
    const T *xp = X + (size_t)min(lane & 15, M - 1) * ldx + (size_t)w0 * GEMM_KSTEP + (lane >> 4) * 8;   // rows beyond M repeat the last row
    f32x4 acc[GEMM_NT];
#pragma unroll
    for (int nt = 0; nt < GEMM_NT; ++nt) acc[nt] = f32x4{0.f, 0.f, 0.f, 0.f};

    int done = 0;
    if (w1 * GEMM_KSTEP <= K && n_w >= PF) {             // no k-step of this wave reaches beyond K: loads need no mask
        u32x4 wr[PF][GEMM_NT], ar[PF];
        auto load_step = [&](int p, int i) {             // k-step w0 + i into ring slot p (p static after unrolling)
#pragma unroll
            for (int nt = 0; nt < GEMM_NT; ++nt) wr[p][nt] = __builtin_nontemporal_load(wp + (size_t)i * (GEMM_NT * 64) + nt * 64);
            ar[p] = *reinterpret_cast<const u32x4 *>(xp + (size_t)i * GEMM_KSTEP);
        };
#pragma unroll
        for (int p = 0; p < PF; ++p) load_step(p, p);
        const int groups = n_w / PF;
        auto group = [&](auto more_tag, int g) {
            constexpr bool MORE = decltype(more_tag)::value;
#pragma unroll
            for (int p = 0; p < PF; ++p) {
                u32x4 w[GEMM_NT];
                const u32x4 a = ar[p];
#pragma unroll
                for (int nt = 0; nt < GEMM_NT; ++nt) w[nt] = wr[p][nt];
                if constexpr (MORE) load_step(p, (g + 1) * PF + p);
#pragma unroll
                for (int nt = 0; nt < GEMM_NT; ++nt) acc[nt] = Mfma<T>::run(a, w[nt], acc[nt]);
                __builtin_amdgcn_sched_barrier(0);       // one k-step at a time: loads stay in ring order
            }
        };
        for (int g = 0; g + 1 < groups; ++g) group(std::true_type{}, g);
        group(std::false_type{}, groups - 1);
        done = groups * PF;
    }
    for (int i = done; i < n_w; ++i) {                   // what the ring did not cover; fragments beyond K are zero
        const bool ok = (w0 + i) * GEMM_KSTEP + (lane >> 4) * 8 < K;
        u32x4 w[GEMM_NT];
#pragma unroll
        for (int nt = 0; nt < GEMM_NT; ++nt) w[nt] = wp[(size_t)i * (GEMM_NT * 64) + nt * 64];
        const u32x4 v = *reinterpret_cast<const u32x4 *>(ok ? xp + (size_t)i * GEMM_KSTEP : xp - (size_t)w0 * GEMM_KSTEP - (lane >> 4) * 8);
        const u32x4 a = ok ? v : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int nt = 0; nt < GEMM_NT; ++nt) acc[nt] = Mfma<T>::run(a, w[nt], acc[nt]);
    }

    const int tph = e.dh >> 5, gh = tile / tph, pi = (tile % tph) * 16 + (lane & 15);   // 32-column tiles per head; the lane's pair
    QkvRows rows;
    if (wave == 0) {
        qkv_rows(e, gh, pi, 0, M, lane, rows);
        qkv_pages(e, gh, rows);
    }
#pragma unroll
    for (int nt = 0; nt < GEMM_NT; ++nt) red[(wave * GEMM_NT + nt) * 64 + lane] = acc[nt];
    __syncthreads();
    qkv_epilogue<T, 1>(red, 4, gh, pi, M, wave, 4, lane, e, rows);
}

// ------------------------------------------------------------------------------------------
// One row: the residual addition and the norm in the product that follows (RowNorm).  As a kernel of its own a row's norm is one
// workgroup and 5.2 us, half of it the boundary between two launches; here every workgroup adds the planes up for itself (S x d x 4
// bytes, 100 to 130 KB at the 8B and 13B shapes, out of the L2s) while its first weights are on their way, and keeps the normed row in
// LDS, where an A fragment of all sixteen rows is one broadcast read: the loop has no staging and no barrier, and 128 KB of weights a CU
// are in flight.  For two rows the planes would be twice as much and the saving the same.  us, stream + norm / so: 13B gate/up 41.9 + 5.2 /
// 44.3, QKV 27.7 + 5.2 / 27.3, 8B gate/up 37.7 + 4.5 / 37.0; a pass of one row of the 13B shape through four layers, 1024 keys, with
// the merge above 631 -> 587.  Groups of four columns, partial sums of squares and their order are epilogue_residual_norm_kernel's
// (wave v of that kernel is a virtual wave here): the same bits.
// The groups are dealt out to W waves: slot s < NV of a wave is virtual wave wave + W s (NV = 16 / W), the slots behind those the same
// virtual waves' second turn (d > 4096); NSL slots are formed, every plane of theirs requested at once (NP planes: slots beyond S re-read
// the last), ahead of the weights, which `ahead` asks for.
static __host__ __device__ __forceinline__ int norm_threads(int d) { return min(1024, (d / 4 + 63) / 64 * 64); }
constexpr int row_slots(int d, int W) { return d <= 4096 ? 16 / W : 16 / W + (d - 4096 + 256 * W - 1) / (256 * W); }

template <typename T, int NP, int NSL, int W, typename Ahead>
__device__ __forceinline__ void row_norm(const RowNorm &p, T *urow, int Kpad, float *red, int tid, bool writer, Ahead ahead) {
    struct __attribute__((aligned(4 * sizeof(T)))) Quad { T t[4]; };
    constexpr int NV = 16 / W;
    static_assert(NV * W == 16 && NSL >= NV && NSL <= 2 * NV, "slots of one or two turns");
    const int wave = tid >> 6, lane = tid & 63, threads = norm_threads(p.d), nvw = threads >> 6;
    const T *bias = static_cast<const T *>(p.bias), *gain = static_cast<const T *>(p.gain);
    auto column = [&](int s) {
        const int vw = wave + W * (s % NV), n = ((s / NV) * threads + vw * 64 + lane) * 4;
        return vw < nvw && n < p.d ? n : -1;
    };
    f32x4 v[NSL][NP], add[NSL];
    Quad bq[NSL], gq[NSL];
#pragma unroll
    for (int j = 0; j < NSL; ++j) {
        const int n = max(column(j), 0);                  // (a slot without columns reads the first ones and drops them)
#pragma unroll
        for (int s = 0; s < NP; ++s) v[j][s] = *reinterpret_cast<const f32x4 *>(p.part + (size_t)min(s, p.S - 1) * p.plane + n);
        add[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (p.residual) add[j] = *reinterpret_cast<const f32x4 *>(p.h + n);
        if (bias) bq[j] = *reinterpret_cast<const Quad *>(bias + n);
        gq[j] = *reinterpret_cast<const Quad *>(gain + n);
    }
    __builtin_amdgcn_sched_barrier(0);
    ahead();
    __builtin_amdgcn_sched_barrier(0);
    f32x4 x[NSL];
#pragma unroll
    for (int j = 0; j < NSL; ++j) {
        f32x4 a = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NP; ++s) if (s < p.S) a += v[j][s];
#pragma unroll
        for (int r = 0; r < 4; ++r) if (bias) add[j][r] += to_f(bq[j].t[r]);
        x[j] = a + add[j];
        const int n = column(j);
        if (writer && n >= 0) *reinterpret_cast<f32x4 *>(p.h_out + n) = x[j];
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        float ss = 0.f;
#pragma unroll
        for (int s = j; s < NSL; s += NV)
            if (column(s) >= 0)
#pragma unroll
                for (int r = 0; r < 4; ++r) ss = fmaf(x[s][r], x[s][r], ss);
        ss = wave_sum(ss);
        if (lane == 0 && wave + W * j < nvw) red[wave + W * j] = ss;
    }
    for (int k = p.d + tid; k < Kpad; k += W * 64) urow[k] = from_f<T>(0.f);    // beyond K the weights are zero
    __syncthreads();
    float sum = 0.f;
    for (int i = 0; i < nvw; ++i) sum += red[i];
    const float rs = 1.0f / sqrtf(sum / (float)p.d + p.eps);
#pragma unroll
    for (int j = 0; j < NSL; ++j) {
        const int n = column(j);
        if (n < 0) continue;
        Quad o;
#pragma unroll
        for (int r = 0; r < 4; ++r) o.t[r] = mul_round<T>(x[j][r] * rs, to_f(gq[j].t[r]));
        *reinterpret_cast<Quad *>(urow + n) = o;
    }
    __syncthreads();
}

// The products of a wave: its NTW column tiles, k-steps [0, n_w) of its stream (whole groups of 8), the row's fragments from LDS.  16 / NTW
// k-steps are in flight, the first of them asked for ahead; k-steps beyond the last repeat it.
constexpr int ROW_PF(int ntw) { return 16 / ntw; }
template <int NTW>
__device__ __forceinline__ void row_fetch(const u32x4 *__restrict__ wp, int ks, int n_w, u32x4 (&w)[NTW]) {
    const u32x4 *src = wp + (size_t)min(ks, n_w - 1) * (GEMM_NT * 64);
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt) w[nt] = __builtin_nontemporal_load(src + nt * 64);
}
template <typename T, int NTW>
__device__ __forceinline__ void row_products(const u32x4 *__restrict__ wp, int n_w, const u32x4 *frag, u32x4 (&wr)[ROW_PF(NTW)][NTW], f32x4 (&acc)[NTW]) {
    constexpr int PF = ROW_PF(NTW);
    auto group = [&](auto more_tag, auto steps_tag, int g) {
        constexpr bool MORE = decltype(more_tag)::value;
        constexpr int STEPS = decltype(steps_tag)::value;
        u32x4 a[STEPS];
#pragma unroll
        for (int p = 0; p < STEPS; ++p) a[p] = frag[(g + p) * 4];
#pragma unroll
        for (int p = 0; p < STEPS; ++p) {
#pragma unroll
            for (int nt = 0; nt < NTW; ++nt) acc[nt] = Mfma<T>::run(a[p], wr[p][nt], acc[nt]);
            if constexpr (MORE) row_fetch<NTW>(wp, g + PF + p, n_w, wr[p]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    int g = 0;
    for (; g + PF < n_w; g += PF) group(std::true_type{}, std::integral_constant<int, PF>{}, g);
    if (n_w - g == PF) group(std::false_type{}, std::integral_constant<int, PF>{}, g);
    else group(std::false_type{}, std::integral_constant<int, KCS>{}, g);       // (PF = 16 and 8 k-steps left)
}

// gate/up, K unsplit: a 128-column tile per workgroup, a 16-column tile per wave.  The gate and the up of a unit then lie in two waves
// and meet in LDS.
constexpr int ROW_SILU_WAVES = 8, ROW_QKV_WAVES = 4;
template <typename T, int NP, int NSL>
__global__ __launch_bounds__(ROW_SILU_WAVES * 64) void gemm_row_silu_kernel(const u32x4 *__restrict__ Wp, RowNorm norm, int ksteps_total,
                                                                            T *__restrict__ act, int F) {
    constexpr int PF = ROW_PF(1);
    extern __shared__ __attribute__((aligned(16))) u32x4 rlds[];        // the row
    __shared__ float red[17], ups[64];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, ngroup = blockIdx.x * 4 + (wave >> 1), nt = wave & 1;
    const u32x4 *wp = Wp + (size_t)ngroup * ksteps_total * (GEMM_NT * 64) + nt * 64 + lane;
    u32x4 wr[PF][1];
    row_norm<T, NP, NSL, ROW_SILU_WAVES>(norm, reinterpret_cast<T *>(rlds), ksteps_total * GEMM_KSTEP, red, tid, blockIdx.x == 0, [&] {
#pragma unroll
        for (int p = 0; p < PF; ++p) row_fetch<1>(wp, p, ksteps_total, wr[p]);
    });
    f32x4 acc[1] = {f32x4{0.f, 0.f, 0.f, 0.f}};
    row_products<T, 1>(wp, ksteps_total, rlds + (lane >> 4), wr, acc);
    if (nt == 1 && lane < 16) ups[(wave >> 1) * 16 + lane] = acc[0][0];        // D tile: row 0 is register 0 of lanes 0 .. 15
    __syncthreads();
    const int f = ngroup * 16 + lane;
    if (nt == 0 && lane < 16 && f < F) {
        const float g = acc[0][0];
        act[f] = mul_round<T>(g / (1.0f + expf(-g)), ups[(wave >> 1) * 16 + lane]);
    }
}

// The QKV projection, a 32-column tile per workgroup, K split inside it: four splits, a wave each, or (NTW = 1) one or two, a pair of
// waves each, which take a 16-column tile (one split: the other pair only norms).
template <typename T, int NP, int NSL, int NTW>
__global__ __launch_bounds__(ROW_QKV_WAVES * 64, 2) void gemm_row_qkv_kernel(const u32x4 *__restrict__ Wp, RowNorm norm, int ksteps_total, QkvEpi e, int S) {
    constexpr int PF = ROW_PF(NTW);
    extern __shared__ __attribute__((aligned(16))) u32x4 rlds[];        // the row; at the end [split][GEMM_NT][64] partial tiles
    __shared__ float red[17];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, tile = blockIdx.x;
    const int split = min(NTW == GEMM_NT ? wave : wave >> 1, S - 1), nt0 = NTW == GEMM_NT ? 0 : wave & 1;
    const bool multiplies = NTW == GEMM_NT || (wave >> 1) < S;          // (wave-uniform)
    const int n_chunks = ksteps_total / KCS, k0 = split * n_chunks / S * KCS, n_w = (split + 1) * n_chunks / S * KCS - k0;
    const u32x4 *wp = Wp + ((size_t)tile * ksteps_total + k0) * (GEMM_NT * 64) + nt0 * 64 + lane;
    u32x4 wr[PF][NTW];
    row_norm<T, NP, NSL, ROW_QKV_WAVES>(norm, reinterpret_cast<T *>(rlds), ksteps_total * GEMM_KSTEP, red, tid, blockIdx.x == 0, [&] {
        if (!multiplies) return;
#pragma unroll
        for (int p = 0; p < PF; ++p) row_fetch<NTW>(wp, p, n_w, wr[p]);
    });
    f32x4 acc[NTW];
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt) acc[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (multiplies) row_products<T, NTW>(wp, n_w, rlds + k0 * 4 + (lane >> 4), wr, acc);
    const int tph = e.dh >> 5, gh = tile / tph, pi = (tile % tph) * 16 + (lane & 15);
    QkvRows rows;
    if (wave == 0) {
        qkv_rows(e, gh, pi, 0, 1, lane, rows);
        qkv_pages(e, gh, rows);
    }
    __syncthreads();                                      // every wave has read its fragments
    f32x4 *tiles = reinterpret_cast<f32x4 *>(rlds);
    if (multiplies) {
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt) tiles[(split * GEMM_NT + nt0 + nt) * 64 + lane] = acc[nt];
    }
    __syncthreads();
    qkv_epilogue<T, 1>(tiles, S, gh, pi, 1, wave, ROW_QKV_WAVES, lane, e, rows);
}

// ------------------------------------------------------------------------------------------
// One product with a ROW-MAJOR matrix (a caller that has no packed weights and calls once): no repacking, no partial planes,
// one launch.  A workgroup takes 16 columns x 16 MT rows; wave s computes K split s - the very splits, and inside them the
// very order, of the streaming kernels - and the splits' tiles are added in split order, so the result is bit for bit that of
// packing, streaming and summing.  A wave brings its own operands into its own corner of LDS (no barrier), two k-steps and
// whole 128-byte lines at a time, in the swizzled order of gemm_tall_kernel: fetched as operands, 64 bytes of 16 rows per
// instruction, the same bytes took the CU's memory pipe twice as long.  NST stages in a ring: four where LDS holds them (few
// splits: few waves to hide the latency), otherwise two.
// With operands just touched, 61 x 1720 x 5000: pack 9.6 + stream 6.1 + sum 3.6 us -> 8.9 us (14.5 fetched as operands into
// registers); 1 x 512 x 512: three launches of 8.0 us -> 2.9 us.  With operands that no cache holds the call gains less: 61 x 1700 x
// 5000 23.7 -> 16.4 us from event to event, 1 x 512 x 512 11.1 -> 6.3.
constexpr int DIRECT_MAX_SPLITS = 16;
__device__ const u32x4 direct_zero = {0u, 0u, 0u, 0u};    // what a lane fetches where its k lies beyond K

template <typename T, int MT, int NST>
__global__ __launch_bounds__(DIRECT_MAX_SPLITS * 64) void gemm_direct_kernel(const T *__restrict__ W, const T *__restrict__ X,
                                                                            float *__restrict__ y, int M, int N, int K, int n_chunks, int mparts) {
    typedef __attribute__((address_space(3))) void *LdsPtr;
    constexpr int TILES = MT + 1, STAGE = TILES * 128;    // 16-row operand tiles of a stage (the last: weights), 16-byte units
    extern __shared__ __attribute__((aligned(1024))) u32x4 dlds[];   // [wave][NST][STAGE]; at the end [wave][MT][64] partial tiles
    const int S = blockDim.x >> 6, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
    // the row parts of a column tile read the same weights: ids equal modulo 8 (one XCD), one after the other
    const int xcd = blockIdx.x & 7, qid = blockIdx.x >> 3;
    const int n0 = ((qid / mparts) * 8 + xcd) * 16, m0 = (qid % mparts) * (16 * MT);
    if (n0 >= N) return;
    const int k0 = wave * n_chunks / S * KCS, k1 = min((wave + 1) * n_chunks / S * KCS, (K + GEMM_KSTEP - 1) / GEMM_KSTEP);
    const int n_st = (k1 - k0 + 1) / 2;                   // stages of two k-steps (what lies beyond K is zero)
    const T *src[TILES][2];                               // load i of a tile: its rows 8 i + lane / 8, eight lanes per row
    int kk[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = i * 8 + (lane >> 3);
        kk[i] = ((lane & 7) ^ tall_x_swizzle(r)) * 8;
#pragma unroll
        for (int t = 0; t < MT; ++t) src[t][i] = X + (size_t)min(m0 + t * 16 + r, M - 1) * K + kk[i];   // rows and columns beyond the
        src[MT][i] = W + (size_t)min(n0 + r, N - 1) * K + kk[i];                                        // matrix repeat the last (never stored)
    }
    const unsigned lds0 = (unsigned)(uintptr_t)(LdsPtr)dlds + (unsigned)(wave * NST * STAGE * 16);
    auto fetch = [&](int st) {
#pragma unroll
        for (int t = 0; t < TILES; ++t)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int k = (k0 + 2 * st) * GEMM_KSTEP;
                const void *p = k + kk[i] < K ? static_cast<const void *>(src[t][i] + k) : static_cast<const void *>(&direct_zero);
                lds_dma16(lds0 + (unsigned)(((st % NST) * STAGE + t * 128 + i * 64) * 16), p);
            }
    };
    f32x4 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    const u32x4 *mine = dlds + wave * NST * STAGE + lr * 8;
    const int swz = tall_x_swizzle(lr);
#pragma unroll
    for (int st = 0; st < NST; ++st) if (st < n_st) fetch(st);
    for (int st = 0; st < n_st; ++st) {
        if (st + NST <= n_st) dma_wait<(NST - 1) * TILES * 2>(); else dma_wait<0>();
        const u32x4 *base = mine + (st % NST) * STAGE;
        u32x4 f[2][TILES];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int t = 0; t < TILES; ++t) f[ks][t] = base[t * 128 + ((ks * 4 + lg) ^ swz)];
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // this stage has been read: its place may be filled again
        if (st + NST < n_st) fetch(st + NST);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[mt] = Mfma<T>::run(f[ks][mt], f[ks][MT], acc[mt]);
    }
    __syncthreads();                                      // every wave is done with its stages
    f32x4 *red = reinterpret_cast<f32x4 *>(dlds);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) red[(wave * MT + mt) * 64 + lane] = acc[mt];
    __syncthreads();
    for (int mt = wave; mt < MT; mt += S) {
        f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int s = 0; s < S; ++s) v += red[(s * MT + mt) * 64 + lane];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = m0 + mt * 16 + lg * 4 + r;
            if (m < M && n0 + lr < N) y[(size_t)m * N + n0 + lr] = v[r];
        }
    }
}

// Does [a, a + an) share a byte with [b, b + bn)?  A kernel that writes its result while other workgroups still read the operands
// must not be given a result that lies over them; through partial planes (every operand is read before the result is written)
// it may.
static bool overlap(const void *a, size_t an, const void *b, size_t bn) {
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return x < y + bn && y < x + an;
}

bool launch_gemm_direct(int dt, const GemmShape &g, const void *W, const void *X, float *y, hipStream_t st) {
    if (dt == DT_F32 || !W || !X || !y || g.M < 1 || g.M > MAX_ROWS || g.N < 1 || g.K < 8 || g.K % 8 || g.S < 1 || g.S > DIRECT_MAX_SPLITS) return false;
    if ((reinterpret_cast<uintptr_t>(W) | reinterpret_cast<uintptr_t>(X)) % 16) return false;      // 16-byte loads to LDS
    const size_t y_bytes = (size_t)g.M * g.N * sizeof(float);
    if (overlap(y, y_bytes, X, (size_t)g.M * g.K * 2) || overlap(y, y_bytes, W, (size_t)g.N * g.K * 2)) return false;
    // two row tiles per workgroup where there are two and the stages fit; the stages of S waves within 160 KB (64 KB asked for
    // with one or two splits leaves room for more than one workgroup per CU)
    const int row_tiles = (g.M + 15) / 16, mt = row_tiles == 1 || g.S > 13 ? 1 : 2, mparts = (row_tiles + mt - 1) / mt, ctiles = (g.N + 15) / 16;
    const size_t stage = (size_t)g.S * (mt + 1) * 128 * 16;
    const int nst = stage * 4 <= 160 * 1024 ? 4 : 2;
    dim3 grid(8 * mparts * ((ctiles + 7) / 8)), block(g.S * 64);
    const int n_chunks = g.Kpad / GEMM_KCHUNK;
#define POSS_DIRECT(T, MT, NST)                                                                                              \
    hipLaunchKernelGGL((gemm_direct_kernel<T, MT, NST>), grid, block, stage * NST, st, static_cast<const T *>(W), static_cast<const T *>(X), y, \
                       g.M, g.N, g.K, n_chunks, mparts)
#define POSS_DIRECT_T(T)                                                                                                     \
    do {                                                                                                                     \
        if (mt == 1) { if (nst == 4) POSS_DIRECT(T, 1, 4); else POSS_DIRECT(T, 1, 2); }                                       \
        else         { if (nst == 4) POSS_DIRECT(T, 2, 4); else POSS_DIRECT(T, 2, 2); }                                       \
    } while (0)
    if (dt == DT_BF16) POSS_DIRECT_T(bf16_t); else POSS_DIRECT_T(f16_t);
#undef POSS_DIRECT_T
#undef POSS_DIRECT
    return true;
}

// ------------------------------------------------------------------------------------------
// Residual epilogue, one workgroup per row: h = sum of planes (+ bias) (+ h); then, because the
// whole row is in this workgroup, the RMSNorm that feeds the next GEMM right away:
// u = T(h / sqrt(mean(h^2) + eps) * gain).  Saves a kernel per norm.
// (16-bit types.)  A thread owns MAXIT groups of four columns (N is a multiple of 4); each operand of a group is
// one load, all of them requested before the first use: one trip to memory (column by column the same loads sat behind branches:
// the round of the 8B shape 6040 -> 5888 us, 76 launches of it; one row of the 13B shape 668 -> 635 us a pass).
template <typename T>
__global__ __launch_bounds__(1024) void epilogue_residual_norm_kernel(const float *__restrict__ part, size_t plane, int S,
                                                                      int Npad, int N, float eps, EpiArgs e) {
    struct __attribute__((aligned(4 * sizeof(T)))) Quad { T t[4]; };
    __shared__ float red[17];
    constexpr int MAXIT = 4;                               // N <= 4 * 4 * 1024
    const int m = blockIdx.x;
    const T *bias = static_cast<const T *>(e.bias), *gain = static_cast<const T *>(e.gain);
    T *u = static_cast<T *>(e.u);
    float *h = e.h + (size_t)m * N, *h_copy = e.h_copy ? e.h_copy + (size_t)m * N : nullptr;
    float *h_user = e.h_user && m < e.h_user_rows ? e.h_user + (size_t)m * N : nullptr;
    f32x4 x[MAXIT], gn[MAXIT];
    float ss = 0.f;
#pragma unroll
    for (int it = 0; it < MAXIT; ++it) {
        const int n = (it * (int)blockDim.x + (int)threadIdx.x) * 4;
        x[it] = f32x4{0.f, 0.f, 0.f, 0.f};
        gn[it] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (n < N) {
            f32x4 add = f32x4{0.f, 0.f, 0.f, 0.f};
            Quad bq, gq;
            if (e.residual) add = *reinterpret_cast<const f32x4 *>(h + n);
            if (bias) bq = *reinterpret_cast<const Quad *>(bias + n);
            if (gain) gq = *reinterpret_cast<const Quad *>(gain + n);
            const f32x4 v = sum_planes4(part, plane, S, (size_t)m * Npad + n);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (bias) add[j] += to_f(bq.t[j]);
                if (gain) gn[it][j] = to_f(gq.t[j]);
            }
            x[it] = v + add;
            *reinterpret_cast<f32x4 *>(h + n) = x[it];
            if (h_copy) *reinterpret_cast<f32x4 *>(h_copy + n) = x[it];
            if (h_user) *reinterpret_cast<f32x4 *>(h_user + n) = x[it];
            if (e.h_stash) {
                Quad o;
#pragma unroll
                for (int j = 0; j < 4; ++j) o.t[j] = from_f<T>(x[it][j]);
                *reinterpret_cast<Quad *>(static_cast<T *>(e.h_stash) + (size_t)m * N + n) = o;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) ss = fmaf(x[it][j], x[it][j], ss);   // (spelt out: which product is rounded on its own is not left to the compiler)
        }
    }
    if (!gain) return;
    ss = block_sum(ss, red);
    const float rs = 1.0f / sqrtf(ss / (float)N + eps);
#pragma unroll
    for (int it = 0; it < MAXIT; ++it) {
        const int n = (it * (int)blockDim.x + (int)threadIdx.x) * 4;
        if (n >= N) continue;
        Quad o;
#pragma unroll
        for (int j = 0; j < 4; ++j) o.t[j] = mul_round<T>(x[it][j] * rs, gn[it][j]);
        *reinterpret_cast<Quad *>(u + (size_t)m * N + n) = o;
    }
}

// ------------------------------------------------------------------------------------------
// float32 storage (reference-precision mode of the small test shape), weights row-major, on v_mfma_f32_16x16x4_f32 (float32
// products and sums).  The products are small and what they cost is latency: a workgroup takes 16 MT rows x 16 NT columns, its
// four waves a quarter of the k-steps of 16 each, straight from memory into registers - a lane fetches four consecutive k of
// one row, and the four MFMAs of a k-step take one of them each, the same permutation of k on both sides - and the four
// partial tiles are added in wave order.  F32_PF k-steps are in flight.  A row's sums depend on K alone.
// 64 x 768 x 256: 36.7 -> 3.7 us, 4 x 256 x 256: 46.7 -> 4.0 us (before: one thread per output, walking k and a row of W of
// its own); 128 x 1700 x 2400 by 32 x 32 tiles: 26 us (40 TFLOP/s).  (8 and 16 waves, 2 to 8 k-steps in flight: within 0.3 us.)
// EPI (NT = 2): the sums are whole, so the epilogue of gate and up (columns 32 b .. are the gates of 16 units, the next 16 their ups)
// or of the QKV projection (columns of 16 rotary pairs of a head: dims 16 j .. and their partners, dh / 2 further) is applied to them
// here, in the operations and the order of the kernels that do it to planes: one launch of 4.4 us instead of 3.8 + 2.9 for gate and up,
// 5.8 instead of 4.0 + 4.4 for QKV (its slots and pages are a chain of three loads), and a boundary between launches less.  A request
// of the 256 wide shape (prompt and first round, with topk_row_kernel): 773 -> 667 us, 163 -> 134 launches.
constexpr int F32_WAVES = 4, F32_PF = 4, F32_KSTEP = 16;
// The residual addition (EPI_RESIDUAL, no norm behind it) is applied to the whole sums as well, and a norm belongs to the product that
// reads the normed rows (NORM): x gain is formed where an operand is used, the sum of squares beside it, by the waves that hold
// the row's k anyway, and the sums are scaled by 1 / rms at the end.  The same request: 134 -> 96 launches, 675 -> 621 and 668 -> 606 us in
// two comparisons (runs of one side differ by 12 and 18 %).  Error against 64 bits over 160 requests, the ratio to norms and
// additions in kernels of their own: logits 0.998 +- 0.002, features 0.999 +- 0.002.
// Every column tile sums the squares again, which wide layers with few rows notice and wide layers with many do not.  Two layers, us, norms in
// kernels of their own / so: drafting six levels, 4 rows 256 wide 325 / 295, 512 389 / 364, 1024 491 / 482, 2048 848 / 865, 4096 1901 / 1940;
// verifying 61 rows 256 130 / 123, 1024 227 / 232, 2048 542 / 536, 4096 1282 / 1260; a prompt of 256 tokens 256 218 / 199, 1024 590 / 582, 2048
// 1536 / 1483, 4096 5411 / 5144, of 1000 tokens 4096 25136 / 24077.  So at every width: a line would have to lie at a number of
// rows, and a row's bits must not hang on how many rows share a pass.
struct F32Epi {
    float *act; int F; QkvEpi qkv;
    float *h, *h_copy, *h_user; int h_user_rows, residual; const float *bias;
    const float *gain; float eps;
};

template <int MT, int NT, bool VEC, int EPI, bool NORM>
__global__ __launch_bounds__(F32_WAVES * 64) void gemm_f32_kernel(const float *__restrict__ W, const float *__restrict__ X, int ldx,
                                                                  float *__restrict__ out, int ld_out, int M, int N, int K, F32Epi epi) {
    static_assert(EPI == EPI_PLAIN || EPI == EPI_RESIDUAL || NT == 2, "a lane holds both columns of a pair");
    __shared__ f32x4 red[F32_WAVES][MT * NT][64];
    __shared__ float squares[F32_WAVES][MT * 16];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
    const int m0 = blockIdx.y * (16 * MT), half = epi.qkv.dh >> 1;
    const int n0 = EPI == EPI_ROPE_KV ? (int)blockIdx.x / (half >> 4) * epi.qkv.dh + (int)blockIdx.x % (half >> 4) * 16
                                      : (int)blockIdx.x * (16 * NT);
    const int n_step = EPI == EPI_ROPE_KV ? half : 16;    // from a column tile to the next
    const float *xp[MT], *wp[NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) xp[mt] = X + (size_t)min(m0 + mt * 16 + lr, M - 1) * ldx;    // rows and columns beyond the
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) wp[nt] = W + (size_t)min(n0 + nt * n_step + lr, N - 1) * K;   // matrix repeat the last (never stored)
    QkvRows rows;
    if constexpr (EPI == EPI_ROPE_KV)
        if (wave < MT) qkv_rows(epi.qkv, n0 / epi.qkv.dh, n0 % epi.qkv.dh + lr, m0 / 16 + wave, M, lane, rows);
    const int n_ks = (K + F32_KSTEP - 1) / F32_KSTEP, k0 = wave * n_ks / F32_WAVES, k1 = (wave + 1) * n_ks / F32_WAVES;
    auto load = [&](const float *row, int ks) {           // four k of this lane; zero beyond K, and from k1 on
        const int k = ks * F32_KSTEP + lg * 4;
        f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
        if constexpr (VEC) {
            const bool ok = ks < k1 && k < K;             // (K is a multiple of 4: all four or none)
            const f32x4 t = *reinterpret_cast<const f32x4 *>(row + (ok ? k : 0));
            if (ok) v = t;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool ok = ks < k1 && k + j < K;
                const float t = row[ok ? k + j : 0];
                if (ok) v[j] = t;
            }
        }
        return v;
    };
    f32x4 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 a[2][F32_PF][MT], b[2][F32_PF][NT], gn[2][F32_PF];
    f32x4 ss[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) ss[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto fetch = [&](int ks, f32x4 (&fa)[F32_PF][MT], f32x4 (&fb)[F32_PF][NT], f32x4 (&fg)[F32_PF]) {
#pragma unroll
        for (int p = 0; p < F32_PF; ++p) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) fa[p][mt] = load(xp[mt], ks + p);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) fb[p][nt] = load(wp[nt], ks + p);
            if constexpr (NORM) fg[p] = load(epi.gain, ks + p);
        }
    };
    auto multiply = [&](const f32x4 (&fa)[F32_PF][MT], const f32x4 (&fb)[F32_PF][NT], const f32x4 (&fg)[F32_PF]) {
#pragma unroll
        for (int p = 0; p < F32_PF; ++p)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    float x = fa[p][mt][j];
                    if constexpr (NORM) { ss[mt][j] = fmaf(x, x, ss[mt][j]); x *= fg[p][j]; }
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, fb[p][nt][j], acc[mt][nt], 0, 0, 0);
                }
    };
    fetch(k0, a[0], b[0], gn[0]);
    if constexpr (EPI == EPI_ROPE_KV)
        if (wave < MT) qkv_pages(epi.qkv, n0 / epi.qkv.dh, rows);
    for (int ks = k0; ks < k1; ks += 2 * F32_PF) {        // (a k-step beyond k1 is all zeros: it changes no sum)
        fetch(ks + F32_PF, a[1], b[1], gn[1]);
        multiply(a[0], b[0], gn[0]);
        if (ks + F32_PF >= k1) break;
        fetch(ks + 2 * F32_PF, a[0], b[0], gn[0]);
        multiply(a[1], b[1], gn[1]);
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) red[wave][mt * NT + nt][lane] = acc[mt][nt];
    if constexpr (NORM) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {                 // of a row: four lanes' shares
            float q = (ss[mt][0] + ss[mt][1]) + (ss[mt][2] + ss[mt][3]), lo, hi;
            swap16(q, lo, hi); q = lo + hi;
            swap32(q, lo, hi); q = lo + hi;
            if (lane < 16) squares[wave][mt * 16 + lane] = q;
        }
    }
    __syncthreads();
    auto sum_of = [&](int t) {                            // tile t = row tile * NT + column tile; register r is row 4 * (lane / 16) + r
        f32x4 v = red[0][t][lane];
#pragma unroll
        for (int w = 1; w < F32_WAVES; ++w) v += red[w][t][lane];
        if constexpr (NORM) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = t / NT * 16 + lg * 4 + r;
                const float q = (squares[0][row] + squares[1][row]) + (squares[2][row] + squares[3][row]);
                static_assert(F32_WAVES == 4, "the sum above");
                v[r] *= 1.0f / sqrtf(q / (float)K + epi.eps);
            }
        }
        return v;
    };
    if constexpr (EPI == EPI_SILU) {
        if (wave >= MT) return;
        const f32x4 g = sum_of(wave * NT);
        const f32x4 up = sum_of(wave * NT + 1);
        const int f = blockIdx.x * 16 + lr;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = m0 + wave * 16 + lg * 4 + r;
            if (m < M && f < epi.F) epi.act[(size_t)m * epi.F + f] = mul_round<float>(g[r] / (1.0f + expf(-g[r])), up[r]);
        }
        return;
    }
    if constexpr (EPI == EPI_ROPE_KV) {
        if (wave >= MT) return;
        const f32x4 a = sum_of(wave * NT);
        const f32x4 b = sum_of(wave * NT + 1);
        qkv_store<float>(epi.qkv, n0 / epi.qkv.dh, n0 % epi.qkv.dh + lr, m0 / 16 + wave, M, lane, a, b, rows);
        return;
    }
    for (int t = wave; t < MT * NT; t += F32_WAVES) {     // D tile: lane -> column lane % 16, register r -> row 4 * (lane / 16) + r
        const f32x4 v = sum_of(t);
        const int n = n0 + (t % NT) * 16 + lr;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = m0 + (t / NT) * 16 + lg * 4 + r;
            if (m >= M || n >= N) continue;
            if constexpr (EPI == EPI_RESIDUAL) {
                const size_t at = (size_t)m * N + n;
                float add = epi.residual ? epi.h[at] : 0.f;
                if (epi.bias) add += epi.bias[n];
                const float x = v[r] + add;
                epi.h[at] = x;
                if (epi.h_copy) epi.h_copy[at] = x;
                if (epi.h_user && m < epi.h_user_rows) epi.h_user[at] = x;
            } else {
                out[(size_t)m * ld_out + n] = v[r];
            }
        }
    }
}

// Two row tiles and two column tiles per workgroup where there are rows for it (half the operand traffic of 16 x 16).
template <int EPI, bool NORM>
static void launch_gemm_f32(const float *W, const float *X, int ldx, float *out, int ld_out, int M, int N, int K, const F32Epi &epi, hipStream_t st,
                            hipEvent_t ev_start, hipEvent_t ev_stop) {
    const bool vec = K % 4 == 0 && ldx % 4 == 0 && reinterpret_cast<uintptr_t>(X) % 16 == 0 && reinterpret_cast<uintptr_t>(W) % 16 == 0 &&
                     (!NORM || reinterpret_cast<uintptr_t>(epi.gain) % 16 == 0);
    constexpr int NT1 = EPI == EPI_PLAIN || EPI == EPI_RESIDUAL ? 1 : 2;
#define POSS_F32(MT, NT, VEC)                                                                                              \
    do {                                                                                                                   \
        dim3 grid((N + 16 * NT - 1) / (16 * NT), (M + 16 * MT - 1) / (16 * MT)), block(F32_WAVES * 64);                    \
        if (ev_start && ev_stop)                                                                                           \
            hipExtLaunchKernelGGL((gemm_f32_kernel<MT, NT, VEC, EPI, NORM>), grid, block, 0, st, ev_start, ev_stop, 0, W, X, ldx, out, ld_out, M, N, K, epi); \
        else                                                                                                               \
            hipLaunchKernelGGL((gemm_f32_kernel<MT, NT, VEC, EPI, NORM>), grid, block, 0, st, W, X, ldx, out, ld_out, M, N, K, epi); \
    } while (0)
    if (M <= 16 || (size_t)M * N < 64 * 1024) { if (vec) POSS_F32(1, NT1, true); else POSS_F32(1, NT1, false); }
    else { if (vec) POSS_F32(2, 2, true); else POSS_F32(2, 2, false); }
#undef POSS_F32
}

// The plain epilogue of every (128-column tile, 16-row block), one workgroup each: sums the split-K planes in split
// order (bitwise repeatable).  32 threads x 4 columns per row, 8 rows per sweep.
__global__ __launch_bounds__(256) void epilogue_kernel(const float *__restrict__ part, size_t plane, int S, int Npad, int N, int M,
                                                       float *out, int ld_out) {
    const int t = threadIdx.x, n = blockIdx.x * GEMM_BLOCK_N + (t & 31) * 4, r0 = blockIdx.y * EPI_ROWS_PLAIN, r1 = min(M, r0 + EPI_ROWS_PLAIN);
    if (n >= N) return;
    for (int r = r0 + (t >> 5); r < r1; r += 8) {
        const f32x4 v = sum_planes4(part, plane, S, (size_t)r * Npad + n);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (n + j < N) out[(size_t)r * ld_out + n + j] = v[j];
    }
}

// The RoPE + KV-write epilogue over several row ranges in one launch, each range into its own cache
// (sequences batched into one GEMM); blockIdx.y runs over the 4-row blocks of all ranges.  A thread takes four consecutive
// rotary pairs of a row, 16 bytes of each half from every plane: one wave for the 4 rows x 128 columns of a workgroup
// (four times 61 rows of the 8B shape: 10.6 us with a pair per thread, now 7.6; 61 rows 4.8, 4.7).
constexpr int ROPE_THREADS = EPI_ROWS_PAIR * 16;
template <typename T>
__global__ __launch_bounds__(ROPE_THREADS) void epilogue_rope_ranges_kernel(const float *__restrict__ part, size_t plane, int S, int Npad,
                                                                            RopeRanges rr, EpiArgs e) {
    struct __attribute__((aligned(4 * sizeof(T)))) Quad { T t[4]; };
    int jr = 0;
    for (int i = 1; i < rr.n; ++i)
        if ((int)blockIdx.y >= rr.blk0[i]) jr = i;
    const int r = rr.r0[jr] + ((int)blockIdx.y - rr.blk0[jr]) * EPI_ROWS_PAIR + ((int)threadIdx.x >> 4);
    const KVCache kv = rr.kv[jr];
    // thread -> pairs i .. i + 3 of one head inside the 128-column tile; pairs are (i, i + dh/2)
    const int half = e.dh >> 1, c = ((int)threadIdx.x & 15) * 4;
    const int hb = (int)blockIdx.x * GEMM_BLOCK_N + (c / half) * e.dh, i = c % half, gh = hb / e.dh;
    if (r >= rr.r1[jr] || gh >= e.hq + 2 * e.hkv || (gh < e.hq && r >= rr.rows_q[jr])) return;
    // columns of the pairs: in the packed order of PackSrc::rope_dh a 32-column group holds dims [16j, 16j+16) followed by their partners
    const int c1 = hb + (i >> 4) * 32 + (i & 15), c2 = c1 + 16;
    float2 cs[4];                                          // requested together with the planes
#pragma unroll
    for (int j = 0; j < 4; ++j) cs[j] = e.cs[r * half + i + j];
    const int sl = e.slot[r];
    const f32x4 x1 = sum_planes4(part, plane, S, (size_t)r * Npad + c1);
    const f32x4 x2 = sum_planes4(part, plane, S, (size_t)r * Npad + c2);
    if (gh >= e.hq + e.hkv) {
        T *vc = static_cast<T *>(kv.vt) + vt_offset(kv, sl, gh - e.hq - e.hkv, e.hkv, e.dh, i);
        const size_t P = (size_t)1 << kv.page_shift;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            vc[j * P] = from_f<T>(x1[j]);
            vc[(j + half) * P] = from_f<T>(x2[j]);
        }
        return;
    }
    Quad o1, o2;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float a, b;
        rope_pair(x1[j], x2[j], cs[j], a, b);
        o1.t[j] = round_f<T>(a);
        o2.t[j] = round_f<T>(b);
    }
    T *dst = gh < e.hq ? static_cast<T *>(e.q) + ((size_t)r * e.hq + gh) * e.dh + i
                       : static_cast<T *>(kv.k) + k_offset(kv, sl, gh - e.hq, e.hkv, e.dh) + i;
    *reinterpret_cast<Quad *>(dst) = o1;
    *reinterpret_cast<Quad *>(dst + half) = o2;
}

void launch_residual_norm(int dt, const float *part, int S, int rows, int N, float eps, const EpiArgs &epi, hipStream_t st) {
    int threads = round_up((N + 3) / 4, 64);
    if (threads > 1024) threads = 1024;
    if (dt == DT_BF16)
        hipLaunchKernelGGL((epilogue_residual_norm_kernel<bf16_t>), dim3(rows), dim3(threads), 0, st, part, (size_t)rows * N, S, N, N, eps, epi);
    else
        hipLaunchKernelGGL((epilogue_residual_norm_kernel<f16_t>), dim3(rows), dim3(threads), 0, st, part, (size_t)rows * N, S, N, N, eps, epi);
}

// ------------------------------------------------------------------------------------------
// Row count of a partial plane as the kernel instantiation writes it.
static int gemm_rows_written(int mpad) {
    const int mt = mpad / 16;
    return (mt <= 2 ? mt : mt <= 4 ? 4 : mt <= 6 ? 6 : mt <= 8 ? 8 : mt <= 12 ? 12 : 16) * 16;
}

GemmShape gemm_plan(int dt, int M, int N, int K, int target_wgs) {
    GemmShape g;
    g.M = M; g.N = N; g.K = K;
    g.Npad = gemm_npad(N);
    g.Kpad = gemm_kpad(dt, K);
    g.Mpad = round_up(M < 1 ? 1 : M, 16);
    if (dt == DT_F32) { g.S = 1; return g; }
    g.Mpad = gemm_rows_written(g.Mpad);       // the kernels are instantiated for 1, 2, 4, 6, 8 or (tall kernel) 12, 16 row tiles
    const int n_blocks = g.Npad / GEMM_BLOCK_N;
    const int n_chunks = g.Kpad / GEMM_KCHUNK;
    // One workgroup per CU (256) at most, as many as fit, chunks dealt out evenly: in every sweep more
    // splits were slower (partial-plane traffic grows, two workgroups on a CU share its LDS and barriers)
    // and fewer leave CUs without a stream.
    if (target_wgs <= 0) target_wgs = 256;
    int S = target_wgs / n_blocks;
    int max_s = n_chunks / 2; if (max_s < 1) max_s = 1;          // at least 512 of K per split
    if (S > max_s) S = max_s;
    if (S < 1) S = 1;
    // The longest stream sets the time: take the fewest splits that keep it (16 chunks over 5 splits
    // is 4 chunks on the busiest; 4 splits do the same with one partial plane less).
    const int longest = (n_chunks + S - 1) / S;
    S = (n_chunks + longest - 1) / longest;
    g.S = S;
    return g;
}

// Two 128-column tiles per workgroup (8 waves sharing one staged activation slice) when the column count alone
// gives every CU work and K is not split.
static bool gemm_wide(const GemmShape &g) {
    return g.S == 1 && g.Mpad <= 96 && g.Npad % (2 * GEMM_BLOCK_N) == 0 && g.Npad / (2 * GEMM_BLOCK_N) >= 256;
}

int gemm_head_segments(const GemmShape &g) { return g.Npad / (GEMM_BLOCK_N * (gemm_wide(g) ? 2 : 1)); }

template <typename T>
static void launch_epilogue_t(const GemmShape &g, const float *part, const EpiArgs &epi, float eps, hipStream_t st) {
    const size_t plane = (size_t)g.Mpad * g.Npad;
    switch (epi.mode) {
        case EPI_RESIDUAL:
            if constexpr (!std::is_same<T, float>::value) {             // (float32: inside gemm_f32_kernel)
                int threads = round_up((g.N + 3) / 4, 64);
                if (threads > 1024) threads = 1024;
                hipLaunchKernelGGL((epilogue_residual_norm_kernel<T>), dim3(g.M), dim3(threads), 0, st, part, plane, g.S, g.Npad, g.N, eps, epi);
            }
            break;
        case EPI_HEAD: break;           // reduced inside the stream kernel
        case EPI_PLANES: break;
        case EPI_SILU: break;           // applied inside the stream kernel
        default:
            if (g.S > 1 || epi.out)     // S == 1 without an output buffer: plane 0 is the result
                hipLaunchKernelGGL(epilogue_kernel, dim3(g.Npad / GEMM_BLOCK_N, (g.M + EPI_ROWS_PLAIN - 1) / EPI_ROWS_PLAIN), dim3(256), 0, st, part,
                                   plane, g.S, g.Npad, g.N, g.M, epi.out, epi.ld_out);
            break;
    }
}

// Is the QKV projection one kernel?  Its workgroups, one per 32 columns, each read all rows over the whole K: these bytes, together,
// are what it pays for the partial planes and the epilogue kernel that it saves (both kernels give the same bits).  Stream and
// epilogue / one kernel, us with the boundaries between launches:
//   4096 -> 6144 (4 splits)   20 rows (50 MB) 13.9 / 13.3, 31 rows (50 MB) 16.2 / 14.0, 47 rows (101 MB) 15.6 / 15.9, 61 rows 15.7 / 17.1
//   5120 -> 15360 (2 splits)  1 row (79 MB) 28.3 / 26.6, 10 rows 28.4 / 26.7, 31 rows (157 MB) 30.0 / 32.0, 61 rows (315 MB) 32.1 / 42.0
//   640 -> 1920 (1 split)     1 row 8.3 / 5.8, 10 rows 8.9 / 6.2, 31 rows 9.3 / 7.4, 61 rows (5 MB) 10.4 / 9.3
//   512 -> 768 (1 split)      1 row 7.0 / 5.0, 10 rows 7.4 / 5.4, 31 rows 7.7 / 6.0, 61 rows (2 MB) 8.6 / 8.1
// Nor with more tiles than CUs and a last round that leaves many of them without one: what they could have streamed meanwhile counts
// (idle CUs x a tile's weights).  The same figures (bf16, a layer's share of a pass, 1 row; up to 31 rows alike):
//   1024 -> 12288 (384 tiles, 8 MB) -2, 13B above (480, 10 MB) -1.7, 1024 -> 9216 (288, 15 MB) 0, 2048 -> 12288 (17 MB) -1.2;
//   2048 -> 10240 (320, 25 MB) +1.4, 4096 -> 12288 (34 MB) +3, 3072 -> 9216 (44 MB) +4.4, 4096 -> 10240 (50 MB) +5.7, 8192 -> 10240 (101 MB) +9.
// Two row tiles pay up to 100 MiB (four layers, us, stream / one kernel): 6144 -> 8192 (96 MiB) 17 rows 558 / 548, 31 rows 585 / 575; 7168 ->
// 7168 (98 MiB) 24 rows 613 / 610; 8192 -> 7168 (112 MiB) 17 rows 671 / 678, 31 rows 674 / 686.  Four do not: the 47 rows above.
constexpr size_t QKV_FUSED_BYTES = (size_t)80 << 20, QKV_FUSED_BYTES_32 = (size_t)100 << 20, QKV_IDLE_BYTES = (size_t)20 << 20;
static bool qkv_fused(const GemmShape &g) {
    const size_t tiles = g.Npad / (GEMM_NT * 16), idle = tiles > 256 ? (256 - tiles % 256) % 256 : 0;
    return g.Mpad <= 64 && g.S <= QKV_MAX_SPLITS && tiles * g.Mpad * g.K * 2 <= (g.Mpad == 32 ? QKV_FUSED_BYTES_32 : QKV_FUSED_BYTES) &&
           idle * (GEMM_NT * 16) * g.K * 2 <= QKV_IDLE_BYTES;
}

// The QKV projection of 16-bit types: one kernel, rotary embedding and cache writes included.
template <typename T>
static void launch_qkv_rope_t(const GemmShape &g, const void *Wp, const void *X, int ldx, const EpiArgs &epi, const RopeRanges &rr,
                              hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
    QkvEpi qe{epi.cs, epi.slot, epi.q, epi.hq, epi.hkv, epi.dh, rr};
    dim3 grid(g.Npad / (GEMM_NT * 16)), block(g.S * 128);
    const int ksteps = g.Kpad / GEMM_KSTEP;
    const u32x4 *w = static_cast<const u32x4 *>(Wp);
    const T *x = static_cast<const T *>(X);
#define POSS_QKV_LAUNCH(MT, NST)                                                                              \
    do {                                                                                                      \
        const size_t lds = (size_t)g.S * NST * QKV_STAGE_BYTES(MT);                                           \
        if (ev_start && ev_stop)                                                                              \
            hipExtLaunchKernelGGL((gemm_qkv_rope_kernel<T, MT, NST>), grid, block, lds, st, ev_start, ev_stop, 0, w, x, ldx, g.M, g.K, ksteps, qe); \
        else                                                                                                  \
            hipLaunchKernelGGL((gemm_qkv_rope_kernel<T, MT, NST>), grid, block, lds, st, w, x, ldx, g.M, g.K, ksteps, qe); \
    } while (0)
    switch (g.Mpad / 16) {
        case 1:
            if (g.S != 4 || ksteps % 32) { POSS_QKV_LAUNCH(1, 6); break; }
            if (ev_start && ev_stop)
                hipExtLaunchKernelGGL((gemm_qkv_row_kernel<T, 8>), grid, dim3(256), 0, st, ev_start, ev_stop, 0, w, x, ldx, g.M, g.K, ksteps, qe);
            else
                hipLaunchKernelGGL((gemm_qkv_row_kernel<T, 8>), grid, dim3(256), 0, st, w, x, ldx, g.M, g.K, ksteps, qe);
            break;
        case 2: POSS_QKV_LAUNCH(2, 5); break;
        default: POSS_QKV_LAUNCH(4, 3); break;
    }
#undef POSS_QKV_LAUNCH
}

template <typename T>
static void launch_gemm_t(const GemmShape &g, const void *Wp, const void *X, int ldx, float *part,
                          const EpiArgs &epi, float eps, hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop, const RopeRanges *rr) {
    if (epi.mode == EPI_ROPE_KV && qkv_fused(g)) {
        launch_qkv_rope_t<T>(g, Wp, X, ldx, epi, *rr, st, ev_start, ev_stop);
        return;
    }
    const bool fuse_silu = epi.mode == EPI_SILU;
    const bool head = epi.mode == EPI_HEAD;
    if (g.Mpad > 128) {                                  // the tall kernel: one 128-column tile of 192 or 256 rows
        HeadEpi he{};
        if (head) he = HeadEpi{epi.head_mode, epi.head_k, g.N, epi.logits, epi.logits_rows, epi.seg_out, epi.pv, epi.pi};
        dim3 grid(g.Npad / GEMM_BLOCK_N, g.S), block(TALL_THREADS);
        const int w_once = (size_t)g.Npad * g.Kpad * sizeof(T) >= TALL_ONCE_BYTES;
        const int ksteps = g.Kpad / GEMM_KSTEP;
        const u32x4 *w = static_cast<const u32x4 *>(Wp);
        const T *x = static_cast<const T *>(X);
        T *act = static_cast<T *>(epi.act);
#define POSS_TALL_LAUNCH_MT(MT, FUSE, HD, FARG)                                                               \
    do {                                                                                                      \
        if (ev_start && ev_stop)                                                                              \
            hipExtLaunchKernelGGL((gemm_tall_kernel<T, MT, FUSE, HD>), grid, block, 0, st, ev_start, ev_stop, 0, w, x, ldx, part, \
                                  g.M, g.K, g.Npad, ksteps, w_once, act, FARG, he);                           \
        else                                                                                                  \
            hipLaunchKernelGGL((gemm_tall_kernel<T, MT, FUSE, HD>), grid, block, 0, st, w, x, ldx, part, g.M, g.K, g.Npad, \
                               ksteps, w_once, act, FARG, he);                                                \
    } while (0)
#define POSS_TALL_LAUNCH(FUSE, HD, FARG)                                                                      \
    do { if (g.Mpad <= 192) POSS_TALL_LAUNCH_MT(12, FUSE, HD, FARG); else POSS_TALL_LAUNCH_MT(16, FUSE, HD, FARG); } while (0)
        if (fuse_silu) POSS_TALL_LAUNCH(true, false, epi.F);
        else if (head) POSS_TALL_LAUNCH(false, true, 0);
        else POSS_TALL_LAUNCH(false, false, 0);
#undef POSS_TALL_LAUNCH_MT
#undef POSS_TALL_LAUNCH
        if (epi.mode == EPI_ROPE_KV) {
            const size_t plane = (size_t)g.Mpad * g.Npad;
            const int blocks = rr->blk0[rr->n - 1] + (rr->r1[rr->n - 1] - rr->r0[rr->n - 1] + EPI_ROWS_PAIR - 1) / EPI_ROWS_PAIR;
            hipLaunchKernelGGL((epilogue_rope_ranges_kernel<T>), dim3(g.Npad / GEMM_BLOCK_N, blocks), dim3(ROPE_THREADS), 0, st, part, plane, g.S,
                               g.Npad, *rr, epi);
            return;
        }
        launch_epilogue_t<T>(g, part, epi, eps, st);
        return;
    }
    // Two tiles per workgroup when the column count alone gives every CU work and K is not split.
    const bool wide = !fuse_silu && gemm_wide(g);
    const int wpb = wide ? 8 : 4;
    HeadEpi he{};
    if (head) he = HeadEpi{epi.head_mode, epi.head_k, g.N, epi.logits, epi.logits_rows, epi.seg_out, epi.pv, epi.pi};
    dim3 grid(g.Npad / (GEMM_NT * 16 * wpb), g.S), block(wpb * 64);
    const int ksteps = g.Kpad / GEMM_KSTEP;
    const u32x4 *w = static_cast<const u32x4 *>(Wp);
    const T *x = static_cast<const T *>(X);
    T *act = static_cast<T *>(epi.act);
    const bool deep = !wide && (int)(grid.x * grid.y) < 256;     // fewer workgroups than CUs: deeper weight ring
    // With a pair of events the launch itself carries them: they take the kernel's own begin and end
    // timestamps (what a profiler reports), not the time of extra packets around it.
    const bool timed = ev_start && ev_stop;
#define POSS_GEMM_LAUNCH(MT, W, FUSE, PFV, HD, FARG)                                                          \
    do {                                                                                                      \
        if (timed)                                                                                            \
            hipExtLaunchKernelGGL((gemm_stream_kernel<T, MT, W, FUSE, PFV, HD>), grid, block, 0, st, ev_start, \
                                  ev_stop, 0, w, x, ldx, part, g.M, g.K, g.Npad, ksteps, act, FARG, he);      \
        else                                                                                                  \
            hipLaunchKernelGGL((gemm_stream_kernel<T, MT, W, FUSE, PFV, HD>), grid, block, 0, st, w, x, ldx, part, \
                               g.M, g.K, g.Npad, ksteps, act, FARG, he);                                      \
    } while (0)
#define POSS_GEMM_CASE(MT)                                                                                    \
    do {                                                                                                      \
        if (fuse_silu) { if (deep) POSS_GEMM_LAUNCH(MT, 4, true, 8, false, epi.F); else POSS_GEMM_LAUNCH(MT, 4, true, 4, false, epi.F); } \
        else if (head) { if (wide) POSS_GEMM_LAUNCH(MT, 8, false, 4, true, 0); else POSS_GEMM_LAUNCH(MT, 4, false, 4, true, 0); } \
        else if (wide) POSS_GEMM_LAUNCH(MT, 8, false, 4, false, 0);                                           \
        else if (deep) POSS_GEMM_LAUNCH(MT, 4, false, 8, false, 0);                                           \
        else POSS_GEMM_LAUNCH(MT, 4, false, 4, false, 0);                                                     \
    } while (0)
    switch (g.Mpad / 16) {
        case 1: POSS_GEMM_CASE(1); break;
        case 2: POSS_GEMM_CASE(2); break;
        case 4: POSS_GEMM_CASE(4); break;
        case 6: POSS_GEMM_CASE(6); break;
        default: POSS_GEMM_CASE(8); break;
    }
#undef POSS_GEMM_CASE
#undef POSS_GEMM_LAUNCH
    if (epi.mode == EPI_ROPE_KV) {                       // rotary + cache writes per row range, one launch
        const size_t plane = (size_t)g.Mpad * g.Npad;
        const int blocks = rr->blk0[rr->n - 1] + (rr->r1[rr->n - 1] - rr->r0[rr->n - 1] + EPI_ROWS_PAIR - 1) / EPI_ROWS_PAIR;
        hipLaunchKernelGGL((epilogue_rope_ranges_kernel<T>), dim3(g.Npad / GEMM_BLOCK_N, blocks), dim3(ROPE_THREADS), 0, st, part, plane, g.S,
                           g.Npad, *rr, epi);
        return;
    }
    launch_epilogue_t<T>(g, part, epi, eps, st);
}

// Refuse, on the host, argument sets that would make a kernel write through a null pointer.
static bool gemm_args_ok(int dt, const GemmShape &g, const void *Wp, const void *X, const float *part, const EpiArgs &e) {
    if (!Wp || !X || !part || g.M < 1 || g.M > LAUNCH_ROWS || g.S < 1) return false;
    if (e.x_gain && dt != DT_F32) return false;
    if (dt == DT_F32) {                                    // norms belong to the products that read them
        if (e.mode == EPI_RESIDUAL) return e.h && !e.gain && e.h != X;
        if ((e.mode == EPI_SILU || e.mode == EPI_ROPE_KV) && !e.x_gain) return false;
    }
    switch (e.mode) {
        case EPI_PLAIN: return e.out || g.S == 1;          // unsplit: plane 0 is the result
        case EPI_ROPE_KV:                                  // caches: checked per range
            return e.q && e.cs && e.slot && (dt == DT_F32 ? e.dh >= 32 && e.dh % 32 == 0 : e.dh == 64 || e.dh == 128);
        case EPI_RESIDUAL: return e.h && (!e.gain || e.u);
        case EPI_PLANES: return dt != DT_F32;
        case EPI_SILU: return e.act && g.S == 1;           // applied to whole sums
        case EPI_HEAD:
            if (g.S != 1 || g.N < 1) return false;
            if (e.head_mode == HEAD_ARGMAX) return e.pv && e.pi;
            return e.head_mode == HEAD_TOPK && e.seg_out && e.head_k >= 1 && e.head_k <= TOPK_MAXK;
        default: return false;
    }
}

static bool ranges_ok(const GemmShape &g, RopeRanges &rr) {
    if (rr.n < 1 || rr.n > ROPE_MAX_RANGES) return false;
    int blocks = 0;
    for (int i = 0; i < rr.n; ++i) {
        if (rr.r0[i] < 0 || rr.r1[i] > g.M || rr.r0[i] >= rr.r1[i]) return false;
        if (!rr.kv[i].k || !rr.kv[i].vt || !rr.kv[i].page_table) return false;
        if (rr.kv[i].page_table != rr.kv[0].page_table || rr.kv[i].page_shift != rr.kv[0].page_shift) return false;   // a context has one
        rr.blk0[i] = blocks;
        blocks += (rr.r1[i] - rr.r0[i] + EPI_ROWS_PAIR - 1) / EPI_ROWS_PAIR;
    }
    return true;
}

bool launch_gemm(int dt, const GemmShape &g, const void *Wp, const void *X, int ldx, float *part,
                 const EpiArgs &epi, float eps, hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop, const RopeRanges *ranges) {
    if (!gemm_args_ok(dt, g, Wp, X, part, epi)) return false;
    if (ranges && epi.mode != EPI_ROPE_KV) return false;               // only that epilogue works by row range
    RopeRanges rr;
    if (epi.mode == EPI_ROPE_KV) {
        if (ranges) rr = *ranges;
        else { rr.n = 1; rr.r0[0] = 0; rr.r1[0] = g.M; rr.rows_q[0] = epi.rows_q; rr.kv[0] = epi.kv; }
        if (!ranges_ok(g, rr)) return false;
    }
    if (dt == DT_F32) {
        if (epi.mode == EPI_HEAD) return false;          // float32 storage reduces its logits with the two-stage kernels
        // the sums are whole: straight to the caller, unless that is over an operand
        const size_t out_bytes = ((size_t)(g.M - 1) * epi.ld_out + g.N) * sizeof(float);
        const bool direct = epi.mode == EPI_PLAIN && epi.out && !overlap(epi.out, out_bytes, X, ((size_t)(g.M - 1) * ldx + g.K) * sizeof(float)) &&
                            !overlap(epi.out, out_bytes, Wp, (size_t)g.N * g.K * sizeof(float));
        const float *w = static_cast<const float *>(Wp), *x = static_cast<const float *>(X);
        F32Epi fe{};
        fe.gain = static_cast<const float *>(epi.x_gain); fe.eps = eps;
        if (epi.mode == EPI_SILU) {
            fe.act = static_cast<float *>(epi.act); fe.F = epi.F;
            launch_gemm_f32<EPI_SILU, true>(w, x, ldx, nullptr, 0, g.M, g.N, g.K, fe, st, ev_start, ev_stop);
            return true;
        }
        if (epi.mode == EPI_ROPE_KV) {
            fe.qkv = QkvEpi{epi.cs, epi.slot, epi.q, epi.hq, epi.hkv, epi.dh, rr};
            launch_gemm_f32<EPI_ROPE_KV, true>(w, x, ldx, nullptr, 0, g.M, g.N, g.K, fe, st, ev_start, ev_stop);
            return true;
        }
        if (epi.mode == EPI_RESIDUAL) {
            fe.h = epi.h; fe.h_copy = epi.h_copy; fe.h_user = epi.h_user; fe.h_user_rows = epi.h_user_rows;
            fe.residual = epi.residual; fe.bias = static_cast<const float *>(epi.bias);
            launch_gemm_f32<EPI_RESIDUAL, false>(w, x, ldx, nullptr, 0, g.M, g.N, g.K, fe, st, ev_start, ev_stop);
            return true;
        }
        float *dst = direct ? epi.out : part;
        const int ld = direct ? epi.ld_out : g.Npad;
        if (epi.x_gain) launch_gemm_f32<EPI_PLAIN, true>(w, x, ldx, dst, ld, g.M, g.N, g.K, fe, st, ev_start, ev_stop);
        else launch_gemm_f32<EPI_PLAIN, false>(w, x, ldx, dst, ld, g.M, g.N, g.K, fe, st, ev_start, ev_stop);
        if (!direct) launch_epilogue_t<float>(g, part, epi, eps, st);
    } else if (dt == DT_BF16) {
        launch_gemm_t<bf16_t>(g, Wp, X, ldx, part, epi, eps, st, ev_start, ev_stop, epi.mode == EPI_ROPE_KV ? &rr : nullptr);
    } else {
        launch_gemm_t<f16_t>(g, Wp, X, ldx, part, epi, eps, st, ev_start, ev_stop, epi.mode == EPI_ROPE_KV ? &rr : nullptr);
    }
    return true;
}

static int longest_split(const GemmShape &g) { return (g.Kpad / GEMM_KCHUNK + g.S - 1) / g.S * GEMM_KCHUNK; }

bool gemm_merged_ok(int dt, const GemmShape &g, const AttnMerge &src) {
    const int k = longest_split(g);
    return dt != DT_F32 && g.M >= 1 && g.M <= 16 && src.n_splits >= 2 && src.n_splits <= 12 && k <= 4096 && g.K == src.hq * src.dh &&
           (size_t)g.M * k * src.n_splits * 4 <= MERGED_BYTES;
}

bool launch_gemm_merged(int dt, const GemmShape &g, const void *Wp, const AttnMerge &src, float *part, const EpiArgs &epi, float eps,
                        hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
    if (!gemm_merged_ok(dt, g, src) || !src.o || !src.ml || (epi.mode != EPI_RESIDUAL && epi.mode != EPI_PLANES) ||
        !gemm_args_ok(dt, g, Wp, src.o, part, epi)) return false;
    dim3 grid(g.Npad / GEMM_BLOCK_N, g.S);
    const size_t lds = (size_t)longest_split(g) / GEMM_KSTEP * 1024;
    const int ksteps = g.Kpad / GEMM_KSTEP;
    const u32x4 *w = static_cast<const u32x4 *>(Wp);
#define POSS_MERGED(T, NR, QB)                                                                                               \
    do {                                                                                                                     \
        if (ev_start && ev_stop)                                                                                             \
            hipExtLaunchKernelGGL((gemm_merged_kernel<T, NR, QB>), grid, dim3(256), lds, st, ev_start, ev_stop, 0, w, src, part, g.M, g.K, g.Npad, ksteps); \
        else                                                                                                                 \
            hipLaunchKernelGGL((gemm_merged_kernel<T, NR, QB>), grid, dim3(256), lds, st, w, src, part, g.M, g.K, g.Npad, ksteps); \
    } while (0)
#define POSS_MERGED_T(T)                                                                                                     \
    do {                                                                                                                     \
        if (src.n_splits <= 4) { if (one) POSS_MERGED(T, 4, 1); else POSS_MERGED(T, 4, 4); }                                 \
        else if (src.n_splits <= 8) { if (one) POSS_MERGED(T, 8, 1); else POSS_MERGED(T, 8, 2); }                            \
        else POSS_MERGED(T, 12, 1);                                                                                          \
    } while (0)
    const bool one = g.M * longest_split(g) <= 4 * 256;   // a quad per thread
    if (dt == DT_BF16) { POSS_MERGED_T(bf16_t); launch_epilogue_t<bf16_t>(g, part, epi, eps, st); }
    else { POSS_MERGED_T(f16_t); launch_epilogue_t<f16_t>(g, part, epi, eps, st); }
#undef POSS_MERGED_T
#undef POSS_MERGED
    return true;
}

// d up to 5120 (QKV) and 6144 (gate/up): a wave's slots times its planes have to fit its registers.
bool gemm_row_ok(int dt, const GemmShape &g, const RowNorm &norm, int mode) {
    if (dt == DT_F32 || g.M != 1 || g.K != norm.d || norm.d % 4 || norm.S < 1 || norm.S > (norm.d <= 4096 ? 8 : 6)) return false;
    if (mode == EPI_SILU) return norm.d <= 6144 && g.S == 1;
    return mode == EPI_ROPE_KV && norm.d <= 5120 && qkv_fused(g) && g.S != 3;
}

bool launch_gemm_row(int dt, const GemmShape &g, const void *Wp, const RowNorm &norm, const EpiArgs &epi, hipStream_t st,
                     hipEvent_t ev_start, hipEvent_t ev_stop) {
    if (!gemm_row_ok(dt, g, norm, epi.mode) || !norm.part || !norm.h_out || norm.h_out == norm.h || !norm.gain || (norm.residual && !norm.h) ||
        !gemm_args_ok(dt, g, Wp, norm.part, const_cast<float *>(norm.part), epi)) return false;
    const int ksteps = g.Kpad / GEMM_KSTEP;
    const u32x4 *w = static_cast<const u32x4 *>(Wp);
    size_t lds = (size_t)ksteps * GEMM_KSTEP * 2;
    QkvEpi qe{};
    if (epi.mode == EPI_ROPE_KV) {
        qe = QkvEpi{epi.cs, epi.slot, epi.q, epi.hq, epi.hkv, epi.dh, RopeRanges{}};
        qe.rr.n = 1; qe.rr.r0[0] = 0; qe.rr.r1[0] = 1; qe.rr.rows_q[0] = epi.rows_q; qe.rr.kv[0] = epi.kv;
        if (!ranges_ok(g, qe.rr)) return false;
        lds = max(lds, (size_t)g.S * GEMM_NT * 64 * sizeof(f32x4));
    }
#define POSS_ROW(KERNEL, GRID, THREADS, ...)                                                                                 \
    do {                                                                                                                     \
        if (ev_start && ev_stop) hipExtLaunchKernelGGL(KERNEL, dim3(GRID), dim3(THREADS), lds, st, ev_start, ev_stop, 0, w, norm, ksteps, __VA_ARGS__); \
        else hipLaunchKernelGGL(KERNEL, dim3(GRID), dim3(THREADS), lds, st, w, norm, ksteps, __VA_ARGS__);                   \
    } while (0)
#define POSS_ROW_SILU(T, NP, NSL) POSS_ROW((gemm_row_silu_kernel<T, NP, NSL>), g.Npad / GEMM_BLOCK_N, ROW_SILU_WAVES * 64, static_cast<T *>(epi.act), epi.F)
#define POSS_ROW_QKV(T, NP, NSL)                                                                                             \
    do {                                                                                                                     \
        if (g.S == QKV_MAX_SPLITS) POSS_ROW((gemm_row_qkv_kernel<T, NP, NSL, GEMM_NT>), g.Npad / (GEMM_NT * 16), ROW_QKV_WAVES * 64, qe, g.S); \
        else POSS_ROW((gemm_row_qkv_kernel<T, NP, NSL, 1>), g.Npad / (GEMM_NT * 16), ROW_QKV_WAVES * 64, qe, g.S);           \
    } while (0)
#define POSS_ROW_T(T)                                                                                                        \
    do {                                                                                                                     \
        if (epi.mode == EPI_SILU) {                                                                                          \
            static_assert(row_slots(4096, ROW_SILU_WAVES) == 2 && row_slots(6144, ROW_SILU_WAVES) == 3, "");                 \
            if (norm.d > 4096) { if (norm.S <= 4) POSS_ROW_SILU(T, 4, 3); else POSS_ROW_SILU(T, 6, 3); }                     \
            else if (norm.S <= 2) POSS_ROW_SILU(T, 2, 2);                                                                    \
            else if (norm.S <= 4) POSS_ROW_SILU(T, 4, 2);                                                                    \
            else POSS_ROW_SILU(T, 8, 2);                                                                                     \
        } else {                                                                                                             \
            static_assert(row_slots(4096, ROW_QKV_WAVES) == 4 && row_slots(5120, ROW_QKV_WAVES) == 5, ""); \
            if (norm.d > 4096) { if (norm.S <= 4) POSS_ROW_QKV(T, 4, 5); else POSS_ROW_QKV(T, 6, 5); }                  \
            else if (norm.S <= 2) POSS_ROW_QKV(T, 2, 4);                                                                     \
            else if (norm.S <= 4) POSS_ROW_QKV(T, 4, 4);                                                                     \
            else POSS_ROW_QKV(T, 8, 4);                                                                                      \
        }                                                                                                                    \
    } while (0)
    if (dt == DT_BF16) POSS_ROW_T(bf16_t); else POSS_ROW_T(f16_t);
#undef POSS_ROW_T
#undef POSS_ROW_QKV
#undef POSS_ROW_SILU
#undef POSS_ROW
    return true;
}

// ------------------------------------------------------------------------------------------
// Repack row-major [rows_i, K] matrices, stacked along N (or gate/up interleaved in groups of 16
// rows), into B-operand order.
__device__ __forceinline__ bool pack_source_row(const PackSrc &src, int n, int &which, int &row) {
    if (src.interleave16) {          // 32 rows = 16 rows of matrix 0, then the same 16 rows of matrix 1
        const int w = n & 31;
        which = w >> 4; row = (n >> 5) * 16 + (w & 15);
        return row < src.rows[which];
    }
    if (src.rope_dh > 0) {           // packed column p of a head -> dim (p / 32) * 16 + p % 16 + (p / 16 % 2) * dh / 2
        const int dh = src.rope_dh, p = n % dh;
        n = n - p + (p >> 5) * 16 + (p & 15) + ((p >> 4) & 1) * (dh >> 1);
    }
    for (which = 0; which < 3; ++which) {
        if (n < src.rows[which]) { row = n; return true; }
        n -= src.rows[which];
    }
    return false;
}

__global__ void pack16_kernel(PackSrc src, int K, int Kpad, int Npad, u32x4 *__restrict__ dst) {
    const size_t unit = (size_t)blockIdx.x * blockDim.x + threadIdx.x;     // one 16-byte unit of dst
    const size_t total = (size_t)Npad * Kpad / 8;
    if (unit >= total) return;
    const int ksteps = Kpad / GEMM_KSTEP;
    const int lane = unit & 63;
    size_t r = unit >> 6;
    const int nt = r % GEMM_NT; r /= GEMM_NT;
    const int ks = r % ksteps;
    const int ngroup = r / ksteps;
    const int n = (ngroup * GEMM_NT + nt) * 16 + (lane & 15);
    const int k = ks * GEMM_KSTEP + (lane >> 4) * 8;
    u32x4 v = u32x4{0u, 0u, 0u, 0u};
    int which, row;
    if (k < K && pack_source_row(src, n, which, row))
        v = *reinterpret_cast<const u32x4 *>(static_cast<const uint16_t *>(src.ptr[which]) + (size_t)row * K + k);
    dst[unit] = v;
}

__global__ void pack32_kernel(PackSrc src, int K, int Npad, float *__restrict__ dst) {
    const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (size_t)Npad * K) return;
    const int n = e / K, k = e % K;
    int which, row;
    dst[e] = pack_source_row(src, n, which, row) ? static_cast<const float *>(src.ptr[which])[(size_t)row * K + k] : 0.f;
}

void launch_pack(int dt, const PackSrc &src, int K, void *dst, hipStream_t st) {
    const int N = src.interleave16 ? gate_up_rows(src.rows[0]) : src.rows[0] + src.rows[1] + src.rows[2];
    const int Npad = gemm_npad(N), Kpad = gemm_kpad(dt, K);
    if (dt == DT_F32) {
        const size_t total = (size_t)Npad * K;
        hipLaunchKernelGGL(pack32_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, src, K, Npad,
                           static_cast<float *>(dst));
    } else {
        const size_t total = (size_t)Npad * Kpad / 8;
        hipLaunchKernelGGL(pack16_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, src, K, Kpad,
                           Npad, static_cast<u32x4 *>(dst));
    }
}

}  // namespace poss
