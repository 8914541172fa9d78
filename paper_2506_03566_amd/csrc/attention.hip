// Tree-masked attention over a paged KV cache.
//
// Every row of a pass sees the `n_prefix` committed cache slots and, of the `region_len` slots
// that follow them (the rows of this round: tree nodes in verification, drafted ancestors in a
// specialist pass, the chunk itself in prefill), those whose bit is set in the row's mask.
//
// 16-bit types: one wave per 16 (or 32) query rows, four waves (one KV head) per key-way and workgroup
// sharing the key/value blocks through LDS, on v_mfma_f32_16x16x32.
// Query rows of the G = Hq/Hkv heads that share a KV head are stacked (rho = m*G + g) so a wave's
// 16 rows reuse every key it loads.  Scores are formed transposed, S^T = K Q^T (keys as MFMA rows):
// a lane then holds 8 scores of ONE query row per 32-key block, which is already the B-operand
// layout of O^T = V^T P^T as long as the keys of a block are contracted in the order the score
// tiles deliver them; the key rows are dealt to the two score tiles so that this order is the
// natural one of V^T, which is cached transposed ([dh][token]).  Blocks go from memory straight
// into LDS (LDS-direct loads), swizzled so that operand reads run at the full LDS rate.
// Softmax is online (running max / sum per query row, float32); partial (max, sum, O) per split
// are merged by a second kernel in fixed order.
#include "attn_split.h"
#include "attn_merge.h"

#include <type_traits>

namespace poss {

static_assert(ATTN_MAX_REGION == MAX_ROWS, "a region's slots are the rows of one sequence in a pass");

typedef float  f32x4 __attribute__((ext_vector_type(4)));
typedef float  f32x16 __attribute__((ext_vector_type(16)));
typedef bf16_t bf16x8 __attribute__((ext_vector_type(8)));
typedef f16_t  f16x8 __attribute__((ext_vector_type(8)));

template <typename T> struct Vec8;
template <> struct Vec8<bf16_t> {
    typedef bf16x8 type;
    static __device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
};
template <> struct Vec8<f16_t> {
    typedef f16x8 type;
    static __device__ __forceinline__ f32x4 mfma(f16x8 a, f16x8 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ f32x16 mfma32(f16x8 a, f16x8 b, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
    }
};

__device__ __forceinline__ bool slot_visible(int slot, int n_prefix, int region_len, uint64_t m0, uint64_t m1) {
    // straight-line: a lane's eight slots would otherwise each cost a divergent branch
    const int j = slot - n_prefix;
    const uint64_t word = j < 64 ? m0 : m1;
    const bool bit = ((word >> (j & 63)) & 1ull) != 0;
    return (j < 0) | (((unsigned)j < (unsigned)region_len) & bit);
}

// Swizzles of the staged blocks.  A block reaches LDS through 16-byte LDS-direct loads: lane l of a wave
// writes base + 16 l, so a row cannot be padded; instead the 16-byte chunk c of row r is kept at position
// c ^ swz(r) of the row (the loading lane simply fetches the chunk that belongs at its position).
// An operand read has its 64 lanes read one row each (lane % 16 picks the row, lane / 16 the chunk).  Measured
// on this GPU with every wave of a CU reading: these two patterns run at 4.0 cycles per ds_read_b128 (256 bytes
// per cycle, the same as consecutive addresses), rows padded by 16 bytes instead (272- or 80-byte strides), a
// three-bit key swizzle, or a value swizzle that also folds in row bit 3, at 8.2 - 8.9 cycles.
// Keys: row kappa of a block (bits 0, 1 and 3, 4 vary over the lanes of a read; bit 2 is the score tile).
template <int DH>
__device__ __forceinline__ int key_swizzle(int kappa) {
    const int l0 = kappa & 1, l1 = (kappa >> 1) & 1, l2 = (kappa >> 3) & 1, l3 = (kappa >> 4) & 1;
    if (DH >= 128) return l0 | (l1 << 1) | (l2 << 2) | (l3 << 3);     // 16 chunks per row: the reading lane's row number
    return l1 | (l2 << 1) | (l3 << 2);                                // 8 chunks per row, two rows per 256 bytes: half of it
}
// Values: row rho of V^T (a dh index; 4 chunks of 8 keys per row, four rows per 256 bytes).
__device__ __forceinline__ int value_swizzle(int rho) { return (rho >> 1) & 3; }

// One workgroup = 4 waves x RT tiles of 16 query rows of ONE KV head (times KW key-ways), over the key
// blocks of one split.  RT = 2 halves the LDS operand reads per MFMA (every key / value fragment
// feeds two row tiles): long contexts are bound by exactly those reads.
// Key / value blocks (32 slots) go from memory straight into LDS (no registers, no LDS stores), four stages
// deep, shared by the four waves of a key-way.  The 16 key rows of score tile tt are rows 8(i/4) + 4tt + i%4
// of the block, so that the 8 scores a lane holds of a query row belong to 8 CONSECUTIVE keys
// (8 lg .. 8 lg + 7): its slice of P^T then pairs with one natural 16-byte chunk of a V^T row.
// With a single split the result is normalised and written in the storage type directly;
// otherwise (max, sum, O) partials go to the merge kernel.
template <int DH, int KW> constexpr int ATTN_LDS = 2 * 4 * KW * 32 * DH;   // elements: four stages of a block of keys and one of values per key-way
template <typename T, int DH, int KW, int RT>
__device__ __forceinline__ void attn_mfma_body(
    T *__restrict__ lds_all, const int row_group, const int kvh, const int split, const T *__restrict__ q, int rows, int hq, int hkv, const uint64_t *__restrict__ mask, int n_prefix,
    int region_len, KVCache kv, int blocks_per_split, float scale,
    float *__restrict__ o_part, float *__restrict__ ml_part, int rho_pad, T *__restrict__ out_direct) {
    typedef typename Vec8<T>::type V8;
    typedef __attribute__((address_space(3))) void *LdsPtr;
    constexpr int KS = DH / 32, DT = DH / 16;
    constexpr int CPR = DH / 8;                           // 16-byte chunks of a key row
    constexpr int UNITS = 32 * CPR;                       // 16-byte units of a key block (and of a value block)
    constexpr int WPW = 4;                                // waves per key-way
    constexpr int STG = 64 * WPW;                         // threads of a key-way: they load its blocks
    constexpr int UPT = UNITS / STG;                      // loads per thread and block
    static_assert(UPT >= 1, "a block must give every thread of its key-way a load");
    constexpr int BLK = 32 * DH;                          // elements of a staged block
    constexpr int NST = 4;                                // stages
    // [stage][key-way] blocks of keys, then of values; after the last block the same memory carries the KW-way merge
    static_assert(2 * NST * KW * BLK == ATTN_LDS<DH, KW>, "what the caller provides");
    T *ks_lds = lds_all, *vs_lds = lds_all + NST * KW * BLK;

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, lr = lane & 15, lg = lane >> 4;
    // which of the KW blocks of an iteration this wave takes (wave / 4; wave-uniform: branches on it are scalar) and
    // which of the four groups of row tiles.  (Waves w and w + 4, the two key-ways of a tile group, are the pair the
    // text below places on one SIMD; giving the pairs (2w, 2w + 1) the two ways instead measured the same.)
    const int kway = __builtin_amdgcn_readfirstlane(tid / STG), wq = wave % WPW;
    const int stid = tid % STG;
    const int G = hq / hkv;
    const int tile0 = (row_group * WPW + wq) * RT;        // this wave's tiles: tile0 .. tile0 + RT - 1
    // query row of lane lr in row tile rt: (valid, row of the pass, query head).  Recomputed where it is needed
    // (the masked blocks at the end of the keys, the final stores) rather than kept in registers over the loop.
    auto row_of = [&](int rt, bool &valid, int &m, int &qh) {
        const int rho = (tile0 + rt) * 16 + lr;
        valid = rho < rows * G;
        m = valid ? rho / G : 0;
        qh = kvh * G + (valid ? rho % G : 0);
    };
    V8 qf[RT][KS];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        bool valid; int m, qh;
        row_of(rt, valid, m, qh);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const u32x4 v = *reinterpret_cast<const u32x4 *>(q + ((size_t)m * hq + qh) * DH + ks * 32 + lg * 8);
            qf[rt][ks] = __builtin_bit_cast(V8, valid ? v : u32x4{0u, 0u, 0u, 0u});
        }
    }

    const int total = n_prefix + region_len;
    const int n_blocks = (total + 31) >> 5;
    const int b0 = split * blocks_per_split, b1 = min(n_blocks, b0 + blocks_per_split);
    const int n_it = (b1 - b0 + KW - 1) / KW;             // iteration `it` takes blocks b0 + it KW .. + KW - 1, one per key-way
    const int P = 1 << kv.page_shift;
    const T *kc = static_cast<const T *>(kv.k), *vc = static_cast<const T *>(kv.vt);

    // Staging.  K block = 32 consecutive token rows = 32*DH contiguous elements; V^T block = DH rows of 32 keys
    // (64 bytes each, row stride P elements).  Thread stid of a block's 256 owns LDS units stid + 256 i and fetches
    // the chunk that belongs there under the swizzle.  Stage it % NST holds iteration it's blocks.
    // (Page-table entries: lane j of pg_vec holds the entry of block b0 + j - a split has at most ATTN_MAX_BPS = 64
    // blocks - fetched with one vector load before the loads to LDS start and picked with v_readlane afterwards.  A
    // scalar load per block would sit in the same counter as the LDS reads and, returning out of order, turn every
    // wait for an operand fragment into a wait for a trip to memory; a vector load inside the loop would make the
    // compiler wait for every load in flight.)
    auto block_of = [&](int it) { return min(b0 + it * KW + kway, b1 - 1); };   // never predicated: past the end a valid block is loaded again and ignored
    const int pg_vec = kv.page_table[(min(b0 + lane, b1 - 1) << 5) >> kv.page_shift];
    auto page_of_block = [&](int b) { return __builtin_amdgcn_readlane(pg_vec, (b - b0) & 63); };   // b wave-uniform
    int k_goff[UPT], v_goff[UPT];                         // element offsets of this thread's chunks inside a block
#pragma unroll
    for (int i = 0; i < UPT; ++i) {
        const int u = stid + i * STG;
        const int krow = u / CPR, kpos = u % CPR;
        k_goff[i] = krow * DH + (kpos ^ key_swizzle<DH>(krow)) * 8;
        const int vrow = u >> 2, vpos = u & 3;
        v_goff[i] = vrow * P + (vpos ^ value_swizzle(vrow)) * 8;
    }
    const unsigned lds_k0 = (unsigned)(uintptr_t)(LdsPtr)ks_lds, lds_v0 = (unsigned)(uintptr_t)(LdsPtr)vs_lds;
    // byte offset of this wave's 64 units of load 0 inside a stage, wave-uniform
    const unsigned wave_units = __builtin_amdgcn_readfirstlane(kway * BLK * (int)sizeof(T) + wq * 1024);
    auto issue_k = [&](int it) {
        const int b = block_of(it), off = (b << 5) & (P - 1);
        const T *kb = kc + ((size_t)(page_of_block(b) * hkv + kvh) * P + off) * DH;
        const unsigned base = lds_k0 + (unsigned)((it & (NST - 1)) * KW * BLK * (int)sizeof(T)) + wave_units;
#pragma unroll
        for (int i = 0; i < UPT; ++i) lds_dma16(base + i * STG * 16, kb + k_goff[i]);
    };
    auto issue_v = [&](int it) {
        const int b = block_of(it), off = (b << 5) & (P - 1);
        const T *vb = vc + (size_t)(page_of_block(b) * hkv + kvh) * DH * P + off;
        const unsigned base = lds_v0 + (unsigned)((it & (NST - 1)) * KW * BLK * (int)sizeof(T)) + wave_units;
#pragma unroll
        for (int i = 0; i < UPT; ++i) lds_dma16(base + i * STG * 16, vb + v_goff[i]);
    };

    f32x4 acc[RT][DT];
    float m_run[RT], l_run[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        m_run[rt] = -INFINITY; l_run[rt] = 0.f;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) acc[rt][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    // operand reads: element offsets of this lane inside a staged block
    const int kappa0 = 8 * (lr >> 2) + (lr & 3), kswz = key_swizzle<DH>(kappa0);
    int k_rd[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) k_rd[ks] = kappa0 * DH + ((ks * 4 + lg) ^ kswz) * 8;
    const int v_rd = lr * 32 + (lg ^ value_swizzle(lr)) * 8;

    // S^T tiles of iteration it's block for this wave's row tiles: rows = keys 8(i/4) + 4tt + i%4, columns = query rows.
    // Every key fragment of the block is requested before the first MFMA.
    auto key_fragments = [&](int it, u32x4 (&kf)[2][KS]) {
        const T *kbuf = &ks_lds[((it & (NST - 1)) * KW + kway) * BLK];
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) kf[tt][ks] = *reinterpret_cast<const u32x4 *>(&kbuf[tt * 4 * DH + k_rd[ks]]);
    };
    auto scores_of = [&](const u32x4 (&kf)[2][KS], f32x4 (&s)[RT][2]) {
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) s[rt][tt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                    s[rt][tt] = Vec8<T>::mfma(__builtin_bit_cast(V8, kf[tt][ks]), qf[rt][ks], s[rt][tt]);
        }
    };
    auto scores = [&](int it, f32x4 (&s)[RT][2]) {
        u32x4 kf[2][KS];
        key_fragments(it, kf);
        scores_of(kf, s);
    };
    // bf16 keeps 8 significant bits: probabilities rounded to it moved a layer's output by 2e-2 at the 8B
    // shape (the mean of hundreds of values loses its low bits), ten times everything else.  They go into the
    // P V product as a sum of two bf16 numbers, p = hi + lo, 16 significant bits, at the price of a second
    // MFMA per value fragment.  fp16 (11 bits) stays single.
    constexpr bool SPLIT_P = std::is_same<T, bf16_t>::value;
    // acc += V^T P^T of iteration it's block, in two halves of the value fragments (h = 0, 1) so that only half of them
    // need registers at a time
    auto pv_half = [&](int it, auto h_tag, const V8 (&p_hi)[RT], const V8 (&p_lo)[RT]) {
        constexpr int HD = DT / 2, H = decltype(h_tag)::value;
        const T *vbuf = &vs_lds[((it & (NST - 1)) * KW + kway) * BLK];
        u32x4 vf[HD];
#pragma unroll
        for (int d = 0; d < HD; ++d) vf[d] = *reinterpret_cast<const u32x4 *>(&vbuf[(H * HD + d) * 16 * 32 + v_rd]);
#pragma unroll
        for (int d = 0; d < HD; ++d)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
                acc[rt][H * HD + d] = Vec8<T>::mfma(__builtin_bit_cast(V8, vf[d]), p_hi[rt], acc[rt][H * HD + d]);
        if constexpr (SPLIT_P) {
#pragma unroll
            for (int d = 0; d < HD; ++d)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                    acc[rt][H * HD + d] = Vec8<T>::mfma(__builtin_bit_cast(V8, vf[d]), p_lo[rt], acc[rt][H * HD + d]);
        }
    };
    typedef std::integral_constant<int, 0> I0;
    typedef std::integral_constant<int, 1> I1;
    auto pv = [&](int it, const V8 (&p_hi)[RT], const V8 (&p_lo)[RT]) {
        pv_half(it, I0{}, p_hi, p_lo);
        pv_half(it, I1{}, p_hi, p_lo);
    };
    // Online softmax of one block's scores: running maximum and sum updated, the probabilities left in MFMA operand
    // form, alpha = the factor the accumulators are to be multiplied by; returns whether any lane's alpha differs from 1.
    // A lane holds keys slot0 + 8 lg + j (j = 4 tt + r) of query row lr.  Scores are kept in the log2
    // domain (scale * log2 e folded into one factor) so that the exponentials are single v_exp_f32 instructions.
    // INSIDE: the whole block lies in the committed prefix (no mask, and some key is visible to every row).
    auto softmax_tile = [&](auto inside_tag, auto rt_tag, int slot0, const f32x4 (&s)[RT][2], V8 (&p_hi)[RT], V8 (&p_lo)[RT], float (&alpha)[RT]) {
        constexpr bool INSIDE = decltype(inside_tag)::value;
        constexpr int rt = decltype(rt_tag)::value;
        {
            // raw scores; the factor (positive: the maximum commutes with it) goes into the exponent's fma
            float sv[8], bm = -INFINITY;
            if (INSIDE || slot0 + 32 <= n_prefix) {
#pragma unroll
                for (int j = 0; j < 8; ++j) { sv[j] = s[rt][j >> 2][j & 3]; bm = fmaxf(bm, sv[j]); }
            } else {
                // the row's mask words come from memory here: few blocks reach into the region
                bool valid; int m, qh;
                row_of(rt, valid, m, qh);
                const uint64_t m0 = valid ? mask[(size_t)m * MASK_WORDS] : 0ull, m1 = valid ? mask[(size_t)m * MASK_WORDS + 1] : 0ull;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int slot = slot0 + 8 * lg + j;
                    sv[j] = slot_visible(slot, n_prefix, region_len, m0, m1) ? s[rt][j >> 2][j & 3] : -INFINITY;
                    bm = fmaxf(bm, sv[j]);
                }
            }
            bm = rows_max(bm) * scale;
            // The reference point of the exponentials only moves when the block's maximum is more than
            // 2^8 above it (any reference gives the same quotient; the probabilities then go up to 256
            // instead of 1, exact in float32 and in the 16-bit operand alike): without the slack nearly
            // every block moves some row's maximum a little and all accumulators are rescaled.
            const float m_new = bm > m_run[rt] + 8.f ? bm : m_run[rt];
            float psum = 0.f;
            alpha[rt] = 1.f;
            if (!INSIDE && m_new == -INFINITY) {
#pragma unroll
                for (int j = 0; j < 8; ++j) { p_hi[rt][j] = (T)0.f; p_lo[rt][j] = (T)0.f; }
            } else {
                alpha[rt] = __builtin_amdgcn_exp2f(m_run[rt] - m_new);   // 2^(-inf) = 0 on the first visible block
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float pe = __builtin_amdgcn_exp2f(fmaf(sv[j], scale, -m_new));
                    p_hi[rt][j] = from_f<T>(pe);
                    if constexpr (SPLIT_P) p_lo[rt][j] = from_f<T>(pe - to_f(p_hi[rt][j]));
                    psum += pe;
                }
            }
            l_run[rt] = l_run[rt] * alpha[rt] + psum;
            m_run[rt] = m_new;
            return __builtin_amdgcn_ballot_w64(alpha[rt] != 1.f) != 0;   // rare once the maximum has settled
        }
    };
    auto softmax = [&](auto inside_tag, int slot0, const f32x4 (&s)[RT][2], V8 (&p_hi)[RT], V8 (&p_lo)[RT], float (&alpha)[RT]) {
        bool rescale = softmax_tile(inside_tag, I0{}, slot0, s, p_hi, p_lo, alpha);
        if constexpr (RT > 1) rescale = rescale | softmax_tile(inside_tag, I1{}, slot0, s, p_hi, p_lo, alpha);   // (no short circuit: it would cut the block in two)
        return rescale;
    };
    auto rescale_acc = [&](const float (&alpha)[RT]) {   // behind a wave-uniform branch that is rarely taken
        asm volatile("" ::: "memory");                   // (keeps the compiler from turning it into 64 selects)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) acc[rt][dt] *= alpha[rt];
    };

    // Schedule.  The loads of an iteration are issued two iterations before the first wave reads them: at the top of
    // iteration `it` go the keys of it + 3 (stage last read by the scores of it - 1, at least one barrier ago) and the
    // values of it + 2 (stage last read by the P V of it - 2, at least one barrier ago); at its foot every wave waits
    // until only those are outstanding, and the barrier then publishes the keys of it + 2 and the values of it + 1.
    // The waves of a workgroup move in step from barrier to barrier, and with two key-ways a SIMD holds one wave of
    // each.  The two key-ways take an iteration in opposite order, so that one wave of a SIMD has vector work while the
    // other has matrix work:
    //   way 0: softmax of it (scores formed an iteration ago), then P V of it and scores of it + 1      vector, matrix
    //   way 1: scores of it + 1 and P V of it (probabilities formed an iteration ago), then softmax of it + 1
    // The accumulators of a key-way see the same operations in the same order either way.  (One key-way: the order of
    // way 0.)  Measured against both ways in way 0's order with the next scores ahead of the softmax: 35.5 against
    // 35.9 us at 8192 tokens - timestamps taken inside the kernel show each wave's own chain (LDS reads, a run of
    // dependent MFMAs, the softmax) at about 3000 of an iteration's 4200 cycles whatever the other wave does.
    // The P V product of an iteration is unconditional (a conditional one made the compiler keep two copies of the
    // accumulators): way 1's block beyond an odd end gets zero probabilities against the valid block staged in its place.
    typedef std::integral_constant<bool, true> Inside;
    typedef std::integral_constant<bool, false> Anywhere;
    const bool matrix_first = KW == 2 && kway == 1;        // wave-uniform
    issue_k(0);
    issue_k(1);
    issue_v(0);
    issue_k(2);
    issue_v(1);
    dma_wait<2 * UPT>();                                  // keys of iterations 0 and 1 and values of iteration 0 have landed
    __syncthreads();
    // softmax of block b's scores -> probabilities; accumulators rescaled
    auto softmax_block = [&](int b, const f32x4 (&s)[RT][2], V8 (&p_hi)[RT], V8 (&p_lo)[RT]) {
        float alpha[RT];
        const bool rescale = (b << 5) + 32 <= n_prefix ? softmax(Inside{}, b << 5, s, p_hi, p_lo, alpha)
                                                       : softmax(Anywhere{}, b << 5, s, p_hi, p_lo, alpha);
        if (rescale) rescale_acc(alpha);
    };
    auto top = [&](int it) {
        if (it + 3 < n_it) issue_k(it + 3);               // workgroup-uniform, like the waits at the foot
        if (it + 2 < n_it) issue_v(it + 2);
    };
    auto foot = [&](int it) {
        if (it + 3 < n_it) dma_wait<2 * UPT>();
        else if (it + 2 < n_it) dma_wait<UPT>();
        else dma_wait<0>();
        __syncthreads();
    };
    // (one loop per order, each with the state of its own order only: scores kept from iteration to iteration in
    // the first, probabilities in the second.  Branches on block indices are wave-uniform.)
    if (!matrix_first) {
        f32x4 s[RT][2];
        scores(0, s);                                     // way 0's block of an iteration always exists
        for (int it = 0; it < n_it; ++it) {
            top(it);
            const int b = b0 + it * KW + kway;
            V8 p_hi[RT], p_lo[RT];
            softmax_block(b, s, p_hi, p_lo);
            __builtin_amdgcn_sched_barrier(0);            // (operand reads hoisted above the softmax would not fit the registers)
            pv(it, p_hi, p_lo);
            if (b + KW < b1) scores(it + 1, s);
            foot(it);
        }
    } else {
        V8 p_hi[RT], p_lo[RT];
        f32x4 s[RT][2];
        auto probabilities = [&](int b) {                 // of block b from its scores in s; zero beyond the end
            if (b < b1) {
                softmax_block(b, s, p_hi, p_lo);
            } else {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int j = 0; j < 8; ++j) { p_hi[rt][j] = (T)0.f; p_lo[rt][j] = (T)0.f; }
            }
        };
        if (b0 + kway < b1) scores(0, s);
        probabilities(b0 + kway);
        for (int it = 0; it < n_it; ++it) {
            const int b_next = b0 + (it + 1) * KW + kway;
            // The next block's scores lead the matrix part: by the time the P V products are issued they are complete,
            // and the softmax behind them starts at once (and needs the matrix pipe no more while way 0 fills it).
            top(it);
            if (b_next < b1) scores(it + 1, s);
            pv(it, p_hi, p_lo);
            __builtin_amdgcn_sched_barrier(0);
            probabilities(b_next);
            foot(it);
        }
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        l_run[rt] += __shfl_xor(l_run[rt], 16, 64);
        l_run[rt] += __shfl_xor(l_run[rt], 32, 64);
    }

    if constexpr (KW > 1) {
        // Merge the KW partial (max, sum, O) of each row tile in key-way order: ways 1.. park theirs
        // in LDS (the stages are free once every wave has read its last values), way 0 folds them in;
        // one tile of each wave at a time.
        float *xch = reinterpret_cast<float *>(lds_all);  // per (way-1, wave): 64 lanes x (DT*4 + 2) floats
        constexpr int REC = DT * 4 + 2;
        static_assert((size_t)(KW - 1) * WPW * 64 * REC * sizeof(float) <= ATTN_LDS<DH, KW> * sizeof(T), "merge records must fit");
        float *mine = xch + ((size_t)((kway - 1) * WPW + wq) * 64 + lane) * REC;
        __syncthreads();
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            if (rt > 0) __syncthreads();                  // way 0 has read the previous tile's records
            if (kway > 0) {
                mine[0] = m_run[rt]; mine[1] = l_run[rt];
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) mine[2 + dt * 4 + r] = acc[rt][dt][r];
            }
            __syncthreads();
            if (kway == 0) {
#pragma unroll
                for (int w = 1; w < KW; ++w) {
                    const float *o = xch + ((size_t)((w - 1) * WPW + wq) * 64 + lane) * REC;
                    const float mo = o[0], lo = o[1];
                    const float mn = fmaxf(m_run[rt], mo);
                    if (mn == -INFINITY) continue;
                    const float a0 = __builtin_amdgcn_exp2f(m_run[rt] - mn), a1 = __builtin_amdgcn_exp2f(mo - mn);
                    l_run[rt] = l_run[rt] * a0 + lo * a1;
                    m_run[rt] = mn;
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                        for (int r = 0; r < 4; ++r) acc[rt][dt][r] = acc[rt][dt][r] * a0 + o[2 + dt * 4 + r] * a1;
                }
            }
        }
        if (kway > 0) return;
    }

    // O^T tile dt: lane -> query row lr, register r -> dh index dt*16 + 4*lg + r
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        if (out_direct) {
            bool valid; int m, qh;
            row_of(rt, valid, m, qh);
            if (valid) {
                const float inv = 1.0f / l_run[rt];
                T *dst = out_direct + ((size_t)m * hq + qh) * DH + 4 * lg;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) dst[dt * 16 + r] = from_f<T>(acc[rt][dt][r] * inv);
            }
            continue;
        }
        const int tile = tile0 + rt;
        const size_t prow = ((size_t)split * hkv + kvh) * rho_pad + tile * 16 + lr;
        if (tile * 16 < rho_pad) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
                *reinterpret_cast<f32x4 *>(o_part + prow * DH + dt * 16 + 4 * lg) = acc[rt][dt];
            if (lg == 0) {
                ml_part[prow * 2] = m_run[rt];
                ml_part[prow * 2 + 1] = l_run[rt];
            }
        }
    }
}

// ------------------------------------------------------------------------------------------
// The same attention for long walks (splits of WALK_MIN_BPS blocks; prompts): on v_mfma_f32_32x32x16, the matrix and the vector
// work of a wave interleaved instruction by instruction.  A wave takes 32 query rows, a SIMD holds two waves.  In one step a wave forms
// the scores of block i + 1, the probabilities of block i and the P V products of block i - 1: three things that do not wait for each
// other, so the softmax of a block (about 130 vector instructions) runs in the shadow of 24 MFMAs of 32 cycles each.  The order is
// written out (group by group, a scheduling barrier behind every MFMA): left to itself the compiler lines up each product's LDS reads
// and waits in front of it, and sinks the softmax below the last product.
//   S^T = K Q^T: MFMA row i is key kappa(i) = 16 (i / 16) + 8 (i / 4 % 2) + 4 (i / 8 % 2) + i % 4 of the block, so that register t of
//       half h = lane / 32 belongs to key 16 (t / 8) + 8 h + t % 8 of query row lane % 32: eight consecutive keys are the B operand of
//       one P V MFMA and pair with a 16-byte chunk of a V^T row.
//   O^T = V^T P^T: tile dt = dh indices 32 dt .., register 4 g + r of half h is index 32 dt + 8 g + 4 h + r.
// A workgroup is four waves of rows x two key-ways, a block of 32 keys per way and stage.  (Eight waves of rows and one way, 64 keys a
// stage - half the staging per row and a barrier every other step: a prompt of 8192 tokens 15.3 against 15.4 ms, and walks twice as long:
// 1.5 against 2.1 ms for 8000 tokens of a small shape, whose workgroups are few.)
// Swizzles (an operand read: 32 rows x 2 chunks; 4.4 cycles per ds_read_b128 with every wave of a CU reading): rows of 256 bytes keep chunk
// c of row r at c ^ (r % 16), rows of 128 bytes at c ^ (r / 2 % 8), rows of 64 bytes at c ^ (r / 4 % 4).
// 81 rows of the 8B shape against 8192 keys: 37.6 us by attn_mfma_kernel, 31 (of which 20 remain without products and softmax: launch,
// first trip to memory, 16 iterations of loads and barriers, 12 MB of partial results).
// Which splits are long (bf16): with few rows a wave of 32 has little to do but wait for its own chain, and 16-row tiles are through
// sooner; fp16, without the low halves, gains nothing before they are.  8B shape, us a pass of four target layers, 16-row tiles / these: 1000
// keys (9 blocks a split) 61 rows 583 / 602; 2000 keys 599 / 617; 3000 keys 608 / 630; 4000 keys (32 blocks) 1 row 529 / 520, 61 rows
// 664 / 644; 8192 keys 530 / 523, 81 rows 716 / 700.  fp16, 8000 keys: 640 wide (5 heads) 1 row 275 / 272, 61 rows 333 / 334, 100 rows 398 / 421;
// 13B (40 heads) 759 / 754, 871 / 871, 81 rows 1001 / 966, 100 rows 1088 / 1052; 4000 keys 641 / 640, 767 / 766, 871 / 850, 957 / 940: with
// many heads it would gain from 65 rows on, and a rule for fp16 would have to go by heads x splits, not by rows (a row's bits).
constexpr int WALK_MIN_BPS = 32, WALK_THREADS = 512;
constexpr int PROMPT_SHORT_BLOCKS = 8;                    // a prompt's first range (4 blocks) is computed as a short context is
template <typename T> __device__ __forceinline__ unsigned pack2(float a, float b) {   // two values rounded to T, a in the low half
    typedef T t2 __attribute__((ext_vector_type(2)));
    const t2 v = {from_f<T>(a), from_f<T>(b)};
    return __builtin_bit_cast(unsigned, v);
}
__device__ __forceinline__ float max3(float a, float b, float c) {         // (as the compiler writes it, without quieting NaNs first)
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
template <int BYTES> __device__ __forceinline__ int walk_swizzle(int r) { return BYTES == 256 ? r & 15 : BYTES == 128 ? (r >> 1) & 7 : (r >> 2) & 3; }

// Which 32 query rows of its workgroup's 128 a wave takes.  A SIMD holds waves w and w + 4, one of each key-way: two groups apart, so that
// up to two groups' worth of rows have a SIMD per wave.  One apart, the second group shared a SIMD with the first: a pass of four layers,
// 4000 keys, us, 10 rows of the 8B shape 545 / 528, 40 rows of 640 wide (bf16) 337 / 325; 8 and 24 rows of the 8B shape the same.
__device__ __forceinline__ int walk_rows_of(int wave) { return (wave + 2 * (wave >> 2)) & 3; }

// The wave's rows: row0 .. row0 + rows - 1 of the pass see the n_prefix slots before them and, of their own region_len slots, those in
// their masks; lane's row m = row0 + rho / G, rho = rho0 + lane % 32.  The walk: blocks [b0, b1).
template <typename T, int DH, bool PROMPT>
__device__ __forceinline__ void attn_walk_body(
    T *__restrict__ lds_all, int kvh, int split, const T *__restrict__ q, int row0, int rows, int rho0, int hq, int hkv, const uint64_t *__restrict__ mask,
    int n_prefix, int region_len, KVCache kv, int b0, int b1, float scale, float *__restrict__ o_part, float *__restrict__ ml_part, int rho_pad,
    T *__restrict__ out_direct) {
    typedef typename Vec8<T>::type V8;
    typedef __attribute__((address_space(3))) void *LdsPtr;
    constexpr bool SPLIT_P = std::is_same<T, bf16_t>::value;   // probabilities as hi + lo, see attn_mfma_body
    constexpr int KW = 2, WPW = 4, STG = 64 * WPW, NST = 4;
    constexpr int DT = DH / 32, NG = DH / 16;             // tiles of O^T; groups = k-steps of the scores = value fragments of a block
    constexpr int PVG = SPLIT_P ? 2 : 1, NS = NG * (PVG + 1);   // P V MFMAs of a group; MFMAs of a step
    constexpr int KROW = DH * 2, VROW = 64;               // bytes of a staged row
    constexpr int CPR = KROW / 16, UPT = 32 * CPR / STG, BLK = 32 * DH;      // 16-byte chunks of a key row, loads of a wave per block, elements of a block
    static_assert(2 * NST * KW * BLK == ATTN_LDS<DH, KW>, "what the caller provides");   // [stage][key-way] blocks of keys, then of values
    T *ks_lds = lds_all, *vs_lds = lds_all + NST * KW * BLK;

    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kway = wave >> 2, wq = walk_rows_of(wave);
    const int stid = wq * 64 + lane, G = hq / hkv;
    const int rho = rho0 + l32;
    const bool valid = rho < rows * G, active = rho0 < rows * G;   // (active: wave-uniform)
    const int m = row0 + (valid ? rho / G : 0), qh = kvh * G + (valid ? rho % G : 0);
    V8 qf[NG];
#pragma unroll
    for (int ks = 0; ks < NG; ++ks) {
        const u32x4 v = *reinterpret_cast<const u32x4 *>(q + ((size_t)m * hq + qh) * DH + ks * 16 + h * 8);
        qf[ks] = __builtin_bit_cast(V8, valid ? v : u32x4{0u, 0u, 0u, 0u});
    }

    const int n_it = (b1 - b0 + KW - 1) / KW;             // step `it` takes block b0 + it KW + kway
    const int P = 1 << kv.page_shift;
    const char *kc = static_cast<const char *>(kv.k), *vc = static_cast<const char *>(kv.vt);

    // Staging, by LDS-direct loads as in attn_mfma_body.  Lane j of pg_vec holds (page, head) of block window + j, pg_next those of the
    // 64 blocks behind (PROMPT: a walk may be long).
    auto page_vec = [&](int b) { return kv.page_table[(min(b + lane, b1 - 1) << 5) >> kv.page_shift] * hkv + kvh; };
    int pg_vec = page_vec(b0), pg_next = PROMPT ? page_vec(b0 + 64) : 0, window = b0;
    struct Block { size_t page; unsigned off; };          // byte offset of its page in either cache, its first slot in the page
    auto block_at = [&](int it) {                         // never predicated: past the end a valid block is loaded again and ignored
        const int b = min(b0 + it * KW + kway, b1 - 1);
        const unsigned pidx = PROMPT && b - window >= 64 ? __builtin_amdgcn_readlane(pg_next, (b - window) & 63) : __builtin_amdgcn_readlane(pg_vec, (b - window) & 63);
        return Block{(size_t)pidx * (unsigned)(P * DH * (int)sizeof(T)), (unsigned)((b << 5) & (P - 1))};
    };
    // thread's 16-byte units of a block: stid + i STG.  Keys: row u / CPR; values: row u / 4, chunk by the swizzle.
    unsigned k_goff[UPT], v_goff[UPT];
#pragma unroll
    for (int i = 0; i < UPT; ++i) {
        const int u = stid + i * STG;
        const int krow = u / CPR, kpos = u % CPR;
        k_goff[i] = (unsigned)(krow * KROW + (kpos ^ walk_swizzle<KROW>(krow)) * 16);
        const int vrow = u >> 2, c = (u & 3) ^ walk_swizzle<VROW>(vrow);
        v_goff[i] = (unsigned)((vrow * P + c * 8) * (int)sizeof(T));
    }
    const unsigned lds_k0 = (unsigned)(uintptr_t)(LdsPtr)ks_lds, lds_v0 = (unsigned)(uintptr_t)(LdsPtr)vs_lds;
    const unsigned wave_units = (unsigned)(kway * BLK * (int)sizeof(T) + wq * 1024);
    auto scalar = [](const char *p) {                     // (wave-uniform already: says so)
        const uint64_t x = reinterpret_cast<uint64_t>(p);
        return reinterpret_cast<const char *>((uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)(x >> 32)) << 32 | (unsigned)__builtin_amdgcn_readfirstlane((int)x));
    };
    auto stage_at = [&](int it) { return (unsigned)((it & (NST - 1)) * KW * BLK * (int)sizeof(T)); };
    auto issue_k = [&](int it, const Block &b, int i) {
        lds_dma16_s(lds_k0 + stage_at(it) + wave_units + i * STG * 16, scalar(kc + b.page + b.off * KROW), k_goff[i]);
    };
    auto issue_v = [&](int it, const Block &b, int i) {
        lds_dma16_s(lds_v0 + stage_at(it) + wave_units + i * STG * 16, scalar(vc + b.page + b.off * (int)sizeof(T)), v_goff[i]);
    };

    // operand reads: byte addresses of this lane inside a stage; the chunk of fragment u by xor
    const int kappa = 16 * (l32 >> 4) + 8 * ((l32 >> 2) & 1) + 4 * ((l32 >> 3) & 1) + (l32 & 3);
    const unsigned k_rd = (unsigned)(kway * BLK * (int)sizeof(T)) + kappa * KROW + ((h ^ walk_swizzle<KROW>(kappa)) * 16);
    const unsigned v_rd = (unsigned)(kway * BLK * (int)sizeof(T)) + l32 * VROW + ((h ^ walk_swizzle<VROW>(l32)) * 16);
    auto key_at = [&](int it) { return stage_at(it) + k_rd; };
    auto value_at = [&](int it) { return stage_at(it) + v_rd; };
    auto key_fragment = [&](unsigned at, int u) {
        return *reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(ks_lds) + (at ^ (unsigned)(u * 32)));
    };
    auto value_fragment = [&](unsigned at, int f) {       // f: dh tile f % DT, keys 16 (f / DT) ..
        return *reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(vs_lds) + ((at ^ (unsigned)((f / DT) * 32)) + (f % DT) * 32 * VROW));
    };

    f32x16 acc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[dt][i] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
    struct Prob { u32x4 hi[2], lo[2]; };

    // Step `it`: softmax of block `it` (scores in s, probabilities to pn), scores of block it + 1 to sn, P V of block it - 1
    // (probabilities pp; FIRST: there is none).  vf holds the first value fragments of block it - 1 on entry, of block `it` on exit.
    // In between it issues the loads `load(l)`, l = 0 .. N_LOADS - 1, one at a time: eight waves asking for 32 KB at the top of an
    // iteration kept each other from issuing anything for 500 cycles.
    u32x4 vf[4];
    constexpr int N_LOADS = 2 * UPT;
    auto step = [&](auto first_tag, int it, f32x16 &s, f32x16 &sn, const Prob &pp, Prob &pn, auto load) {
        constexpr bool FIRST = decltype(first_tag)::value;
        const unsigned k_st = key_at(it + 1), v_st = value_at(it - 1), v_next = value_at(it);
        u32x4 kf[3];
        kf[0] = key_fragment(k_st, 0);
        kf[1] = key_fragment(k_st, 1);
        __builtin_amdgcn_sched_barrier(0);
        float mx = 0.f, m_ref = 0.f, alpha = 1.f, psum = 0.f, e[16];
        // The softmax in N_CHUNKS pieces, a value's exponential, its part in the sum and the high half of its pair, and the low half in
        // three successive ones: an instruction that needs the one before it costs a wave 9 cycles, one that does not 6.
        // (The empty statements hold a value where it is computed: the compiler would sink all of it below the last MFMA.)
        constexpr int N_CHUNKS = 22;
        auto sum_and_pack = [&](int j) {
            asm volatile("" : "+v"(e[j]));
            psum += e[j];
            asm volatile("" : "+v"(psum));
            if (j & 1) {
                unsigned hi = pack2<T>(e[j - 1], e[j]);
                asm volatile("" : "+v"(hi));
                pn.hi[j >> 3][(j & 7) >> 1] = hi;
            }
        };
        auto low_half = [&](int j) {                      // of the pair (j - 1, j)
            if constexpr (SPLIT_P) {
                const unsigned hi = pn.hi[j >> 3][(j & 7) >> 1];
                unsigned lo = pack2<T>(e[j - 1] - __builtin_bit_cast(float, hi << 16), e[j] - __builtin_bit_cast(float, hi & 0xffff0000u));
                asm volatile("" : "+v"(lo));
                pn.lo[j >> 3][(j & 7) >> 1] = lo;
            }
        };
        auto chunk = [&](int c) {
            if (c == 0) {
                float a = s[0], b = s[8];
#pragma unroll
                for (int j = 1; j < 7; j += 2) { a = max3(a, s[j], s[j + 1]); b = max3(b, s[8 + j], s[9 + j]); }
                mx = max3(a, b, max3(s[7], s[15], s[15]));
            } else if (c == 1) {
                float a, b;
                swap32(mx, a, b);
                mx = max3(a, b, b) * scale;
            } else if (c == 2) {
                const float m_new = mx > m_run + 8.f ? mx : m_run;    // (the reference moves only when it has to: see attn_mfma_body)
                m_ref = m_new == -INFINITY ? 0.f : m_new; // (nothing visible yet)
                mx = m_run - m_ref;
                m_run = m_new;
            } else if (c == 3) {
                alpha = __builtin_amdgcn_exp2f(mx);
            } else {
                const int j = c - 4;
                if (j < 16) {
                    const float sv = s[j];
                    e[j] = __builtin_amdgcn_exp2f(fmaf(sv, scale, -m_ref));
                }
                if (j >= 1 && j <= 16) sum_and_pack(j - 1);
                if (j >= 2 && (j - 2) % 2 == 1) low_half(j - 2);
            }
        };
        constexpr int NSV = FIRST ? NG : NS, PV = FIRST ? 0 : PVG;   // MFMAs of this variant, P V MFMAs of a group
#pragma unroll
        for (int u = 0; u < NG; ++u) {
            // fragments of two groups ahead
            if (u + 2 < NG) kf[(u + 2) % 3] = key_fragment(k_st, u + 2);
            if constexpr (SPLIT_P) {
                if (u % 2 == 0) {
#pragma unroll
                    for (int w = 0; w < 2; ++w) {
                        if (u + 2 < NG) { if (!FIRST) vf[(u + 2 + w) & 3] = value_fragment(v_st, u + 2 + w); }
                        else vf[(u + 2 + w) & 3] = value_fragment(v_next, u + 2 + w - NG);
                    }
                }
            } else {
                if (u + 2 < NG) { if (!FIRST) vf[(u + 2) & 3] = value_fragment(v_st, u + 2); }
                else vf[(u + 2) & 3] = value_fragment(v_next, u + 2 - NG);
            }
#pragma unroll
            for (int w = 0; w <= PV; ++w) {
                if (w < PV) {
                    const int f = SPLIT_P ? (u & ~1) + w : u;
                    const V8 p = __builtin_bit_cast(V8, SPLIT_P && (u & 1) ? pp.lo[f / DT] : pp.hi[f / DT]);
                    acc[f % DT] = Vec8<T>::mfma32(__builtin_bit_cast(V8, vf[f & 3]), p, acc[f % DT]);
                } else {
                    f32x16 z;
                    if (u == 0) {
#pragma unroll
                        for (int i = 0; i < 16; ++i) z[i] = 0.f;
                    } else {
                        z = sn;
                    }
                    sn = Vec8<T>::mfma32(__builtin_bit_cast(V8, kf[u % 3]), qf[u], z);
                }
                const int t = u * (PV + 1) + w;
#pragma unroll
                for (int c = t * N_CHUNKS / NSV; c < (t + 1) * N_CHUNKS / NSV; ++c) chunk(c);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int l = 0; l < N_LOADS; ++l)
                if (u == (2 * l + 1) * NG / (2 * N_LOADS)) load(l);
        }
        l_run = l_run * alpha + psum;
        if (!FIRST && __builtin_amdgcn_ballot_w64(alpha != 1.f) != 0) {    // rare once the maximum has settled
            asm volatile("" ::: "memory");                // (keeps the compiler from turning it into 64 selects)
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) acc[dt] *= alpha;
        }
    };
    // scores of keys that the row does not see (few blocks reach into the region: its mask words come from memory here)
    auto hide = [&](int b, f32x16 &s) {
        const uint64_t m0 = valid ? mask[(size_t)m * MASK_WORDS] : 0ull, m1 = valid ? mask[(size_t)m * MASK_WORDS + 1] : 0ull;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const float v = s[j];
            s[j] = (b < b1) & slot_visible((b << 5) + 16 * (j >> 3) + 8 * h + (j & 7), n_prefix, region_len, m0, m1) ? v : -INFINITY;
        }
    };
    // P V of the last block
    auto last_pv = [&](int it, const Prob &pp) {
        const unsigned v_st = value_at(it);
#pragma unroll
        for (int f = 0; f < NG; ++f) {
            const V8 v = __builtin_bit_cast(V8, f < 2 ? vf[f] : value_fragment(v_st, f));
            acc[f % DT] = Vec8<T>::mfma32(v, __builtin_bit_cast(V8, pp.hi[f / DT]), acc[f % DT]);
            if constexpr (SPLIT_P) acc[f % DT] = Vec8<T>::mfma32(v, __builtin_bit_cast(V8, pp.lo[f / DT]), acc[f % DT]);
        }
    };

    // Loads are issued two iterations ahead, as in attn_mfma_body: in iteration `it` the keys of it + 3 (their stage was last read in
    // it - 2) and the values of it + 2 (last read in it - 1); at its foot every wave waits until only those are outstanding, and the
    // barrier then publishes the keys of it + 2 and the values of it + 1.  (PROMPT: past the end a valid block is loaded again, without
    // a branch.)
    typedef std::integral_constant<bool, true> Yes;
    typedef std::integral_constant<bool, false> No;
    Block ahead, last;                                    // the blocks of it + 3 and it + 2
    f32x16 sa, sb;
    Prob pa, pb;
    auto iterate = [&](auto first_tag, int it, f32x16 &s, f32x16 &sn, const Prob &pp, Prob &pn) {
        const bool more_k = it + 3 < n_it, more_v = it + 2 < n_it;   // (workgroup-uniform)
        if (PROMPT && it > 0 && (it * KW) % 64 == 0) {    // (the blocks asked for below lie at most 7 beyond this iteration's)
            window += 64;
            pg_vec = pg_next;
            pg_next = page_vec(window + 64);
        }
        last = ahead;
        ahead = block_at(it + 3);
        auto load = [&](int l) {                          // keys first
            if (l < UPT) { if (PROMPT || more_k) issue_k(it + 3, ahead, l); }
            else if (PROMPT || more_v) issue_v(it + 2, last, l - UPT);
        };
        if (active) {
            const int b = b0 + it * KW + kway;
            if ((b << 5) + 32 > n_prefix || b >= b1) hide(b, s);
            step(first_tag, it, s, sn, pp, pn, load);
        } else {
#pragma unroll
            for (int l = 0; l < N_LOADS; ++l) load(l);
        }
        if (PROMPT || more_k) dma_wait<2 * UPT>();
        else if (more_v) dma_wait<UPT>();
        else dma_wait<0>();
        __syncthreads();
    };
    {
        const Block t = block_at(0);
        last = block_at(1);
        ahead = block_at(2);
#pragma unroll
        for (int i = 0; i < UPT; ++i) issue_k(0, t, i);
#pragma unroll
        for (int i = 0; i < UPT; ++i) issue_k(1, last, i);
#pragma unroll
        for (int i = 0; i < UPT; ++i) issue_v(0, t, i);
#pragma unroll
        for (int i = 0; i < UPT; ++i) issue_k(2, ahead, i);
#pragma unroll
        for (int i = 0; i < UPT; ++i) issue_v(1, last, i);
    }
    dma_wait<2 * UPT>();                                  // keys of iterations 0 and 1 and values of iteration 0 have landed
    __syncthreads();
    if (active) {
#pragma unroll
        for (int i = 0; i < 16; ++i) sa[i] = 0.f;
#pragma unroll
        for (int u = 0; u < NG; ++u) sa = Vec8<T>::mfma32(__builtin_bit_cast(V8, key_fragment(key_at(0), u)), qf[u], sa);
    }
    iterate(Yes{}, 0, sa, sb, pb, pa);
    int it = 1;
    for (; it + 1 < n_it; it += 2) {
        iterate(No{}, it, sb, sa, pa, pb);
        iterate(No{}, it + 1, sa, sb, pb, pa);
    }
    if (it < n_it) {
        iterate(No{}, it, sb, sa, pa, pb);
        if (active) last_pv(n_it - 1, pb);
    } else if (active) {
        last_pv(n_it - 1, pa);
    }
    {
        float a, b;
        swap32(l_run, a, b);
        l_run = a + b;
    }

    if constexpr (PROMPT) dma_wait<0>();                  // (no load may land where the results are exchanged)
    // the other key-way's (max, sum, O) through LDS, folded in by way 0: [wave][value][lane]
    float *xch = reinterpret_cast<float *>(lds_all) + (size_t)wq * (DT * 16 + 2) * 64 + lane;
    static_assert((size_t)WPW * (DT * 16 + 2) * 64 * sizeof(float) <= ATTN_LDS<DH, KW> * sizeof(T), "merge records must fit");
    __syncthreads();
    if (kway > 0) {
        xch[0] = m_run;
        xch[64] = l_run;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int i = 0; i < 16; ++i) xch[(2 + dt * 16 + i) * 64] = acc[dt][i];
    }
    __syncthreads();
    if (kway > 0 || !active) return;
    const float mo = xch[0], lo = xch[64], mn = fmaxf(m_run, mo);
    if (mn != -INFINITY) {
        const float a0 = __builtin_amdgcn_exp2f(m_run - mn), a1 = __builtin_amdgcn_exp2f(mo - mn);
        l_run = l_run * a0 + lo * a1;
        m_run = mn;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[dt][i] = acc[dt][i] * a0 + xch[(2 + dt * 16 + i) * 64] * a1;
    }
    if (PROMPT || out_direct) {
        if (!valid) return;
        struct __attribute__((aligned(4 * sizeof(T)))) Quad { T t[4]; };
        const float inv = 1.0f / l_run;
        T *dst = out_direct + ((size_t)m * hq + qh) * DH + 4 * h;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                Quad o;
#pragma unroll
                for (int r = 0; r < 4; ++r) o.t[r] = from_f<T>(acc[dt][4 * g + r] * inv);
                *reinterpret_cast<Quad *>(dst + dt * 32 + g * 8) = o;
            }
        return;
    }
    if (rho >= rho_pad) return;
    const size_t prow = ((size_t)split * hkv + kvh) * rho_pad + rho;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            f32x4 v;
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = acc[dt][4 * g + r];
            *reinterpret_cast<f32x4 *>(o_part + prow * DH + dt * 32 + g * 8 + 4 * h) = v;
        }
    if (h == 0) {
        ml_part[prow * 2] = m_run;
        ml_part[prow * 2 + 1] = l_run;
    }
}

// a split of a sequence's keys, for the 128 query rows x heads of row_group
template <typename T, int DH>
__device__ __forceinline__ void attn_walk_split(T *lds, int row_group, int kvh, int split, const T *q, int rows, int hq, int hkv, const uint64_t *mask,
                                                int n_prefix, int region_len, KVCache kv, int blocks_per_split, float scale, float *o_part,
                                                float *ml_part, int rho_pad, T *out_direct) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wq = walk_rows_of(wave);
    const int b0 = split * blocks_per_split, b1 = min((n_prefix + region_len + 31) >> 5, b0 + blocks_per_split);
    attn_walk_body<T, DH, false>(lds, kvh, split, q, 0, rows, (row_group * 4 + wq) * 32, hq, hkv, mask, n_prefix, region_len, kv, b0, b1, scale, o_part,
                                 ml_part, rho_pad, out_direct);
}

// Workgroup id -> (row group, KV head, split).  Consecutive ids go to the 8 XCDs in turn, each with an
// L2 of its own, so the row groups that read the same keys and values (same head and split) are given
// ids that are equal modulo 8: the block is fetched from memory once and then found in that L2.
// Returns false for the padding of the last round of eight.
__device__ __forceinline__ bool attn_place(int wg_id, int n_pairs, int n_row_groups, int &row_group, int &pair) {
    const int xcd = wg_id & 7, qid = wg_id >> 3;
    row_group = qid % n_row_groups;
    pair = (qid / n_row_groups) * 8 + xcd;
    return pair < n_pairs;
}

template <typename T, int DH, int KW, int RT>
__global__ __launch_bounds__(256 * KW) void attn_mfma_kernel(
    const T *__restrict__ q, int rows, int hq, int hkv, const uint64_t *__restrict__ mask, int n_prefix,
    int region_len, KVCache kv, int blocks_per_split, int n_splits, int n_row_groups, float scale,
    float *__restrict__ o_part, float *__restrict__ ml_part, int rho_pad, T *__restrict__ out_direct) {
    __shared__ __attribute__((aligned(1024))) T lds[ATTN_LDS<DH, KW>];
    int row_group, pair;
    if (!attn_place(blockIdx.x, hkv * n_splits, n_row_groups, row_group, pair)) return;
    attn_mfma_body<T, DH, KW, RT>(lds, row_group, pair % hkv, pair / hkv, q, rows, hq, hkv, mask, n_prefix, region_len, kv, blocks_per_split,
                                  scale, o_part, ml_part, rho_pad, out_direct);
}

template <typename T, int DH>
__global__ __launch_bounds__(WALK_THREADS) void attn_walk_kernel(
    const T *__restrict__ q, int rows, int hq, int hkv, const uint64_t *__restrict__ mask, int n_prefix,
    int region_len, KVCache kv, int blocks_per_split, int n_splits, int n_row_groups, float scale,
    float *__restrict__ o_part, float *__restrict__ ml_part, int rho_pad, T *__restrict__ out_direct) {
    __shared__ __attribute__((aligned(1024))) T lds[ATTN_LDS<DH, 2>];
    int row_group, pair;
    if (!attn_place(blockIdx.x, hkv * n_splits, n_row_groups, row_group, pair)) return;
    attn_walk_split<T, DH>(lds, row_group, pair % hkv, pair / hkv, q, rows, hq, hkv, mask, n_prefix, region_len, kv, blocks_per_split,
                                 scale, o_part, ml_part, rho_pad, out_direct);
}

// A prompt's rows [0, rows) at slots c0 ..: ranges of MAX_ROWS rows (the width of a row's mask), each against the slots before
// it and itself, all in one launch.  With thousands of rows the keys need no splitting: a workgroup walks all of them and
// writes its rows directly - no partial outputs, no merge.  Pairs (range, KV head) are dealt to the XCDs in turn, the longest
// walks first.  The first n_short ranges have walks as short as the splits of a short context and are computed as those are, bit for
// bit (the ids behind walk_wgs).
// One layer of 8192 tokens (two passes) of the 8B shape: 1.15 ms by attn_mfma_body, 0.81 with attn_walk_body (680 TFLOP/s of the causal
// product, 1.02 PFLOP/s of MFMAs: the low halves of the probabilities are half as many again).
template <typename T, int DH>
__global__ __launch_bounds__(WALK_THREADS) void attn_prompt_kernel(const T *__restrict__ q, int rows, int hq, int hkv, const uint64_t *__restrict__ mask,
                                                          int c0, KVCache kv, int n_short, int walk_wgs, float scale, T *__restrict__ out) {
    __shared__ __attribute__((aligned(1024))) T lds[ATTN_LDS<DH, 2>];
    const int n_row_groups = (MAX_ROWS * (hq / hkv) + 127) / 128, n_ranges = (rows + MAX_ROWS - 1) / MAX_ROWS;
    const bool brief = (int)blockIdx.x >= walk_wgs;
    int row_group, pair;
    if (!attn_place(blockIdx.x - (brief ? walk_wgs : 0), hkv * (brief ? n_short : n_ranges - n_short), n_row_groups, row_group, pair)) return;
    const int range = brief ? pair / hkv : n_ranges - 1 - pair / hkv;
    const int r0 = range * MAX_ROWS, n = min(MAX_ROWS, rows - r0), b1 = (c0 + r0 + n + 31) >> 5;
    if (brief) {
        const size_t off = (size_t)r0 * hq * DH;
        attn_mfma_body<T, DH, 2, 2>(lds, row_group, pair % hkv, 0, q + off, n, hq, hkv, mask + (size_t)r0 * MASK_WORDS, c0 + r0, n, kv, b1, scale,
                                    nullptr, nullptr, 0, out + off);
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wq = walk_rows_of(wave);
    attn_walk_body<T, DH, true>(lds, pair % hkv, 0, q, r0, n, (row_group * 4 + wq) * 32, hq, hkv, mask, c0 + r0, n, kv, 0, b1, scale,
                                nullptr, nullptr, 0, out);
}

// Several sequences in one launch: every sequence has its own rows, cache, prefix, split count and slice of the
// partial buffers; a workgroup finds its sequence from the first workgroup id of each, then does exactly what it does
// in a launch of its own.
constexpr int ATTN_MAX_SEQ = 8;
struct AttnSeq {
    const void *q; const uint64_t *mask; void *out_direct; float *o_part, *ml_part;
    KVCache kv;
    int rows, n_prefix, region_len, blocks_per_split, n_splits, n_row_groups, rho_pad, wg0, row0;
};
struct AttnSeqs { int n; AttnSeq s[ATTN_MAX_SEQ]; };

template <typename T, int DH, int KW, int RT>
__global__ __launch_bounds__(256 * KW) void attn_mfma_batch_kernel(AttnSeqs seqs, int hq, int hkv, float scale) {
    __shared__ __attribute__((aligned(1024))) T lds[ATTN_LDS<DH, KW>];
    int i = 0;
    for (int j = 1; j < seqs.n; ++j)
        if ((int)blockIdx.x >= seqs.s[j].wg0) i = j;
    const AttnSeq &a = seqs.s[i];
    int row_group, pair;
    if (!attn_place(blockIdx.x - a.wg0, hkv * a.n_splits, a.n_row_groups, row_group, pair)) return;
    attn_mfma_body<T, DH, KW, RT>(lds, row_group, pair % hkv, pair / hkv, static_cast<const T *>(a.q), a.rows, hq, hkv, a.mask, a.n_prefix,
                                  a.region_len, a.kv, a.blocks_per_split, scale, a.o_part, a.ml_part, a.rho_pad,
                                  static_cast<T *>(a.out_direct));
}

template <typename T, int DH>
__global__ __launch_bounds__(WALK_THREADS) void attn_walk_batch_kernel(AttnSeqs seqs, int hq, int hkv, float scale) {
    __shared__ __attribute__((aligned(1024))) T lds[ATTN_LDS<DH, 2>];
    int i = 0;
    for (int j = 1; j < seqs.n; ++j)
        if ((int)blockIdx.x >= seqs.s[j].wg0) i = j;
    const AttnSeq &a = seqs.s[i];
    int row_group, pair;
    if (!attn_place(blockIdx.x - a.wg0, hkv * a.n_splits, a.n_row_groups, row_group, pair)) return;
    attn_walk_split<T, DH>(lds, row_group, pair % hkv, pair / hkv, static_cast<const T *>(a.q), a.rows, hq, hkv, a.mask, a.n_prefix,
                                 a.region_len, a.kv, a.blocks_per_split, scale, a.o_part, a.ml_part, a.rho_pad,
                                 static_cast<T *>(a.out_direct));
}

// out[m][qh][:] = sum_s e^{m_s - M} O_s / sum_s e^{m_s - M} l_s, splits in order, for the rows of every sequence of a launch
// (sequences whose keys fit one split wrote their rows directly and are skipped).  dh / 4 lanes per (row, query head), four
// columns each; a workgroup stays within one row, so that which sequence it belongs to is scalar (looked up per lane, the
// sequence's pointers cost a trip to memory of their own: 5.6 us in the round of the 8B shape).  Up to NR splits (the usual case, NR = 4, 8, 12): everything in registers and every load requested before the first
// use - one trip to memory, no LDS, no barrier; each lane forms the weights itself (the (max, sum) pairs are the same addresses for
// the group) and slots beyond n_splits re-read the last split and are not used.  NR = 0: any number of splits, two passes over
// the (max, sum) pairs.  Four times 61 rows of the 8B shape, four
// splits: 9.5 -> 5.9 us; 61 rows: 4.6 -> 4.5 (before: a workgroup per (row, head),
// a column per lane).
constexpr int MERGE_THREADS = 256;
template <typename T, int NR>
__global__ __launch_bounds__(MERGE_THREADS) void attn_merge_kernel(AttnSeqs seqs, int hq, int hkv, int dh, T *__restrict__ out) {
    struct __attribute__((aligned(8))) Quad { T t[4]; };
    const int lanes = dh >> 2, row = blockIdx.x, qh = blockIdx.y * (MERGE_THREADS / lanes) + (int)threadIdx.x / lanes;
    const int i = ((int)threadIdx.x % lanes) * 4;
    int si = 0;
    for (int j = 1; j < seqs.n; ++j)
        if (row >= seqs.s[j].row0) si = j;
    const AttnSeq &a = seqs.s[si];
    const int m = row - a.row0, n_splits = a.n_splits;
    if (m >= a.rows || n_splits == 1 || qh >= hq) return;
    const int G = hq / hkv, kvh = qh / G, rho = m * G + qh % G;
    const size_t stride = (size_t)hkv * a.rho_pad;        // rows between consecutive splits
    const size_t row0 = (size_t)kvh * a.rho_pad + rho;
    const float *src = a.o_part + row0 * dh + i, *ml = a.ml_part + row0 * 2;
    float den = 0.f;
    f32x4 num = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (NR > 0) {
        MergeQuad<NR> mq;
        mq.load(src, ml, stride, dh, n_splits);
        mq.merge(n_splits, num, den);
    } else {
        float M = -INFINITY;
        for (int s = 0; s < n_splits; ++s) M = fmaxf(M, ml[(size_t)s * stride * 2]);
#pragma unroll 4
        for (int s = 0; s < n_splits; ++s) {
            const float2 x = *reinterpret_cast<const float2 *>(ml + (size_t)s * stride * 2);
            const float w = x.x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(x.x - M);
            den += w * x.y;
            num += w * *reinterpret_cast<const f32x4 *>(src + (size_t)s * stride * dh);
        }
    }
    Quad o;
#pragma unroll
    for (int j = 0; j < 4; ++j) o.t[j] = from_f<T>(num[j] / den);
    *reinterpret_cast<Quad *>(out + ((size_t)row * hq + qh) * dh + i) = o;
}

// n_rows: rows that `out` holds for the sequences of the launch
template <typename T>
static void launch_merge_t(const ModelDims &md, const AttnSeqs &seqs, int n_rows, T *out, hipStream_t st) {
    int most = 0;
    for (int i = 0; i < seqs.n; ++i) if (seqs.s[i].n_splits > most) most = seqs.s[i].n_splits;
    const int per = MERGE_THREADS / (md.dh >> 2);
    dim3 grid(n_rows, (md.hq + per - 1) / per), block(MERGE_THREADS);
#define POSS_MERGE(NR) hipLaunchKernelGGL((attn_merge_kernel<T, NR>), grid, block, 0, st, seqs, md.hq, md.hkv, md.dh, out)
    if (most <= 4) POSS_MERGE(4); else if (most <= 8) POSS_MERGE(8); else if (most <= 12) POSS_MERGE(12); else POSS_MERGE(0);
#undef POSS_MERGE
}

// float32 storage: one workgroup per (row, query head); exact two-pass softmax.  A thread takes whole keys for the scores
// (16 bytes at a time), then the threads split into 256 / dh2 groups over the keys for P V (dh2: dh rounded up to a power of two),
// whose partial sums are added in group order.  4 rows of four heads over 89 keys: 19.3 -> 6.5 us (before: one wave, dh
// scalar loads per key and one dependent load per key in P V).
constexpr int AF32_THREADS = 256;
__global__ __launch_bounds__(AF32_THREADS) void attn_f32_kernel(const float *__restrict__ q, int hq, int hkv, int dh, int dh2,
                                                                const uint64_t *__restrict__ mask, int n_prefix, int region_len,
                                                                KVCache kv, float scale, float *__restrict__ out) {
    extern __shared__ float sc[];                         // max(keys, AF32_THREADS) floats
    __shared__ float red[17];
    const int m = blockIdx.x, qh = blockIdx.y, kvh = qh / (hq / hkv), tid = threadIdx.x;
    const float *qr = q + ((size_t)m * hq + qh) * dh;
    const uint64_t m0 = mask[(size_t)m * MASK_WORDS], m1 = mask[(size_t)m * MASK_WORDS + 1];
    const int total = n_prefix + region_len;
    const float *kc = static_cast<const float *>(kv.k), *vc = static_cast<const float *>(kv.vt);
    float mx = -INFINITY;
    for (int sl = tid; sl < total; sl += AF32_THREADS) {
        float x = -INFINITY;
        if (slot_visible(sl, n_prefix, region_len, m0, m1)) {
            const float *kr = kc + k_offset(kv, sl, kvh, hkv, dh);
            float a = 0.f;
#pragma unroll 8
            for (int i = 0; i < dh; i += 4) {             // (dh is a multiple of 32)
                const f32x4 k4 = *reinterpret_cast<const f32x4 *>(kr + i), q4 = *reinterpret_cast<const f32x4 *>(qr + i);
#pragma unroll
                for (int j = 0; j < 4; ++j) a = fmaf(q4[j], k4[j], a);
            }
            x = a * scale;
        }
        sc[sl] = x;
        mx = fmaxf(mx, x);
    }
    mx = wave_max(mx);
    if ((tid & 63) == 0) red[tid >> 6] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    float sum = 0.f;
    for (int sl = tid; sl < total; sl += AF32_THREADS) {
        const float p = expf(sc[sl] - mx);
        sc[sl] = p;
        sum += p;
    }
    sum = block_sum(sum, red);                            // (its barriers also publish sc)
    const int groups = AF32_THREADS / dh2, i = tid & (dh2 - 1), gi = tid / dh2;
    const int per = ((total + groups - 1) / groups + 3) & ~3, s0 = min(total, gi * per), s1 = min(total, s0 + per);
    float a = 0.f;
    if (i < dh) {
        int sl = s0;
        for (; sl + 4 <= s1; sl += 4) {                   // four consecutive slots, s0 a multiple of 4: one page
            const f32x4 v = *reinterpret_cast<const f32x4 *>(vc + vt_offset(kv, sl, kvh, hkv, dh, i));
#pragma unroll
            for (int j = 0; j < 4; ++j) a = fmaf(sc[sl + j], v[j], a);
        }
        for (; sl < s1; ++sl) a = fmaf(sc[sl], vc[vt_offset(kv, sl, kvh, hkv, dh, i)], a);
    }
    __syncthreads();                                      // every score has been read
    sc[tid] = a;
    __syncthreads();
    if (tid < dh) {
        float o = 0.f;
        for (int g = 0; g < groups; ++g) o += sc[g * dh2 + tid];
        out[((size_t)m * hq + qh) * dh + tid] = o / sum;
    }
}

// Launch shape of one sequence's attention: the split rule, key-ways and row tiles per wave.
// Key-ways follow the split size (so, like it, the committed prefix only); the number of row tiles per wave may follow
// the row count: it does not change any row's arithmetic.
struct AttnShape { int bps, n_splits, kw, rt, n_row_groups, rho_pad, n_wgs; bool walk; };
static AttnShape attention_shape(const ModelDims &md, int rows, int n_prefix, int region_len, int keys_per_split,
                                 bool crowded = false) {
    AttnShape a;
    const int G = md.hq / md.hkv;
    const int tiles = (rows * G + 15) / 16;
    a.rho_pad = tiles * 16;
    const int n_blocks = (n_prefix + region_len + 31) / 32;
    a.bps = attn_blocks_per_split(n_prefix, keys_per_split);
    a.n_splits = (n_blocks + a.bps - 1) / a.bps;
    a.kw = a.bps >= 4 ? 2 : 1;
    a.walk = md.dt == DT_BF16 && a.bps >= WALK_MIN_BPS;
    // Two row tiles a wave where one would put more workgroups in the launch than the chip has CUs (a workgroup fills a CU's LDS: the
    // surplus would run as a second round).  Otherwise the keys are staged twice as often, by twice as many CUs: 61 rows of the 8B
    // shape, us a pass of four layers, two tiles / one: 1000 keys 600 / 583, 2000 623 / 599, 3000 648 / 608; 100 rows of 640 wide, fp16, 1000
    // keys 379 / 358, 4000 435 / 398, 8000 437 / 397.  At the line, 280 workgroups of 5 blocks (100 rows of the 8B shape, 600 keys), a launch
    // takes 14.3 / 14.1.
    const int pairs = 8 * ((md.hkv * a.n_splits + 7) / 8);
    a.rt = a.walk || (tiles > 4 && (crowded || (tiles + 3) / 4 * pairs > 256)) ? 2 : 1;
    a.n_row_groups = (tiles + 4 * a.rt - 1) / (4 * a.rt);
    a.n_wgs = a.n_row_groups * pairs;
    return a;
}

template <typename T>
static void launch_attention_t(const ModelDims &md, const void *q, int rows, const RowMeta &rm, int n_prefix,
                               int region_len, const KVCache &kv, int keys_per_split, const AttnScratch &sc,
                               void *out, hipStream_t st, bool merge) {
    const AttnShape a = attention_shape(md, rows, n_prefix, region_len, keys_per_split);
    const float scale = 1.4426950408889634f / sqrtf((float)md.dh);     // log2(e) / sqrt(dh): scores in the log2 domain
    T *direct = a.n_splits == 1 ? static_cast<T *>(out) : nullptr;
#define POSS_ATTN(DH, KW, RT)                                                                                     \
    hipLaunchKernelGGL((attn_mfma_kernel<T, DH, KW, RT>), dim3(a.n_wgs), dim3(256 * KW), 0, st,                  \
                       static_cast<const T *>(q), rows, md.hq, md.hkv, rm.mask, n_prefix, region_len, kv, a.bps,  \
                       a.n_splits, a.n_row_groups, scale, sc.o, sc.ml, a.rho_pad, direct)
#define POSS_ATTN_DH(DH)                                                                                         \
    do {                                                                                                         \
        if constexpr (std::is_same<T, bf16_t>::value) if (a.walk) {                                              \
            hipLaunchKernelGGL((attn_walk_kernel<T, DH>), dim3(a.n_wgs), dim3(WALK_THREADS), 0, st,              \
                               static_cast<const T *>(q), rows, md.hq, md.hkv, rm.mask, n_prefix, region_len, kv, a.bps, \
                               a.n_splits, a.n_row_groups, scale, sc.o, sc.ml, a.rho_pad, direct);               \
            break;                                                                                               \
        }                                                                                                        \
        if (a.kw == 2) { if (a.rt == 2) POSS_ATTN(DH, 2, 2); else POSS_ATTN(DH, 2, 1); }                         \
        else           { if (a.rt == 2) POSS_ATTN(DH, 1, 2); else POSS_ATTN(DH, 1, 1); }                         \
    } while (0)
    if (md.dh == 128) POSS_ATTN_DH(128); else POSS_ATTN_DH(64);
#undef POSS_ATTN_DH
#undef POSS_ATTN
    if (a.n_splits > 1 && merge) {
        AttnSeqs one;
        one.n = 1;
        one.s[0] = AttnSeq{q, rm.mask, direct, sc.o, sc.ml, kv, rows, n_prefix, region_len, a.bps, a.n_splits, a.n_row_groups, a.rho_pad, 0, 0};
        launch_merge_t<T>(md, one, rows, static_cast<T *>(out), st);
    }
}

template <typename T>
static void launch_attention_batch_t(const ModelDims &md, const void *q, const RowMeta &rm, const AttnSeg *segs, int n,
                                     int keys_per_split, const AttnScratch &sc, void *out, hipStream_t st) {
    const float scale = 1.4426950408889634f / sqrtf((float)md.dh);
    const size_t qd = (size_t)md.hq * md.dh;
    AttnShape shp[ATTN_MAX_SEQ];
    AttnSeq all[ATTN_MAX_SEQ];
    size_t o_off = 0, ml_off = 0;
    bool any_split = false;
    int wgs_all = 0;
    for (int i = 0; i < n; ++i)
        wgs_all += attention_shape(md, segs[i].rows, segs[i].n_prefix, segs[i].region_len, keys_per_split).n_wgs;
    const bool crowded = wgs_all > 256;
    for (int i = 0; i < n; ++i) {
        const AttnSeg &g = segs[i];
        shp[i] = attention_shape(md, g.rows, g.n_prefix, g.region_len, keys_per_split, crowded);
        AttnSeq &a = all[i];
        a.q = static_cast<const T *>(q) + g.row0 * qd;
        a.mask = rm.mask + (size_t)g.row0 * MASK_WORDS;
        a.out_direct = shp[i].n_splits == 1 ? static_cast<T *>(out) + g.row0 * qd : nullptr;
        a.o_part = sc.o + o_off; a.ml_part = sc.ml + ml_off;
        o_off += (size_t)shp[i].n_splits * md.hkv * shp[i].rho_pad * md.dh;
        ml_off += (size_t)shp[i].n_splits * md.hkv * shp[i].rho_pad * 2;
        a.kv = *g.kv;
        a.rows = g.rows; a.n_prefix = g.n_prefix; a.region_len = g.region_len;
        a.blocks_per_split = shp[i].bps; a.n_splits = shp[i].n_splits; a.n_row_groups = shp[i].n_row_groups;
        a.rho_pad = shp[i].rho_pad; a.wg0 = 0; a.row0 = g.row0;
        any_split = any_split || shp[i].n_splits > 1;
    }
    // one launch per kind of kernel that occurs (long walk, or key-ways and row tiles): as a rule one
    for (int kind = 0; kind < 5; ++kind) {
        const bool walk = kind == 4;
        const int kw = (kind >> 1) + 1, rt = (kind & 1) + 1;
        AttnSeqs grp;
        grp.n = 0;
        int wgs = 0;
        for (int i = 0; i < n; ++i)
            if (shp[i].walk == walk && (walk || (shp[i].kw == kw && shp[i].rt == rt))) {
                grp.s[grp.n] = all[i];
                grp.s[grp.n].wg0 = wgs;
                wgs += shp[i].n_wgs;
                ++grp.n;
            }
        if (grp.n == 0) continue;
#define POSS_ATTNB(DH, KW, RT)                                                                                   \
    hipLaunchKernelGGL((attn_mfma_batch_kernel<T, DH, KW, RT>), dim3(wgs), dim3(256 * KW), 0, st, grp, md.hq, md.hkv, scale)
#define POSS_ATTNB_DH(DH)                                                                                        \
    do {                                                                                                         \
        if constexpr (std::is_same<T, bf16_t>::value) if (walk) {                                                \
            hipLaunchKernelGGL((attn_walk_batch_kernel<T, DH>), dim3(wgs), dim3(WALK_THREADS), 0, st, grp, md.hq, md.hkv, scale); \
            break;                                                                                               \
        }                                                                                                        \
        if (kw == 2) { if (rt == 2) POSS_ATTNB(DH, 2, 2); else POSS_ATTNB(DH, 2, 1); }                      \
        else              { if (rt == 2) POSS_ATTNB(DH, 1, 2); else POSS_ATTNB(DH, 1, 1); }                      \
    } while (0)
        if (md.dh == 128) POSS_ATTNB_DH(128); else POSS_ATTNB_DH(64);
#undef POSS_ATTNB_DH
#undef POSS_ATTNB
    }
    if (any_split) {
        AttnSeqs grp;
        grp.n = n;
        for (int i = 0; i < n; ++i) grp.s[i] = all[i];
        launch_merge_t<T>(md, grp, segs[n - 1].row0 + segs[n - 1].rows, static_cast<T *>(out), st);      // (sequences are in row order)
    }
}

void launch_attention_batch(const ModelDims &md, const void *q, const RowMeta &rm, const AttnSeg *segs, int n,
                            int keys_per_split, const AttnScratch &sc, void *out, hipStream_t st) {
    if (n == 1 || md.dt == DT_F32 || n > ATTN_MAX_SEQ) {       // one sequence: the launch of its own; float32: the exact kernel
        const size_t row_bytes = (size_t)md.hq * md.dh * dtype_size(md.dt);
        for (int i = 0; i < n; ++i) {
            const AttnSeg &g = segs[i];
            const RowMeta srm{rm.pos + g.row0, rm.slot + g.row0, rm.mask + (size_t)g.row0 * MASK_WORDS};
            launch_attention(md, static_cast<const char *>(q) + g.row0 * row_bytes, g.rows, srm, g.n_prefix, g.region_len, *g.kv,
                             keys_per_split, sc, static_cast<char *>(out) + g.row0 * row_bytes, st);
        }
        return;
    }
    if (md.dt == DT_BF16) launch_attention_batch_t<bf16_t>(md, q, rm, segs, n, keys_per_split, sc, out, st);
    else launch_attention_batch_t<f16_t>(md, q, rm, segs, n, keys_per_split, sc, out, st);
}

template <typename T>
static void launch_attention_prompt_t(const ModelDims &md, const void *q, int rows, const uint64_t *mask, int c0, const KVCache &kv,
                                      void *out, hipStream_t st) {
    const int n_ranges = (rows + MAX_ROWS - 1) / MAX_ROWS, n_row_groups = (MAX_ROWS * (md.hq / md.hkv) + 127) / 128;
    int n_short = 0;                                                     // ranges that walk fewer than PROMPT_SHORT_BLOCKS blocks
    while (n_short < n_ranges && (c0 + (rows < (n_short + 1) * MAX_ROWS ? rows : (n_short + 1) * MAX_ROWS) + 31) / 32 < PROMPT_SHORT_BLOCKS) ++n_short;
    const int walk_wgs = 8 * n_row_groups * ((md.hkv * (n_ranges - n_short) + 7) / 8), short_wgs = 8 * n_row_groups * ((md.hkv * n_short + 7) / 8);
    const float scale = 1.4426950408889634f / sqrtf((float)md.dh);
#define POSS_PROMPT(DH)                                                                                                              \
    hipLaunchKernelGGL((attn_prompt_kernel<T, DH>), dim3(walk_wgs + short_wgs), dim3(WALK_THREADS), 0, st, static_cast<const T *>(q), rows, \
                       md.hq, md.hkv, mask, c0, kv, n_short, walk_wgs, scale, static_cast<T *>(out))
    if (md.dh == 128) POSS_PROMPT(128); else POSS_PROMPT(64);
#undef POSS_PROMPT
}

void launch_attention_prompt(const ModelDims &md, const void *q, int rows, const uint64_t *mask, int c0, const KVCache &kv, void *out,
                             hipStream_t st) {
    if (md.dt == DT_BF16) launch_attention_prompt_t<bf16_t>(md, q, rows, mask, c0, kv, out, st);
    else launch_attention_prompt_t<f16_t>(md, q, rows, mask, c0, kv, out, st);
}

AttnMerge attention_partials(const ModelDims &md, int rows, int n_prefix, int region_len, int keys_per_split, const AttnScratch &sc) {
    if (md.dt == DT_F32) return AttnMerge{nullptr, nullptr, 1, 0, md.hq, md.hkv, md.dh};
    const AttnShape a = attention_shape(md, rows, n_prefix, region_len, keys_per_split);
    return AttnMerge{sc.o, sc.ml, a.n_splits, a.rho_pad, md.hq, md.hkv, md.dh};
}

int attention_splits(int total_keys, int keys_per_split) {
    int bps = keys_per_split / 32; if (bps < 1) bps = 1;
    return ((total_keys + 31) / 32 + bps - 1) / bps;
}

void launch_attention(const ModelDims &md, const void *q, int rows, const RowMeta &rm, int n_prefix,
                      int region_len, const KVCache &kv, int keys_per_split, const AttnScratch &sc,
                      void *out, hipStream_t st, bool merge) {
    if (md.dt == DT_F32) {
        const int keys = n_prefix + region_len;
        const size_t lds = (size_t)(keys < AF32_THREADS ? AF32_THREADS : keys) * sizeof(float);
        int dh2 = 2;
        while (dh2 < md.dh) dh2 *= 2;                     // (dh is at most 256)
        const float scale = 1.0f / sqrtf((float)md.dh);
        const float *qf = static_cast<const float *>(q);
        float *of = static_cast<float *>(out);
        hipLaunchKernelGGL(attn_f32_kernel, dim3(rows, md.hq), dim3(AF32_THREADS), lds, st, qf, md.hq, md.hkv, md.dh, dh2, rm.mask, n_prefix,
                           region_len, kv, scale, of);
    } else if (md.dt == DT_BF16) {
        launch_attention_t<bf16_t>(md, q, rows, rm, n_prefix, region_len, kv, keys_per_split, sc, out, st, merge);
    } else {
        launch_attention_t<f16_t>(md, q, rows, rm, n_prefix, region_len, kv, keys_per_split, sc, out, st, merge);
    }
}

}  // namespace poss
