// Device-side helpers: storage conversions, block reductions, cache addressing.
#pragma once
#include "common.h"

namespace poss {

template <typename T> __device__ __forceinline__ float to_f(T v) { return (float)v; }
template <typename T> __device__ __forceinline__ T from_f(float v) { return (T)v; }   // round to nearest even
// Where several kernels form the same value they must round alike, and in fp16 the plain conversion does not: the compiler folds a
// float32 product or multiply-add into it (v_fma_mixlo_f16: rounded once, from the exact result) in one kernel and converts the
// float32 result (rounded twice) in the next, as its vectoriser decides.  The two differ in one value of ten thousand.
// round_f: the float32 value, rounded.  mul_round: the product, rounded once (bf16 and float32: as float32 arithmetic gives it).
template <typename T> __device__ __forceinline__ T round_f(float v) { return (T)v; }
template <> __device__ __forceinline__ f16_t round_f<f16_t>(float v) {
    asm("" : "+v"(v));                                    // the value itself, not what it was computed from
    return (f16_t)v;
}
template <typename T> __device__ __forceinline__ T mul_round(float a, float b) { return (T)(a * b); }
template <> __device__ __forceinline__ f16_t mul_round<f16_t>(float a, float b) {
    f16_t r = (f16_t)(a * b);                             // v_fma_mixlo_f16, unless several conversions are made one
    asm("" : "+v"(r));
    return r;
}

// x of lane l ^ OFF as a second operand: bits 5 and 4 by the row-swap instructions of gfx950 (see rows_max below), the
// others by DPP.  Nothing goes through the LDS crossbar, as a shuffle would (about 100 cycles a step).  Every lane of the wave
// must be active.
template <int CTRL, int BANKS = 0xf>
__device__ __forceinline__ float dpp(float old, float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old), __builtin_bit_cast(int, x), CTRL, 0xf, BANKS, false));
}
// the pairs (x[l], x[l ^ 32]) resp. (x[l], x[l ^ 16]) of a lane, in the order (lower, upper)
__device__ __forceinline__ void swap32(float x, float &a, float &b) {
    a = x; b = x;
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ void swap16(float x, float &a, float &b) {
    a = x; b = x;
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ float xor8(float x) { return dpp<0x128>(x, x); }                          // row_ror:8
__device__ __forceinline__ float xor4(float x) { return dpp<0x114, 0xa>(dpp<0x104, 0x5>(x, x), x); } // row_shl:4 | row_shr:4
__device__ __forceinline__ float xor2(float x) { return dpp<0x4e>(x, x); }                           // quad_perm 2 3 0 1
__device__ __forceinline__ float xor1(float x) { return dpp<0xb1>(x, x); }                           // quad_perm 1 0 3 2

__device__ __forceinline__ float wave_sum(float v) {      // butterfly over 32, 16, .. 1
    float a, b;
    swap32(v, a, b); v = a + b;
    swap16(v, a, b); v = a + b;
    v += xor8(v); v += xor4(v); v += xor2(v); v += xor1(v);
    return v;
}
__device__ __forceinline__ float wave_max(float v) {
    float a, b;
    swap32(v, a, b); v = fmaxf(a, b);
    swap16(v, a, b); v = fmaxf(a, b);
    v = fmaxf(v, xor8(v)); v = fmaxf(v, xor4(v)); v = fmaxf(v, xor2(v)); v = fmaxf(v, xor1(v));
    return v;
}
__device__ __forceinline__ float lane_value(float v, int lane) {       // lane wave-uniform
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}

// What a lane of this wave wrote to LDS before it is what every lane reads behind it (LDS operations of a wave complete in
// order: no instruction comes of this, it orders the compiler's accesses).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Sum over a workgroup of up to 1024 threads, identical in every thread; fixed order.
__device__ __forceinline__ float block_sum(float v, float *red /* >= 17 floats of LDS */) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    v = wave_sum(v);
    __syncthreads();                      // red may still be read from an earlier call
    if (lane == 0) red[wave] = v;
    __syncthreads();
    float s = 0.f;
    for (int i = 0; i < nw; ++i) s += red[i];
    return s;
}

// One 16-byte LDS-direct load per lane: lane l's 16 bytes from `g` land at LDS byte address lds_base + 16 l
// (lds_base wave-uniform).  Written as assembly because the compiler, which cannot tell which LDS reads a
// load it knows of may alias, would wait for ALL such loads before every LDS read; counted waits
// (dma_wait) are placed by hand instead.  M0 is set in the same statement and nothing else in these kernels uses it.
__device__ __forceinline__ void lds_dma16(unsigned lds_base, const void *g) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_base), "v"(g) : "memory");
}
// The same for bytes that no other workgroup will want: non-temporal, so that they do not push out of the L2 what others share.
__device__ __forceinline__ void lds_dma16_nt(unsigned lds_base, const void *g) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt" ::"s"(lds_base), "v"(g) : "memory");
}
// The same with a scalar base and a byte offset per lane.
__device__ __forceinline__ void lds_dma16_s(unsigned lds_base, const void *g, unsigned off) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_base), "v"(off), "s"(g) : "memory");
}
// Wait until at most N of this wave's vector-memory loads are outstanding (they complete in order).
template <int N>
__device__ __forceinline__ void dma_wait() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// A token id that came out of arithmetic indexes the embedding table only through this: an argmax over a row of
// logits that are all NaN finds no entry that compares and leaves the id of "no entry" (0x7fffffff) - a bad number
// must not become a bad address.  Such a row reads token 0.
__device__ __forceinline__ int embedding_row(int token, int vocab) { return (unsigned)token < (unsigned)vocab ? token : 0; }

// (value, index) ordering used by every argmax / top-k here: larger value first, then lower index.
__device__ __forceinline__ bool better(float v, int i, float bv, int bi) {
    return (v > bv) || (v == bv && i < bi);
}

// One step of an argmax butterfly: the pair of lane l ^ OFF (OFF = 8, 4, 2, 1 by DPP; 16, 32 by the row swaps).
__device__ __forceinline__ int as_int(float x) { return __builtin_bit_cast(int, x); }
__device__ __forceinline__ float as_float(int x) { return __builtin_bit_cast(float, x); }
template <int OFF>
__device__ __forceinline__ void argmax_step(float &v, int &i) {
    float ov; int oi;
    if constexpr (OFF >= 16) {
        float v2, i1, i2;
        if constexpr (OFF == 32) { swap32(v, ov, v2); swap32(as_float(i), i1, i2); } else { swap16(v, ov, v2); swap16(as_float(i), i1, i2); }
        oi = as_int(i1); v = v2; i = as_int(i2);          // the pair in the order (lower lane, upper lane)
    } else {
        const float fi = as_float(i);
        ov = OFF == 8 ? xor8(v) : OFF == 4 ? xor4(v) : OFF == 2 ? xor2(v) : xor1(v);
        oi = as_int(OFF == 8 ? xor8(fi) : OFF == 4 ? xor4(fi) : OFF == 2 ? xor2(fi) : xor1(fi));
    }
    if (better(ov, oi, v, i)) { v = ov; i = oi; }
}
// over the 32 lanes of a half wave (all of them active; the other half need not be)
__device__ __forceinline__ void half_argmax(float &v, int &i) {
    argmax_step<16>(v, i); argmax_step<8>(v, i); argmax_step<4>(v, i); argmax_step<2>(v, i); argmax_step<1>(v, i);
}
__device__ __forceinline__ float half_max(float v) {
    float a, b;
    swap16(v, a, b); v = fmaxf(a, b);
    v = fmaxf(v, xor8(v)); v = fmaxf(v, xor4(v)); v = fmaxf(v, xor2(v)); v = fmaxf(v, xor1(v));
    return v;
}
__device__ __forceinline__ int half_min(int x) {
    float a, b;
    swap16(as_float(x), a, b); x = min(as_int(a), as_int(b));
    x = min(x, as_int(xor8(as_float(x)))); x = min(x, as_int(xor4(as_float(x))));
    x = min(x, as_int(xor2(as_float(x)))); x = min(x, as_int(xor1(as_float(x))));
    return x;
}
__device__ __forceinline__ float half_sum(float v) {
    float a, b;
    swap16(v, a, b); v = a + b;
    v += xor8(v); v += xor4(v); v += xor2(v); v += xor1(v);
    return v;
}
__device__ __forceinline__ void wave_argmax(float &v, int &i) {
    argmax_step<32>(v, i);
    half_argmax(v, i);
}

// Workgroup-wide argmax; result valid in every thread.  red_v/red_i: >= 17 entries of LDS each.
__device__ __forceinline__ void block_argmax(float &v, int &i, float *red_v, int *red_i) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    wave_argmax(v, i);
    __syncthreads();
    if (lane == 0) { red_v[wave] = v; red_i[wave] = i; }
    __syncthreads();
    if (threadIdx.x == 0) {
        float bv = red_v[0]; int bi = red_i[0];
        for (int w = 1; w < nw; ++w)
            if (better(red_v[w], red_i[w], bv, bi)) { bv = red_v[w]; bi = red_i[w]; }
        red_v[16] = bv; red_i[16] = bi;
    }
    __syncthreads();
    v = red_v[16]; i = red_i[16];
}

// Maximum over the four 16-lane rows of a wave (lanes l, l^16, l^32, l^48), left in every lane.  The two
// row-swap instructions of gfx950 stay in the vector ALU (v_permlane16_swap: [A.r0 B.r0 A.r2 B.r2] and
// [A.r1 B.r1 A.r3 B.r3] from rows r0..r3 of registers A and B; v_permlane32_swap: [A.lo B.lo] and
// [A.hi B.hi]); a shuffle would go through the LDS crossbar and wait for it.  Written as assembly with both
// registers as in/out operands: through the builtin, this compiler reads the second result from the first
// register.  (The s_nop covers the wait states a swap needs behind the VALU write of its operands.)
// Every lane of the wave must be active.
__device__ __forceinline__ float rows_max(float x) {
    float a, b;
    swap16(x, a, b);
    x = fmaxf(a, b);
    swap32(x, a, b);
    return fmaxf(a, b);
}

// Rotary table of one row, by `half` threads of the row's workgroup starting at first_thread:
// cs[i] = (cos, sin)(pos * theta^(-2i/dh)).  The angle is formed in float64 so that positions in the
// thousands keep float32-accurate sines; one table serves every layer of the pass.
__device__ __forceinline__ void rope_table_row(int pos, const double *__restrict__ inv_freq, int half,
                                               float2 *__restrict__ cs_row, int first_thread = 0) {
    const int i = (int)threadIdx.x - first_thread;
    if (i < 0 || i >= half) return;
    double s, c;
    sincos((double)pos * inv_freq[i], &s, &c);
    cs_row[i] = make_float2((float)c, (float)s);
}

// Rotation of one rotary pair, spelt out operation by operation (two products, two fused multiply-adds): the kernels
// that apply it must round alike, so nothing is left to the compiler's choice of what to contract.
__device__ __forceinline__ void rope_pair(float x1, float x2, float2 cs, float &o1, float &o2) {
#pragma clang fp contract(off)
    const float p = x2 * cs.y, q = x1 * cs.y;
    o1 = __builtin_fmaf(x1, cs.x, -p);
    o2 = __builtin_fmaf(x2, cs.x, q);
}

// Element offsets into the paged caches; _in: with the slot's physical page already looked up.
__device__ __forceinline__ size_t k_offset_in(const KVCache &kv, int pg, int slot, int head, int hkv, int dh) {
    const int P = 1 << kv.page_shift;
    return ((size_t)(pg * hkv + head) * P + (slot & (P - 1))) * dh;
}
__device__ __forceinline__ size_t vt_offset_in(const KVCache &kv, int pg, int slot, int head, int hkv, int dh, int row) {
    const int P = 1 << kv.page_shift;
    return ((size_t)(pg * hkv + head) * dh + row) * P + (slot & (P - 1));
}
__device__ __forceinline__ size_t k_offset(const KVCache &kv, int slot, int head, int hkv, int dh) {
    return k_offset_in(kv, kv.page_table[slot >> kv.page_shift], slot, head, hkv, dh);
}
__device__ __forceinline__ size_t vt_offset(const KVCache &kv, int slot, int head, int hkv, int dh, int row) {
    return vt_offset_in(kv, kv.page_table[slot >> kv.page_shift], slot, head, hkv, dh, row);
}

}  // namespace poss
