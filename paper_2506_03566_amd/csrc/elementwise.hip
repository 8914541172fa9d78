// Small kernels around the GEMMs: embedding gather + first RMSNorm, rotary table, argmax, row copies.  All arithmetic in
// float32; values become the storage type only where they are the next GEMM's operand.
#include "device_utils.h"
#include "quotient.h"

#include <type_traits>

namespace poss {

#define POSS_DISPATCH(dt, ...)                                               \
    switch (dt) {                                                            \
        case DT_F32:  { using T = float;  __VA_ARGS__; } break;              \
        case DT_BF16: { using T = bf16_t; __VA_ARGS__; } break;              \
        default:      { using T = f16_t;  __VA_ARGS__; } break;              \
    }

// ------------------------------------------------------------------ h = emb[token]; u = T(rmsnorm(h) g)
// (and the row's rotary table, which every layer of the pass uses; no u in float32 storage, whose products norm the rows they read)
template <typename T>
__global__ __launch_bounds__(256) void embed_norm_kernel(const T *__restrict__ embed, const int32_t *__restrict__ tokens,
                                                         int vocab, int d, float eps, const T *__restrict__ gain,
                                                         float *__restrict__ h, T *__restrict__ u,
                                                         const int32_t *__restrict__ pos,
                                                         const double *__restrict__ inv_freq, int half,
                                                         float2 *__restrict__ cs) {
    constexpr bool NORM = !std::is_same<T, float>::value;
    __shared__ float red[17];
    const int row = blockIdx.x;
    // the rotary table by the last wave, so that the first ones start on the embedding row at once
    rope_table_row(pos[row], inv_freq, half, cs + (size_t)row * half, half <= 64 && blockDim.x >= 128 ? (int)blockDim.x - 64 : 0);
    const T *e = embed + (size_t)embedding_row(tokens[row], vocab) * d;
    constexpr int VE = 16 / (int)sizeof(T);               // elements per 16-byte access
    constexpr int MAXV = 4;                                // 16-byte pieces a thread keeps (d <= 4 * 256 * VE)
    if (d % VE == 0 && d <= MAXV * 256 * VE && blockDim.x == 256) {
        // one trip to memory: the row and the gains are loaded in 16-byte pieces and kept in registers
        union Piece { uint4 q; T t[VE]; };
        Piece ev[MAXV], gv[MAXV];
        const int nv = d / VE;
#pragma unroll
        for (int j = 0; j < MAXV; ++j) {
            const int p = threadIdx.x + j * 256;
            if (p < nv) {
                ev[j].q = reinterpret_cast<const uint4 *>(e)[p];
                if constexpr (NORM) gv[j].q = reinterpret_cast<const uint4 *>(gain)[p];
            }
        }
        float ss = 0.f;                                    // fixed order: a thread's pieces one after the other, element by element
#pragma unroll
        for (int j = 0; j < MAXV; ++j) {
            const int p = threadIdx.x + j * 256;
            if (p < nv) {
#pragma unroll
                for (int x = 0; x < VE; ++x) {
                    const float v = to_f(ev[j].t[x]);
                    h[(size_t)row * d + (size_t)p * VE + x] = v;
                    ss += v * v;
                }
            }
        }
        if constexpr (!NORM) return;
        ss = block_sum(ss, red);
        const float rs = 1.0f / sqrtf(ss / (float)d + eps);
#pragma unroll
        for (int j = 0; j < MAXV; ++j) {
            const int p = threadIdx.x + j * 256;
            if (p < nv) {
                Piece o;
#pragma unroll
                for (int x = 0; x < VE; ++x) o.t[x] = from_f<T>(to_f(ev[j].t[x]) * rs * to_f(gv[j].t[x]));
                reinterpret_cast<uint4 *>(u + (size_t)row * d)[p] = o.q;
            }
        }
        return;
    }
    float ss = 0.f;
    for (int i = threadIdx.x; i < d; i += blockDim.x) {
        const float v = to_f(e[i]);
        h[(size_t)row * d + i] = v;
        ss += v * v;
    }
    if constexpr (!NORM) return;
    ss = block_sum(ss, red);
    const float rs = 1.0f / sqrtf(ss / (float)d + eps);
    for (int i = threadIdx.x; i < d; i += blockDim.x)
        u[(size_t)row * d + i] = from_f<T>(to_f(e[i]) * rs * to_f(gain[i]));
}

void launch_embed_norm(const ModelDims &md, const void *embed, const int32_t *tokens, int rows,
                       const void *gain, float *h, void *u, const int32_t *pos, const double *inv_freq,
                       float2 *cs, hipStream_t st) {
    POSS_DISPATCH(md.dt, hipLaunchKernelGGL((embed_norm_kernel<T>), dim3(rows), dim3(256), 0, st,
                                            static_cast<const T *>(embed), tokens, md.vocab, md.d, md.eps,
                                            static_cast<const T *>(gain), h, static_cast<T *>(u), pos, inv_freq,
                                            md.dh / 2, cs));
}

// ------------------------------------------------------------------ u = T(rmsnorm(h) g), stash = T(h), many rows
// Bound by memory: a row is read once, in 16-byte pieces kept in registers, and its 16-bit rows are written 8 bytes at a time.
template <typename T>
__global__ __launch_bounds__(1024) void norm_rows_kernel(const float *__restrict__ h, int d, float eps, const T *__restrict__ gain,
                                                         T *__restrict__ u, T *__restrict__ stash) {
    __shared__ float red[17];
    constexpr int MAXV = 4;                                // four columns each: d <= 16 * blockDim.x
    struct __attribute__((aligned(4 * sizeof(T)))) Quad { T t[4]; };
    const size_t row = blockIdx.x;
    const float4 *src = reinterpret_cast<const float4 *>(h + row * d);
    const int nv = d / 4;
    float4 v[MAXV];
    Quad gv[MAXV];
    float ss = 0.f;
#pragma unroll
    for (int j = 0; j < MAXV; ++j) {
        const int p = threadIdx.x + j * blockDim.x;
        v[j] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (p < nv) { v[j] = src[p]; gv[j] = reinterpret_cast<const Quad *>(gain)[p]; }
        ss = fmaf(v[j].x, v[j].x, ss); ss = fmaf(v[j].y, v[j].y, ss);      // as the residual + norm epilogue does
        ss = fmaf(v[j].z, v[j].z, ss); ss = fmaf(v[j].w, v[j].w, ss);
    }
    ss = block_sum(ss, red);
    const float rs = 1.0f / sqrtf(ss / (float)d + eps);
#pragma unroll
    for (int j = 0; j < MAXV; ++j) {
        const int p = threadIdx.x + j * blockDim.x;
        if (p >= nv) continue;
        const float x[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
        Quad o;
#pragma unroll
        for (int i = 0; i < 4; ++i) o.t[i] = mul_round<T>(x[i] * rs, to_f(gv[j].t[i]));
        reinterpret_cast<Quad *>(u + row * d)[p] = o;
        if (stash) {
#pragma unroll
            for (int i = 0; i < 4; ++i) o.t[i] = from_f<T>(x[i]);
            reinterpret_cast<Quad *>(stash + row * d)[p] = o;
        }
    }
}

void launch_norm_rows(const ModelDims &md, const float *h, int rows, const void *gain, void *u, void *stash, hipStream_t st) {
    const int threads = md.d <= 4096 ? 256 : md.d <= 8192 ? 512 : 1024;
    POSS_DISPATCH(md.dt, hipLaunchKernelGGL((norm_rows_kernel<T>), dim3(rows), dim3(threads), 0, st, h, md.d, md.eps,
                                            static_cast<const T *>(gain), static_cast<T *>(u), static_cast<T *>(stash)));
}

// ------------------------------------------------------------------ argmax per row (lowest index on ties)
// Two stages so that a 128K-entry row is not one workgroup's serial scan: (segment, row) partial
// winners, then one small workgroup per row over the partials.  A row of one segment is finished by the first stage (25 rows of 4096
// ids, two launches: 7.3 + 4.7 us; one, its ids requested in one trip: 4.0).
__device__ __forceinline__ void argmax_out(int bi, int rowi, int32_t *__restrict__ out, int32_t *__restrict__ host_out) {
    if (bi == 0x7fffffff) bi = 0;                         // no logit of the row compared (all NaN): token 0, not an id outside the vocabulary
    out[rowi] = bi;
    if (host_out) host_out[rowi] = bi;
}

constexpr int ARGMAX_SEG = 4096;
__global__ __launch_bounds__(256) void argmax_seg_kernel(const float *__restrict__ logits, int ld, int vocab, int n_seg, float *__restrict__ pv,
                                                         int *__restrict__ pi, int32_t *__restrict__ out, int32_t *__restrict__ host_out) {
    constexpr int NV = ARGMAX_SEG / 256;
    __shared__ float red_v[17];
    __shared__ int red_i[17];
    const int seg = blockIdx.x, rowi = blockIdx.y, i0 = seg * ARGMAX_SEG + (int)threadIdx.x;
    const float *row = logits + (size_t)rowi * ld;
    float v[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) v[j] = row[min(i0 + j * 256, vocab - 1)];       // one trip; ids beyond the vocabulary do not compete
    float bv = -INFINITY; int bi = 0x7fffffff;
#pragma unroll
    for (int j = 0; j < NV; ++j)
        if (i0 + j * 256 < vocab && better(v[j], i0 + j * 256, bv, bi)) { bv = v[j]; bi = i0 + j * 256; }
    block_argmax(bv, bi, red_v, red_i);
    if (threadIdx.x != 0) return;
    if (n_seg == 1) argmax_out(bi, rowi, out, host_out);
    else { pv[rowi * n_seg + seg] = bv; pi[rowi * n_seg + seg] = bi; }
}

__global__ __launch_bounds__(64) void argmax_merge_kernel(const float *__restrict__ pv, const int *__restrict__ pi, int n_seg,
                                                          int32_t *__restrict__ out, int32_t *__restrict__ host_out) {
    const int rowi = blockIdx.x;
    float bv = -INFINITY; int bi = 0x7fffffff;
    for (int s = threadIdx.x; s < n_seg; s += 64) {
        const float v = pv[rowi * n_seg + s]; const int i = pi[rowi * n_seg + s];
        if (better(v, i, bv, bi)) { bv = v; bi = i; }
    }
    wave_argmax(bv, bi);
    if (threadIdx.x == 0) argmax_out(bi, rowi, out, host_out);
}

size_t argmax_scratch_floats(int rows, int vocab) { return (size_t)2 * rows * head_segments_max(vocab); }   // finest segmentation: the Head GEMM's tiles

void launch_argmax_merge(const float *pv, const int *pi, int n_seg, int rows, int32_t *out, int32_t *host_out, hipStream_t st) {
    hipLaunchKernelGGL(argmax_merge_kernel, dim3(rows), dim3(64), 0, st, pv, pi, n_seg, out, host_out);
}

void launch_argmax(const float *logits, int ld, int rows, int vocab, float *scratch, int32_t *out, int32_t *host_out, hipStream_t st) {
    const int n_seg = (vocab + ARGMAX_SEG - 1) / ARGMAX_SEG;
    float *pv = scratch;
    int *pi = reinterpret_cast<int *>(scratch + (size_t)rows * n_seg);
    hipLaunchKernelGGL(argmax_seg_kernel, dim3(n_seg, rows), dim3(256), 0, st, logits, ld, vocab, n_seg, pv, pi, out, host_out);
    if (n_seg > 1) launch_argmax_merge(pv, pi, n_seg, rows, out, host_out, st);
}

// ------------------------------------------------------------------ temperature sampling per row
// The token after a row is drawn from softmax(logits / T) by inverse CDF in vocabulary order: the first
// id whose cumulative probability exceeds u.  Stage 1: per (segment, row) the maximum and the sum of
// exp((l - max) / T).  Stage 2: one workgroup per row picks the segment in which u * Z falls, then the
// id inside it.  All sums run in a fixed order: the same inputs give the same token on every run.
constexpr int SAMPLE_SEG = 4096, SAMPLE_PER_THREAD = SAMPLE_SEG / 256;
constexpr int SAMPLE_MAX_SEGS = 1024;

__global__ __launch_bounds__(256) void sample_seg_kernel(const float *__restrict__ logits, int ld, int vocab, int n_seg,
                                                         float inv_t, float *__restrict__ pm, float *__restrict__ pe) {
    __shared__ float red[17];
    const int seg = blockIdx.x, rowi = blockIdx.y;
    const float *row = logits + (size_t)rowi * ld;
    const int i0 = seg * SAMPLE_SEG + threadIdx.x * SAMPLE_PER_THREAD;       // a contiguous run per thread
    float v[SAMPLE_PER_THREAD], mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < SAMPLE_PER_THREAD; ++j) {
        v[j] = i0 + j < vocab ? row[i0 + j] : -INFINITY;
        mx = fmaxf(mx, v[j]);
    }
    mx = wave_max(mx);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    float se = 0.f;
#pragma unroll
    for (int j = 0; j < SAMPLE_PER_THREAD; ++j) se += v[j] > -INFINITY ? expf((v[j] - mx) * inv_t) : 0.f;
    se = block_sum(se, red);
    if (threadIdx.x == 0) { pm[rowi * n_seg + seg] = mx; pe[rowi * n_seg + seg] = se; }
}

__global__ __launch_bounds__(256) void sample_pick_kernel(const float *__restrict__ logits, int ld, int vocab, int n_seg,
                                                          float inv_t, const float *__restrict__ pm,
                                                          const float *__restrict__ pe, const float *__restrict__ u_by_depth,
                                                          const int32_t *__restrict__ depth, int32_t *__restrict__ out) {
    __shared__ float w[SAMPLE_MAX_SEGS];
    __shared__ float tsum[256];
    __shared__ float red[17];
    __shared__ int s_seg, s_first, s_last;
    __shared__ float s_rest;
    const int rowi = blockIdx.x, tid = threadIdx.x;
    const float u = u_by_depth[depth ? depth[rowi] : 0];
    float mx = -INFINITY;
    for (int s = tid; s < n_seg; s += 256) mx = fmaxf(mx, pm[rowi * n_seg + s]);
    mx = wave_max(mx);
    if ((tid & 63) == 0) red[tid >> 6] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    for (int s = tid; s < n_seg; s += 256) {
        const float m = pm[rowi * n_seg + s];
        w[s] = m > -INFINITY ? pe[rowi * n_seg + s] * expf((m - mx) * inv_t) : 0.f;
    }
    __syncthreads();
    if (tid == 0) {                                       // at most a few dozen segments: one thread, fixed order
        float z = 0.f;
        for (int s = 0; s < n_seg; ++s) z += w[s];
        const float target = u * z;
        float cum = 0.f;
        int pick = -1, last = 0;
        for (int s = 0; s < n_seg; ++s) {
            if (w[s] > 0.f) last = s;
            if (pick < 0 && cum + w[s] > target) { pick = s; s_rest = target - cum; }
            if (pick < 0) cum += w[s];
        }
        if (pick < 0) { pick = last; s_rest = INFINITY; }  // rounding pushed u * Z past the total: last id with mass
        s_seg = pick; s_first = 0x7fffffff; s_last = -1;
    }
    __syncthreads();
    const int seg = s_seg;
    const float rest = s_rest;
    const float *row = logits + (size_t)rowi * ld;
    const int i0 = seg * SAMPLE_SEG + tid * SAMPLE_PER_THREAD;
    float x[SAMPLE_PER_THREAD], ts = 0.f;
#pragma unroll
    for (int j = 0; j < SAMPLE_PER_THREAD; ++j) {
        x[j] = i0 + j < vocab ? expf((row[i0 + j] - mx) * inv_t) : 0.f;
        ts += x[j];
    }
    tsum[tid] = ts;
    __syncthreads();
    float before = 0.f;                                   // mass of the threads before this one, summed in order
    for (int t = 0; t < tid; ++t) before += tsum[t];
    int mine = 0x7fffffff, last_mass = -1;
    float cum = before;
#pragma unroll
    for (int j = 0; j < SAMPLE_PER_THREAD; ++j) {
        if (x[j] > 0.f) last_mass = i0 + j;
        cum += x[j];
        if (mine == 0x7fffffff && cum > rest) mine = i0 + j;
    }
    if (mine != 0x7fffffff) atomicMin(&s_first, mine);
    if (last_mass >= 0) atomicMax(&s_last, last_mass);
    __syncthreads();
    // nothing crossed (rounding pushed the target past the segment's mass): the last id with mass in the segment
    if (tid == 0) out[rowi] = s_first != 0x7fffffff ? s_first : (s_last >= 0 ? s_last : 0);
}

size_t sample_scratch_floats(int rows, int vocab) { return (size_t)2 * rows * ((vocab + SAMPLE_SEG - 1) / SAMPLE_SEG); }

bool launch_sample(const float *logits, int ld, int rows, int vocab, float temperature, const float *u_by_depth,
                   const int32_t *depth, float *scratch, int32_t *out, hipStream_t st) {
    const int n_seg = (vocab + SAMPLE_SEG - 1) / SAMPLE_SEG;
    if (n_seg > SAMPLE_MAX_SEGS || !(temperature > 0.f)) return false;
    float *pm = scratch, *pe = scratch + (size_t)rows * n_seg;
    const float inv_t = 1.0f / temperature;
    hipLaunchKernelGGL(sample_seg_kernel, dim3(n_seg, rows), dim3(256), 0, st, logits, ld, vocab, n_seg, inv_t, pm, pe);
    hipLaunchKernelGGL(sample_pick_kernel, dim3(rows), dim3(256), 0, st, logits, ld, vocab, n_seg, inv_t, pm, pe, u_by_depth,
                       depth, out);
    return true;
}

// ------------------------------------------------------------------ drawn children and the rejection rule
// A draw is "the first id whose cumulative mass exceeds u times the total", masses exp((l - max) / T).  The vocabulary is cut
// into blocks of 256 ids (one float4 per lane of a wave: coalesced); a draw finds the block (a scan over the block sums), then
// the id inside it (a scan over the lanes of one wave).  Every sum is formed in one fixed order, so a run is repeatable - and the
// order decides draws (an id of a 128K-entry vocabulary owns 8e-6 of the mass, the rounding of a prefix sum is a tenth of that),
// so all that follows keeps it: block sums by wave_sum; a scan over the shares of 1024 "threads" (ceil(blocks / 1024) blocks each),
// 64 at a time, the sixteen totals added one after the other; the drafter's total over its row by the same 1024 threads.
// Two launches over the whole chip (draw_max_kernel, draw_mass_kernel) leave, per row, the maximum, the masses and the block
// sums; a draw is one wave's work: no barriers, one trip to memory for all draws as a rule, and a drawn id changes
// one scan.  Ten children of ten rows of 128256: 21.8 us (31 with scans and shares in registers, a trip to memory a draw and scans
// by shuffles), and 10 for the two launches.  It is a serial chain: about 3500 cycles a draw, of which the two scans are 800.
constexpr int DRAW_THREADS = 1024, DRAW_BLOCK = 256, DRAW_MAX_BLOCKS = 8192, DRAW_SEG = 4096;
constexpr int DRAW_UNROLL = 4, DRAW_WAVES = DRAW_THREADS / 64, DRAW_MAX_K = 16;
typedef float f32x4e __attribute__((ext_vector_type(4)));

static inline int draw_blocks(int vocab) { return (vocab + DRAW_BLOCK - 1) / DRAW_BLOCK; }
static inline int draw_segs(int vocab) { return (vocab + DRAW_SEG - 1) / DRAW_SEG; }

// pm[row][seg] = the largest of row[seg * DRAW_SEG ..]
__global__ __launch_bounds__(256) void draw_max_kernel(const float *__restrict__ logits, int ld, int vocab, int n_seg, float *__restrict__ pm) {
    __shared__ float red[4];
    const int seg = blockIdx.x, rowi = blockIdx.y, tid = threadIdx.x;
    const float *row = logits + (size_t)rowi * ld;
    float v[DRAW_SEG / 256], mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < DRAW_SEG / 256; ++j) {            // requested together, never predicated (a repeated id changes no maximum)
        const int i = seg * DRAW_SEG + j * 256 + tid;
        v[j] = row[i < vocab ? i : vocab - 1];
    }
#pragma unroll
    for (int j = 0; j < DRAW_SEG / 256; ++j) mx = fmaxf(mx, v[j]);
    mx = wave_max(mx);
    if ((tid & 63) == 0) red[tid >> 6] = mx;
    __syncthreads();
    if (tid == 0) pm[(size_t)rowi * n_seg + seg] = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

// mass[row][id] = exp((l - max) / T) (0 from the vocabulary's end to the row's), bsum[row][block], mx[row]; a wave takes four blocks
__global__ __launch_bounds__(256) void draw_mass_kernel(const float *__restrict__ logits, int ld, int vocab, int n_seg, int nblk, float inv_t,
                                                        const float *__restrict__ pm, float *__restrict__ mass, float *__restrict__ bsum,
                                                        float *__restrict__ mx_out) {
    const int rowi = blockIdx.y, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, b0 = (blockIdx.x * 4 + wave) * 4;
    const float *row = logits + (size_t)rowi * ld;
    f32x4e v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int id0 = (b0 + u) * DRAW_BLOCK + lane * 4;
        v[u] = *reinterpret_cast<const f32x4e *>(row + (id0 + 3 < ld ? id0 : 0));
    }
    float mx = -INFINITY;
    for (int s = lane; s < n_seg; s += 64) mx = fmaxf(mx, pm[(size_t)rowi * n_seg + s]);
    mx = wave_max(mx);
    if (b0 == 0 && lane == 0) mx_out[rowi] = mx;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int id0 = (b0 + u) * DRAW_BLOCK + lane * 4;
#pragma unroll
        for (int j = 0; j < 4; ++j) v[u][j] = id0 + j < vocab ? expf((v[u][j] - mx) * inv_t) : 0.f;
        if (id0 + 3 < ld) *reinterpret_cast<f32x4e *>(mass + (size_t)rowi * ld + id0) = v[u];
        const float s = wave_sum(((v[u][0] + v[u][1]) + v[u][2]) + v[u][3]);
        if (lane == 0 && b0 + u < nblk) bsum[(size_t)rowi * nblk + b0 + u] = s;
    }
}

void launch_draw_masses(const float *logits, int ld, int rows, int vocab, float temperature, const DrawMasses &m, hipStream_t st) {
    const int n_seg = draw_segs(vocab), nblk = draw_blocks(vocab);
    hipLaunchKernelGGL(draw_max_kernel, dim3(n_seg, rows), dim3(256), 0, st, logits, ld, vocab, n_seg, m.pm);
    hipLaunchKernelGGL(draw_mass_kernel, dim3((nblk + 15) / 16, rows), dim3(256), 0, st, logits, ld, vocab, n_seg, nblk, 1.0f / temperature,
                       m.pm, m.mass, m.bsum, m.mx);
}

size_t draw_pm_floats(int rows, int vocab) { return (size_t)rows * draw_segs(vocab); }
size_t draw_bsum_floats(int rows, int vocab) { return (size_t)rows * draw_blocks(vocab); }

struct DrawLds {
    float bsum[DRAW_MAX_BLOCKS];       // mass of every block
    float cum[DRAW_THREADS];           // inclusive scan over the threads' shares of bsum
    float red[17];
    float wave_off[17];
    float f[4]; int i[4];
    int removed[16];
};

// Inclusive scan of one value per thread over the workgroup, in a fixed order: inside a wave by shuffles, the 16 wave
// totals by thread 0.  Returns the inclusive value; *total = the sum of all.
__device__ __forceinline__ float block_scan(float v, DrawLds &L, float *total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const float t = __shfl_up(v, o, 64);
        if (lane >= o) v += t;
    }
    __syncthreads();
    if (lane == 63) L.red[wave] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        float a = 0.f;
        for (int w = 0; w < DRAW_THREADS / 64; ++w) { L.wave_off[w] = a; a += L.red[w]; }
        L.wave_off[16] = a;
    }
    __syncthreads();
    *total = L.wave_off[16];
    return v + L.wave_off[wave];
}

// The block that holds u * (total mass): the first whose inclusive cumulative sum exceeds it; blocks without mass are never
// chosen; if rounding pushed the target past the total, the last block with mass (*before = -inf then).  Every thread
// gets the result.
__device__ __forceinline__ int find_block(DrawLds &L, int nblk, float u, float *before, float *total_out) {
    const int tid = threadIdx.x, per = (nblk + DRAW_THREADS - 1) / DRAW_THREADS, b0 = tid * per, b1 = min(nblk, b0 + per);
    float s = 0.f;
    int last_mass = -1;
    for (int b = b0; b < b1; ++b) { s += L.bsum[b]; if (L.bsum[b] > 0.f) last_mass = b; }
    float total;
    const float incl = block_scan(s, L, &total);
    L.cum[tid] = incl;
    if (tid == 0) { L.i[0] = -1; L.i[1] = -1; }
    __syncthreads();
    const float target = u * total, prev = tid ? L.cum[tid - 1] : 0.f;
    if (last_mass >= 0) atomicMax(&L.i[1], last_mass);
    if (s > 0.f && prev <= target && target < incl) {
        // (prev + the shares one by one may round differently from incl: the last share with mass takes what is left)
        float cumb = prev;
        for (int b = b0; b < b1; ++b) {
            const float w = L.bsum[b];
            if (w > 0.f && (cumb + w > target || b == last_mass)) { L.i[0] = b; L.f[0] = cumb; break; }
            cumb += w;
        }
    }
    __syncthreads();
    *total_out = total;
    if (L.i[0] >= 0) { *before = L.f[0]; return L.i[0]; }
    *before = -INFINITY;
    return L.i[1] < 0 ? 0 : L.i[1];
}

// Inclusive scan of non-negative values over a wave: for o = 1, 2, .. 32, v[l] += v[l - o] where there is such a lane (0 elsewhere, which
// adds nothing).  Up to 8 lanes by DPP (wave_shr:1, o times), 16 and 32 by the row swaps: about 350 cycles; six shuffles through the LDS
// crossbar took 1000 in these kernels.
__device__ __forceinline__ float wave_shr1(float x) { return dpp<0x138>(0.f, x); }
__device__ __forceinline__ float wave_scan(float v) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
        float t = v;
#pragma unroll
        for (int i = 0; i < o; ++i) t = wave_shr1(t);
        v += t;
    }
    float lo, hi, lo2, hi2;
    swap16(v, lo, hi);                                    // rows (0 0 2 2) and (1 1 3 3)
    swap32(hi, lo2, hi2);                                 // lo2: row 1 everywhere
    v += lane < 16 ? 0.f : (lane >> 4) == 2 ? lo2 : lo;
    swap32(v, lo, hi);
    v += lane < 32 ? 0.f : lo;
    return v;
}

// By one wave: the id inside block b at which the cumulative mass (m: the lane's four ids, in id order) exceeds `rest`; with
// take_last or nothing crossing, the last id with mass (the block's first if none has any).
__device__ __forceinline__ int pick_in_block(int b, float rest, bool take_last, f32x4e m) {
    const int lane = threadIdx.x & 63;
    const float ls = ((m[0] + m[1]) + m[2]) + m[3];
    const float incl = wave_scan(ls);
    const float prev = incl - ls;                         // (exclusive prefix of this lane)
    int last = -1;
#pragma unroll
    for (int j = 0; j < 4; ++j) if (m[j] > 0.f) last = b * DRAW_BLOCK + lane * 4 + j;
    int mine = -1;
    if (!take_last && ls > 0.f && incl > rest) {          // the crossing falls into this lane's four ids
        float c = prev;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            c += m[j];
            if (mine < 0 && m[j] > 0.f && c > rest) mine = b * DRAW_BLOCK + lane * 4 + j;
        }
        if (mine < 0) mine = last;                        // (prev + the four masses rounded below incl)
    }
    // first crossing lane wins; otherwise the last id with mass
    const unsigned long long crossed = __ballot(mine >= 0);
    int pick;
    if (crossed) {
        const int src = __ffsll((long long)crossed) - 1;
        pick = __builtin_amdgcn_readlane(mine, src);
    } else {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) last = max(last, __shfl_xor(last, o, 64));
        pick = last;
    }
    return pick < 0 ? b * DRAW_BLOCK : pick;
}

// the masses of lane's four ids of block b, of a row of masses (0 where the row ends)
__device__ __forceinline__ f32x4e load_masses(const float *mass, int ld, int b, int lane) {
    const int id0 = b * DRAW_BLOCK + lane * 4;
    f32x4e v = f32x4e{0.f, 0.f, 0.f, 0.f};
    if (id0 + 3 < ld) v = *reinterpret_cast<const f32x4e *>(mass + id0);
    return v;
}

// One workgroup per row: wave 0 draws k ids without replacement; the others sum the row meanwhile (z: the total the rejection
// walk divides by), as block_sum over all sixteen would: wave 1 takes the share of wave 0 besides its own.
__global__ __launch_bounds__(DRAW_THREADS) void sample_children_kernel(const float *__restrict__ logits, int ld, int vocab, int nblk, int k,
                                                                       float inv_t, DrawMasses dm, const float *__restrict__ u,
                                                                       int32_t *__restrict__ out_id, float *__restrict__ out_logp) {
    typedef __attribute__((address_space(3))) void *LdsPtr;
    __shared__ float bsum[DRAW_MAX_BLOCKS];
    __shared__ float red[17];
    __shared__ float scans[DRAW_THREADS];
    __shared__ __attribute__((aligned(1024))) float fetched[DRAW_MAX_K][DRAW_BLOCK];
    const int rowi = blockIdx.x, tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const float *mass = dm.mass + (size_t)rowi * ld;
    const int per = (nblk + DRAW_THREADS - 1) / DRAW_THREADS;
    if (wave == 0) {
        const float uu = lane < k ? u[rowi * k + lane] : 0.f, mx = dm.mx[rowi];
        for (int b0 = lane; b0 < nblk; b0 += 64 * 8) {    // (eight at a time on their way)
            float t[8];
#pragma unroll
            for (int x = 0; x < 8; ++x) t[x] = dm.bsum[(size_t)rowi * nblk + min(b0 + 64 * x, nblk - 1)];
#pragma unroll
            for (int x = 0; x < 8; ++x) if (b0 + 64 * x < nblk) bsum[b0 + 64 * x] = t[x];
        }
        wave_lds_sync();
        // share t = blocks [t per, (t + 1) per); scan w is over the shares 64 w ..: scans[] holds them, lane w of `totals` the total of
        // scan w, lane w of `ends` the sum of the totals up to and with it.  (Scans behind the last block hold nothing.  Scans and
        // shares in registers, sixteen of each, meant sixteen copies of the code of every step, the sixteen scans of the start 22 K cycles
        // of 65 K, mostly for fetching it.)
        const int n_w = (nblk + per * 64 - 1) / (per * 64);
        auto share = [&](int t) {
            if (per == 1) return t < nblk ? bsum[t] : 0.f;
            float s = 0.f;
            for (int b = t * per; b < min(nblk, (t + 1) * per); ++b) s += bsum[b];
            return s;
        };
        float totals = 0.f, ends = 0.f;
        auto scan_shares = [&](int w) {
            const float sc = wave_scan(share(w * 64 + lane));
            scans[w * 64 + lane] = sc;
            const float all = lane_value(sc, 63);
            if (lane == w) totals = all;
        };
        auto add_totals = [&]() {                         // one after the other
            float sum = 0.f;
            for (int w0 = 0; w0 < n_w; w0 += 4)
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    sum += lane_value(totals, w0 + w);
                    if (lane == w0 + w) ends = sum;
                }
            return sum;
        };
        for (int w = 0; w < n_w; ++w) scan_shares(w);
        wave_lds_sync();
        float total = add_totals();
        const float log_z = logf(total);                  // the normaliser of the full distribution
        // The blocks that the draws would come from if none took anything out, fetched in one trip (a draw from elsewhere makes a trip of
        // its own): of the first share whose inclusive prefix exceeds lane j's target; one block per share up to DRAW_THREADS blocks.
        int guess = 0;
        {
            const float aim = uu * total;
            float before = 0.f;
            int w = 0;
            for (int x = 0; x < n_w - 1; ++x) {
                const float end = lane_value(ends, x);
                if (end <= aim) { w = x + 1; before = end; }
            }
            guess = w * 64;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) if (scans[guess + o - 1] + before <= aim) guess += o;
            guess = min(guess * per, nblk - 1);
        }
        const unsigned lds0 = (unsigned)(uintptr_t)(LdsPtr)&fetched[0][0];
        for (int j = 0; j < k; ++j) {
            const int id0 = __builtin_amdgcn_readlane(guess, j) * DRAW_BLOCK + lane * 4;
            lds_dma16(lds0 + j * (DRAW_BLOCK * 4), mass + (id0 + 3 < ld ? id0 : 0));
        }
        dma_wait<0>();
        wave_lds_sync();
        int mine = 0;                                     // lane j < k: the j-th id drawn
        for (int d = 0; d < k; ++d) {
            if (d > 0) total = add_totals();
            const float target = lane_value(uu, d) * total;
            // the scan that holds the target, the share inside it, the block inside the share
            int b = -1;
            float before = -INFINITY;
            const int w = __popcll(__ballot(lane < n_w && ends <= target));
            if (w < n_w) {
                const float start = w ? lane_value(ends, w - 1) : 0.f;
                const float incl = scans[w * 64 + lane] + start, prev = lane ? scans[w * 64 + max(lane, 1) - 1] + start : start;
                const unsigned long long hit = __ballot(share(w * 64 + lane) > 0.f && prev <= target && target < incl);
                if (hit) {
                    const int l = __ffsll((long long)hit) - 1, t = w * 64 + l;
                    before = lane_value(prev, l);
                    if (per == 1) {                       // its mass is above 0
                        b = t;
                    } else {
                        int last_mass = -1;
                        for (int x = t * per; x < min(nblk, (t + 1) * per); ++x) if (bsum[x] > 0.f) last_mass = x;
                        for (int x = t * per; x < min(nblk, (t + 1) * per); ++x) {
                            const float m = bsum[x];
                            if (m > 0.f && (before + m > target || x == last_mass)) { b = x; break; }
                            before += m;
                        }
                    }
                }
            }
            if (b < 0) {                                  // rounding pushed the target past the total: the last block with mass
                before = -INFINITY;
                int last = 0;
                for (int x = lane; x < nblk; x += 64) if (bsum[x] > 0.f) last = x;
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) last = max(last, __shfl_xor(last, o, 64));
                b = last;
            }
            b = __builtin_amdgcn_readfirstlane(b);
            // its masses without the ids already drawn: they are taken out of the fetched copy as they are drawn
            const unsigned long long at = __ballot(lane < k && guess == b);
            const int slot = at ? __ffsll((long long)at) - 1 : -1;
            f32x4e m;
            const int id0 = b * DRAW_BLOCK + lane * 4;
            if (slot >= 0) {
                m = *reinterpret_cast<const f32x4e *>(&fetched[slot][lane * 4]);
                if (id0 + 3 >= ld) m = f32x4e{0.f, 0.f, 0.f, 0.f};
            } else {
                m = load_masses(mass, ld, b, lane);
                for (int j = 0; j < d; ++j) {
                    const int r = __builtin_amdgcn_readlane(mine, j) - id0;
#pragma unroll
                    for (int x = 0; x < 4; ++x) if (r == x) m[x] = 0.f;
                }
            }
            const int c = pick_in_block(b, target - before, before == -INFINITY, m);
            if (lane == d) mine = c;
#pragma unroll
            for (int x = 0; x < 4; ++x) if (c - id0 == x) m[x] = 0.f;
            const float s = wave_sum(((m[0] + m[1]) + m[2]) + m[3]);      // the block's mass without the id just drawn, formed afresh
            if (lane == 0) {
                bsum[b] = s;
                if (slot >= 0) fetched[slot][c - b * DRAW_BLOCK] = 0.f;      // (c lies in block b)
            }
            wave_lds_sync();
            scan_shares((per == 1 ? b : b / per) >> 6);
            wave_lds_sync();
        }
        if (lane < k) {
            out_id[rowi * k + lane] = mine;
            out_logp[rowi * k + lane] = (logits[(size_t)rowi * ld + mine] - mx) * inv_t - log_z;
        }
    }
    auto share_of = [&](int w) {
        float sq = 0.f;
        for (int b0 = w; b0 < nblk; b0 += DRAW_WAVES * DRAW_UNROLL) {
            f32x4e v[DRAW_UNROLL];
#pragma unroll
            for (int x = 0; x < DRAW_UNROLL; ++x) v[x] = load_masses(mass, ld, min(b0 + x * DRAW_WAVES, nblk - 1), lane);
#pragma unroll
            for (int x = 0; x < DRAW_UNROLL; ++x) {
                if (b0 + x * DRAW_WAVES >= nblk) break;   // wave-uniform
                sq += ((v[x][0] + v[x][1]) + v[x][2]) + v[x][3];
            }
        }
        sq = wave_sum(sq);
        if (lane == 0) red[w] = sq;
    };
    if (wave > 0) share_of(wave);
    if (wave == 1) share_of(0);
    __syncthreads();
    if (tid == 0) {
        float z = 0.f;
        for (int w = 0; w < DRAW_WAVES; ++w) z += red[w];
        dm.z[rowi] = z;
    }
}

void launch_sample_children(const float *logits, int ld, int rows, int vocab, int k, float temperature, const DrawMasses &m, const float *u,
                            int32_t *out_id, float *out_logp, hipStream_t st) {
    launch_draw_masses(logits, ld, rows, vocab, temperature, m, st);
    hipLaunchKernelGGL(sample_children_kernel, dim3(rows), dim3(DRAW_THREADS), 0, st, logits, ld, vocab, draw_blocks(vocab), k, 1.0f / temperature,
                       m, u, out_id, out_logp);
}

// the masses and totals alone (no draws)
void launch_draft_masses(const float *logits, int ld, int rows, int vocab, float temperature, const DrawMasses &m, hipStream_t st) {
    launch_sample_children(logits, ld, rows, vocab, 0, temperature, m, nullptr, nullptr, nullptr, st);
}

// The walk, one workgroup.  The masses of the target's rows and the drafter's are there (draw_mass_kernel), so a rejection is one
// pass that reads two rows, P and Q, and writes the residual with its block sums (before: two exponentials and two divisions per
// id as well, and four passes per node for maxima and totals).  One round over 128256 ids: 401 -> 41 us, and 16 for the masses of
// the tree's 61 rows.
__global__ __launch_bounds__(DRAW_THREADS) void rejection_walk_kernel(TreeDev td, int k, int L_depth, int vocab, int nblk, DrawMasses target,
                                                                      DrawMasses draft, int ld, const float *__restrict__ ua,
                                                                      float *__restrict__ resid, int32_t *__restrict__ g) {
    __shared__ DrawLds L;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    // a token from the block sums in L.bsum: found by all threads, picked by wave 0, given to every thread
    auto draw_token = [&](float un, const float *mass) {
        float before, total;
        const int b = find_block(L, nblk, un, &before, &total);
        if (wave == 0) {
            const int c = pick_in_block(b, un * total - before, before == -INFINITY, load_masses(mass, ld, b, lane));
            if (lane == 0) L.i[2] = c;
        }
        __syncthreads();
        return L.i[2];
    };
    // what a row of the drafter's holds without the first n removed ids
    auto mass_left = [&](const float *Q, int n) {
        float s = 0.f;
        for (int b = wave; b < nblk; b += DRAW_WAVES) {
            f32x4e m = load_masses(Q, ld, b, lane);
            const int id0 = b * DRAW_BLOCK + lane * 4;
            for (int j = 0; j < n; ++j) {
                const int r = L.removed[j] - id0;
                if (r >= 0 && r < 4) m[r] = 0.f;
            }
            s += ((m[0] + m[1]) + m[2]) + m[3];
        }
        return block_sum(s, L.red);
    };
    const int n_nodes = td.n_nodes[0];
    for (int i = tid; i < n_nodes; i += DRAW_THREADS) g[i] = -1;
    int cur = 0;
    for (int step = 0; step <= L_depth; ++step) {         // at most L accepted children, then the last token
        const int d = td.depth[cur];
        const float *P = target.mass + (size_t)cur * ld;
        // which drafter row expanded this node, and where its drawn children sit in the pool
        int e = -1, cbase = 0;
        if (cur == 0) { e = 0; cbase = 0; }
        else if (d < L_depth) {
            const int pv = td.node_pool[cur];
            for (int r = 0; r < k; ++r)
                if (td.fr_pool[d * k + r] == pv) { e = 1 + (d - 1) * k + r; cbase = k + (d - 1) * k * k + r * k; }
        }
        for (int b = tid; b < nblk; b += DRAW_THREADS) L.bsum[b] = target.bsum[(size_t)cur * nblk + b];
        __syncthreads();
        if (e < 0) {                                      // no drawn children: the target's own token ends the walk
            const int c = draw_token(ua[d * (k + 1) + k], P);
            if (tid == 0) g[cur] = c;
            return;
        }
        float before_unused, zp;                          // zp: the total of P (p = P / zp)
        (void)find_block(L, nblk, 0.f, &before_unused, &zp);
        const float *Q = draft.mass + (size_t)e * ld;
        float zq = draft.z[e];
        bool have_resid = false;
        int next = -1, last_tok = -1;
        for (int i = 0; i < k; ++i) {
            const int c = td.pool_token[cbase + i];
            const float ec = Q[c];
            // At a low temperature fewer than k ids may have any mass in float32: the slots behind them hold an id without mass, or one
            // drawn before, and no child.
            bool drawn = ec > 0.f;
            for (int j = 0; j < i; ++j) drawn = drawn && L.removed[j] != c;
            if (!drawn) break;
            const float pc = (have_resid ? resid[c] : P[c]) / zp, qc = ec / zq;
            const float a = fminf(1.f, pc / qc);
            if (ua[d * (k + 1) + i] < a) {                // accepted (every thread takes the same decision)
                const int node = td.pool_node[cbase + i];
                if (tid == 0) g[cur] = c;
                if (node >= 0) next = node; else last_tok = c;
                break;
            }
            // rejected: P <- max(P / zp - Q / zq, 0) with its block sums, zp <- their total; the candidate leaves q
            __syncthreads();                              // resid[c] has been read by every thread
            const float *from = have_resid ? resid : P;
            const float yp = 1.0f / zp, yq = 1.0f / zq;
            const bool by_reciprocal = quotient_divisor(zp) && quotient_divisor(zq);      // (what is left of q can be nothing)
            for (int b0 = wave; b0 < nblk; b0 += DRAW_WAVES * DRAW_UNROLL) {
                f32x4e pv[DRAW_UNROLL], qv[DRAW_UNROLL];
#pragma unroll
                for (int x = 0; x < DRAW_UNROLL; ++x) {
                    const int b = min(b0 + x * DRAW_WAVES, nblk - 1);
                    pv[x] = load_masses(from, ld, b, lane);
                    qv[x] = load_masses(Q, ld, b, lane);
                }
#pragma unroll
                for (int x = 0; x < DRAW_UNROLL; ++x) {
                    const int b = b0 + x * DRAW_WAVES;
                    if (b >= nblk) break;                 // wave-uniform
                    const int id0 = b * DRAW_BLOCK + lane * 4;
                    f32x4e qm = qv[x];
                    for (int j = 0; j < i; ++j) {
                        const int r = L.removed[j] - id0;
                        if (r >= 0 && r < 4) qm[r] = 0.f;
                    }
                    f32x4e r4;
                    unsigned least = ~0u;
#pragma unroll
                    for (int j = 0; j < 4; ++j) least = min(least, min(quotient_key(pv[x][j]), quotient_key(qm[j])));
                    if (by_reciprocal && !__any(least < QUOTIENT_LEAST)) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) r4[j] = fmaxf(quotient(pv[x][j], zp, yp) - quotient(qm[j], zq, yq), 0.f);
                    } else {                              // masses of 1e-30 and below (a low temperature), or no divisor for it
#pragma unroll
                        for (int j = 0; j < 4; ++j) r4[j] = fmaxf(pv[x][j] / zp - qm[j] / zq, 0.f);
                    }
                    if (id0 + 3 < ld) *reinterpret_cast<f32x4e *>(resid + id0) = r4;
                    const float s = wave_sum(((r4[0] + r4[1]) + r4[2]) + r4[3]);
                    if (lane == 0) L.bsum[b] = s;
                }
            }
            if (tid == 0) L.removed[i] = c;
            __syncthreads();
            (void)find_block(L, nblk, 0.f, &before_unused, &zp);   // (its barriers also publish resid[])
            zq -= ec;
            if (!(zq > 0.f)) zq = mass_left(Q, i + 1);    // (the candidate had all the mass that float32 sees beside it)
            have_resid = true;
            if (!(zp > 0.f)) break;                       // p and q alike to the last bit: nothing to draw from but p
        }
        if (next < 0 && last_tok < 0) {                   // every candidate rejected: draw from the last residual
            const bool from_resid = have_resid && zp > 0.f;
            if (have_resid && !from_resid) {
                __syncthreads();
                for (int b = tid; b < nblk; b += DRAW_THREADS) L.bsum[b] = target.bsum[(size_t)cur * nblk + b];
                __syncthreads();
            }
            const int c = draw_token(ua[d * (k + 1) + k], from_resid ? resid : P);
            if (tid == 0) g[cur] = c;
            // a child that carries the token all the same (the id of an empty slot) is where the commit goes on
            for (int i = 0; i < k && next < 0; ++i)
                if (td.pool_token[cbase + i] == c && td.pool_node[cbase + i] >= 0) next = td.pool_node[cbase + i];
        }
        if (next < 0) return;
        cur = next;
    }
}

void launch_rejection_walk(const TreeDev &td, int k, int L, int vocab, const DrawMasses &target, const DrawMasses &draft, int ld,
                           const float *ua, float *resid, int32_t *g, hipStream_t st) {
    hipLaunchKernelGGL(rejection_walk_kernel, dim3(1), dim3(DRAW_THREADS), 0, st, td, k, L, vocab, draw_blocks(vocab), target, draft, ld, ua,
                       resid, g);
}

__global__ void copy_rows_f32_kernel(const float *__restrict__ src, int ld_src, float *__restrict__ dst, int ld_dst,
                                     int cols) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c < cols) dst[(size_t)blockIdx.y * ld_dst + c] = src[(size_t)blockIdx.y * ld_src + c];
}

void launch_copy_rows_f32(const float *src, int ld_src, float *dst, int ld_dst, int rows, int cols,
                          hipStream_t st) {
    hipLaunchKernelGGL(copy_rows_f32_kernel, dim3((cols + 255) / 256, rows), dim3(256), 0, st, src, ld_src, dst,
                       ld_dst, cols);
}

__global__ void fill_u32_kernel(uint32_t *p, size_t n, uint32_t v) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

void launch_fill_u32(uint32_t *p, size_t n, uint32_t v, hipStream_t st) {
    if (n == 0) return;
    size_t blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)blocks), dim3(256), 0, st, p, n, v);
}

// ------------------------------------------------------------------ debug: cache slots -> float arrays
template <typename T>
__global__ void read_kv_kernel(KVCache kv, int hkv, int dh, int slot0, float *__restrict__ k_out,
                               float *__restrict__ v_out) {
    const int j = blockIdx.x, sl = slot0 + j;
    const T *kc = static_cast<const T *>(kv.k), *vc = static_cast<const T *>(kv.vt);
    for (int p = threadIdx.x; p < hkv * dh; p += blockDim.x) {
        const int h = p / dh, i = p % dh;
        k_out[(size_t)j * hkv * dh + p] = to_f(kc[k_offset(kv, sl, h, hkv, dh) + i]);
        v_out[(size_t)j * hkv * dh + p] = to_f(vc[vt_offset(kv, sl, h, hkv, dh, i)]);
    }
}

void launch_read_kv(const ModelDims &md, const KVCache &kv, int slot0, int n, float *k_out, float *v_out,
                    hipStream_t st) {
    POSS_DISPATCH(md.dt, hipLaunchKernelGGL((read_kv_kernel<T>), dim3(n), dim3(256), 0, st, kv, md.hkv, md.dh,
                                            slot0, k_out, v_out));
}

}  // namespace poss
