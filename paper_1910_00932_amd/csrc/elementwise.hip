// BatchNorm (training mode) / ReLU / residual-tail kernels and small utilities,
// channels-innermost frames [rows][C].  The paper names BatchNorm only in its
// training setting (section 4.1); the standard definition is used: batch mean
// and biased batch variance over all N*T frames, y_hat = (y-mean)*rstd,
// z = gamma*y_hat + beta.  All of these are HBM-bound: 16-byte vectors, one
// pass per tensor, per-channel reductions in registers -> LDS -> fp64 atomics.
#include "internal.h"

namespace tsm {

template <typename T, int V> struct alignas(sizeof(T) * V) Pack { T v[V]; };

// Stores of results that the caches cannot hold until their next use go past them (16-byte packs only).
template <typename T, int V>
__device__ __forceinline__ void store_pack(T* p, const Pack<T, V>& v, bool stream) {
    typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
    if (sizeof(T) * V == 16 && stream)
        __builtin_nontemporal_store(*(const u32x4_t*)&v, (u32x4_t*)p);
    else
        *(Pack<T, V>*)p = v;
}
static inline bool stream_result(long rows, int C, int dtype) { return rows * C * (long)dtype_size(dtype) > (64L << 20); }

// ---------------------------------------------------------------------------------
// 16-byte stores over the aligned body, 4-byte stores over the (at most three) words in front of it and behind it.
__global__ void __launch_bounds__(256) fill_zero_kernel(uint32_t* p, int nhead, uint4* body, size_t n16, uint32_t* tail, int ntail) {
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * 256;
    for (; i < n16; i += stride) body[i] = make_uint4(0u, 0u, 0u, 0u);
    if (blockIdx.x == 0) {
        if ((int)threadIdx.x < nhead) p[threadIdx.x] = 0u;
        if ((int)threadIdx.x < ntail) tail[threadIdx.x] = 0u;
    }
}

// p: 4-byte aligned, bytes: a multiple of 4 (rounded up otherwise: every caller's buffer ends on a word)
int fill_zero(void* p, size_t bytes, hipStream_t s) {
    if (bytes == 0) return TSM_OK;
    size_t words = (bytes + 3) / 4;
    uint32_t* w = (uint32_t*)p;
    size_t nhead = ((16 - ((uintptr_t)p & 15)) & 15) / 4;
    if (nhead > words) nhead = words;
    words -= nhead;
    const size_t n16 = words / 4;
    const int ntail = (int)(words - n16 * 4);
    const size_t want = (n16 + 255) / 256;
    const unsigned blocks = (unsigned)(want < 1 ? 1 : (want < 16384 ? want : 16384));
    fill_zero_kernel<<<dim3(blocks), dim3(256), 0, s>>>(w, (int)nhead, (uint4*)(w + nhead), n16, w + nhead + n16 * 4, ntail);
    return check_launch("fill_zero");
}

// ---- launch shape shared by every per-channel kernel ---------------------------------------
// Threads (tx, ty): tx walks channel vectors, ty walks rows; every thread keeps one
// channel vector for its whole life, so per-channel coefficients and partial sums
// stay in registers and consecutive lanes touch consecutive 16-byte pieces of a row.
struct RowShape {
    dim3 grid, block;
    int cv;
};

static RowShape row_shape(long rows, int C, int V, int rows_per_thread, int max_gx, int nt = 256) {
    RowShape r;
    r.cv = C / V;
    int bx = r.cv < nt ? r.cv : nt;
    int by = nt / bx;
    if (by < 1) by = 1;
    long gx = (rows + (long)by * rows_per_thread - 1) / ((long)by * rows_per_thread);
    if (gx < 1) gx = 1;
    if (gx > max_gx) gx = max_gx;
    r.block = dim3(bx, by);
    r.grid = dim3((unsigned)gx, (unsigned)((r.cv + bx - 1) / bx));
    return r;
}

static inline int vec_of(int dtype, int C) {
    const int v = dtype == TSM_F32 ? 4 : 8;
    return C % v == 0 ? v : 1;
}

static constexpr int RED_ROWS_PER_THREAD = 8, RED_MAX_GX = 512;
// Elementwise passes: one row per thread and 128-thread blocks (measured: a grid-stride loop over some twenty rows
// per thread costs 5 % on bn_bwd_apply and 10 % on the block tail, 256-thread blocks another 2 %).
static constexpr int EW_ROWS_PER_THREAD = 1, EW_MAX_GX = 1 << 22, EW_THREADS = 128;

// Number of per-block partial rows the reduction kernels write for this tensor.
int red_blocks(long rows, int C, int dtype) {
    return (int)row_shape(rows, C, vec_of(dtype, C), RED_ROWS_PER_THREAD, RED_MAX_GX).grid.x;
}

// Sums the per-thread partials a[V], b[V] over ty and stores them into this block's
// row of the partial buffer: prow[c] and prow[C + c].  No atomics: deterministic.
template <int V>
__device__ __forceinline__ void block_partial_2(const float* a, const float* b, int cvi, int cv, int C, float* prow) {
    __shared__ float red[2][256 * V];
    const int tx = threadIdx.x, ty = threadIdx.y, bx = blockDim.x, by = blockDim.y;
#pragma unroll
    for (int j = 0; j < V; ++j) {
        red[0][(ty * bx + tx) * V + j] = a[j];
        red[1][(ty * bx + tx) * V + j] = b[j];
    }
    __syncthreads();
    if (ty == 0 && cvi < cv) {
#pragma unroll
        for (int j = 0; j < V; ++j) {
            float sa = 0.f, sb = 0.f;
            for (int r = 0; r < by; ++r) {
                sa += red[0][(r * bx + tx) * V + j];
                sb += red[1][(r * bx + tx) * V + j];
            }
            prow[cvi * V + j] = sa;
            prow[C + cvi * V + j] = sb;
        }
    }
}

// ---- per-channel sum and sum of squares -------------------------------------------------
template <typename T, int V>
__global__ void __launch_bounds__(256) channel_stats_kernel(const T* __restrict__ y, long rows, int C, int cv,
                                                            float* __restrict__ partial) {
    const int cvi = blockIdx.y * blockDim.x + threadIdx.x;
    float s1[V], s2[V];
#pragma unroll
    for (int j = 0; j < V; ++j) s1[j] = s2[j] = 0.f;
    if (cvi < cv) {
        for (long r = (long)blockIdx.x * blockDim.y + threadIdx.y; r < rows; r += (long)gridDim.x * blockDim.y) {
            Pack<T, V> pk = *(const Pack<T, V>*)(y + r * C + (long)cvi * V);
#pragma unroll
            for (int j = 0; j < V; ++j) {
                float v = Elem<T>::ld(pk.v[j]);
                s1[j] += v;
                s2[j] = fmaf(v, v, s2[j]);
            }
        }
    }
    block_partial_2<V>(s1, s2, cvi, cv, C, partial + (size_t)blockIdx.x * 2 * C);
}

template <typename T, int V>
static int channel_stats_tv(const T* y, long rows, int C, float* partial, hipStream_t s) {
    RowShape r = row_shape(rows, C, V, RED_ROWS_PER_THREAD, RED_MAX_GX);
    channel_stats_kernel<T, V><<<r.grid, r.block, 0, s>>>(y, rows, C, r.cv, partial);
    return check_launch("channel_stats");
}

// partial: fp32 [red_blocks(rows, C, dtype)][2*C]
int channel_stats(int dtype, const void* y, long rows, int C, float* partial, hipStream_t s) {
    const int v = vec_of(dtype, C);
    if (dtype == TSM_F32)
        return v == 4 ? channel_stats_tv<float, 4>((const float*)y, rows, C, partial, s)
                      : channel_stats_tv<float, 1>((const float*)y, rows, C, partial, s);
    return v == 8 ? channel_stats_tv<bf16_t, 8>((const bf16_t*)y, rows, C, partial, s)
                  : channel_stats_tv<bf16_t, 1>((const bf16_t*)y, rows, C, partial, s);
}

// Adds up the rows of a partial buffer for channel c = blockIdx.x*16 + threadIdx.x.  This kernel is pure latency (it
// sits between two dependent launches of every BatchNorm, forward and backward), so the rows are split over 64 ty
// lanes of a (16 x 64) block and a lane issues the loads of its first four rows together: up to 256 rows cost one
// memory round trip.  The lanes meet in a fixed order: the four ty lanes of a wavefront by two shuffles, the sixteen
// wavefronts through LDS.  The totals are valid on the threads with threadIdx.y == 0.
static constexpr int SP_C = 16, SP_R = 64;
__device__ __forceinline__ void sum_partials(const float* __restrict__ partial, int nblocks, int C, int c,
                                             double* out1, double* out2) {
    __shared__ double red[2][SP_R / 4][SP_C];
    double s1 = 0.0, s2 = 0.0;
    if (c < C) {
        float a[4] = {0.f, 0.f, 0.f, 0.f}, b[4] = {0.f, 0.f, 0.f, 0.f};
        for (int b0 = threadIdx.y; b0 < nblocks; b0 += 4 * SP_R) {
            float va[4], vb[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {   // rows beyond the end re-read the last row and count as zero: no branch around the loads
                const int r = b0 + k * SP_R;
                const size_t at = (size_t)(r < nblocks ? r : nblocks - 1) * 2 * C + c;
                va[k] = partial[at];
                vb[k] = partial[at + C];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const bool in = b0 + k * SP_R < nblocks;
                a[k] += in ? va[k] : 0.f;
                b[k] += in ? vb[k] : 0.f;
            }
        }
        s1 = ((double)a[0] + (double)a[1]) + ((double)a[2] + (double)a[3]);
        s2 = ((double)b[0] + (double)b[1]) + ((double)b[2] + (double)b[3]);
    }
    // thread (tx, ty) is lane (ty % 4) * 16 + tx of wavefront ty / 4
    s1 += __shfl_xor(s1, 16);
    s2 += __shfl_xor(s2, 16);
    s1 += __shfl_xor(s1, 32);
    s2 += __shfl_xor(s2, 32);
    if ((threadIdx.y & 3) == 0) {
        red[0][threadIdx.y >> 2][threadIdx.x] = s1;
        red[1][threadIdx.y >> 2][threadIdx.x] = s2;
    }
    __syncthreads();
    double t1 = 0.0, t2 = 0.0;
    if (threadIdx.y == 0) {
#pragma unroll
        for (int r = 0; r < SP_R / 4; ++r) {
            t1 += red[0][r][threadIdx.x];
            t2 += red[1][r][threadIdx.x];
        }
    }
    *out1 = t1;
    *out2 = t2;
}

// ---- partial statistics -> per-channel vectors ------------------------------------------------------
struct BnMoments { float mean, rstd; double var; };
__device__ __forceinline__ BnMoments bn_moments(double s1, double s2, double inv_m, float eps) {
    const double mean = s1 * inv_m;
    double var = s2 * inv_m - mean * mean;
    if (var < 0) var = 0;
    return {(float)mean, (float)(1.0 / sqrt(var + (double)eps)), var};
}
__device__ __forceinline__ void bn_store(const BnVec& o, float* run_mean, float* run_var, int c, const BnMoments& m, float scale,
                                         float shift, double unbias, float momentum) {
    o.mean[c] = m.mean;
    o.rstd[c] = m.rstd;
    o.scale[c] = scale;
    o.shift[c] = shift;
    if (run_mean) {
        run_mean[c] = (1.f - momentum) * run_mean[c] + momentum * m.mean;
        run_var[c] = (1.f - momentum) * run_var[c] + momentum * (float)(m.var * unbias);
    }
}

__global__ void __launch_bounds__(SP_C * SP_R) bn_finalize_kernel(const float* __restrict__ partial, int nblocks, double inv_m, double unbias, int C,
                                   const float* __restrict__ gamma, const float* __restrict__ beta, float eps,
                                   BnVec o, float* run_mean, float* run_var, float momentum) {
    const int c = blockIdx.x * SP_C + threadIdx.x;
    double s1, s2;
    sum_partials(partial, nblocks, C, c, &s1, &s2);
    if (c >= C || threadIdx.y != 0) return;
    const BnMoments m = bn_moments(s1, s2, inv_m, eps);
    const float g = gamma ? gamma[c] : 1.f;
    const float b = beta ? beta[c] : 0.f;
    bn_store(o, run_mean, run_var, c, m, g * m.rstd, b - m.mean * g * m.rstd, unbias, momentum);
}

int bn_finalize(const float* partial, int nblocks, long rows, int C, const float* gamma, const float* beta, float eps,
                BnVec out, float* run_mean, float* run_var, float momentum, hipStream_t s) {
    const double inv_m = rows > 0 ? 1.0 / (double)rows : 0.0;
    const double unbias = rows > 1 ? (double)rows / (double)(rows - 1) : 1.0;
    bn_finalize_kernel<<<dim3(cdiv(C, SP_C)), dim3(SP_C, SP_R), 0, s>>>(partial, nblocks, inv_m, unbias, C, gamma, beta, eps,
                                                                out, run_mean, run_var, momentum);
    return check_launch("bn_finalize");
}

__global__ void __launch_bounds__(SP_C * SP_R) stats_to_float_kernel(const float* __restrict__ partial, int nblocks, int C, float* sum, float* sumsq) {
    const int c = blockIdx.x * SP_C + threadIdx.x;
    double s1, s2;
    sum_partials(partial, nblocks, C, c, &s1, &s2);
    if (c >= C || threadIdx.y != 0) return;
    sum[c] = (float)s1;
    sumsq[c] = (float)s2;
}

int stats_to_float(const float* partial, int nblocks, int C, float* sum, float* sumsq, hipStream_t s) {
    stats_to_float_kernel<<<dim3(cdiv(C, SP_C)), dim3(SP_C, SP_R), 0, s>>>(partial, nblocks, C, sum, sumsq);
    return check_launch("stats_to_float");
}

// ---- z = relu(scale*y + shift) ------------------------------------------------------------------
template <typename T, int V>
__global__ void __launch_bounds__(256) bn_relu_kernel(const T* __restrict__ y, long rows, int C, int cv,
                                                      const float* __restrict__ scale,
                                                      const float* __restrict__ shift, T* __restrict__ z) {
    const int cvi = blockIdx.y * blockDim.x + threadIdx.x;
    if (cvi >= cv) return;
    float sc[V], sh[V];
#pragma unroll
    for (int j = 0; j < V; ++j) {
        sc[j] = scale[cvi * V + j];
        sh[j] = shift[cvi * V + j];
    }
    for (long r = (long)blockIdx.x * blockDim.y + threadIdx.y; r < rows; r += (long)gridDim.x * blockDim.y) {
        const long off = r * C + (long)cvi * V;
        Pack<T, V> in = *(const Pack<T, V>*)(y + off), out;
#pragma unroll
        for (int j = 0; j < V; ++j) {
            float v = fmaf(Elem<T>::ld(in.v[j]), sc[j], sh[j]);
            out.v[j] = Elem<T>::st(v > 0.f ? v : 0.f);
        }
        *(Pack<T, V>*)(z + off) = out;
    }
}

template <typename T, int V>
static int bn_relu_tv(const T* y, long rows, int C, const float* scale, const float* shift, T* z, hipStream_t s) {
    RowShape r = row_shape(rows, C, V, EW_ROWS_PER_THREAD, EW_MAX_GX, EW_THREADS);
    bn_relu_kernel<T, V><<<r.grid, r.block, 0, s>>>(y, rows, C, r.cv, scale, shift, z);
    return check_launch("bn_relu_apply");
}

int bn_relu_apply(int dtype, const void* y, long rows, int C, const float* scale, const float* shift, void* z,
                  hipStream_t s) {
    if (rows == 0) return TSM_OK;
    const int v = vec_of(dtype, C);
    if (dtype == TSM_F32)
        return v == 4 ? bn_relu_tv<float, 4>((const float*)y, rows, C, scale, shift, (float*)z, s)
                      : bn_relu_tv<float, 1>((const float*)y, rows, C, scale, shift, (float*)z, s);
    return v == 8 ? bn_relu_tv<bf16_t, 8>((const bf16_t*)y, rows, C, scale, shift, (bf16_t*)z, s)
                  : bn_relu_tv<bf16_t, 1>((const bf16_t*)y, rows, C, scale, shift, (bf16_t*)z, s);
}

// ---- out = relu(scale*y + shift + shortcut') -------------------------------------------------------
template <typename T, int V, bool PROJ>
__global__ void __launch_bounds__(256) tail_kernel(const T* __restrict__ y, long rows, int C, int cv,
                                                   const float* __restrict__ scale, const float* __restrict__ shift,
                                                   const T* __restrict__ sc, const float* __restrict__ scale_d,
                                                   const float* __restrict__ shift_d, T* __restrict__ out, bool stream,
                                                   uint8_t* __restrict__ bits) {
    const int cvi = blockIdx.y * blockDim.x + threadIdx.x;
    if (cvi >= cv) return;
    float s0[V], h0[V], s1[V], h1[V];
#pragma unroll
    for (int j = 0; j < V; ++j) {
        s0[j] = scale[cvi * V + j];
        h0[j] = shift[cvi * V + j];
        s1[j] = PROJ ? scale_d[cvi * V + j] : 1.f;
        h1[j] = PROJ ? shift_d[cvi * V + j] : 0.f;
    }
    for (long r = (long)blockIdx.x * blockDim.y + threadIdx.y; r < rows; r += (long)gridDim.x * blockDim.y) {
        const long off = r * C + (long)cvi * V;
        Pack<T, V> a = *(const Pack<T, V>*)(y + off), b = *(const Pack<T, V>*)(sc + off), o;
#pragma unroll
        for (int j = 0; j < V; ++j) {
            float rr = Elem<T>::ld(b.v[j]);
            if (PROJ) rr = fmaf(rr, s1[j], h1[j]);
            const float v = fmaf(Elem<T>::ld(a.v[j]), s0[j], h0[j]) + rr;
            o.v[j] = Elem<T>::st(v > 0.f ? v : 0.f);
        }
        store_pack<T, V>(out + off, o, stream);
        if (V == 8 && bits) {   // which of the eight stored values are positive: the ReLU decisions, one byte per vector
            unsigned m = 0;
#pragma unroll
            for (int j = 0; j < V; ++j) m |= (Elem<T>::ld(o.v[j]) > 0.f ? 1u : 0u) << j;
            bits[r * cv + cvi] = (uint8_t)m;
        }
    }
}

template <typename T, int V>
static int tail_tv(const T* y, long rows, int C, const float* scale, const float* shift, const T* sc,
                   const float* scale_d, const float* shift_d, T* out, uint8_t* bits, hipStream_t s) {
    RowShape r = row_shape(rows, C, V, EW_ROWS_PER_THREAD, EW_MAX_GX, EW_THREADS);
    const bool st = stream_result(rows, C, sizeof(T) == 2 ? TSM_BF16 : TSM_F32);
    if (scale_d)
        tail_kernel<T, V, true><<<r.grid, r.block, 0, s>>>(y, rows, C, r.cv, scale, shift, sc, scale_d, shift_d, out, st, bits);
    else
        tail_kernel<T, V, false><<<r.grid, r.block, 0, s>>>(y, rows, C, r.cv, scale, shift, sc, scale_d, shift_d, out, st, bits);
    return check_launch("block_tail_fwd");
}

bool block_tail_writes_bits(int dtype, int C) { return dtype == TSM_BF16 && C % 8 == 0; }

int block_tail_fwd(int dtype, const void* y, long rows, int C, const float* scale, const float* shift,
                   const void* shortcut, const float* scale_d, const float* shift_d, void* out, hipStream_t s,
                   uint8_t* out_bits) {
    if (rows == 0) return TSM_OK;
    const int v = vec_of(dtype, C);
    if (out_bits && !block_tail_writes_bits(dtype, C)) return fail(TSM_ERR_UNSUPPORTED, "block tail: decision bits need bf16 and channels % 8 == 0");
    if (dtype == TSM_F32)
        return v == 4 ? tail_tv<float, 4>((const float*)y, rows, C, scale, shift, (const float*)shortcut, scale_d, shift_d, (float*)out, nullptr, s)
                      : tail_tv<float, 1>((const float*)y, rows, C, scale, shift, (const float*)shortcut, scale_d, shift_d, (float*)out, nullptr, s);
    return v == 8 ? tail_tv<bf16_t, 8>((const bf16_t*)y, rows, C, scale, shift, (const bf16_t*)shortcut, scale_d, shift_d, (bf16_t*)out, out_bits, s)
                  : tail_tv<bf16_t, 1>((const bf16_t*)y, rows, C, scale, shift, (const bf16_t*)shortcut, scale_d, shift_d, (bf16_t*)out, nullptr, s);
}

// ---- backward, pass A: ReLU mask + the two BatchNorm reductions -------------------------------------
// Up to five streams of memory with few wavefronts (512 blocks: every block is a partial row): what it runs at is how many
// loads each has in flight.  Rows ahead, us, five tensors of 200704 x 256 bf16 and the five launches of a 64-clip step: none 135
// and 1060 (3.8 TB/s), two 111 and 868 (4.6), four 122 and 892; 1024 blocks 112 and 925 - 1037, and more rows to add up.
static constexpr int RBR_UR = 2;
template <typename T, int V>
__global__ void __launch_bounds__(256) relu_bn_bwd_reduce_kernel(
    const T* __restrict__ dout, const T* __restrict__ act, const T* __restrict__ y, long rows, int C, int cv,
    const float* __restrict__ mean, const float* __restrict__ rstd, T* __restrict__ dz_out,
    float* __restrict__ partial, const T* __restrict__ y2, const float* __restrict__ mean2,
    const float* __restrict__ rstd2, float* __restrict__ partial2) {
    const int cvi = blockIdx.y * blockDim.x + threadIdx.x;
    float s1[V], s2[V], s3[V], mu[V], rs[V], mu2[V], rs2[V];
#pragma unroll
    for (int j = 0; j < V; ++j) s1[j] = s2[j] = s3[j] = mu[j] = rs[j] = mu2[j] = rs2[j] = 0.f;
    if (cvi < cv) {
#pragma unroll
        for (int j = 0; j < V; ++j) {
            mu[j] = mean[cvi * V + j];
            rs[j] = rstd[cvi * V + j];
            if (y2) {
                mu2[j] = mean2[cvi * V + j];
                rs2[j] = rstd2[cvi * V + j];
            }
        }
        // the next RBR_UR rows are on their way while these are added up (rows beyond the end re-read the last one)
        const long step = (long)gridDim.x * blockDim.y, first = (long)blockIdx.x * blockDim.y + threadIdx.y;
        Pack<T, V> d[RBR_UR], a[RBR_UR], yy[RBR_UR], yy2[RBR_UR];
        auto load = [&](long r0) {
#pragma unroll
            for (int u = 0; u < RBR_UR; ++u) {
                const long r = r0 + u * step, off = (r < rows ? r : rows - 1) * C + (long)cvi * V;
                d[u] = *(const Pack<T, V>*)(dout + off);
                yy[u] = *(const Pack<T, V>*)(y + off);
                if (act) a[u] = *(const Pack<T, V>*)(act + off);
                if (y2) yy2[u] = *(const Pack<T, V>*)(y2 + off);
            }
        };
        if (first < rows) load(first);
        for (long r0 = first; r0 < rows; r0 += RBR_UR * step) {
            Pack<T, V> o[RBR_UR];
#pragma unroll
            for (int u = 0; u < RBR_UR; ++u) {
                const bool in = r0 + u * step < rows;
#pragma unroll
                for (int j = 0; j < V; ++j) {
                    const float dz = in && (!act || Elem<T>::ld(a[u].v[j]) > 0.f) ? Elem<T>::ld(d[u].v[j]) : 0.f;
                    o[u].v[j] = Elem<T>::st(dz);
                    s1[j] += dz;
                    s2[j] = fmaf(dz, (Elem<T>::ld(yy[u].v[j]) - mu[j]) * rs[j], s2[j]);
                    if (y2) s3[j] = fmaf(dz, (Elem<T>::ld(yy2[u].v[j]) - mu2[j]) * rs2[j], s3[j]);
                }
            }
            const long rn = r0 + RBR_UR * step;
            if (rn < rows) load(rn);
            if (dz_out) {
#pragma unroll
                for (int u = 0; u < RBR_UR; ++u)
                    if (r0 + u * step < rows) *(Pack<T, V>*)(dz_out + (r0 + u * step) * C + (long)cvi * V) = o[u];
            }
        }
    }
    block_partial_2<V>(s1, s2, cvi, cv, C, partial + (size_t)blockIdx.x * 2 * C);
    if (y2) {
        __syncthreads();
        block_partial_2<V>(s1, s3, cvi, cv, C, partial2 + (size_t)blockIdx.x * 2 * C);
    }
}

template <typename T, int V>
static int relu_bn_bwd_reduce_tv(const T* dout, const T* act, const T* y, long rows, int C, const float* mean,
                                 const float* rstd, T* dz_out, float* partial, const T* y2, const float* mean2,
                                 const float* rstd2, float* partial2, hipStream_t s) {
    RowShape r = row_shape(rows, C, V, RED_ROWS_PER_THREAD, RED_MAX_GX);
    relu_bn_bwd_reduce_kernel<T, V><<<r.grid, r.block, 0, s>>>(dout, act, y, rows, C, r.cv, mean, rstd, dz_out, partial,
                                                                y2, mean2, rstd2, partial2);
    return check_launch("relu_bn_bwd_reduce");
}

// partial / partial2: fp32 [red_blocks(rows, C, dtype)][2*C]
int relu_bn_bwd_reduce(int dtype, const void* dout, const void* act, const void* y, long rows, int C,
                       const float* mean, const float* rstd, void* dz_out, float* partial, const void* y2,
                       const float* mean2, const float* rstd2, float* partial2, hipStream_t s) {
    if (rows == 0) return TSM_OK;
    const int v = vec_of(dtype, C);
#define TSM_RBR(T, V)                                                                                                \
    relu_bn_bwd_reduce_tv<T, V>((const T*)dout, (const T*)act, (const T*)y, rows, C, mean, rstd, (T*)dz_out, partial, \
                                (const T*)y2, mean2, rstd2, partial2, s)
    if (dtype == TSM_F32) return v == 4 ? TSM_RBR(float, 4) : TSM_RBR(float, 1);
    return v == 8 ? TSM_RBR(bf16_t, 8) : TSM_RBR(bf16_t, 1);
#undef TSM_RBR
}

// ---- backward, between the passes: sums -> per-channel coefficients ---------------------------------------
// dy = gamma*rstd*(dz - S1/m - yhat*S2/m), yhat = (y-mean)*rstd, rewritten as dy = a*dz + b*y + c with
//   a = gamma*rstd,  b = -gamma*rstd^2*S2/m,  c = gamma*rstd*(mean*rstd*S2/m - S1/m);
// dbeta = S1, dgamma = S2.
struct BnCoef { float a, b, c; };
__device__ __forceinline__ BnCoef bn_coef(double s1, double s2, double inv_m, float g, float mu, float rs) {
    const float m1 = (float)(s1 * inv_m), m2 = (float)(s2 * inv_m);
    return {g * rs, -g * rs * rs * m2, g * rs * (mu * rs * m2 - m1)};
}

__global__ void __launch_bounds__(SP_C * SP_R) bn_bwd_coeffs_kernel(const float* __restrict__ partial, int nblocks, double inv_m, int C,
                                     const float* __restrict__ mean, const float* __restrict__ rstd,
                                     const float* __restrict__ gamma, float* __restrict__ coef,
                                     float* __restrict__ dgamma, float* __restrict__ dbeta) {
    const int c = blockIdx.x * SP_C + threadIdx.x;
    double s1, s2;
    sum_partials(partial, nblocks, C, c, &s1, &s2);
    if (c >= C || threadIdx.y != 0) return;
    const BnCoef k = bn_coef(s1, s2, inv_m, gamma ? gamma[c] : 1.f, mean[c], rstd[c]);
    coef[c] = k.a;
    coef[C + c] = k.b;
    coef[2 * C + c] = k.c;
    if (dbeta) dbeta[c] = (float)s1;
    if (dgamma) dgamma[c] = (float)s2;
}

int bn_bwd_coeffs(const float* partial, int nblocks, long rows, int C, const float* mean, const float* rstd,
                  const float* gamma, float* coef, float* dgamma, float* dbeta, hipStream_t s) {
    const double inv_m = rows > 0 ? 1.0 / (double)rows : 0.0;
    bn_bwd_coeffs_kernel<<<dim3(cdiv(C, SP_C)), dim3(SP_C, SP_R), 0, s>>>(partial, nblocks, inv_m, C, mean, rstd, gamma, coef,
                                                                  dgamma, dbeta);
    return check_launch("bn_bwd_coeffs");
}

// ---- backward, pass B: dy = a*dz + b*y + c ------------------------------------------------------------------
template <typename T, int V>
__global__ void __launch_bounds__(256) bn_bwd_apply_kernel(const T* __restrict__ dz, const T* __restrict__ y,
                                                           long rows, int C, int cv, const float* __restrict__ coef,
                                                           T* __restrict__ dy) {
    const int cvi = blockIdx.y * blockDim.x + threadIdx.x;
    if (cvi >= cv) return;
    float ka[V], kb[V], kc[V];
#pragma unroll
    for (int j = 0; j < V; ++j) {
        ka[j] = coef[cvi * V + j];
        kb[j] = coef[C + cvi * V + j];
        kc[j] = coef[2 * C + cvi * V + j];
    }
    for (long r = (long)blockIdx.x * blockDim.y + threadIdx.y; r < rows; r += (long)gridDim.x * blockDim.y) {
        const long off = r * C + (long)cvi * V;
        Pack<T, V> a = *(const Pack<T, V>*)(dz + off), b = *(const Pack<T, V>*)(y + off), o;
#pragma unroll
        for (int j = 0; j < V; ++j)
            o.v[j] = Elem<T>::st(fmaf(ka[j], Elem<T>::ld(a.v[j]), fmaf(kb[j], Elem<T>::ld(b.v[j]), kc[j])));
        *(Pack<T, V>*)(dy + off) = o;   // (read again right away by two kernels: a nontemporal store measured slower)
    }
}

template <typename T, int V>
static int bn_bwd_apply_tv(const T* dz, const T* y, long rows, int C, const float* coef, T* dy, hipStream_t s) {
    RowShape r = row_shape(rows, C, V, EW_ROWS_PER_THREAD, EW_MAX_GX, EW_THREADS);
    bn_bwd_apply_kernel<T, V><<<r.grid, r.block, 0, s>>>(dz, y, rows, C, r.cv, coef, dy);
    return check_launch("bn_bwd_apply");
}

// Two BatchNorms that share one upstream gradient (the last stage of a block and its projection shortcut):
// dy1 = a1*dz + b1*y1 + c1 and dy2 = a2*dz + b2*y2 + c2 from one read of dz.
template <typename T, int V>
__global__ void __launch_bounds__(256) bn_bwd_apply2_kernel(const T* __restrict__ dz, const T* __restrict__ y1,
                                                            const T* __restrict__ y2, long rows, int C, int cv,
                                                            const float* __restrict__ coef1, const float* __restrict__ coef2,
                                                            T* __restrict__ dy1, T* __restrict__ dy2) {
    const int cvi = blockIdx.y * blockDim.x + threadIdx.x;
    if (cvi >= cv) return;
    float ka[V], kb[V], kc[V], la[V], lb[V], lc[V];
#pragma unroll
    for (int j = 0; j < V; ++j) {
        ka[j] = coef1[cvi * V + j];
        kb[j] = coef1[C + cvi * V + j];
        kc[j] = coef1[2 * C + cvi * V + j];
        la[j] = coef2[cvi * V + j];
        lb[j] = coef2[C + cvi * V + j];
        lc[j] = coef2[2 * C + cvi * V + j];
    }
    for (long r = (long)blockIdx.x * blockDim.y + threadIdx.y; r < rows; r += (long)gridDim.x * blockDim.y) {
        const long off = r * C + (long)cvi * V;
        Pack<T, V> a = *(const Pack<T, V>*)(dz + off), b = *(const Pack<T, V>*)(y1 + off), c = *(const Pack<T, V>*)(y2 + off), o, p;
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const float g = Elem<T>::ld(a.v[j]);
            o.v[j] = Elem<T>::st(fmaf(ka[j], g, fmaf(kb[j], Elem<T>::ld(b.v[j]), kc[j])));
            p.v[j] = Elem<T>::st(fmaf(la[j], g, fmaf(lb[j], Elem<T>::ld(c.v[j]), lc[j])));
        }
        *(Pack<T, V>*)(dy1 + off) = o;
        *(Pack<T, V>*)(dy2 + off) = p;
    }
}

template <typename T, int V>
static int bn_bwd_apply2_tv(const T* dz, const T* y1, const T* y2, long rows, int C, const float* coef1, const float* coef2,
                            T* dy1, T* dy2, hipStream_t s) {
    RowShape r = row_shape(rows, C, V, EW_ROWS_PER_THREAD, EW_MAX_GX, EW_THREADS);
    bn_bwd_apply2_kernel<T, V><<<r.grid, r.block, 0, s>>>(dz, y1, y2, rows, C, r.cv, coef1, coef2, dy1, dy2);
    return check_launch("bn_bwd_apply");
}

int bn_bwd_apply2(int dtype, const void* dz, const void* y1, const float* coef1, void* dy1, const void* y2,
                  const float* coef2, void* dy2, long rows, int C, hipStream_t s) {
    if (rows == 0) return TSM_OK;
    const int v = vec_of(dtype, C);
    if (dtype == TSM_F32)
        return v == 4 ? bn_bwd_apply2_tv<float, 4>((const float*)dz, (const float*)y1, (const float*)y2, rows, C, coef1, coef2, (float*)dy1, (float*)dy2, s)
                      : bn_bwd_apply2_tv<float, 1>((const float*)dz, (const float*)y1, (const float*)y2, rows, C, coef1, coef2, (float*)dy1, (float*)dy2, s);
    return v == 8 ? bn_bwd_apply2_tv<bf16_t, 8>((const bf16_t*)dz, (const bf16_t*)y1, (const bf16_t*)y2, rows, C, coef1, coef2, (bf16_t*)dy1, (bf16_t*)dy2, s)
                  : bn_bwd_apply2_tv<bf16_t, 1>((const bf16_t*)dz, (const bf16_t*)y1, (const bf16_t*)y2, rows, C, coef1, coef2, (bf16_t*)dy1, (bf16_t*)dy2, s);
}

// coef: fp32 [3*C] from bn_bwd_coeffs
int bn_bwd_apply(int dtype, const void* dz, const void* y, long rows, int C, const float* coef, void* dy,
                 hipStream_t s) {
    if (rows == 0) return TSM_OK;
    const int v = vec_of(dtype, C);
    if (dtype == TSM_F32)
        return v == 4 ? bn_bwd_apply_tv<float, 4>((const float*)dz, (const float*)y, rows, C, coef, (float*)dy, s)
                      : bn_bwd_apply_tv<float, 1>((const float*)dz, (const float*)y, rows, C, coef, (float*)dy, s);
    return v == 8 ? bn_bwd_apply_tv<bf16_t, 8>((const bf16_t*)dz, (const bf16_t*)y, rows, C, coef, (bf16_t*)dy, s)
                  : bn_bwd_apply_tv<bf16_t, 1>((const bf16_t*)dz, (const bf16_t*)y, rows, C, coef, (bf16_t*)dy, s);
}

// ---- BatchNorm's sums finished inside the pass that needs them ---------------------------------------------------------
// Between two convolutions stand the sums of the first's partial rows (bn_finalize, bn_bwd_coeffs: a launch of pure latency)
// and the elementwise pass that waits for them.  Where the rows are few, every block of the elementwise pass adds them up
// itself for its slab of 128 bytes of channels, in fp64 and in one fixed order (so all blocks hold the same coefficients),
// after it has requested its first rows; the first block of a slab leaves the vectors behind that later kernels read.  Latency is
// what bounds it: 4.5 us at 6400 x 128 bf16 where the two launches took 3.8 and 2.8.
static constexpr int FOLD_TX = 8, FOLD_TY = 32, FOLD_UR = 4;   // threads along a row and rows; rows per thread in flight
static constexpr int FOLD_NT = FOLD_TX * FOLD_TY;
enum { FOLD_RELU, FOLD_TAIL, FOLD_TAIL_PROJ, FOLD_BWD, FOLD_BWD2 };

struct FoldArgs {
    BnSums bn[2];
    double inv_m, unbias;
    float eps, momentum;
    long rows;
    int C;
    const void *in0, *in1, *in2;   // RELU: y; TAIL: y, shortcut; BWD: dz, y; BWD2: dz, y1, y2
    void *out0, *out1;
    uint8_t* bits;
    bool stream;
};

// Totals of the slab's channels c0 .. c0 + CS: s_tot[0..CS) first, s_tot[CS..2*CS) second sums.  Ends with a barrier.
template <int CS>
__device__ __forceinline__ void fold_sums(const float* partial, int nrows, int C, int c0, double (*s_red)[2 * CS], double* s_tot) {
    constexpr int Q = 2 * CS / 4, RL = FOLD_NT / Q, U = 16;   // 16-byte pieces of a row, rows read side by side, in flight
    const int tid = threadIdx.x, q = tid % Q, rl = tid / Q;
    const float* p = partial + (q / (CS / 4)) * C + c0 + (q % (CS / 4)) * 4;
    double t[4] = {0.0, 0.0, 0.0, 0.0};
    for (int r0 = rl; r0 < nrows; r0 += U * RL) {
        float4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {   // rows beyond the end re-read the last one and count as zero: no branch around the loads
            const int r = r0 + u * RL;
            v[u] = *(const float4*)(p + (size_t)(r < nrows ? r : nrows - 1) * 2 * C);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool in = r0 + u * RL < nrows;
            t[0] += in ? (double)v[u].x : 0.0;
            t[1] += in ? (double)v[u].y : 0.0;
            t[2] += in ? (double)v[u].z : 0.0;
            t[3] += in ? (double)v[u].w : 0.0;
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) s_red[rl][q * 4 + k] = t[k];
    __syncthreads();
    if (tid < 2 * CS) {
        double v = 0.0;
#pragma unroll
        for (int l = 0; l < RL; ++l) v += s_red[l][tid];
        s_tot[tid] = v;
    }
    __syncthreads();
}

template <typename T, int V, int MODE>
__global__ void __launch_bounds__(FOLD_NT) bn_fold_kernel(FoldArgs a) {
    constexpr int CS = FOLD_TX * V;
    constexpr bool FWD = MODE <= FOLD_TAIL_PROJ;
    constexpr int NBN = MODE == FOLD_TAIL_PROJ || MODE == FOLD_BWD2 ? 2 : 1;
    constexpr int NIN = MODE == FOLD_RELU ? 1 : MODE == FOLD_BWD2 ? 3 : 2;
    __shared__ double s_red[FOLD_NT / (CS / 2)][2 * CS], s_tot[2 * CS];
    __shared__ float s_co[NBN][3][CS];
    typedef Pack<T, V> P;
    const int tid = threadIdx.x, tx = tid % FOLD_TX, ty = tid / FOLD_TX;
    const int c0 = blockIdx.y * CS, C = a.C;
    const void* const src[3] = {a.in0, a.in1, a.in2};
    const long step = (long)gridDim.x * (FOLD_TY * FOLD_UR);
    long r0 = (long)blockIdx.x * (FOLD_TY * FOLD_UR) + ty;
    P in[NIN][FOLD_UR];
    auto load = [&](long r0) {
#pragma unroll
        for (int u = 0; u < FOLD_UR; ++u) {   // (rows beyond the end read the last one and are not stored)
            const long r = r0 + u * FOLD_TY;
            const long off = (r < a.rows ? r : a.rows - 1) * C + c0 + tx * V;
#pragma unroll
            for (int k = 0; k < NIN; ++k) in[k][u] = *(const P*)((const T*)src[k] + off);
        }
    };
    load(r0);
#pragma unroll
    for (int n = 0; n < NBN; ++n) {
        const BnSums& b = a.bn[n];
        fold_sums<CS>(b.partial, b.nrows, C, c0, s_red, s_tot);
        if (tid < CS) {
            const int c = c0 + tid;
            const double s1 = s_tot[tid], s2 = s_tot[CS + tid];
            const bool first = blockIdx.x == 0;
            if (FWD) {
                const BnMoments m = bn_moments(s1, s2, a.inv_m, a.eps);
                const float g = b.gamma ? b.gamma[c] : 1.f, be = b.beta ? b.beta[c] : 0.f;
                const float sc = g * m.rstd, sh = be - m.mean * g * m.rstd;
                s_co[n][0][tid] = sc;
                s_co[n][1][tid] = sh;
                if (first) bn_store(b.vec, b.run_mean, b.run_var, c, m, sc, sh, a.unbias, a.momentum);
            } else {
                const BnCoef k = bn_coef(s1, s2, a.inv_m, b.gamma ? b.gamma[c] : 1.f, b.vec.mean[c], b.vec.rstd[c]);
                s_co[n][0][tid] = k.a;
                s_co[n][1][tid] = k.b;
                s_co[n][2][tid] = k.c;
                if (first && b.dbeta) b.dbeta[c] = (float)s1;
                if (first && b.dgamma) b.dgamma[c] = (float)s2;
            }
        }
        __syncthreads();
    }
    float co[NBN][3][V];
#pragma unroll
    for (int n = 0; n < NBN; ++n)
#pragma unroll
        for (int k = 0; k < (FWD ? 2 : 3); ++k)
#pragma unroll
            for (int j = 0; j < V; ++j) co[n][k][j] = s_co[n][k][tx * V + j];
    for (; r0 < a.rows + ty; r0 += step) {   // (every thread of a block makes the same number of turns)
        P o0[FOLD_UR], o1[MODE == FOLD_BWD2 ? FOLD_UR : 1];
        unsigned m[FOLD_UR];
#pragma unroll
        for (int u = 0; u < FOLD_UR; ++u) {
            m[u] = 0;
#pragma unroll
            for (int j = 0; j < V; ++j) {
                const float x0 = Elem<T>::ld(in[0][u].v[j]);
                if constexpr (MODE == FOLD_RELU) {
                    const float v = fmaf(x0, co[0][0][j], co[0][1][j]);
                    o0[u].v[j] = Elem<T>::st(v > 0.f ? v : 0.f);
                } else if constexpr (FWD) {
                    float rr = Elem<T>::ld(in[1][u].v[j]);
                    if (MODE == FOLD_TAIL_PROJ) rr = fmaf(rr, co[NBN - 1][0][j], co[NBN - 1][1][j]);
                    const float v = fmaf(x0, co[0][0][j], co[0][1][j]) + rr;
                    o0[u].v[j] = Elem<T>::st(v > 0.f ? v : 0.f);
                    m[u] |= (Elem<T>::ld(o0[u].v[j]) > 0.f ? 1u : 0u) << j;
                } else {
                    o0[u].v[j] = Elem<T>::st(fmaf(co[0][0][j], x0, fmaf(co[0][1][j], Elem<T>::ld(in[1][u].v[j]), co[0][2][j])));
                    if constexpr (MODE == FOLD_BWD2)
                        o1[u].v[j] = Elem<T>::st(fmaf(co[1][0][j], x0, fmaf(co[1][1][j], Elem<T>::ld(in[2][u].v[j]), co[1][2][j])));
                }
            }
        }
        const long rn = r0 + step;
        if (rn - ty < a.rows) load(rn);
#pragma unroll
        for (int u = 0; u < FOLD_UR; ++u) {
            const long r = r0 + u * FOLD_TY;
            if (r >= a.rows) continue;
            const long off = r * C + c0 + tx * V;
            store_pack<T, V>((T*)a.out0 + off, o0[u], FWD && a.stream);
            if constexpr (MODE == FOLD_BWD2) *(P*)((T*)a.out1 + off) = o1[u];
            if constexpr (V == 8 && (MODE == FOLD_TAIL || MODE == FOLD_TAIL_PROJ))
                if (a.bits) a.bits[off / 8] = (uint8_t)m[u];
        }
    }
}

// Up to FOLD_ROWS partial rows a block's own sums cost less than the launch they replace (4 - 5 us; of the 106 per train step 72 go
// at 2 clips of 160 x 160, 10 at 8 clips of 224 x 224 and none at 64, where the ring kernel's blocks write a row each).
// Train step of 2 clips of 160 x 160, four micro-batches, us by the line's place: no folding 11837, 64 rows 11554, 128 11488, 256
// 11582, 512 11667; 8 clips of 224 x 224 6657, 6659, 6649, 6731, 6744 (256 rows of 64 channels are 128 KB per block).
static constexpr int FOLD_ROWS = 128, FOLD_BLOCKS = 512;
bool bn_fold_use(int dtype, int nrows, long rows, int C) {
    return C % (FOLD_TX * (dtype == TSM_F32 ? 4 : 8)) == 0 && rows > 0 && nrows > 0 && nrows <= FOLD_ROWS;
}

template <typename T, int V, int MODE>
static int fold_launch(FoldArgs& a, hipStream_t s, const char* what) {
    const int slabs = a.C / (FOLD_TX * V);
    long gx = (a.rows + FOLD_TY * FOLD_UR - 1) / (FOLD_TY * FOLD_UR);
    const long most = FOLD_BLOCKS / slabs > 1 ? FOLD_BLOCKS / slabs : 1;
    if (gx > most) gx = most;
    bn_fold_kernel<T, V, MODE><<<dim3((unsigned)gx, (unsigned)slabs), dim3(FOLD_NT), 0, s>>>(a);
    return check_launch(what);
}

static FoldArgs fold_args(const BnSums& b0, const BnSums* b1, long rows, int C, int dtype) {
    FoldArgs a = {};
    a.bn[0] = b0;
    if (b1) a.bn[1] = *b1;
    a.rows = rows; a.C = C;
    a.inv_m = 1.0 / (double)rows;
    a.unbias = rows > 1 ? (double)rows / (double)(rows - 1) : 1.0;
    a.stream = stream_result(rows, C, dtype);
    return a;
}

int bn_fold_relu(int dtype, const BnSums& b, float eps, float momentum, const void* y, long rows, int C, void* z, hipStream_t s) {
    FoldArgs a = fold_args(b, nullptr, rows, C, dtype);
    a.eps = eps; a.momentum = momentum; a.in0 = y; a.out0 = z; a.stream = false;
    return dtype == TSM_F32 ? fold_launch<float, 4, FOLD_RELU>(a, s, "bn_fold_relu") : fold_launch<bf16_t, 8, FOLD_RELU>(a, s, "bn_fold_relu");
}

int bn_fold_tail(int dtype, const BnSums& b, const BnSums* bd, float eps, float momentum, const void* y, const void* shortcut,
                 long rows, int C, void* out, uint8_t* out_bits, hipStream_t s) {
    FoldArgs a = fold_args(b, bd, rows, C, dtype);
    a.eps = eps; a.momentum = momentum; a.in0 = y; a.in1 = shortcut; a.out0 = out; a.bits = out_bits;
    if (dtype == TSM_F32) return bd ? fold_launch<float, 4, FOLD_TAIL_PROJ>(a, s, "bn_fold_tail") : fold_launch<float, 4, FOLD_TAIL>(a, s, "bn_fold_tail");
    return bd ? fold_launch<bf16_t, 8, FOLD_TAIL_PROJ>(a, s, "bn_fold_tail") : fold_launch<bf16_t, 8, FOLD_TAIL>(a, s, "bn_fold_tail");
}

int bn_fold_bwd(int dtype, const BnSums& b, const void* dz, const void* y, long rows, int C, void* dy, hipStream_t s) {
    FoldArgs a = fold_args(b, nullptr, rows, C, dtype);
    a.in0 = dz; a.in1 = y; a.out0 = dy;
    return dtype == TSM_F32 ? fold_launch<float, 4, FOLD_BWD>(a, s, "bn_fold_bwd") : fold_launch<bf16_t, 8, FOLD_BWD>(a, s, "bn_fold_bwd");
}

int bn_fold_bwd2(int dtype, const BnSums& b1, const BnSums& b2, const void* dz, const void* y1, void* dy1, const void* y2, void* dy2,
                 long rows, int C, hipStream_t s) {
    FoldArgs a = fold_args(b1, &b2, rows, C, dtype);
    a.in0 = dz; a.in1 = y1; a.in2 = y2; a.out0 = dy1; a.out1 = dy2;
    return dtype == TSM_F32 ? fold_launch<float, 4, FOLD_BWD2>(a, s, "bn_fold_bwd") : fold_launch<bf16_t, 8, FOLD_BWD2>(a, s, "bn_fold_bwd");
}

// ---- out = a + b ------------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(256) add_kernel(const T* __restrict__ a, const T* __restrict__ b, T* __restrict__ o,
                                                  size_t n) {
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) o[i] = Elem<T>::st(Elem<T>::ld(a[i]) + Elem<T>::ld(b[i]));
}

int add_tensors(int dtype, const void* a, const void* b, void* out, size_t n, hipStream_t s) {
    if (n == 0) return TSM_OK;
    unsigned blocks = (unsigned)((n + 255) / 256);
    if (dtype == TSM_F32)
        add_kernel<float><<<dim3(blocks), dim3(256), 0, s>>>((const float*)a, (const float*)b, (float*)out, n);
    else
        add_kernel<bf16_t><<<dim3(blocks), dim3(256), 0, s>>>((const bf16_t*)a, (const bf16_t*)b, (bf16_t*)out, n);
    return check_launch("add_tensors");
}

// ---- weight repacking ----------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(256) pack_fwd_kernel(const T* __restrict__ w, bf16_t* __restrict__ out, int Cout,
                                                       int Cin, int taps, int CinP) {
    long i = (long)blockIdx.x * 256 + threadIdx.x;  // out index: [co][tap][ci padded to CinP]
    if (i >= (long)Cout * CinP * taps) return;
    const int ci = (int)(i % CinP);
    const int tap = (int)((i / CinP) % taps);
    const int co = (int)(i / ((long)CinP * taps));
    out[i] = ci < Cin ? f32_to_bf16(Elem<T>::ld(w[((long)co * Cin + ci) * taps + tap])) : (bf16_t)0;
}

int pack_weights_fwd(int dtype, const void* w, bf16_t* out, int Cout, int Cin, int taps, int CinP, hipStream_t s) {
    long n = (long)Cout * CinP * taps;
    if (dtype == TSM_F32)
        pack_fwd_kernel<float><<<dim3(cdiv(n, 256)), dim3(256), 0, s>>>((const float*)w, out, Cout, Cin, taps, CinP);
    else
        pack_fwd_kernel<bf16_t><<<dim3(cdiv(n, 256)), dim3(256), 0, s>>>((const bf16_t*)w, out, Cout, Cin, taps, CinP);
    return check_launch("pack_weights_fwd");
}

template <typename T>
__global__ void __launch_bounds__(256) pack_dgrad_kernel(const T* __restrict__ w, bf16_t* __restrict__ out, int Cout,
                                                         int Cin, int KT, int KH, int KW) {
    const int taps = KT * KH * KW;
    long i = (long)blockIdx.x * 256 + threadIdx.x;  // out index: [ci][flipped tap][co]
    if (i >= (long)Cout * Cin * taps) return;
    const int co = (int)(i % Cout);
    const int ftap = (int)((i / Cout) % taps);
    const int ci = (int)(i / ((long)Cout * taps));
    const int kw = KW - 1 - ftap % KW, kh = KH - 1 - (ftap / KW) % KH, kt = KT - 1 - ftap / (KW * KH);
    const int tap = (kt * KH + kh) * KW + kw;
    out[i] = f32_to_bf16(Elem<T>::ld(w[((long)co * Cin + ci) * taps + tap]));
}

int pack_weights_dgrad(int dtype, const void* w, bf16_t* out, int Cout, int Cin, int KT, int KH, int KW,
                       hipStream_t s) {
    long n = (long)Cout * Cin * KT * KH * KW;
    if (dtype == TSM_F32)
        pack_dgrad_kernel<float><<<dim3(cdiv(n, 256)), dim3(256), 0, s>>>((const float*)w, out, Cout, Cin, KT, KH, KW);
    else
        pack_dgrad_kernel<bf16_t><<<dim3(cdiv(n, 256)), dim3(256), 0, s>>>((const bf16_t*)w, out, Cout, Cin, KT, KH, KW);
    return check_launch("pack_weights_dgrad");
}

// A block's weights are a few megabytes: what a launch of its own costs each of them is the launch (serving one res4 block
// of 8 clips: three maps and three packings in six launches of 80 us, 15 us of it in front of the first convolution).
static constexpr int PREP_PER_BLOCK = 1024;
template <typename T>
__global__ void __launch_bounds__(256) block_prep_kernel(BlockPrep t, float eps) {
    if (blockIdx.x >= t.blocks) {   // one thread block per BatchNorm behind the items
        const BlockPrep::Bn& b = t.bn[blockIdx.x - t.blocks];
        for (int c = threadIdx.x; c < b.C; c += 256) {
            const float sc = b.gamma[c] / sqrtf(b.var[c] + eps);
            b.scale[c] = sc;
            b.shift[c] = fmaf(-b.mean[c], sc, b.beta[c]);
        }
        return;
    }
    int l = 0;
    while (l + 1 < t.nitem && blockIdx.x >= t.item[l + 1].first) ++l;
    const BlockPrep::Item& it = t.item[l];
    const long i0 = (long)(blockIdx.x - it.first) * PREP_PER_BLOCK + threadIdx.x;
    const int taps = it.KT * it.KH * it.KW;
#pragma unroll
    for (int u = 0; u < PREP_PER_BLOCK / 256; ++u) {
        const long i = i0 + u * 256;
        if (i >= it.total) return;
        if (it.in == nullptr) {
            ((uint32_t*)it.out)[i] = 0u;
            continue;
        }
        const unsigned row = (unsigned)(i / it.CP);
        const int c = (int)(i - (long)row * it.CP), tap = (int)(row % (unsigned)taps), n = (int)(row / (unsigned)taps);
        const int co = it.dgrad ? c : n, ci = it.dgrad ? n : c;
        T v = Elem<T>::st(0.f);
        if (c < (it.dgrad ? it.Cout : it.Cin)) v = ((const T*)it.in)[((long)co * it.Cin + ci) * taps + (it.dgrad ? taps - 1 - tap : tap)];
        ((T*)it.out)[i] = v;
    }
}

void BlockPrep::pack(const ConvP& p, int CP, bool dgrad, const void* w, void* out) {
    Item& it = item[nitem++];
    it = Item{w, out, (long)(dgrad ? p.Cin : p.Cout) * p.taps() * CP, p.Cout, p.Cin, p.KT, p.KH, p.KW, CP, dgrad ? 1 : 0, blocks};
    blocks += (unsigned)((it.total + PREP_PER_BLOCK - 1) / PREP_PER_BLOCK);
}
void BlockPrep::fill(void* out, long words) {
    Item& it = item[nitem++];
    it = Item{nullptr, out, words, 0, 0, 1, 1, 1, 1, 0, blocks};
    blocks += (unsigned)((words + PREP_PER_BLOCK - 1) / PREP_PER_BLOCK);
}
void BlockPrep::affine(const float* gamma, const float* beta, const float* mean, const float* var, float* scale, float* shift, int C) {
    bn[nbn++] = Bn{gamma, beta, mean, var, scale, shift, C};
}

int block_prep(int dtype, const BlockPrep& t, float eps, hipStream_t s) {
    const unsigned grid = t.blocks + (unsigned)t.nbn;
    if (grid == 0) return TSM_OK;
    if (dtype == TSM_F32) block_prep_kernel<float><<<dim3(grid), dim3(256), 0, s>>>(t, eps);
    else block_prep_kernel<bf16_t><<<dim3(grid), dim3(256), 0, s>>>(t, eps);
    return check_launch("block_prep");
}

__global__ void __launch_bounds__(256) unpack_wgrad_kernel(const float* __restrict__ packed, float* __restrict__ dw,
                                                           int Cout, int Cin, int taps, int CinP, int accumulate) {
    long i = (long)blockIdx.x * 256 + threadIdx.x;  // dw index: [co][ci][tap]
    if (i >= (long)Cout * Cin * taps) return;
    const int tap = (int)(i % taps);
    const int ci = (int)((i / taps) % Cin);
    const int co = (int)(i / ((long)Cin * taps));
    const float v = packed[((long)co * taps + tap) * CinP + ci];
    dw[i] = accumulate ? dw[i] + v : v;
}

int unpack_wgrad(const float* packed, float* dw, int Cout, int Cin, int taps, int CinP, int accumulate,
                 hipStream_t s) {
    long n = (long)Cout * Cin * taps;
    unpack_wgrad_kernel<<<dim3(cdiv(n, 256)), dim3(256), 0, s>>>(packed, dw, Cout, Cin, taps, CinP, accumulate);
    return check_launch("unpack_wgrad");
}

}  // namespace tsm
