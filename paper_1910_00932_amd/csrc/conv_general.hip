// Implicit-GEMM convolutions for what the 64-channel kernels of conv_mfma.hip do not take: fp32 storage with any
// channel counts, and bf16 storage whose channel counts or shift groups are not multiples of eight.
//
// Both storage types run the same code: a K step is 128 bytes of every tile row (32 floats or 64 bf16), staged through
// LDS, and only the instruction that multiplies a 16-byte fragment pair differs -- v_mfma_f32_32x32x16_bf16, or four
// v_mfma_f32_32x32x2_f32 (fp32 products and sums: no precision is given up against a scalar fmaf loop).  The fp32 weight gradient
// forms its products of bf16 parts (split_f32.h).
//
// What bounds them: forward and data gradient in fp32 the matrix cores' fp32 rate (140 TFLOP/s measured; 64 cycles per instruction
// and 4 KB of LDS fragments per 4096 of those cycles: neither LDS nor memory comes close), of which a barrier per step that stops
// all four wavefronts at once leaves 57 TFLOP/s (6272 x 2304 -> 256; conv_ksplit.hip, without that barrier, 92 with the same
// instructions).  Tiles are chosen for how well they fill the last round.
//
// Against one thread per output element (1.2 TFLOP/s whatever the layer; those kernels are kept in direct.hip for strides
// beyond 2 and filters beyond 8): fp32 train step at 4 clips of 8 x 224^2 655 -> 16.1 ms; bf16 72 -> 200 channels 3x3 at
// 4 clips of 8 x 29^2, all three directions, 17.7 ms -> 211 us.  Forward and data gradients have since moved to
// conv_ksplit.hip (12.9 ms and 157 us) except where channel counts are no multiple of a 16-byte vector, a tensor
// exceeds the 2 GiB of a buffer's offsets or a large bf16 layer reads a shifted copy; the weight gradients are here.
//
// The shift is index arithmetic as in conv_mfma.hip.  A 16-byte vector of channels that straddles two shift groups is
// put together from one masked load per group; where rows are not 16-byte aligned (channel counts that are no multiple
// of the vector) it is loaded element by element.
#include <algorithm>
#include <type_traits>
#include "internal.h"
#include "taps_inside.h"
#include "split_f32.h"

namespace tsm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

static constexpr int KB = 128;          // bytes of every tile row per K step
static constexpr int PITCH = KB + 16;   // LDS row pitch: rows 36 banks apart

struct GenArgs {
    const void* src;       // x (fwd) or dy (dgrad), channels innermost
    const void* wp;        // packed weights [Cd][taps][CsP]
    void* dst;
    const void* addend;    // dgrad: added to dx (nullable)
    float* stats;          // fwd: [mtiles][2*Cd] partial sums of y and y^2 (nullable)
    int F, T;
    int Hs, Ws, Cs, CsP;   // source frame; CsP = channels per tap in wp, a multiple of the vector
    int Hd, Wd, Cd;
    int KT, KH, KW, stride, padh, padw;
    int fold;              // fwd: shift of source channels; dgrad: adjoint shift of destination channels
    int shifted;           // fwd: fold of a source that is S(x) already
    int Kp;                // taps * CsP
    int ntiles, mtiles;
    // parity classes of destination pixels (see IgemmArgs in conv_mfma.hip)
    int ncls, cstep;
    int ph[4], pw[4], hc[4], wc[4], mt0[5];
    int a0h[4], nth[4], a0w[4], ntw[4];
};

__device__ __forceinline__ int grp_dt(int c, int fold) { return c < fold ? 1 : (c < 2 * fold ? -1 : 0); }

// Bits of a 16-byte vector that belong to elements lo <= e < hi.
template <typename T>
__device__ __forceinline__ u32x4 elem_mask(int lo, int hi) {
    u32x4 m;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (sizeof(T) == 4)
            m[q] = (q >= lo && q < hi) ? 0xffffffffu : 0u;
        else
            m[q] = ((2 * q >= lo && 2 * q < hi) ? 0xffffu : 0u) | ((2 * q + 1 >= lo && 2 * q + 1 < hi) ? 0xffff0000u : 0u);
    }
    return m;
}

// Channels ch .. ch+VE-1 of S(x) at one pixel: `p` points at channel 0 of the pixel in the row's own frame (it may lie
// outside the tensor: nothing is read unless the masks allow it), `sp_ok` tells whether the tap lies inside the frame,
// tmask has bit 30 / 31 set where frame t+1 / t-1 is in the clip, d0 is the frame offset of a temporal tap.
template <typename T, bool RAG>
__device__ __forceinline__ u32x4 load_shifted(const T* p, bool sp_ok, uint32_t tmask, int ch, int C, int fold, int d0, long frame) {
    constexpr int VE = 16 / sizeof(T);
    auto in_clip = [&](int d) { return d == 0 || (d > 0 ? (tmask >> 30) & 1u : tmask >> 31) != 0; };
    u32x4 v = {0u, 0u, 0u, 0u};
    if (!sp_ok) return v;
    if (!RAG) {
        const int d = d0 + grp_dt(ch, fold);
        if (in_clip(d)) v = *(const u32x4*)(p + d * frame + ch);
        return v;
    }
    if (C % VE == 0) {
        if (ch < fold && in_clip(1)) v = *(const u32x4*)(p + frame + ch) & elem_mask<T>(0, fold - ch);
        if (ch < 2 * fold && ch + VE > fold && in_clip(-1)) v |= *(const u32x4*)(p - frame + ch) & elem_mask<T>(fold - ch, 2 * fold - ch);
        if (ch + VE > 2 * fold && in_clip(d0)) v |= *(const u32x4*)(p + d0 * frame + ch) & elem_mask<T>(2 * fold - ch, VE);
        return v;
    }
#pragma unroll
    for (int e = 0; e < VE; ++e) {
        const int c = ch + e;
        const int d = d0 + grp_dt(c, fold);
        if (c < C && in_clip(d)) {
            const T* q = p + d * frame + c;
            if (sizeof(T) == 4)
                v[e & 3] = *(const uint32_t*)q;
            else
                v[(e >> 1) & 3] |= (uint32_t)*(const bf16_t*)q << (16 * (e & 1));
        }
    }
    return v;
}

// One 16-byte fragment pair per (i, j): lane = row lane % 32 of the operand, K elements of its half (lane / 32).
template <typename T, int MI, int NJ>
__device__ __forceinline__ void mma(const u32x4* a, const u32x4* b, f32x16 (&acc)[MI][NJ]) {
    if constexpr (sizeof(T) == 2) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[i]), __builtin_bit_cast(bf16x8, b[j]), acc[i][j], 0, 0, 0);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[i][e]), __uint_as_float(b[j][e]), acc[i][j], 0, 0, 0);
    }
}

// The accumulators of a lane that hold NaN, and a new value for one of them.
template <int MI, int NJ, typename Acc>
__device__ __forceinline__ uint64_t nan_mask(const Acc (&acc)[MI][NJ]) {
    constexpr int RN = sizeof(Acc) / 4;
    static_assert(MI * NJ * RN <= 64, "one bit each");
    uint64_t m = 0;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int r = 0; r < RN; ++r)
                if (acc[i][j][r] != acc[i][j][r]) m |= 1ull << ((i * NJ + j) * RN + r);
    return m;
}
template <int MI, int NJ, typename Acc>
__device__ __forceinline__ void set_at(Acc (&acc)[MI][NJ], int at, float v) {
    constexpr int RN = sizeof(Acc) / 4;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int r = 0; r < RN; ++r)
                acc[i][j][r] = at == (i * NJ + j) * RN + r ? v : acc[i][j][r];
}

struct GenRow {
    long off;        // element offset of the row's tap origin, channel 0 (only used for taps inside the frame)
    uint32_t mask;   // bits 0..7 / 8..15: tap rows / columns inside the frame; 30 / 31: frame t+1 / t-1 in the clip
    int dst;         // destination row, -1 beyond the last one
};

// D[pixels x channels], one tile per block.
template <typename T, int BM, int BN, int WM, int WN, bool DGRAD, bool RAG, bool BUF>
__global__ void __launch_bounds__(256, 2) gen_igemm_kernel(GenArgs a) {
    static_assert(!BUF || (!RAG && !DGRAD), "whole vectors of one shift group, paddings that are not negative");   // (and KT == 1, see gen_launch)
    static_assert(WM * WN == 4, "four wavefronts");
    constexpr int TM = BM / WM, TN = BN / WN;
    constexpr int MI = TM / 32, NJ = TN / 32;
    constexpr int VE = 16 / (int)sizeof(T);
    constexpr int KV = KB / 16, KE = KB / (int)sizeof(T);
    constexpr int RPP = 256 / KV;
    constexpr int PA = BM / RPP, PB = BN / RPP;
    __shared__ __attribute__((aligned(16))) unsigned char smem[2 * (BM + BN) * PITCH];
    __shared__ GenRow s_row[BM];
    static_assert(2 * WM * 2 * BN * 4 <= 2 * (BM + BN) * PITCH, "the statistics slots reuse the stages");

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    const int kvec = tid % KV, lrow = tid / KV;

    // tiles that share their pixels have indices 8 apart: one XCD, one L2
    const int bid = (int)blockIdx.x;
    const int mt = ((bid >> 3) / a.ntiles) * 8 + (bid & 7);
    if (mt >= a.mtiles) return;
    const int n0 = ((bid >> 3) % a.ntiles) * BN;
    int cls = 0;
    while (cls + 1 < a.ncls && mt >= a.mt0[cls + 1]) ++cls;
    const int nth = a.nth[cls], ntw = a.ntw[cls];
    const long frame = (long)a.Hs * a.Ws * a.Cs;

    if (tid < BM) {
        const int hc = a.hc[cls], wc = a.wc[cls];
        const long m = (long)(mt - a.mt0[cls]) * BM + tid;
        GenRow r;
        r.off = 0; r.mask = 0; r.dst = -1;
        if (m < (long)a.F * hc * wc) {
            const int f = (int)(m / (hc * wc));
            const int q = (int)(m - (long)f * (hc * wc));
            const int qh = q / wc, qw = q - qh * wc;
            const int dh = qh * a.cstep + a.ph[cls], dw = qw * a.cstep + a.pw[cls];
            const int oh = DGRAD ? (dh - a.padh + a.a0h[cls]) / a.cstep : dh * a.stride - a.padh;
            const int ow = DGRAD ? (dw - a.padw + a.a0w[cls]) / a.cstep : dw * a.stride - a.padw;
            const int t = f % a.T;
            for (int th = 0; th < nth; ++th)
                if (oh + th >= 0 && oh + th < a.Hs) r.mask |= 1u << th;
            for (int tw = 0; tw < ntw; ++tw)
                if (ow + tw >= 0 && ow + tw < a.Ws) r.mask |= 1u << (8 + tw);
            if (t + 1 < a.T) r.mask |= 1u << 30;
            if (t >= 1) r.mask |= 1u << 31;
            r.off = ((long)f * a.Hs * a.Ws + (long)oh * a.Ws + ow) * a.Cs;
            r.dst = (f * a.Hd + dh) * a.Wd + dw;
        }
        s_row[tid] = r;
    }
    __syncthreads();

    const T* aptr[PA];
    uint32_t amask[PA];
#pragma unroll
    for (int i = 0; i < PA; ++i) {
        const GenRow r = s_row[i * RPP + lrow];
        aptr[i] = (const T*)a.src + r.off;
        amask[i] = r.mask;
    }
    const T* bptr[PB];
#pragma unroll
    for (int j = 0; j < PB; ++j) {
        const int n = n0 + j * RPP + lrow;
        bptr[j] = n < a.Cd ? (const T*)a.wp + (long)n * a.Kp : nullptr;
    }
    const int ntaps = a.KT * nth * ntw;
    const int nk = (ntaps * a.CsP + KE - 1) / KE;
    int kt = 0, th = 0, tw = 0, ltap = 0, ch = kvec * VE;   // position of this thread's vector in the K range
    auto wrap = [&]() {
        while (ch >= a.CsP) {
            ch -= a.CsP;
            ++ltap;
            if (++tw >= ntw) { tw = 0; if (++th >= nth) { th = 0; ++kt; } }
        }
    };
    wrap();

    // BUF: buffer loads, padding lanes beyond the end: no load stands under a condition, where it would be awaited at once (us
    // without and with: 26912 x 648 -> 200 28 and 24, 50176 x 1080 -> 64 29 and 24, 25600 x 2808 -> 312 122 and 92 = 486 TFLOP/s)
    constexpr uint32_t OOB = 0x80000000u;
    constexpr int ES = (int)sizeof(T);
    const uint32_t bias = BUF ? (uint32_t)(((long)a.padh * a.Ws + a.padw) * a.Cs * ES) : 0u;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)a.src - bias), 0, (int)((uint32_t)(a.F * frame * ES) + bias), 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)a.wp, 0, (int)(uint32_t)((long)a.Cd * a.Kp * ES), 0x00020000);
    u32x4 areg[PA], breg[PB];
    auto load = [&]() {
        const bool kvalid = ltap < ntaps;
        if constexpr (BUF) {
            const int d = grp_dt(ch, a.fold);
            const uint32_t need = (1u << th) | (1u << (8 + tw)) | (d > 0 ? 1u << 30 : 0u) | (d < 0 ? 1u << 31 : 0u);
            const uint32_t va = (uint32_t)(((th * a.Ws + tw) * a.Cs + ch + d * (int)frame) * ES) + bias;
            const uint32_t vb = (uint32_t)(((th * a.KW + tw) * a.CsP + ch) * ES);
#pragma unroll
            for (int i = 0; i < PA; ++i)
                areg[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(kvalid && (amask[i] & need) == need ? (uint32_t)((const char*)aptr[i] - (const char*)a.src) + va : OOB), 0, 0);
#pragma unroll
            for (int j = 0; j < PB; ++j)
                breg[j] = __builtin_amdgcn_raw_buffer_load_b128(rw, (int)(kvalid && bptr[j] ? (uint32_t)((const char*)bptr[j] - (const char*)a.wp) + vb : OOB), 0, 0);
            ch += KE;
            wrap();
            return;
        }
        const uint32_t need = (1u << th) | (1u << (8 + tw));
        const int d0 = kt - a.KT / 2;
        const int toff = (th * a.Ws + tw) * a.Cs;
#pragma unroll
        for (int i = 0; i < PA; ++i)
            areg[i] = load_shifted<T, RAG>(aptr[i] + toff, kvalid && (amask[i] & need) == need, amask[i], ch, a.Cs, DGRAD ? 0 : a.fold, d0, frame);
        const int woff = ((kt * a.KH + a.a0h[cls] + th * a.cstep) * a.KW + a.a0w[cls] + tw * a.cstep) * a.CsP + ch;
#pragma unroll
        for (int j = 0; j < PB; ++j) breg[j] = (kvalid && bptr[j]) ? *(const u32x4*)(bptr[j] + woff) : u32x4{0u, 0u, 0u, 0u};
        ch += KE;
        wrap();
    };
    auto store = [&](int buf) {
        unsigned char* A = smem + buf * (BM + BN) * PITCH;
#pragma unroll
        for (int i = 0; i < PA; ++i) *(u32x4*)(A + (i * RPP + lrow) * PITCH + kvec * 16) = areg[i];
#pragma unroll
        for (int j = 0; j < PB; ++j) *(u32x4*)(A + (BM + j * RPP + lrow) * PITCH + kvec * 16) = breg[j];
    };

    f32x16 acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    if (nk > 0) {
        load();
        store(0);
        __syncthreads();
    }
    for (int k = 0; k < nk; ++k) {
        const int buf = k & 1;
        if (k + 1 < nk) load();
        const unsigned char* A = smem + buf * (BM + BN) * PITCH + (wm * TM + (lane & 31)) * PITCH + 16 * (lane >> 5);
        const unsigned char* B = smem + buf * (BM + BN) * PITCH + (BM + wn * TN + (lane & 31)) * PITCH + 16 * (lane >> 5);
#pragma unroll
        for (int ks = 0; ks < KB / 32; ++ks) {
            u32x4 af[MI], bf[NJ];
#pragma unroll
            for (int i = 0; i < MI; ++i) af[i] = *(const u32x4*)(A + i * 32 * PITCH + ks * 32);
#pragma unroll
            for (int j = 0; j < NJ; ++j) bf[j] = *(const u32x4*)(B + j * 32 * PITCH + ks * 32);
            mma<T, MI, NJ>(af, bf, acc);
        }
        if (k + 1 < nk) store(buf ^ 1);
        __syncthreads();
    }

    uint64_t nan = nan_mask(acc);   // (see taps_inside.h)
    while (__builtin_expect(nan != 0, 0)) {
        const int at = __ffsll((long long)nan) - 1, i = at / (NJ * 16), j = at / 16 % NJ, r = at % 16;
        nan &= nan - 1;
        const GenRow row = s_row[wm * TM + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)];
        const int col = n0 + wn * TN + j * 32 + (lane & 31);
        if (row.dst >= 0 && col < a.Cd)
            set_at(acc, at, sum_taps_inside<T, DGRAD>(a, cls, (const T*)a.src + row.off, row.mask, (const T*)a.wp + (long)col * a.Kp, a.CsP));
    }

    // ---- epilogue: lane = channel lane % 32, register r = row 8*(r/4) + 4*(lane/32) + r%4 of the 32x32 block; a
    // half-wavefront stores 32 consecutive channels of one pixel
    float* s_part = (float*)smem;   // [2][WM*2][BN]
    const int hw_d = a.Hd * a.Wd;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int cl = wn * TN + j * 32 + (lane & 31), col = n0 + cl;
        float s1 = 0.f, s2 = 0.f;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = wm * TM + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                const int m = s_row[row].dst;
                if (m < 0 || col >= a.Cd) continue;
                T* const dst = (T*)a.dst;
                if (!DGRAD) {
                    const T q = Elem<T>::st(acc[i][j][r]);
                    const float v = Elem<T>::ld(q);
                    s1 += v;
                    s2 = fmaf(v, v, s2);
                    dst[(long)m * a.Cd + col] = q;
                } else {
                    const int dt = grp_dt(col, a.fold);
                    auto emit = [&](long mr, float v) {
                        const long at = mr * a.Cd + col;
                        // (rounded once before the addition, like the kernels that stage the result)
                        if (a.addend) v = Elem<T>::ld(Elem<T>::st(v)) + Elem<T>::ld(((const T*)a.addend)[at]);
                        dst[at] = Elem<T>::st(v);
                    };
                    if (dt == 0) {
                        emit(m, acc[i][j][r]);
                    } else {
                        const uint32_t mask = s_row[row].mask;
                        const bool next = (mask >> 30) & 1u, prev = mask >> 31;   // frame t+1 / t-1 is in the clip
                        if (dt > 0 ? next : prev) emit(m + (long)dt * hw_d, acc[i][j][r]);
                        // the frame that receives nothing from inside the clip
                        if (dt > 0 ? !prev : !next) emit(m, 0.f);
                    }
                }
            }
        }
        if (!DGRAD && a.stats) {
            const int slot = wm * 2 + (lane >> 5);
            s_part[slot * BN + cl] = s1;
            s_part[(WM * 2 + slot) * BN + cl] = s2;
        }
    }
    if (!DGRAD && a.stats) {
        __syncthreads();
        if (tid < 2 * BN) {
            const int stat = tid / BN, cl = tid % BN;
            float v = 0.f;
#pragma unroll
            for (int sl = 0; sl < WM * 2; ++sl) v += s_part[(stat * WM * 2 + sl) * BN + cl];
            if (n0 + cl < a.Cd) a.stats[(size_t)mt * 2 * a.Cd + stat * a.Cd + n0 + cl] = v;
        }
    }
}

// ---- weight gradient: D[Cout x (tap, Cin)], reduced over a chunk of output pixels, fp32 atomics -------------------
struct GenWgradArgs {
    const void* x;
    const void* dy;
    float* dw;             // element (co, ci, tap) at co*so + ci*si + tap*st
    long so;
    int si, st;
    int F, T, H, W, Cin, CinP, Ho, Wo, Cout;
    int KT, KH, KW, stride, pad, fold;
    int shifted;           // fold of an x that is S(x) already
    int inside_only;       // pixels whose tap lies outside add nothing whatever dy is (see taps_inside.h)
    long M, chunk;
    int K;                 // taps * CinP: columns of D, padded per tap
    int col_tiles;
};

static constexpr int GPX = 32;   // pixels per step

// (Buffer loads and 32-bit divisions in the decode instead of conditional loads and 64-bit ones: 26912 pixels 72 -> 200 3x3
// bf16 49.3 -> 46.2 us, 115200 pixels 160 -> 128 129.3 -> 112.1, 51200 pixels 264 -> 264 242.8 -> 206.1.)
// Operand rows go to LDS as loaded, [pixel][channel], padded by 64 bytes so that the four pixels that a wavefront reads together
// fall into different banks.  fp32: a lane reads its channel of eight pixels and cuts them into three parts; the vector
// instructions for that take as long as the matrix instructions they feed (us with fp32 instructions and now: 6272 pixels 256 ->
// 256 3x3 92 and 74, 1568 pixels 512 -> 512 3x3 95 and 78, 1568 pixels 2048 -> 512 53 and 51, 100352 pixels 64 -> 64 3x3 110 and
// 113).  bf16: the transposing read.
//
// Two groups of four wavefronts with LDS of their own take half of a block's pixels each and meet in LDS at the end: as many
// wavefronts per CU as two blocks, half the atomic additions, which were up to a third of the time (us with one group, with its
// additions as plain stores, with two groups: 26912 pixels 72 -> 200 3x3 bf16 45.8, 30.1, 39.6, 25088 pixels 128 -> 128 3x3 fp32 79.7,
// 60.8, 72.5, 25088 pixels 512 -> 128 1x1 44.3, 36.1, 41.9).
template <typename T, int BCO, int BCI, int GW_GROUPS>
struct GenWgradLds {
    static constexpr int PADB = 64;
    static constexpr int ROWA = BCO * (int)sizeof(T) + PADB, ROWB = BCI * (int)sizeof(T) + PADB;
    static constexpr int STAGE = GPX * (ROWA + ROWB);
    __attribute__((aligned(16))) unsigned char mem[GW_GROUPS][2 * STAGE];
    GenRow row[GW_GROUPS][3][GPX];
    int lossy[2];          // fp32: set by any wavefront, behind the first step and behind the last
};

// EXACT: fp32 products by fp32 instructions.  Without it, fp32: false, and nothing added, where the parts of an operand do not hold
// it or a sum leaves the range (see split_f32.h); the same for all threads of a block.
template <typename T, int BCO, int BCI, int WM, int WN, int GW_GROUPS, bool RAG, bool EXACT>
__device__ __forceinline__ bool gen_wgrad_block(const GenWgradArgs& a, GenWgradLds<T, BCO, BCI, GW_GROUPS>& lds, const int thread) {
    static_assert(WM * WN == 4, "four wavefronts");
    typedef GenWgradLds<T, BCO, BCI, GW_GROUPS> Lds;
    constexpr int TM = BCO / WM, TN = BCI / WN;
    constexpr bool SPLIT = sizeof(T) == 4;             // fp32 on the bf16 matrix cores (see split_f32.h)
    constexpr int TB = SPLIT ? 16 : 32, RN = SPLIT ? 4 : 16;   // result blocks of TB x TB, RN values per lane
    constexpr int MI = TM / TB, NJ = TN / TB;
    typedef std::conditional_t<SPLIT, f32x4, f32x16> Acc;
    auto row_of = [](int lane, int r) { return SPLIT ? 4 * (lane >> 4) + r : 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); };
    constexpr int VE = 16 / (int)sizeof(T);
    constexpr int ROWA = Lds::ROWA, ROWB = Lds::ROWB, STAGE = Lds::STAGE;
    constexpr int AV = BCO / VE, BV = BCI / VE;
    constexpr int RA = 256 / AV, RB = 256 / BV;        // rows per load pass
    constexpr int PA = GPX / RA, PB = GPX / RB;
    static_assert(256 % AV == 0 && 256 % BV == 0 && GPX % RA == 0 && GPX % RB == 0, "tile / thread mismatch");
    constexpr int NR = MI * NJ * RN;                   // sums per lane
    static_assert(GW_GROUPS == 1 || (GW_GROUPS == 2 && NR / 2 * 256 * 4 <= 2 * STAGE && (MI % 2 == 0 || NJ == 1)), "half of them travel through the group's stages");
    const int grp = GW_GROUPS == 1 ? 0 : __builtin_amdgcn_readfirstlane(thread >> 8);
    const int tid = thread & 255, lane = tid & 63, wave = tid >> 6;
    unsigned char* const smem = lds.mem[grp];
    GenRow (*const s_pix)[GPX] = lds.row[grp];
    const int wm = wave / WN, wn = wave % WN;
    const int co0 = ((int)blockIdx.y / a.col_tiles) * BCO;
    const int j0 = ((int)blockIdx.y % a.col_tiles) * BCI;
    // steps of each group: the block's pixels, fewer than a chunk in a layer's last block, over the groups (beyond the last pixel
    // they add zeros)
    const long left = a.M - (long)blockIdx.x * a.chunk;
    const int nsteps = (int)(((left < a.chunk ? left : a.chunk) + GW_GROUPS * GPX - 1) / (GW_GROUPS * GPX));
    const long mbeg = (long)blockIdx.x * a.chunk + (long)grp * nsteps * GPX;
    long mend = mbeg + (long)nsteps * GPX;
    if (mend > a.M) mend = a.M;
    const int hw = a.Ho * a.Wo;
    const long frame = (long)a.H * a.W * a.Cin;

    const int avec = tid % AV, arow = tid / AV;
    const int bvec = tid % BV, brow = tid / BV;
    // this thread's column vector: (tap, first channel) for life
    const int jb = j0 + bvec * VE;
    const bool col_ok = jb < a.K;
    const int tap = col_ok ? jb / a.CinP : 0, ch = col_ok ? jb - tap * a.CinP : 0;
    const int kw = tap % a.KW, kh = (tap / a.KW) % a.KH, kt = tap / (a.KW * a.KH);
    const uint32_t need = (1u << kh) | (1u << (8 + kw));
    const int d0 = kt - a.KT / 2;
    const int toff = (kh * a.W + kw) * a.Cin;
    // not RAG: the column's frame offset and what it needs are fixed as well
    const int dcol = d0 + grp_dt(ch, a.fold);
    const uint32_t needt = need | (dcol > 0 ? 1u << 30 : 0u) | (dcol < 0 ? 1u << 31 : 0u);
    const long tcol = toff + ch + (long)dcol * frame;

    // Whole vectors of one shift group (not RAG) are fetched by buffer loads: padding lanes pass an offset beyond the
    // buffer and receive zeros, so that no load stands under a condition; the buffer of x starts at the most negative tap
    // origin.
    constexpr uint32_t OOB = 0x80000000u;
    const uint32_t bias = RAG ? 0u : (uint32_t)(((long)a.pad * a.W + a.pad) * a.Cin * (long)sizeof(T));
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)a.x - bias), 0,
                                                                        (int)((uint32_t)(a.F * (long)a.H * a.W * a.Cin * (long)sizeof(T)) + bias), 0x00020000);
    const __amdgpu_buffer_rsrc_t rdy = __builtin_amdgcn_make_buffer_rsrc((void*)a.dy, 0, (int)(uint32_t)(a.M * a.Cout * (long)sizeof(T)), 0x00020000);
    // (row counts are below 2^31: 32-bit divisions)
    auto decode = [&](int st) {
        if (tid < GPX) {
            const long m = mbeg + (long)st * GPX + tid;
            GenRow r;
            r.off = 0; r.mask = 0; r.dst = 0;
            if (m < mend) {
                const int f = (int)((unsigned)m / (unsigned)hw);
                const int pix = (int)((unsigned)m - (unsigned)f * (unsigned)hw);
                const int oh = (int)((unsigned)pix / (unsigned)a.Wo), ow = pix - oh * a.Wo;
                const int ih = oh * a.stride - a.pad, iw = ow * a.stride - a.pad;
                const int t = f % a.T;
                for (int h = 0; h < a.KH; ++h)
                    if (ih + h >= 0 && ih + h < a.H) r.mask |= 1u << h;
                for (int w = 0; w < a.KW; ++w)
                    if (iw + w >= 0 && iw + w < a.W) r.mask |= 1u << (8 + w);
                if (t + 1 < a.T) r.mask |= 1u << 30;
                if (t >= 1) r.mask |= 1u << 31;
                r.off = ((long)f * a.H * a.W + (long)ih * a.W + iw) * a.Cin;
            }
            s_pix[st % 3][tid] = r;
        }
    };
    u32x4 ar[PA], br[PB];
    auto load = [&](int st) {
#pragma unroll
        for (int i = 0; i < PA; ++i) {
            const long m = mbeg + (long)st * GPX + arow + i * RA;
            if constexpr (!RAG)
                ar[i] = __builtin_amdgcn_raw_buffer_load_b128(rdy, (int)((m < mend && co0 + avec * VE < a.Cout) ? (uint32_t)(m * a.Cout + co0 + avec * VE) * (uint32_t)sizeof(T) : OOB), 0, 0);
            else
                ar[i] = load_shifted<T, RAG>((const T*)a.dy + m * a.Cout, m < mend && co0 + avec * VE < a.Cout, 0u, co0 + avec * VE, a.Cout, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < PB; ++i) {
            const GenRow r = s_pix[st % 3][brow + i * RB];
            if constexpr (!RAG)
                br[i] = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)((col_ok && (r.mask & needt) == needt) ? (uint32_t)(r.off + tcol) * (uint32_t)sizeof(T) + bias : OOB), 0, 0);
            else
                br[i] = load_shifted<T, RAG>((const T*)a.x + r.off + toff, col_ok && (r.mask & need) == need, r.mask, ch, a.Cin, a.fold, d0, frame);
        }
    };
    // fp32: twice the bits, less one, of the smallest operand other than zero.  Taken as they are stored, once in a block: a
    // comparison where they are cut, twice in the large tile, costs that tile's loop spills.
    uint32_t least = ~0u;
    // Every other step's sums are formed of -dy (see mma_split_b), and the blocks and groups of a tile begin with different signs, so
    // that odd numbers of steps leave nothing over either.
    auto negated = [&](int st) { return ((st + (int)blockIdx.x + grp) & 1) != 0; };
    auto store = [&](int buf, int st) {
        unsigned char* S = smem + buf * STAGE;
        if constexpr (SPLIT && !EXACT) {
#pragma unroll
            for (int i = 0; i < PA; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) least = min(least, (ar[i][q] << 1) - 1u);
#pragma unroll
            for (int i = 0; i < PB; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) least = min(least, (br[i][q] << 1) - 1u);
        }
#pragma unroll
        for (int i = 0; i < PA; ++i) {
            if constexpr (SPLIT && !EXACT) ar[i] ^= negated(st) ? 0x80000000u : 0u;
            *(u32x4*)(S + (arow + i * RA) * ROWA + avec * 16) = ar[i];
        }
#pragma unroll
        for (int i = 0; i < PB; ++i) *(u32x4*)(S + GPX * ROWA + (brow + i * RB) * ROWB + bvec * 16) = br[i];
    };

    // fp32: every step's 32 pixels are a sum of their own, added to the others in fp32 (523 pixels at 1568 x 512 -> 512 3x3: one
    // chain over them is off by 2.6e-7 against 64 bits, two levels of sums by 1.1e-7).
    Acc acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int r = 0; r < RN; ++r) acc[i][j][r] = 0.f;

    auto multiply = [&](int buf, float sign) {
        const unsigned char* A = smem + buf * STAGE;
        const unsigned char* B = A + GPX * ROWA;
        if constexpr (SPLIT && EXACT) {
            auto value = [&](const unsigned char* base, int row, int chan, int e) {
                return *(const float*)(base + ((lane >> 4) + 4 * e) * row + (chan + (lane & 15)) * 4);
            };
#pragma unroll
            for (int i = 0; i < MI; ++i)
                mma_exact<NJ>([&](int, int e) { return value(A, ROWA, wm * TM + i * 16, e); },
                              [&](int j, int e) { return value(B, ROWB, wn * TN + j * 16, e); }, acc[i]);
        } else if constexpr (SPLIT) {
            // a lane supplies pixels lane/16 + {0, 4, .. 28} of its channel, to both operands
            auto frag = [&](const unsigned char* base, int row, int chan) {
                const unsigned char* p = base + (lane >> 4) * row + (chan + (lane & 15)) * 4;
                float f[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) f[e] = *(const float*)(p + 4 * e * row);
                return split3(f);
            };
            static_assert(GPX == 32, "one chain per step");
            Split3 bf[NJ];
#pragma unroll
            for (int j = 0; j < NJ; ++j) bf[j] = frag(B, ROWB, wn * TN + j * 16);
#pragma unroll
            for (int i = 0; i < MI; ++i) mma_split_b<NJ>(frag(A, ROWA, wm * TM + i * 16), bf, sign, acc[i]);
        } else {
            // lane = 32*kg + 16*mblk + 4*e + c supplies channels 4c.. of pixel 8*kg + e and receives four pixels of one channel
            const int c = lane & 3, e = (lane >> 2) & 3, mblk = (lane >> 4) & 1, kg = lane >> 5;
            auto frag = [&](const unsigned char* base, int row, int chan) {
                const unsigned char* p = base + (8 * kg + e) * row + (chan + 16 * mblk + 4 * c) * 2;
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p);
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p + 4 * row));
                return __builtin_bit_cast(u32x4, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            };
#pragma unroll
            for (int k = 0; k < GPX; k += 16) {
                u32x4 af[MI], bf[NJ];
#pragma unroll
                for (int i = 0; i < MI; ++i) af[i] = frag(A + k * ROWA, ROWA, wm * TM + i * 32);
#pragma unroll
                for (int j = 0; j < NJ; ++j) bf[j] = frag(B + k * ROWB, ROWB, wn * TN + j * 32);
                mma<T, MI, NJ>(af, bf, acc);
            }
        }
    };

    if (SPLIT && !EXACT && thread == 0) lds.lossy[0] = lds.lossy[1] = 0;
    decode(0);
    if (nsteps > 1) decode(1);
    __syncthreads();
    load(0);
    store(0, 0);
    if (SPLIT && !EXACT && __any(least < SPLIT_LEAST)) lds.lossy[0] = 1;
    __syncthreads();
    // (where such operands are many, the steps are not worth while)
    if (SPLIT && !EXACT && lds.lossy[0]) return false;
    for (int st = 0; st < nsteps; ++st) {
        const int buf = st & 1;
        if (st + 2 < nsteps) decode(st + 2);
        if (st + 1 < nsteps) load(st + 1);
        multiply(buf, negated(st) ? -1.f : 1.f);
        if (st + 1 < nsteps) store(buf ^ 1, st + 1);
        __syncthreads();
    }
    if constexpr (SPLIT && !EXACT) {
        if (__any(least < SPLIT_LEAST || !split_finite(acc))) lds.lossy[1] = 1;
        __syncthreads();
        if (lds.lossy[1]) return false;
    }
    uint64_t nan = a.inside_only ? nan_mask(acc) : 0ull;
    while (__builtin_expect(nan != 0, 0)) {
        const int at = __ffsll((long long)nan) - 1, i = at / (NJ * RN), j = at / RN % NJ, r = at % RN;
        nan &= nan - 1;
        const int col = j0 + wn * TN + j * TB + lane % TB, co = co0 + wm * TM + i * TB + row_of(lane, r);
        const int tp = col / a.CinP, ci = col - tp * a.CinP;
        if (col >= a.K || ci >= a.Cin || co >= a.Cout) continue;
        const int w_ = tp % a.KW, h_ = tp / a.KW % a.KH, dk = tp / (a.KW * a.KH) - a.KT / 2;
        const int d = dk + tap_group_dt(ci, a.fold + a.shifted);   // (one of them is zero)
        float v = 0.f;
#pragma unroll 1
        for (long m = mbeg; m < mend && v == v; ++m) {
            const int f = (int)(m / hw), pix = (int)(m - (long)f * hw), t = f % a.T;
            const int ih = pix / a.Wo * a.stride - a.pad + h_, iw = pix % a.Wo * a.stride - a.pad + w_;
            if (ih < 0 || ih >= a.H || iw < 0 || iw >= a.W || t + d < 0 || t + d >= a.T) continue;
            v = fmaf(Elem<T>::ld(((const T*)a.dy)[m * a.Cout + co]),
                     Elem<T>::ld(((const T*)a.x)[(((long)f + (a.shifted ? dk : d)) * a.H * a.W + (long)ih * a.W + iw) * a.Cin + ci]), v);
        }
        set_at(acc, at, v);
    }
    // a group keeps the first or the second half of its sums and hands over the other
    constexpr int NK = NR / GW_GROUPS;
    auto at = [&](int k) { return acc[k / (NJ * RN)][k / RN % NJ][k % RN]; };
    const float* const theirs = (const float*)lds.mem[GW_GROUPS - 1 - grp];
    if constexpr (GW_GROUPS == 2) {
        float* const mine = (float*)smem;
#pragma unroll
        for (int k = 0; k < NK; ++k) mine[k * 256 + tid] = grp == 0 ? at(k + NK) : at(k);
        __syncthreads();
    }
    bool ok[NJ];
    long off[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int col = j0 + wn * TN + j * TB + lane % TB;
        const int tp = col / a.CinP, ci = col - tp * a.CinP;
        ok[j] = col < a.K && ci < a.Cin;
        off[j] = (long)ci * a.si + (long)tp * a.st;
    }
#pragma unroll
    for (int k = 0; k < NK; ++k) {
        const float v = GW_GROUPS == 1 ? at(k) : (grp == 0 ? at(k) : at((k + NK) % NR)) + theirs[k * 256 + tid];
        const int idx = k + grp * NK, i = idx / (NJ * RN), r = idx % RN, j = k / RN % NJ;
        const int co = co0 + wm * TM + i * TB + row_of(lane, r);
        if (ok[j] && co < a.Cout) atomicAdd(a.dw + (long)co * a.so + off[j], v);
    }
    return true;
}

template <typename T, int BCO, int BCI, int WM, int WN, int GW_GROUPS, bool RAG>
__global__ void __launch_bounds__(256 * GW_GROUPS, 2) gen_wgrad_kernel(GenWgradArgs a) {
    __shared__ GenWgradLds<T, BCO, BCI, GW_GROUPS> lds;
    if (gen_wgrad_block<T, BCO, BCI, WM, WN, GW_GROUPS, RAG, false>(a, lds, (int)threadIdx.x)) return;
    if constexpr (sizeof(T) == 4) {
        int thread = (int)threadIdx.x;
        asm volatile("" : "+v"(thread));   // shares no address register with the code above, which has none to spare
        gen_wgrad_block<T, BCO, BCI, WM, WN, GW_GROUPS, RAG, true>(a, lds, thread);
    }
}

// ---- weights: ABI [Cout][Cin][taps] -> [Cout][taps][CinP] (fwd) or [Cin][flipped taps][CoutP] (dgrad), padding zero
template <typename T, bool DGRAD>
__global__ void __launch_bounds__(256) gen_pack_kernel(const T* __restrict__ w, T* __restrict__ out, int Cout, int Cin, int KT,
                                                       int KH, int KW, int CP, long total) {
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    const int taps = KT * KH * KW;
    const int c = (int)(i % CP), tap = (int)(i / CP % taps), n = (int)(i / ((long)CP * taps));
    const int co = DGRAD ? c : n, ci = DGRAD ? n : c;
    T v = Elem<T>::st(0.f);
    if (c < (DGRAD ? Cout : Cin)) {
        int src = tap;
        if (DGRAD) {   // spatial taps are flipped and so is the temporal one
            const int kw = tap % KW, kh = tap / KW % KH, kt = tap / (KW * KH);
            src = ((KT - 1 - kt) * KH + (KH - 1 - kh)) * KW + (KW - 1 - kw);
        }
        v = w[((long)co * Cin + ci) * taps + src];
    }
    out[i] = v;
}

// ---- host side ----------------------------------------------------------------------------------------------------
static int cu_count() {
    static int n = 0;
    if (n == 0) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess) n = v;
        if (n <= 0) n = 256;
    }
    return n;
}
static int pad_vec(int c, int dtype) { const int v = dtype == TSM_F32 ? 4 : 8; return (c + v - 1) / v * v; }

bool gen_conv_supported(const ConvP& p) {
    if (p.pitch && p.pitch != p.Cin) return false;
    if (p.stride > 2 || p.KH > 8 || p.KW > 8) return false;   // four parity classes, eight mask bits each way
    if (p.KT > 1 && p.fold > 0) return false;                 // frame offsets stay within one frame either way
    if (p.Cin > 65536 || p.Cout > 65536 || (long)p.taps() * (p.Cin + 8) > 0x3fffffffL || (long)p.taps() * (p.Cout + 8) > 0x3fffffffL) return false;
    if (p.rows_in() > 0x3fffffffL || p.rows_out() > 0x3fffffffL) return false;
    if ((long)p.H * p.W * p.Cin > 0x3fffffffL || (long)p.Ho * p.Wo * p.Cout > 0x3fffffffL) return false;
    if (((long)p.KH * p.W + p.KW) * p.Cin > 0x3fffffffL || ((long)p.KH * p.Wo + p.KW) * p.Cout > 0x3fffffffL) return false;   // offset of a tap
    if ((p.rows_in() / 64 + 40) * ((p.Cin + 63) / 64) > 0x7fffffffL || (p.rows_out() / 64 + 40) * ((p.Cout + 63) / 64) > 0x7fffffffL) return false;
    return true;
}

// Elements of the packed weights each direction needs; 0: the ABI order serves as it is.
size_t gen_pack_elems(const ConvP& p, int dtype, bool dgrad) {
    if (dgrad) return (size_t)p.Cin * p.taps() * pad_vec(p.Cout, dtype);
    if (p.taps() == 1 && pad_vec(p.Cin, dtype) == p.Cin) return 0;
    return (size_t)p.Cout * p.taps() * pad_vec(p.Cin, dtype);
}

int gen_pack_weights(const ConvP& p, int dtype, bool dgrad, const void* w, void* out, hipStream_t s) {
    const long total = (long)gen_pack_elems(p, dtype, dgrad);
    const int CP = pad_vec(dgrad ? p.Cout : p.Cin, dtype);
    const dim3 grid((unsigned)((total + 255) / 256));
    if (dtype == TSM_F32) {
        if (dgrad) gen_pack_kernel<float, true><<<grid, dim3(256), 0, s>>>((const float*)w, (float*)out, p.Cout, p.Cin, p.KT, p.KH, p.KW, CP, total);
        else gen_pack_kernel<float, false><<<grid, dim3(256), 0, s>>>((const float*)w, (float*)out, p.Cout, p.Cin, p.KT, p.KH, p.KW, CP, total);
    } else {
        if (dgrad) gen_pack_kernel<bf16_t, true><<<grid, dim3(256), 0, s>>>((const bf16_t*)w, (bf16_t*)out, p.Cout, p.Cin, p.KT, p.KH, p.KW, CP, total);
        else gen_pack_kernel<bf16_t, false><<<grid, dim3(256), 0, s>>>((const bf16_t*)w, (bf16_t*)out, p.Cout, p.Cin, p.KT, p.KH, p.KW, CP, total);
    }
    return check_launch("gen_pack");
}

static void gen_classes(GenArgs& a, bool dgrad, int BM) {
    if (!dgrad || a.stride == 1) {
        a.ncls = 1; a.cstep = 1;
        a.ph[0] = a.pw[0] = 0; a.hc[0] = a.Hd; a.wc[0] = a.Wd;
        a.a0h[0] = a.a0w[0] = 0; a.nth[0] = a.KH; a.ntw[0] = a.KW;
    } else {
        const int st = a.stride;
        a.ncls = st * st; a.cstep = st;
        for (int c = 0; c < a.ncls; ++c) {
            a.ph[c] = c / st; a.pw[c] = c % st;
            a.hc[c] = (a.Hd - a.ph[c] + st - 1) / st;
            a.wc[c] = (a.Wd - a.pw[c] + st - 1) / st;
            a.a0h[c] = (((a.padh - a.ph[c]) % st) + st) % st;
            a.a0w[c] = (((a.padw - a.pw[c]) % st) + st) % st;
            a.nth[c] = a.a0h[c] < a.KH ? (a.KH - a.a0h[c] + st - 1) / st : 0;
            a.ntw[c] = a.a0w[c] < a.KW ? (a.KW - a.a0w[c] + st - 1) / st : 0;
            if (a.nth[c] == 0 || a.ntw[c] == 0) a.nth[c] = a.ntw[c] = 0;
        }
    }
    a.mt0[0] = 0;
    for (int c = 0; c < a.ncls; ++c) a.mt0[c + 1] = a.mt0[c] + (int)(((long)a.F * a.hc[c] * a.wc[c] + BM - 1) / BM);
    a.mtiles = a.mt0[a.ncls];
}

// Tile by the time the fullest CU needs: rounds of tiles times tile area, the smaller tiles charged for the operand
// bytes they read more often.
struct GenTile { int bm, bn; };
static GenTile gen_tile(long rows, int Cd) {
    static const struct { int bm, bn; double cost; } opt[3] = {{128, 128, 1.0}, {128, 64, 1.06}, {64, 64, 1.15}};
    GenTile best{64, 64};
    double tbest = 0;
    for (const auto& o : opt) {
        const long tiles = ((rows + o.bm - 1) / o.bm) * ((Cd + o.bn - 1) / o.bn);
        const long rounds = (tiles + cu_count() - 1) / cu_count();
        const double t = (double)rounds * o.bm * o.bn * o.cost;
        if (tbest == 0 || t < tbest) { tbest = t; best = {o.bm, o.bn}; }
    }
    return best;
}

template <typename T, bool DGRAD, bool RAG>
static int gen_launch(GenArgs& a, hipStream_t s) {
    const GenTile t = gen_tile((long)a.F * a.Hd * a.Wd, a.Cd);
    gen_classes(a, DGRAD, t.bm);
    a.ntiles = (a.Cd + t.bn - 1) / t.bn;
    const dim3 grid((unsigned)((a.mtiles + 7) / 8 * 8 * a.ntiles));
    auto run = [&](auto buf) {
        constexpr bool BUF = decltype(buf)::value;
        if (t.bm == 128 && t.bn == 128) gen_igemm_kernel<T, 128, 128, 2, 2, DGRAD, RAG, BUF><<<grid, dim3(256), 0, s>>>(a);
        else if (t.bm == 128) gen_igemm_kernel<T, 128, 64, 2, 2, DGRAD, RAG, BUF><<<grid, dim3(256), 0, s>>>(a);
        else gen_igemm_kernel<T, 64, 64, 2, 2, DGRAD, RAG, BUF><<<grid, dim3(256), 0, s>>>(a);
    };
    // bf16 layers on a shifted copy, below 2 GiB with the padding in front of the first pixel and the taps behind the last
    const long es = (long)sizeof(T), src = (long)a.F * a.Hs * a.Ws * a.Cs * es;
    const long edge = 2 * (((long)a.KH + a.padh) * a.Ws + a.KW + a.padw) * a.Cs * es;
    if constexpr (sizeof(T) == 2 && !DGRAD && !RAG) {
        if (a.KT == 1 && src + edge < 0x7ff00000L && (long)a.Cd * a.Kp * es < 0x7ff00000L) run(std::true_type());
        else run(std::false_type());
    } else {
        run(std::false_type());
    }
    if (sizeof(T) == 4) return check_launch(DGRAD ? "gen_dgrad_f32" : "gen_fwd_f32");
    return check_launch(DGRAD ? "gen_dgrad_bf16" : "gen_fwd_bf16");
}

int gen_fwd_blocks(const ConvP& p, int dtype) {
    if (ksplit_use(p, dtype, false)) return ksplit_rows(p, dtype, false);
    const int bm = gen_tile(p.rows_out(), p.Cout).bm;
    return (int)((p.rows_out() + bm - 1) / bm);
}

static void gen_common(GenArgs& a, const ConvP& p) {
    a.addend = nullptr; a.stats = nullptr;
    a.F = p.F; a.T = p.T; a.KT = p.KT; a.KH = p.KH; a.KW = p.KW; a.stride = p.stride; a.fold = p.fold; a.shifted = p.shifted;
}

int gen_conv_fwd(const ConvP& p, int dtype, const void* x, const void* wp, void* y, float* stats, hipStream_t s) {
    if (p.rows_out() == 0) return TSM_OK;
    if (ksplit_use(p, dtype, false)) return ksplit_fwd(p, dtype, x, wp, y, stats, nullptr, s);
    GenArgs a;
    gen_common(a, p);
    a.src = x; a.wp = wp; a.dst = y; a.stats = stats;
    a.Hs = p.H; a.Ws = p.W; a.Cs = p.Cin; a.CsP = pad_vec(p.Cin, dtype);
    a.Hd = p.Ho; a.Wd = p.Wo; a.Cd = p.Cout;
    a.padh = a.padw = p.pad;
    a.Kp = p.taps() * a.CsP;
    const bool rag = a.CsP != a.Cs || p.fold % (dtype == TSM_F32 ? 4 : 8) != 0;
    if (dtype == TSM_F32) return rag ? gen_launch<float, false, true>(a, s) : gen_launch<float, false, false>(a, s);
    return rag ? gen_launch<bf16_t, false, true>(a, s) : gen_launch<bf16_t, false, false>(a, s);
}

int gen_conv_dgrad(const ConvP& p, int dtype, const void* dy, const void* wd, void* dx, const void* addend, hipStream_t s) {
    if (p.rows_in() == 0) return TSM_OK;
    if (ksplit_use(p, dtype, true)) return ksplit_dgrad(p, dtype, dy, wd, dx, addend, 1, nullptr, s);
    GenArgs a;
    gen_common(a, p);
    a.src = dy; a.wp = wd; a.dst = dx; a.addend = addend;
    a.Hs = p.Ho; a.Ws = p.Wo; a.Cs = p.Cout; a.CsP = pad_vec(p.Cout, dtype);
    a.Hd = p.H; a.Wd = p.W; a.Cd = p.Cin;
    a.padh = p.KH - 1 - p.pad; a.padw = p.KW - 1 - p.pad;
    a.Kp = p.taps() * a.CsP;
    const bool rag = a.CsP != a.Cs;
    if (dtype == TSM_F32) return rag ? gen_launch<float, true, true>(a, s) : gen_launch<float, true, false>(a, s);
    return rag ? gen_launch<bf16_t, true, true>(a, s) : gen_launch<bf16_t, true, false>(a, s);
}

template <typename T, bool RAG>
static int gen_wgrad_launch(GenWgradArgs& a, hipStream_t s) {
    const long cus = cu_count();
    // Large tiles are 128 x 128, and 64 x 128 where fp32 is loaded element by element: addresses and operands of the square one do
    // not fit the registers then.  Those layers take the small tile where it leaves a block fewer than eight steps.  Us with 128 x
    // 128, 64 x 128, 64 x 64: 3136 pixels 33 -> 65 3x3 51.9, 34.7, 20.6, 12544 130 -> 70 3x3 104, 77.0, 87.9, 25088 127 -> 255 3x3 257,
    // 218, 282, 392 255 -> 513 1x1 53, 32.1, 18.5; around the line 392 511 -> 257 3x3 (9 steps) 57, 40.6, 42.1, 12544 3 -> 67 7x7 (6
    // steps) 53, 39.5, 30.5.  (No more than 64 results: 25088 63 -> 61 3x3 62.9 with 64 x 128, 55.7.)  The longest pay for the smaller tile's
    // loads: 4704 1512 -> 426 3x3 1109 with fp32 instructions on 128 x 128, 1228 with 64 x 128, 25088 127 -> 255 221, 219.
    constexpr bool TALL = sizeof(T) == 4 && RAG;
    const long small_tiles = (long)cdiv(a.Cout, 64) * cdiv(a.K, 64);
    const bool big = a.Cout > 64 && a.K > 64 && (!TALL || small_tiles * a.M >= 8L * GPX * 2 * cus);
    const int bco = big && !TALL ? 128 : 64, bci = big ? 128 : 64;
    a.col_tiles = cdiv(a.K, bci);
    const long tiles = (long)cdiv(a.Cout, bco) * a.col_tiles;
    // one round of blocks, eight wavefronts per CU, and at least eight steps per block against the atomics of its tile.  Two groups
    // per block with the small tile for layers of a few steps (3136 pixels 64 -> 64 3x3 fp32 15.3 and 12.0 us, but 100352 pixels
    // 108 and 116), and with the large one in bf16 where they leave no more CUs without one than single groups do (25600 pixels
    // 312 -> 312 3x3, 66 tiles: 140 and 157) and at most 150 steps per block share the atomics' time among them (us with one and with two:
    // 50176 pixels 72 -> 200 3x3, 37 steps, 66, 57, 200704, 149 steps, 169, 170, 200704 96 -> 520 3x3, 448 steps, 438, 456, 37632 288 -> 1408
    // 3x3, 588 steps, 585, 614).  Large fp32 layers run beside data gradients, which find room between small
    // blocks: alone 80 and 71 us (figures above), in the step at 4 clips 10.43 and 10.76 ms.
    // Layers loaded element by element wait for their loads, which eight wavefronts at one barrier do together: beyond four tiles and
    // ten steps they take two groups only where the tiles that read one stretch of pixels then spread over fewer XCDs (blocks go to the XCDs in
    // turn, so over 8 / gcd(8, blocks per tile)) and find it in their L2.  Us with one and with two, blocks per tile:  140 -> 140 3x3
    // 6272 pixels (9 steps) 65, 60, 12544 106, 120, 200704 1475, 1778 (23, 11); 28 -> 430 3x3 12544 70, 66, 50176 233, 248, 200704 852,
    // 946 (42, 21); 526 -> 238 3x3 50176 1390, 1515 (6, 3); 250 -> 250 3x3 50176 622, 641 (14, 7); but 130 -> 256 3x3 50176 285, 266 (25,
    // 12), 100 -> 300 3x3 50176 448, 432 (21, 10), 200704 1753, 1692, 36 -> 200 3x3 50176 114, 98 (85, 42); two to four tiles: 20 -> 100 3x3
    // 200704 172, 158, 70 -> 330 1x1 243, 231, 200 -> 250 1x1 218, 209.
    auto splits = [&](long slots) { return std::max(1L, slots / tiles); };
    auto filled = [&](long slots) { const long n = splits(slots) * tiles; return (double)n / (double)((n + slots - 1) / slots * slots); };
    auto together = [&](long slots) { const long n = splits(slots); return std::min(8L, n & -n); };
    const long steps = cdiv(a.M, GPX * splits(2 * cus));
    const bool beside = RAG ? tiles <= 4 || steps <= 10 || together(cus) > together(2 * cus) : steps <= 150;
    const bool two = big ? sizeof(T) == 2 && beside && filled(cus) >= 0.95 * filled(2 * cus) : a.M <= 8L * GPX * splits(2 * cus);
    const long want = splits(two ? cus : 2 * cus), unit = two ? 2L * GPX : (long)GPX;
    a.chunk = (std::max((a.M + want - 1) / want, 8L * GPX) + unit - 1) / unit * unit;
    const dim3 grid((unsigned)((a.M + a.chunk - 1) / a.chunk), (unsigned)tiles), block(two ? 512 : 256);
    if constexpr (sizeof(T) == 2)
        if (big && two) gen_wgrad_kernel<T, 128, 128, 2, 2, 2, RAG><<<grid, block, 0, s>>>(a);
    if (big && !two) gen_wgrad_kernel<T, TALL ? 64 : 128, 128, 2, 2, 1, RAG><<<grid, block, 0, s>>>(a);
    if (!big && two) gen_wgrad_kernel<T, 64, 64, 2, 2, 2, RAG><<<grid, block, 0, s>>>(a);
    if (!big && !two) gen_wgrad_kernel<T, 64, 64, 2, 2, 1, RAG><<<grid, block, 0, s>>>(a);
    return check_launch(sizeof(T) == 4 ? "gen_wgrad_f32" : "gen_wgrad_bf16");
}

// dw is added to; packed: [Cout][taps][Cin], otherwise the ABI order [Cout][Cin][taps].
int gen_conv_wgrad(const ConvP& p, int dtype, const void* x, const void* dy, float* dw, bool packed, hipStream_t s) {
    if (p.rows_out() == 0) return TSM_OK;
    GenWgradArgs a;
    a.x = x; a.dy = dy; a.dw = dw;
    a.so = (long)p.K(); a.si = packed ? 1 : p.taps(); a.st = packed ? p.Cin : 1;
    a.F = p.F; a.T = p.T; a.H = p.H; a.W = p.W; a.Cin = p.Cin; a.CinP = pad_vec(p.Cin, dtype);
    a.Ho = p.Ho; a.Wo = p.Wo; a.Cout = p.Cout;
    a.KT = p.KT; a.KH = p.KH; a.KW = p.KW; a.stride = p.stride; a.pad = p.pad; a.fold = p.fold;
    a.shifted = p.shifted; a.inside_only = dtype == TSM_F32 || !mfma_conv_supported(p);
    a.M = p.rows_out();
    a.K = p.taps() * a.CinP;
    const int ve = dtype == TSM_F32 ? 4 : 8;
    // (a buffer load's offset stays below 2 GiB)
    const long es = (long)dtype_size(dtype), limit = 0x7ff00000L;
    const long edge = std::max(2 * ((long)p.KH * p.W + p.KW), (long)p.pad * p.W + p.pad) * p.Cin * es;   // taps behind the last pixel, padding before the first
    const bool rag = p.Cin % ve || p.Cout % ve || p.fold % ve || p.rows_in() * p.Cin * es + edge >= limit || p.rows_out() * p.Cout * es >= limit;
    if (dtype == TSM_F32) return rag ? gen_wgrad_launch<float, true>(a, s) : gen_wgrad_launch<float, false>(a, s);
    return rag ? gen_wgrad_launch<bf16_t, true>(a, s) : gen_wgrad_launch<bf16_t, false>(a, s);
}

}  // namespace tsm
