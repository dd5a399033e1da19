// Implicit-GEMM convolutions whose K range is split over the wavefronts of a block: small problems in either storage
// type, and fp32 storage at every size.
//
// What bounds them elsewhere: a layer with fewer output tiles than the chip has CUs is one long chain of K steps per tile,
// each a gather, a barrier and a few MFMAs, and a CU fetches no faster than about 30 B/clk for it (392 x 4608 -> 512 on
// 64 CUs: 39 us, 0.5 us per step of 64).  Here the wavefronts of a block take every KS-th chunk of 128 bytes of K each,
// with LDS of their own, so that no barrier stands in the loop and eight chunks are in flight per CU; their partial tiles
// meet in LDS once at the end (fp32, added in a fixed order).  One tile per block, no persistence: what fills the chip at
// small sizes is tiles of 32 or 64 rows.  fp32 layers run here at every size; their products are six bf16 products each
// (split_f32.h), which a wavefront cuts its operands for as it reads them out of LDS: 6.5 vector instructions per value, as long as
// the matrix instructions they feed, is what bounds them then (us with the fp32 instructions, which bound them at 140 TFLOP/s, and
// now: 100352 x 576 -> 64 97 and 84, 25088 x 1152 -> 128 87 and 76, 6272 x 2304 -> 256 85 and 73 = 102 TFLOP/s, 1568 x 4608 -> 512
// 85 and 71; 7 to 9 % of it for the comparison that finds operands which cannot be cut).  Two chunks in flight per wavefront instead of one change nothing on the small layers: bytes per CU, not
// latency, are what is left (392 x 4608 -> 512 in 32 x 32 tiles reads 590 KB per CU).
#include <stdlib.h>
#include <algorithm>
#include "internal.h"
#include "taps_inside.h"
#include "split_f32.h"

namespace tsm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

static constexpr uint32_t OOB = 0x80000000u;   // beyond every buffer: a load there returns zeros

struct KsArgs {
    const void* src;       // x (fwd) or dy (dgrad), channels innermost
    const void* wp;        // packed weights [Cd][taps][Cs]
    void* dst;
    const void* addend;    // dgrad: added to dx (nullable); add_stride 2: compact form, see IgemmArgs in conv_mfma.hip
    int add_stride, add_ho, add_wo;
    float* stats;          // [mtiles][2*Cd]: one row per pixel tile (fwd: sums of y and y^2; dgrad: BatchNorm-backward sums)
    const void* act;       // dgrad: ReLU mask source, BatchNorm input and statistics (nullable), as in IgemmArgs
    const void* ybn;
    const float* bn_mean;
    const float* bn_rstd;
    const uint8_t* act_bits;
    const float* ep_scale; // fwd, bf16: affine epilogue (nullable), as in IgemmArgs
    const float* ep_shift;
    const void* ep_res;
    int ep_relu;
    int F, T;
    int Hs, Ws, Cs;
    int Hd, Wd, Cd;
    int KT, KH, KW;
    int stride, padh, padw;
    int fold;              // fwd: shift of source channels; dgrad: adjoint shift of destination channels
    int shifted;           // fwd: fold of a source that is S(x) already
    int inside_only;       // taps outside add nothing whatever they are multiplied with (see taps_inside.h)
    uint32_t wrow;         // bytes of one weight row
    uint32_t src_bytes, w_bytes, bias_bytes;
    int ntiles, mtiles, by_n;
    // parity classes of destination pixels (see IgemmArgs)
    int ncls, cstep;
    int ph[4], pw[4], hc[4], wc[4], mt0[5];
    int a0h[4], nth[4], a0w[4], ntw[4];
};

__device__ __forceinline__ int ks_group_dt(int c, int fold) { return c < fold ? 1 : (c < 2 * fold ? -1 : 0); }
__device__ __forceinline__ __amdgpu_buffer_rsrc_t ks_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)bytes, 0x00020000);
}
// Orders the LDS accesses of one wavefront, which the LDS serves in program order, for the compiler.
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

struct KsRow {
    uint32_t off;    // byte offset of the row's tap origin in the biased buffer
    uint32_t mask;   // bits 0..7 / 8..15: tap rows / columns inside the frame; 30 / 31: frame t+1 / t-1 in the clip
    int dst;         // destination row, -1 beyond the last one
    int arow;        // row of a compact addend, -1: none
};

// 16-byte vector of T <-> floats
template <typename T> __device__ __forceinline__ void unpack(const u32x4& v, float* f) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if constexpr (sizeof(T) == 2) {
            f[2 * q] = __uint_as_float(v[q] << 16);
            f[2 * q + 1] = __uint_as_float(v[q] & 0xffff0000u);
        } else {
            f[q] = __uint_as_float(v[q]);
        }
    }
}
template <typename T> __device__ __forceinline__ u32x4 pack(const float* f) {
    u32x4 v;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if constexpr (sizeof(T) == 2) v[q] = pack_bf16x2(f[2 * q], f[2 * q + 1]);
        else v[q] = __float_as_uint(f[q]);
    }
    return v;
}

// One tile of 32*MI pixels x 32*NJ channels per block; wavefront w multiplies the K chunks (128 bytes of every tile row)
// w, w + KS, w + 2*KS, ... of it.  RAG: source channels that are no multiple of a chunk (they are one of the vector), and bf16
// layers with inside_only.
template <typename T, int MI, int NJ, int KS, bool DGRAD, bool RAG>
__global__ void __launch_bounds__(KS * 64, MI * NJ == 1 ? 4 : 2) ksplit_kernel(KsArgs a) {
    constexpr int NT = KS * 64;
    constexpr int TM = 32 * MI, TN = 32 * NJ;
    constexpr int ES = (int)sizeof(T), VE = 16 / ES, KE = 128 / ES;
    constexpr int STAGE = (TM + TN) * 128;          // bytes per wavefront
    constexpr int PA = TM / 8, PB = TN / 8;         // 16-byte pieces per lane and chunk
    constexpr int SL = TN / 4;                      // 16-byte slots per row of a partial tile
    constexpr bool CHECK = ES == 4 || RAG;          // takes layers with inside_only
    static_assert(TM * TN * 4 <= STAGE, "a partial tile takes the place of its wavefront's operands");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    KsRow* s_row = (KsRow*)(smem + KS * STAGE);
    float* s_part = (float*)(s_row + TM);           // [2][KS][TN]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // workgroups go to the eight XCDs round-robin by index: each XCD gets a contiguous eighth of the tiles, enumerated so
    // that those which read the same pixels, or those which read the same weights, whichever operand is the larger, are
    // neighbours and find it in their L2
    // (with several parity classes, whose tiles differ in length, an XCD takes every eighth pixel tile instead)
    const int g8 = (int)blockIdx.x >> 3, x8 = (int)blockIdx.x & 7;
    const int id = x8 * ((int)gridDim.x >> 3) + g8;
    const int mt = a.ncls > 1 ? g8 / a.ntiles * 8 + x8 : a.by_n ? id % a.mtiles : id / a.ntiles;
    const int nt = a.ncls > 1 ? g8 % a.ntiles : a.by_n ? id / a.mtiles : id % a.ntiles;
    if (mt >= a.mtiles || nt >= a.ntiles) return;
    const int n0 = nt * TN;
    int cls = 0;
    while (cls + 1 < a.ncls && mt >= a.mt0[cls + 1]) ++cls;
    const int nth = a.nth[cls], ntw = a.ntw[cls], ntaps = a.KT * nth * ntw;
    const int hw_d = a.Hd * a.Wd;
    const int frame_bytes = a.Hs * a.Ws * a.Cs * ES;

    if (tid < TM) {
        const int hc = a.hc[cls], wc = a.wc[cls];
        const unsigned m = (unsigned)(mt - a.mt0[cls]) * TM + tid;
        KsRow r;
        r.off = 0; r.mask = 0; r.dst = -1; r.arow = -1;
        if (m < (unsigned)a.F * (unsigned)(hc * wc)) {
            const int f = (int)(m / (unsigned)(hc * wc));
            const int q = (int)(m - (unsigned)f * (unsigned)(hc * wc));
            const int qh = (int)((unsigned)q / (unsigned)wc), qw = q - qh * wc;
            const int dh = qh * a.cstep + a.ph[cls], dw = qw * a.cstep + a.pw[cls];
            const int sh = a.cstep == 2 ? 1 : 0;    // (divides the numerators exactly, negative ones included)
            const int oh = DGRAD ? (dh - a.padh + a.a0h[cls]) >> sh : dh * a.stride - a.padh;
            const int ow = DGRAD ? (dw - a.padw + a.a0w[cls]) >> sh : dw * a.stride - a.padw;
            const int t = f % a.T;
            for (int th = 0; th < nth; ++th)
                if (oh + th >= 0 && oh + th < a.Hs) r.mask |= 1u << th;
            for (int tw = 0; tw < ntw; ++tw)
                if (ow + tw >= 0 && ow + tw < a.Ws) r.mask |= 1u << (8 + tw);
            if (t + 1 < a.T) r.mask |= 1u << 30;
            if (t >= 1) r.mask |= 1u << 31;
            r.off = (uint32_t)(((long)f * a.Hs * a.Ws + (long)oh * a.Ws + ow) * a.Cs * ES + a.bias_bytes);
            r.dst = (f * a.Hd + dh) * a.Wd + dw;
            if (DGRAD && a.add_stride == 2 && ((dh | dw) & 1) == 0) r.arow = (f * a.add_ho + (dh >> 1)) * a.add_wo + (dw >> 1);
        }
        s_row[tid] = r;
    }
    __syncthreads();

    // Operands: 8 lanes fetch the 128 bytes of a row, the row of piece i is 2*(lane/8) + i%2 + 16*(i/2).  Position p of
    // row r in LDS holds its vector p ^ ((r/2) % 8): the fragment reads of 16 consecutive rows hit different banks, and
    // all pieces of a lane carry the same vector of the chunk.
    const __amdgpu_buffer_rsrc_t ra = ks_rsrc((const char*)a.src - a.bias_bytes, a.src_bytes + a.bias_bytes);
    const __amdgpu_buffer_rsrc_t rb = ks_rsrc(a.wp, a.w_bytes);
    const int lr = lane >> 3, kvec = (lane & 7) ^ lr;
    uint32_t aoff[PA], amask[PA], boff[PB];
#pragma unroll
    for (int i = 0; i < PA; ++i) {
        const KsRow r = s_row[2 * lr + (i & 1) + 16 * (i >> 1)];
        aoff[i] = r.off + (RAG ? 0 : kvec * 16);
        amask[i] = r.mask;
    }
#pragma unroll
    for (int j = 0; j < PB; ++j) {
        const int n = n0 + 2 * lr + (j & 1) + 16 * (j >> 1);
        boff[j] = n < a.Cd ? (uint32_t)n * a.wrow + (RAG ? 0 : kvec * 16) : OOB;
    }

    const int nch = RAG ? (ntaps * a.Cs + KE - 1) / KE : ntaps * (a.Cs / KE);
    const int cpt = RAG ? 1 : a.Cs / KE;            // chunks per tap
    u32x4 areg[PA], breg[PB];
    // position of the next chunk to fetch (not RAG): tap and chunk of the tap
    int kt = 0, th = 0, tw = 0, cb = wave;
    auto wrap = [&]() {
        while (cb >= cpt) {
            cb -= cpt;
            if (++tw >= ntw) { tw = 0; if (++th >= nth) { th = 0; ++kt; } }
        }
    };
    if (!RAG && wave < nch) wrap();
    auto load = [&](int q) {
        if constexpr (RAG) {
            const unsigned e = (unsigned)(q * 8 + kvec) * VE;          // first element of the lane's vector in the K range
            const unsigned tap = e / (unsigned)a.Cs;
            const int ch = (int)(e - tap * (unsigned)a.Cs);
            const bool ok = (int)tap < ntaps;
            const int w_ = (int)(tap % (unsigned)ntw), hk = (int)(tap / (unsigned)ntw);
            const int h_ = (int)((unsigned)hk % (unsigned)nth), k_ = (int)((unsigned)hk / (unsigned)nth);
            const int d = k_ - a.KT / 2 + (DGRAD ? 0 : ks_group_dt(ch, a.fold));
            const uint32_t need = (1u << h_) | (1u << (8 + w_)) | (d > 0 ? 1u << 30 : 0u) | (d < 0 ? 1u << 31 : 0u);
            const uint32_t va = (uint32_t)(((h_ * a.Ws + w_) * a.Cs + ch) * ES + d * frame_bytes);
            const uint32_t vb = (uint32_t)((((k_ * a.KH + a.a0h[cls] + h_ * a.cstep) * a.KW + a.a0w[cls] + w_ * a.cstep) * a.Cs + ch) * ES);
#pragma unroll
            for (int i = 0; i < PA; ++i)
                areg[i] = __builtin_amdgcn_raw_buffer_load_b128(ra, (int)((ok && (amask[i] & need) == need) ? aoff[i] + va : OOB), 0, 0);
#pragma unroll
            for (int j = 0; j < PB; ++j) breg[j] = __builtin_amdgcn_raw_buffer_load_b128(rb, (int)((ok && boff[j] != OOB) ? boff[j] + vb : OOB), 0, 0);
        } else {
            const int chb = cb * KE;
            const int d0 = kt - a.KT / 2;
            const int d = d0 + ((!DGRAD && chb < 2 * a.fold) ? ks_group_dt(chb + kvec * VE, a.fold) : 0);
            const uint32_t need = (1u << th) | (1u << (8 + tw)) | (d > 0 ? 1u << 30 : 0u) | (d < 0 ? 1u << 31 : 0u);
            const uint32_t dl = (uint32_t)(d * frame_bytes);
            const int sa = ((th * a.Ws + tw) * a.Cs + chb) * ES;
            const int sb = (((kt * a.KH + a.a0h[cls] + th * a.cstep) * a.KW + a.a0w[cls] + tw * a.cstep) * a.Cs + chb) * ES;
#pragma unroll
            for (int i = 0; i < PA; ++i)
                areg[i] = __builtin_amdgcn_raw_buffer_load_b128(ra, (int)((amask[i] & need) == need ? aoff[i] + dl : OOB), sa, 0);
#pragma unroll
            for (int j = 0; j < PB; ++j) breg[j] = __builtin_amdgcn_raw_buffer_load_b128(rb, (int)boff[j], sb, 0);
            cb += KS;
            wrap();
        }
    };

    f32x16 acc[ES == 2 ? MI : 1][ES == 2 ? NJ : 1];         // bf16: blocks of 32 x 32
    f32x4 sums[ES == 4 ? 2 * MI : 1][ES == 4 ? 2 * NJ : 1];   // fp32: of 16 x 16
    if constexpr (ES == 2) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    } else {
#pragma unroll
        for (int i = 0; i < 2 * MI; ++i)
#pragma unroll
            for (int j = 0; j < 2 * NJ; ++j) sums[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    unsigned char* const st = smem + wave * STAGE;
    auto stage = [&]() {
        const int wr = lr * 256 + (lane & 7) * 16;
#pragma unroll
        for (int i = 0; i < PA; ++i) *(u32x4*)(st + wr + (i & 1) * 128 + (i >> 1) * 2048) = areg[i];
#pragma unroll
        for (int j = 0; j < PB; ++j) *(u32x4*)(st + TM * 128 + wr + (j & 1) * 128 + (j >> 1) * 2048) = breg[j];
    };
    bool lossy = false;    // fp32: an operand whose parts do not hold it, or a sum beyond the range (see split_f32.h)
    if (wave < nch) {
        load(wave);
        for (int q = wave; q < nch; q += KS) {
            stage();
            wave_lds_order();
            if (q + KS < nch) load(q + KS);
            if constexpr (ES == 2) {
                const int r = lane & 31, hi = lane >> 5, sw = (r >> 1) & 7;
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    const int pos = ((2 * ks + hi) ^ sw) * 16;
                    u32x4 af[MI], bf[NJ];
#pragma unroll
                    for (int i = 0; i < MI; ++i) af[i] = *(const u32x4*)(st + (i * 32 + r) * 128 + pos);
#pragma unroll
                    for (int j = 0; j < NJ; ++j) bf[j] = *(const u32x4*)(st + (TM + j * 32 + r) * 128 + pos);
                    // (result blocks are [channel][pixel]: a lane holds four consecutive channels of one pixel per quad)
#pragma unroll
                    for (int i = 0; i < MI; ++i)
#pragma unroll
                        for (int j = 0; j < NJ; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, bf[j]), __builtin_bit_cast(bf16x8, af[i]), acc[i][j], 0, 0, 0);
                }
            } else {
                // two vectors of a row, four apart, are the eight values a lane supplies to 32 products (both operands alike)
                const int r = lane & 15, g = lane >> 4;
                auto frag = [&](int row, bool negate) {
                    const int sw = (row >> 1) & 7;
                    const f32x4 u = *(const f32x4*)(st + row * 128 + (g ^ sw) * 16), v = *(const f32x4*)(st + row * 128 + ((g + 4) ^ sw) * 16);
                    const float f[8] = {u[0], u[1], u[2], u[3], v[0], v[1], v[2], v[3]};
                    return split3(f, lossy, negate);
                };
                Split3 bf[2 * NJ];
#pragma unroll
                for (int j = 0; j < 2 * NJ; ++j) bf[j] = frag(TM + j * 16 + r, false);
#pragma unroll
                for (int i = 0; i < 2 * MI; ++i) mma_split<2 * NJ>(bf, frag(i * 16 + r, (i & 1) != 0), sums[i]);
            }
            wave_lds_order();
            if constexpr (ES == 4) if (__builtin_expect(__any(lossy), 0)) break;
        }
        if constexpr (ES == 4) {
            // The matrix core's sums lean towards minus infinity.  Every other 16 pixels are the sums of -x, so that what is added up
            // over pixels later (BatchNorm's sums, weight gradients) does not lean with them.
#pragma unroll
            for (int i = 1; i < 2 * MI; i += 2)
#pragma unroll
                for (int j = 0; j < 2 * NJ; ++j) sums[i][j] = -sums[i][j];
            lossy |= split_overflow(sums);   // (an instruction per two sums: tiles of one or two chunks per wavefront notice four)
        }
    }
    const int nact = nch < KS ? nch : KS;
    // the wavefront's partial tile, rows of SL 16-byte slots, slot s of row r at position s ^ (r % SL)
    auto put = [&](int row, int slot, const f32x4& v) { *(f32x4*)(st + row * (TN * 4) + ((slot ^ (row & (SL - 1))) * 16)) = v; };
    auto put_tile = [&]() {
        if constexpr (ES == 2) {
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        put(i * 32 + (lane & 31), j * 8 + 2 * q + (lane >> 5), f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]});
        } else {
#pragma unroll
            for (int i = 0; i < 2 * MI; ++i)
#pragma unroll
                for (int j = 0; j < 2 * NJ; ++j) put(i * 16 + (lane & 15), j * 4 + (lane >> 4), sums[i][j]);
        }
    };
    if (wave < nact) {
        put_tile();
        // Such a tile is formed again by fp32 instructions.  Behind the store, where the loop above, which has no register to
        // spare, shares nothing with it: inside the loop it costs spills.
        if constexpr (ES == 4) if (__builtin_expect(__any(lossy), 0)) {
            wave_lds_order();
#pragma unroll
            for (int i = 0; i < 2 * MI; ++i)
#pragma unroll
                for (int j = 0; j < 2 * NJ; ++j) sums[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            kt = th = tw = 0;
            cb = wave;
            if (!RAG) wrap();
            load(wave);
            for (int q = wave; q < nch; q += KS) {
                stage();
                wave_lds_order();
                if (q + KS < nch) load(q + KS);
                const int r = lane & 15, g = lane >> 4;
                auto value = [&](int row, int e) { return *(const float*)(st + row * 128 + ((g + (e & 4)) ^ ((row >> 1) & 7)) * 16 + (e & 3) * 4); };
#pragma unroll
                for (int i = 0; i < 2 * MI; ++i)
                    mma_exact<2 * NJ>([&](int j, int e) { return value(TM + j * 16 + r, e); }, [&](int, int e) { return value(i * 16 + r, e); }, sums[i]);
                wave_lds_order();
            }
            put_tile();
        }
    }

    // ---- epilogue: thread = CV-th vector of VE channels of every (NT/CV)-th row
    constexpr int CV = TN / VE, NV = (TM * CV + NT - 1) / NT, RPS = NT / CV;
    static_assert(NV == 1 || TM * CV % NT == 0, "tile / thread mismatch");
    const int vcol = tid % CV, r0 = (tid / CV) % TM, col = n0 + vcol * VE;
    const bool colok = col < a.Cd && tid / CV < TM;      // (small tiles have fewer vectors than threads)
    const bool fuse_mask = DGRAD && (a.act_bits != nullptr || a.act != nullptr);
    const bool fuse_bn = fuse_mask && a.ybn != nullptr;
    const bool affine = !DGRAD && ES == 2 && a.ep_scale != nullptr;
    const int dt = DGRAD ? ks_group_dt(col, a.fold) : 0;
    const bool straddle = DGRAD && ks_group_dt(col + VE - 1, a.fold) != dt;
    // what the epilogue reads is requested before the partial tiles are exchanged; rows that are not stored read zeros
    long mr[NV], mz[NV];
    u32x4 ad[NV], ac[NV], yy[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const KsRow r = s_row[v * RPS + r0];
        const bool live = r.dst >= 0 && colok;
        const u32x4 zero = {0u, 0u, 0u, 0u};
        ad[v] = ac[v] = yy[v] = zero;
        mz[v] = -1;
        if (!DGRAD) {
            mr[v] = live ? r.dst : -1;
            if (affine && a.ep_res && live) ad[v] = *(const u32x4*)((const T*)a.ep_res + (long)r.dst * a.Cd + col);
        } else {
            const bool next = (r.mask >> 30) & 1u, prev = r.mask >> 31;
            const bool in_clip = dt == 0 || (dt > 0 ? next : prev);
            mr[v] = live && in_clip && !straddle ? (long)r.dst + (long)dt * hw_d : -1;
            mz[v] = live && !straddle && dt != 0 && !(dt > 0 ? prev : next) ? r.dst : -1;
            if (mr[v] >= 0) {
                const long e = mr[v] * a.Cd + col;
                if (a.addend) {
                    if (a.add_stride == 2) {
                        if (r.arow >= 0) ad[v] = *(const u32x4*)((const T*)a.addend + ((long)r.arow + (long)dt * (a.add_ho * a.add_wo)) * a.Cd + col);
                    } else {
                        ad[v] = *(const u32x4*)((const T*)a.addend + e);
                    }
                }
                if (fuse_mask) {
                    if (a.act_bits) ac[v][0] = a.act_bits[e / 8];
                    else ac[v] = *(const u32x4*)((const T*)a.act + e);
                }
                if (fuse_bn) yy[v] = *(const u32x4*)((const T*)a.ybn + e);
            }
        }
    }
    float mu[VE], rs[VE], f1[VE], f2[VE];
#pragma unroll
    for (int q = 0; q < VE; ++q) {
        f1[q] = f2[q] = 0.f;
        mu[q] = rs[q] = 0.f;
        if ((fuse_bn || affine) && colok) {
            mu[q] = DGRAD ? a.bn_mean[col + q] : a.ep_scale[col + q];
            rs[q] = DGRAD ? a.bn_rstd[col + q] : a.ep_shift[col + q];
        }
    }
    __syncthreads();
    auto add_up = [&](int v, float* f) {
        const int row = v * RPS + r0;
#pragma unroll
        for (int q = 0; q < VE; ++q) f[q] = 0.f;
        for (int w = 0; w < nact; ++w) {
            const unsigned char* p = smem + w * STAGE + row * (TN * 4);
#pragma unroll
            for (int h = 0; h < VE / 4; ++h) {
                const f32x4 x = *(const f32x4*)(p + (((vcol * (VE / 4) + h) ^ (row & (SL - 1))) * 16));
#pragma unroll
                for (int q = 0; q < 4; ++q) f[4 * h + q] += x[q];
            }
        }
    };
    float sum[CHECK ? NV : 1][VE];
    if constexpr (CHECK) {
#pragma unroll
        for (int v = 0; v < NV; ++v) add_up(v, sum[v]);
    }
    if constexpr (CHECK) if (a.inside_only && colok) {
        uint32_t nan = 0;
        static_assert(NV * VE <= 32, "one bit each");
#pragma unroll
        for (int e = 0; e < NV * VE; e += 2)
            if (__builtin_isunordered(sum[e / VE][e % VE], sum[e / VE][e % VE + 1])) nan |= 3u << e;
        while (__builtin_expect(nan != 0, 0)) {
            const int at = __ffs((int)nan) - 1, c = col + at % VE;
            nan &= nan - 1;
            const KsRow r = s_row[at / VE * RPS + r0];
            if (r.dst < 0) continue;
            const float f = sum_taps_inside<T, DGRAD>(a, cls, (const T*)((const char*)a.src + ((long)r.off - (long)a.bias_bytes)), r.mask,
                                                      (const T*)((const char*)a.wp + (size_t)c * a.wrow), a.Cs);
#pragma unroll
            for (int e = 0; e < NV * VE; ++e) sum[e / VE][e % VE] = e == at ? f : sum[e / VE][e % VE];
        }
    }
    T* const dst = (T*)a.dst;
    // value (rounded once) -> addend -> ReLU mask and BatchNorm sums -> store
    auto finish = [&](long m, float* f, const u32x4& adv, const u32x4& acv, const u32x4& yyv) {
        if (a.addend) {
            float g[VE];
            unpack<T>(adv, g);
#pragma unroll
            for (int q = 0; q < VE; ++q) f[q] += g[q];
            const u32x4 o = pack<T>(f);
            unpack<T>(o, f);
        }
        if (fuse_mask) {
            float m_[VE], y_[VE];
            unpack<T>(acv, m_);
            unpack<T>(yyv, y_);
#pragma unroll
            for (int q = 0; q < VE; ++q) {
                const bool on = a.act_bits ? ((acv[0] >> q) & 1u) != 0 : m_[q] > 0.f;
                f[q] = on ? f[q] : 0.f;
                f1[q] += f[q];
                f2[q] = fmaf(f[q], (y_[q] - mu[q]) * rs[q], f2[q]);
            }
        }
        *(u32x4*)(dst + m * a.Cd + col) = pack<T>(f);
    };
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const int row = v * RPS + r0;
        float f[VE];
        if constexpr (CHECK) {
            unpack<T>(pack<T>(sum[v]), f);
        } else {
            add_up(v, f);
            const u32x4 o = pack<T>(f);
            unpack<T>(o, f);
        }
        if constexpr (!DGRAD) {
            if (mr[v] < 0) continue;
            if (a.stats) {
#pragma unroll
                for (int q = 0; q < VE; ++q) {
                    f1[q] += f[q];
                    f2[q] = fmaf(f[q], f[q], f2[q]);
                }
            }
            if (affine) {
                float g[VE];
                unpack<T>(ad[v], g);
#pragma unroll
                for (int q = 0; q < VE; ++q) {
                    f[q] = fmaf(f[q], mu[q], rs[q]) + g[q];
                    if (a.ep_relu) f[q] = f[q] > 0.f ? f[q] : 0.f;
                }
            }
            *(u32x4*)(dst + mr[v] * a.Cd + col) = pack<T>(f);
        } else {
            if (mz[v] >= 0) {   // the frame that receives nothing from inside the clip
                const long e = mz[v] * a.Cd + col;
                u32x4 zad = {0u, 0u, 0u, 0u}, zac = zad, zyy = zad;
                if (a.addend) {
                    if (a.add_stride == 2) {
                        const int arow = s_row[row].arow;
                        if (arow >= 0) zad = *(const u32x4*)((const T*)a.addend + (long)arow * a.Cd + col);
                    } else {
                        zad = *(const u32x4*)((const T*)a.addend + e);
                    }
                }
                if (fuse_mask) {
                    if (a.act_bits) zac[0] = a.act_bits[e / 8];
                    else zac = *(const u32x4*)((const T*)a.act + e);
                }
                if (fuse_bn) zyy = *(const u32x4*)((const T*)a.ybn + e);
                float z[VE];
#pragma unroll
                for (int q = 0; q < VE; ++q) z[q] = 0.f;
                finish(mz[v], z, zad, zac, zyy);
            }
            if (mr[v] >= 0) finish(mr[v], f, ad[v], ac[v], yy[v]);
            if (straddle && colok && s_row[row].dst >= 0) {   // (dense addend, no mask: checked on the host)
                const KsRow r = s_row[row];
                const bool next = (r.mask >> 30) & 1u, prev = r.mask >> 31;
#pragma unroll
                for (int q = 0; q < VE; ++q) {
                    const int d = ks_group_dt(col + q, a.fold);
                    auto put = [&](long m, float val) {
                        const long at = m * a.Cd + col + q;
                        if (a.addend) val += Elem<T>::ld(((const T*)a.addend)[at]);
                        dst[at] = Elem<T>::st(val);
                    };
                    if (d == 0 || (d > 0 ? next : prev)) put((long)r.dst + (long)d * hw_d, f[q]);
                    if (d != 0 && !(d > 0 ? prev : next)) put(r.dst, 0.f);
                }
            }
        }
    }
    if (a.stats) {   // lanes CV apart hold the same channels; one slot per wavefront, added in a fixed order
#pragma unroll
        for (int q = 0; q < VE; ++q) {
#pragma unroll
            for (int off = CV; off < 64; off <<= 1) {
                f1[q] += __shfl_xor(f1[q], off);
                f2[q] += __shfl_xor(f2[q], off);
            }
        }
        if (lane < CV) {
#pragma unroll
            for (int q = 0; q < VE; ++q) {
                s_part[wave * TN + lane * VE + q] = f1[q];
                s_part[(KS + wave) * TN + lane * VE + q] = f2[q];
            }
        }
        __syncthreads();
        for (int i = tid; i < 2 * TN; i += NT) {
            const int stat = i / TN, c = i % TN;
            float v = 0.f;
#pragma unroll
            for (int w = 0; w < KS; ++w) v += s_part[(stat * KS + w) * TN + c];
            if (n0 + c < a.Cd) a.stats[(size_t)mt * 2 * a.Cd + stat * a.Cd + n0 + c] = v;
        }
    }
}

// ---- host side ----------------------------------------------------------------------------------------------------
static int ks_cus() {
    static int n = 0;
    if (n == 0) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess) n = v;
        if (n <= 0) n = 256;
    }
    return n;
}

struct KsTile { int bm, bn, ks; };

// Rows of a direction's destination, per parity class.
static int ks_classes(KsArgs& a, bool dgrad, int BM) {
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
    return a.mt0[a.ncls];
}

static void ks_geometry(KsArgs& a, const ConvP& p, int dtype, bool dgrad) {
    const long es = (long)dtype_size(dtype);
    a.F = p.F; a.T = p.T; a.KT = p.KT; a.KH = p.KH; a.KW = p.KW; a.stride = p.stride; a.fold = p.fold;
    a.shifted = p.shifted; a.inside_only = dtype == TSM_F32 || !mfma_conv_supported(p);
    if (!dgrad) {
        a.Hs = p.H; a.Ws = p.W; a.Cs = p.Cin; a.Hd = p.Ho; a.Wd = p.Wo; a.Cd = p.Cout;
        a.padh = a.padw = p.pad;
    } else {
        a.Hs = p.Ho; a.Ws = p.Wo; a.Cs = p.Cout; a.Hd = p.H; a.Wd = p.W; a.Cd = p.Cin;
        a.padh = p.KH - 1 - p.pad; a.padw = p.KW - 1 - p.pad;
    }
    a.wrow = (uint32_t)(p.taps() * a.Cs * es);
    a.w_bytes = (uint32_t)(a.wrow * (long)a.Cd);
    a.src_bytes = (uint32_t)((long)a.F * a.Hs * a.Ws * a.Cs * es);
    a.bias_bytes = (uint32_t)(((long)std::max(a.padh, 0) * a.Ws + std::max(a.padw, 0)) * a.Cs * es);
}

// Whether the kernel can run a direction of a layer at all.
static bool ks_supported(const ConvP& p, int dtype, bool dgrad) {
    const int ve = dtype == TSM_F32 ? 4 : 8;
    const long es = (long)dtype_size(dtype), limit = 0x7ff00000L;   // 32-bit buffer offsets below OOB
    if (p.pitch && p.pitch != p.Cin) return false;
    if (p.Cin % ve || p.Cout % ve || p.stride > 2 || p.KH > 8 || p.KW > 8) return false;
    if (p.KT > 1 && p.fold > 0) return false;
    if (!dgrad && p.fold % ve) return false;           // a vector's channels come from one frame
    // offsets run from the padding in front of the first pixel (the bias of ks_geometry) to the last tap behind the last one
    const long cs = dgrad ? p.Cout : p.Cin, cd = dgrad ? p.Cin : p.Cout, ws = dgrad ? p.Wo : p.W;
    const long padh = dgrad ? p.KH - 1 - p.pad : p.pad, padw = dgrad ? p.KW - 1 - p.pad : p.pad;
    const long src = (dgrad ? p.rows_out() : p.rows_in()) * cs * es, span = ((long)p.KH * ws + p.KW) * cs * es;
    const long bias = (std::max(padh, 0L) * ws + std::max(padw, 0L)) * cs * es;
    if (src + 2 * span >= limit || src + bias >= limit || (long)p.taps() * cs * cd * es >= limit) return false;
    if (p.rows_in() > 0x3fffffffL || p.rows_out() > 0x3fffffffL) return false;
    return p.rows_in() > 0 && p.rows_out() > 0;
}

template <typename T, int MI, int NJ, int KS, bool DGRAD, bool RAG>
static int ks_launch(KsArgs& a, hipStream_t s) {
    constexpr int TM = 32 * MI, TN = 32 * NJ;
    constexpr size_t smem = (size_t)KS * (TM + TN) * 128 + TM * sizeof(KsRow) + 2 * KS * TN * sizeof(float);
    static_assert(smem <= 160 * 1024, "LDS budget");
    auto kern = ksplit_kernel<T, MI, NJ, KS, DGRAD, RAG>;
    static bool configured = false;
    if (!configured) {
        if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
            return fail(TSM_ERR_LAUNCH, "ksplit: cannot raise dynamic LDS limit");
        configured = true;
    }
    a.mtiles = ks_classes(a, DGRAD, TM);
    a.ntiles = (a.Cd + TN - 1) / TN;
    a.by_n = a.w_bytes > a.src_bytes;
    const long grid = a.ncls > 1 ? (long)(a.mtiles + 7) / 8 * 8 * a.ntiles : ((long)a.mtiles * a.ntiles + 7) / 8 * 8;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(KS * 64), smem, s, a);
    if (sizeof(T) == 4) return check_launch(DGRAD ? "ksplit_dgrad_f32" : "ksplit_fwd_f32");
    return check_launch(DGRAD ? "ksplit_dgrad_bf16" : "ksplit_fwd_bf16");
}

// 64 x 64 tiles of a direction that have something to multiply; *idle: of those that only store zeros or an addend (a strided
// 1x1 layer's data gradient has parity classes without taps).
static long ks_tiles(const ConvP& p, int dtype, bool dgrad, long* idle = nullptr) {
    KsArgs a;
    ks_geometry(a, p, dtype, dgrad);
    ks_classes(a, dgrad, 64);
    long mt = 0;
    for (int c = 0; c < a.ncls; ++c)
        if (a.nth[c] > 0) mt += a.mt0[c + 1] - a.mt0[c];
    if (idle) *idle = (a.mt0[a.ncls] - mt) * ((a.Cd + 63) / 64);
    return mt * ((a.Cd + 63) / 64);
}

// Tile and split by how many 64 x 64 tiles there are for the CUs, which all hold eight wavefronts of the kernel:
// the fewer, the smaller the tile and the more wavefronts share one.  Measured, us (fp32, then bf16; rows x K -> N):
// (fp32: with the fp32 instructions)
//   tiles / CU > 2.5     64x64, 2 wavefronts: 25088 x 1152 -> 128 fp32 82 (4 wavefronts: 90, 8: 97)
//   tiles / CU > 1       64x64, 4: 6272 x 2304 -> 256 fp32 83 (2: 147, 8: 88), bf16 21 (8: 24)
//   tiles / CU > 1/2     64x64, 8: 1568 x 4608 -> 512 fp32 83 (4: 90, 32x32: 93), 6272 x 1152 -> 128 bf16 11.0 (11.5, 20)
//   tiles / CU > 1/4     32x64, 8: 1568 x 2304 -> 256 bf16 12.6 (64x64: 13.4, 32x32: 16)
//   fewer                32x32, 8: 392 x 4608 -> 512 bf16 13.3 (64x64: 18.5, 32x64: 16), fp32 29 (80, 45)
static KsTile ks_tile(const ConvP& p, int dtype, bool dgrad) {
    const long cus = ks_cus(), n = ks_tiles(p, dtype, dgrad);
    if (2 * n > 5 * cus) return {64, 64, 2};
    if (n > cus) return {64, 64, 4};
    if (2 * n > cus) return {64, 64, 8};
    if (4 * n > cus) return {32, 64, 8};
    return {32, 32, 8};
}

template <typename T, bool DGRAD>
static int ks_dispatch(KsArgs& a, KsTile t, hipStream_t s) {
    const bool rag = a.Cs % (128 / (int)sizeof(T)) != 0 || (sizeof(T) == 2 && a.inside_only);
#define KS_CASE(BM, BN, KS_) \
    if (t.bm == BM && t.bn == BN && t.ks == KS_) return rag ? ks_launch<T, BM / 32, BN / 32, KS_, DGRAD, true>(a, s) : ks_launch<T, BM / 32, BN / 32, KS_, DGRAD, false>(a, s)
    KS_CASE(64, 64, 4);
    KS_CASE(64, 64, 8);
    KS_CASE(32, 64, 8);
    KS_CASE(32, 32, 8);
    KS_CASE(64, 64, 2);
#undef KS_CASE
    return fail(TSM_ERR_UNSUPPORTED, "ksplit: no such tile");
}

// fp32 layers, and bf16 layers that conv_mfma.hip does not take, run here whenever they can: the alternative is the block-
// wide schedule of conv_general.hip (fp32 6272 x 2304 -> 256: 129 us there, 73 here; 25088 x 1152 -> 128: 106, 76; bf16
// data gradient 26912 x 1800 -> 72 with split shift groups: 56, 36).  bf16 layers that it does take change over where
// there are at most two 64 x 64 tiles per CU, and so do forward layers that read a shifted copy (26912 x 648 -> 200, 1684 tiles:
// its three directions together 132.1 us with the general kernel, 140.0 with this one).  Measured on both sides of the line, us there -> here: 6272 x 2304 -> 256 (392
// tiles) 25.4 -> 20.7, 6272 x 1024 -> 256 (392) 16.4 -> 14.0, 392 x 4608 -> 512 (56) 39 -> 13, 25088 x 64 -> 64 (392) 8.6 -> 7.4;
// 12544 x 1024 -> 256 (784) 18.9 -> 22.4, 6272 x 128 -> 512 (784) 9.5 -> 13.5, 25088 x 64 -> 256 (1568) 12.2 -> 15.
// Data gradients with idle tiles (strided 1x1 layers): more of those than CUs cost more than the split saves unless K is long.
// Us there -> here, K and tiles in all: 128 224 10.6 -> 10.7, 64 392 10.9 -> 13.3, 128 416 10.7 -> 13.7, 512 400 13.5 -> 15.9,
// 256 448 11.7 -> 15.6; 1024 400 16.9 -> 15.0, 2048 800 33.7 -> 26.1.
// TSM_KSPLIT=0 leaves every layer to the other kernels, TSM_KSPLIT=1 takes the layers with whole_k as well, and
// TSM_KSPLIT_MAX_TILES=<n> moves the line (all read at every call: tests and comparisons set them).
bool ksplit_use(const ConvP& p, int dtype, bool dgrad) {
    if (!ks_supported(p, dtype, dgrad)) return false;
    const char* e = getenv("TSM_KSPLIT");
    if (e && e[0] == '0') return false;
    if (dtype == TSM_F32 || (!mfma_conv_supported(p) && (dgrad || !p.shifted))) return true;
    if (p.whole_k && !(e && e[0] == '1')) return false;
    const char* m = getenv("TSM_KSPLIT_MAX_TILES");
    long idle = 0;
    const long tiles = ks_tiles(p, dtype, dgrad, &idle);
    if (idle > 0 && tiles + idle > ks_cus() && p.Cout < 1024) return false;
    return tiles <= (m ? atol(m) : 2L * ks_cus());
}

int ksplit_rows(const ConvP& p, int dtype, bool dgrad) {
    KsArgs a;
    ks_geometry(a, p, dtype, dgrad);
    return ks_classes(a, dgrad, ks_tile(p, dtype, dgrad).bm);
}

int ksplit_fwd(const ConvP& p, int dtype, const void* x, const void* wp, void* y, float* stats, const FwdEpilogue* ep, hipStream_t s) {
    KsArgs a = {};
    ks_geometry(a, p, dtype, false);
    a.src = x; a.wp = wp; a.dst = y; a.stats = stats; a.add_stride = 1;
    if (ep && dtype != TSM_BF16) return fail(TSM_ERR_UNSUPPORTED, "ksplit: the affine epilogue is for bf16 layers");
    if (ep) { a.ep_scale = ep->scale; a.ep_shift = ep->shift; a.ep_res = ep->res; a.ep_relu = ep->relu; }
    const KsTile t = ks_tile(p, dtype, false);
    return dtype == TSM_F32 ? ks_dispatch<float, false>(a, t, s) : ks_dispatch<bf16_t, false>(a, t, s);
}

int ksplit_dgrad(const ConvP& p, int dtype, const void* dy, const void* wd, void* dx, const void* addend, int addend_stride,
                 const DgradFuse* fuse, hipStream_t s) {
    KsArgs a = {};
    ks_geometry(a, p, dtype, true);
    a.src = dy; a.wp = wd; a.dst = dx; a.addend = addend; a.add_stride = 1;
    if (addend && addend_stride == 2) { a.add_stride = 2; a.add_ho = (p.H + 1) / 2; a.add_wo = (p.W + 1) / 2; }
    if (fuse) {
        // (y == nullptr: only the ReLU mask of `act` is applied, no sums)
        a.act = fuse->act; a.ybn = fuse->y; a.bn_mean = fuse->mean; a.bn_rstd = fuse->rstd;
        a.stats = fuse->y ? fuse->partial : nullptr;
        if (dtype == TSM_BF16) a.act_bits = fuse->act_bits;
    }
    if (p.fold % (dtype == TSM_F32 ? 4 : 8) && (fuse || a.add_stride == 2)) return fail(TSM_ERR_UNSUPPORTED, "ksplit: shift groups that split a vector take no fused epilogue");
    const KsTile t = ks_tile(p, dtype, true);
    return dtype == TSM_F32 ? ks_dispatch<float, true>(a, t, s) : ks_dispatch<bf16_t, true>(a, t, s);
}

}  // namespace tsm
