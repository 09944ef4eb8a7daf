// Windowed cross-attention of the projector with the values projected AFTER the pooling (the other order is in qformer.hip, which
// says when which is taken):
//     sum_t p[j, h, t] (w_v[h] h_t)  =  w_v[h] (sum_t p[j, h, t] h_t).
// A window of 15 frames has n_q x 16 = 48 (query, head) pairs, and a head needs its own 64 rows of w_v only: 3.1 M
// multiply-adds per window for the projection and 0.8 M for the pooling instead of 15.7 M, and no values in memory.  The pooled
// states of 16 windows would be 1.5 MB, so they go from one product to the next through LDS.
//
// A workgroup takes 16 windows; its eight wavefronts each pool two windows for all heads and project two heads for all windows,
// in units of 32 state columns and a query:
//   pool     D[cols, heads] = H^T P^T over the frames of a window.  A product takes 32 k and a window has at most 16 frames: the
//            probabilities are bf16 pairs hi + lo, hi against k 0..15 and lo against k 16..31 of twice the same frames (bf16 as
//            stored).  H^T fragments come from the transposing LDS read.
//   exchange the sums, again as bf16 pairs hi + lo, go to LDS in fragment order: a lane that held one head then reads one window
//   project  O[dims, windows] += w_v[h] (hi + lo), w_v as stored in a fragment-ordered copy, straight from the L2
// A pair has 16 significant bits and the range of fp32, where the other order rounds the values to IEEE half (11 bits, 65504): nothing
// is clamped here, whatever the scales of states and w_v, and NaN stays NaN.  Relative error of g against 64 bits (1300 windows, states of
// unit spread, four times and a twentieth of it): 2.717e-3, 3.574e-3 and 2.343e-3; the other order 2.725e-3, 3.581e-3 and 2.352e-3
// (bf16 results and score rows: 2.7e-3, 3.6e-3 and 2.3e-3 of each).
// What bounds it: nothing alone.  32 columns are 60 products a wavefront (1920 cycles of the matrix cores), 64 KB of weights (1024
// cycles of the address path), 225 KB through LDS (1760 cycles) and 336 conversions; the parts overlap in half.  At 198 K frames (842
// workgroups, 3.3 rounds over the CUs) 346 us under a trace and 94 us for the scores, against 578 us for scores and values in one product
// and 114 us for the pooling.  Sums as half values (36 products, 130 KB) are 254 us there, but lose what is outside their range.
#include "gemm_core.h"
#include "ssd_internal.h"

namespace ssd {

constexpr int QV_WINDOWS = 16, QV_WAVES = 8, QV_HEADS = 16, QV_DIM = 64;
constexpr int QV_HEAD_BYTES = 2048 + 16;                   // hi | lo of one head: 16 windows x 32 columns each; padded for the writes
constexpr int QV_SLOT_BYTES = QV_HEADS * QV_HEAD_BYTES;    // the sums of one query and 32 columns
constexpr int QV_SLOTS = 4;                                // two are read while the other two are written
constexpr int QV_H_BYTES = 2 * 16 * 64;                    // two windows x 16 frames x 32 state columns of one wavefront
template <int NQ> constexpr int qv_lds_bytes() {
    constexpr int loop = QV_SLOTS * QV_SLOT_BYTES + QV_WAVES * QV_H_BYTES, out = QV_WINDOWS * (NQ * QV_HEADS * QV_DIM * 2 + 16);
    return loop > out ? loop : out;
}

bool qformer_values_supported(int n_q, int n_heads, int d_h, int d_enc, int window) {
    return n_q <= 3 && n_heads == QV_HEADS && d_h == QV_HEADS * QV_DIM && d_enc % 64 == 0 && window <= 16;
}

typedef short v4i16_t __attribute__((ext_vector_type(4)));
typedef short v8i16_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) v4i16_t lds_v4i16_t;

__device__ __forceinline__ uint32_t cvt_pk_bf16(float a, float b) { return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){a, b}, bf16x2_t)); }
// a pair of values as bf16 pairs: hi, and lo = what hi left out
__device__ __forceinline__ void split_bf16(float a, float b, uint32_t& hi, uint32_t& lo) {
    hi = cvt_pk_bf16(a, b);
    lo = cvt_pk_bf16(a - bf16_lo(hi), b - bf16_hi(hi));
}

// w_v [d_h, d_enc] in the order of the operand fragments: unit ((c * 16 + head) * 4 + n) * 64 + lane holds
// w_v[64 head + 16 n + lane % 16][32 c + 8 (lane / 16) .. + 7]
__global__ void __launch_bounds__(256) qformer_value_fragments_kernel(const bf16_t* __restrict__ w_v, int d_enc, uint4* __restrict__ out) {
    const int u = blockIdx.x * 256 + threadIdx.x;
    if (u >= QV_HEADS * QV_DIM * (d_enc / 8)) return;
    const int lane = u % 64, n = (u / 64) % 4, head = (u / 256) % QV_HEADS, c = u / (256 * QV_HEADS);
    const bf16_t* src = w_v + (int64_t)(head * QV_DIM + n * 16 + lane % 16) * d_enc + 32 * c + 8 * (lane / 16);
    uint32_t v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = (uint32_t)src[2 * e] | ((uint32_t)src[2 * e + 1] << 16);
    out[u] = make_uint4(v[0], v[1], v[2], v[3]);
}
void launch_qformer_value_fragments(const uint16_t* w_v, int d_enc, uint16_t* out, hipStream_t st) {
    const int units = QV_HEADS * QV_DIM * (d_enc / 8);
    hipLaunchKernelGGL(qformer_value_fragments_kernel, dim3((units + 255) / 256), dim3(256), 0, st, w_v, d_enc, reinterpret_cast<uint4*>(out));
}

template <int NQ>
__global__ void __launch_bounds__(64 * QV_WAVES) qformer_values_kernel(const bf16_t* __restrict__ enc_h, const float* __restrict__ scores,
                                                                     const bf16_t* __restrict__ w_frag, const QWindow* __restrict__ wins, int n_windows,
                                                                     int d_enc, bf16_t* __restrict__ o, int32_t* __restrict__ flags) {
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* x_lds = smem;
    const int lane = threadIdx.x % 64, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int m = lane % 16, g = lane / 16;
    const int w0 = blockIdx.x * QV_WINDOWS;
    unsigned char* h_lds = smem + QV_SLOTS * QV_SLOT_BYTES + wave * QV_H_BYTES;
    QWindow win[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const QWindow t = wins[min(w0 + 2 * wave + i, n_windows - 1)];
        win[i].frame0 = __builtin_amdgcn_readfirstlane(t.frame0);
        win[i].n_frames = __builtin_amdgcn_readfirstlane(t.n_frames);
    }

    // ---- H: 32 columns of the two windows' frames, global -> registers -> LDS, rows of 64 bytes
    // (the transposing reads take 32 bytes of rows r .. r + 3 and r + 8 .. r + 11 at a time: the halves of rows 8 .. 15 are exchanged.
    // Through registers because the compiler lets every other LDS access wait for all direct loads to LDS in flight: 2 us a step.)
    const __amdgpu_buffer_rsrc_t h_rsrc = make_rsrc(enc_h), w_rsrc = make_rsrc(w_frag);
    auto row_offset = [&](int i, int frame) { return (unsigned)(win[i].frame0 + frame) * (unsigned)d_enc * 2u + (unsigned)(((lane % 4) ^ (2 * (lane / 32))) * 16); };
    unsigned h_off[2];                                       // lane / 4: the frame
#pragma unroll
    for (int i = 0; i < 2; ++i) h_off[i] = row_offset(i, min(lane / 4, win[i].n_frames - 1));
    const int n32 = d_enc / 32;
    uint4 h_reg[2][2];                                       // two steps ahead of the fragments
    auto load_h = [&](int c, uint4 (&dst)[2]) {
#pragma unroll
        for (int i = 0; i < 2; ++i) dst[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(h_rsrc, h_off[i], min(c, n32 - 1) * 64, 0));
    };
    load_h(0, h_reg[0]);
    load_h(1, h_reg[1]);

    // ---- probabilities: lane (head m, frames 8 (g % 2) .. + 7), hi for g < 2 and lo for the others.  The lanes with g < 2 make the
    // first window's pairs and the others the second window's; half of each is exchanged.
    f16x8_t p_frag[2][NQ];
    bool lost;                                               // a frame has no finite score
    {
        const int f0 = g < 2 ? win[0].frame0 : win[1].frame0, nf = g < 2 ? win[0].n_frames : win[1].n_frames;
        float s[NQ][8];
#pragma unroll
        for (int j = 0; j < NQ; ++j)
#pragma unroll
            for (int e = 0; e < 8; ++e) s[j][e] = scores[(int64_t)(f0 + min(8 * (g % 2) + e, nf - 1)) * QF_SCORE_COLS + j * QV_HEADS + m];
        unsigned finite[2] = {0, 0};                         // frames of the two windows that have a finite score
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            bool any = false;
#pragma unroll
            for (int j = 0; j < NQ; ++j) any |= fabsf(s[j][e]) < INFINITY;
            const unsigned long long lanes = __ballot(any);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if ((lanes >> (16 * q)) & 0xffff) finite[q / 2] |= 1u << (8 * (q % 2) + e);
        }
        // Such a frame has an infinite or NaN state, and each of its probabilities is 0 or in a column of NaN.  Another frame's states
        // take its place in the sums: 0 times infinity would reach the queries that give it no weight.
        lost = (finite[0] & finite[1]) != 0xffffu;
        if (lost) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
                if (finite[i] && !(finite[i] >> (lane / 4) & 1)) h_off[i] = row_offset(i, __ffs(finite[i]) - 1);
            load_h(0, h_reg[0]);
            load_h(1, h_reg[1]);
        }
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            float mx = -INFINITY, sum = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if (8 * (g % 2) + e >= nf) s[j][e] = -INFINITY;
                mx = fmaxf(mx, s[j][e]);
            }
            mx = fmaxf(mx, __shfl_xor(mx, 16));
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                s[j][e] = __expf(s[j][e] - mx);
                sum += s[j][e];
            }
            sum += __shfl_xor(sum, 16);
            const float inv = 1.0f / sum;
            uint32_t v[2][4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uint32_t hi, lo;
                split_bf16(s[j][2 * e] * inv, s[j][2 * e + 1] * inv, hi, lo);
                const uint32_t other = (uint32_t)__shfl_xor((int)(g < 2 ? lo : hi), 32);
                v[0][e] = g < 2 ? hi : other;
                v[1][e] = g < 2 ? other : lo;
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) p_frag[i][j] = as_f16x8(make_uint4(v[i][0], v[i][1], v[i][2], v[i][3]));
        }
    }

    // ---- pool: H^T fragments of 32 columns (two windows, two blocks of 16 columns), the products with query j, their way to an X buffer
    int h_rd[2];                                             // transposing reads of frames 8 (g % 2) + 4 t .. + 3 (lane i: row i / 4, four columns)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int r = 8 * (g % 2) + 4 * t + m / 4;
        h_rd[t] = r * 64 + (r / 8) * 32 + (m % 4) * 8;       // columns 0 .. 15; the others are at this xor 32
    }
    f16x8_t h_frag[2][2];
    auto read_h = [&](const uint4 (&src)[2]) {
#pragma unroll
        for (int i = 0; i < 2; ++i) *reinterpret_cast<uint4*>(h_lds + i * 1024 + lane * 16) = src[i];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                v4i16_t part[2];
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    part[t] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(h_lds + i * 1024 + (h_rd[t] ^ (n * 32))));
                h_frag[i][n] = __builtin_bit_cast(f16x8_t, __builtin_shufflevector(part[0], part[1], 0, 1, 2, 3, 4, 5, 6, 7));
            }
    };
    unsigned char* x_wr = x_lds + m * QV_HEAD_BYTES + (g / 2) * 256 + (g % 2) * 8 + 2 * wave * 16;
    f32x4_t sums[2][2];                                      // lane: head m, state columns 16 n + 4 g .. + 3
    auto pool = [&](int j) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int n = 0; n < 2; ++n) sums[i][n] = mfma_16x16x32<true>(h_frag[i][n], p_frag[i][j], (f32x4_t){0.f, 0.f, 0.f, 0.f});
    };
    auto store_sums = [&](int slot) {                        // slot: byte offset
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                const f32x4_t d = sums[i][n];
                uint2 hi, lo;
                split_bf16(d[0], d[1], hi.x, lo.x);
                split_bf16(d[2], d[3], hi.y, lo.y);
                *reinterpret_cast<uint2*>(x_wr + slot + n * 512 + i * 16) = hi;
                *reinterpret_cast<uint2*>(x_wr + slot + n * 512 + i * 16 + 1024) = lo;
            }
    };

    // ---- project
    f32x4_t acc[2][NQ][4];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < NQ; ++j)
#pragma unroll
            for (int n = 0; n < 4; ++n) acc[h][j][n] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    f16x8_t w[2][4];
    auto load_w = [&](int c, int h) {
        const int base = __builtin_amdgcn_readfirstlane((min(c, n32 - 1) * QV_HEADS + 2 * wave) * 4096);
#pragma unroll
        for (int n = 0; n < 4; ++n) w[h][n] = __builtin_bit_cast(f16x8_t, __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, lane * 16 + (h * 4 + n) * 1024, base, 0));
    };
    f16x8_t x[2][2];                                         // head, hi | lo
    const unsigned char* x_rd = x_lds + 2 * wave * QV_HEAD_BYTES + lane * 16;
    auto read_x = [&](int h, int slot) {
#pragma unroll
        for (int e = 0; e < 2; ++e) x[h][e] = as_f16x8(*reinterpret_cast<const uint4*>(x_rd + slot + h * QV_HEAD_BYTES + e * 1024));
    };
    auto project = [&](int h, int j) {
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int n = 0; n < 4; ++n) acc[h][j][n] = mfma_16x16x32<true>(w[h][n], x[h][e], acc[h][j][n]);
    };

    // Unit u: 32 columns c = u / NQ and a query j = u % NQ.  It projects the sums of u from one slot, forms those of u + 2 and puts
    // them into another; two units a barrier.  (The last units form sums of columns that they repeat; nobody reads them.)
    auto frames = [&](int c, int odd) {                      // fragments of columns c; request of c + 2
        read_h(h_reg[odd]);
        load_h(c + 2, h_reg[odd]);
    };
    load_w(0, 0);
    load_w(0, 1);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        if (t % NQ == 0) frames(t / NQ, t / NQ % 2);
        pool(t % NQ);
        store_sums(t * QV_SLOT_BYTES);
    }
    __syncthreads();
    if (2 % NQ == 0) frames(2 / NQ, 2 / NQ % 2);
    int rd = 0, wr = 2 * QV_SLOT_BYTES;                      // slots of the units being projected and being formed
    read_x(0, 0);
    read_x(1, 0);
    for (int c0 = 0; c0 < n32; c0 += 2) {                    // (n32 is even)
#pragma unroll
        for (int u = 0; u < 2 * NQ; ++u) {
            const int j = u % NQ, t = u + 2, k = u % 2;
            __builtin_amdgcn_sched_barrier(0);
            pool(t % NQ);
            __builtin_amdgcn_sched_barrier(0);
            project(0, j);
            if (k == 0) read_x(0, rd + QV_SLOT_BYTES);
            if (j == NQ - 1) load_w(c0 + u / NQ + 1, 0);
            project(1, j);
            store_sums(wr + k * QV_SLOT_BYTES);
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (k == 0) read_x(1, rd + QV_SLOT_BYTES);
            if (j == NQ - 1) load_w(c0 + u / NQ + 1, 1);
            if ((t + 1) % NQ == 0) frames(c0 + (t + 1) / NQ, (t + 1) / NQ % 2);
            if (k == 1) {
                __syncthreads();
                const int was = rd;
                rd = wr;
                wr = was;
                read_x(0, rd);
                read_x(1, rd);
            }
        }
    }
    __syncthreads();                                         // the first sums of a unit that does not exist have been read
    float finite = 0.f;                                      // 0, or NaN if a result is not finite
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < NQ; ++j)
#pragma unroll
            for (int n = 0; n < 4; ++n)
#pragma unroll
                for (int r = 0; r < 4; ++r) finite = fmaf(acc[h][j][n][r], 0.f, finite);
    if (lost || finite != 0.f) raise_flag(flags, SSD_FLAG_ACT_OVERFLOW);

    // ---- out: the rows of the 16 windows are one contiguous piece; a lane's four dims go through LDS into it
    // (lane: window m, dims 16 n + 4 g .. + 3 of head 2 wave + h; the rows of a window are 16 bytes apart from a multiple of the banks)
    constexpr int ROW = QV_HEADS * QV_DIM * 2, WIN = NQ * ROW + 16;
#pragma unroll
    for (int j = 0; j < NQ; ++j)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                const f32x4_t a = acc[h][j][n];
                *reinterpret_cast<uint2*>(smem + m * WIN + j * ROW + ((2 * wave + h) * QV_DIM + n * 16 + 4 * g) * 2) =
                    make_uint2(pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]));
            }
    __syncthreads();
    unsigned char* dst = reinterpret_cast<unsigned char*>(o) + (int64_t)w0 * (NQ * ROW);
    const int windows = min(QV_WINDOWS, n_windows - w0);
    for (int i = wave; i < windows * NQ; i += QV_WAVES)
#pragma unroll
        for (int q = 0; q < ROW / 1024; ++q)
            *reinterpret_cast<uint4*>(dst + i * ROW + q * 1024 + lane * 16) = *reinterpret_cast<const uint4*>(smem + i / NQ * WIN + i % NQ * ROW + q * 1024 + lane * 16);
}

template <int NQ>
static void launch_values(const uint16_t* enc_h, const float* scores, const uint16_t* w_frag, const QWindow* wins, int n_windows, int d_enc,
                          uint16_t* o, int32_t* flags, hipStream_t st) {
    auto kern = qformer_values_kernel<NQ>;
    constexpr int lds = qv_lds_bytes<NQ>();
    static_assert(lds <= 160 * 1024, "LDS of a compute unit");
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3((n_windows + QV_WINDOWS - 1) / QV_WINDOWS), dim3(64 * QV_WAVES), lds, st, enc_h, scores, w_frag, wins, n_windows, d_enc, o, flags);
}
void launch_qformer_values(const uint16_t* enc_h, const float* scores, const uint16_t* w_frag, const QWindow* wins, int n_windows, int n_q,
                           int d_enc, uint16_t* o, int32_t* flags, hipStream_t st) {
    if (n_windows <= 0) return;
#define SSD_QV(NQ) launch_values<NQ>(enc_h, scores, w_frag, wins, n_windows, d_enc, o, flags, st)
    if (n_q == 1) SSD_QV(1); else if (n_q == 2) SSD_QV(2); else SSD_QV(3);
#undef SSD_QV
}

}  // namespace ssd
