// Weight-streaming GEMM for at most 32 rows (the auto-regressive steps, the last rows of a short utterance):
//   acc[M,64] = A[M,K] * W[n0 .. n0+63, K]^T.
// With so few rows the projection is one pass over the weight matrix, and what bounds it is the number
// of weight bytes a compute unit keeps in flight and the number of cache lines a load instruction
// touches.  W is therefore read from a second copy of the weights in "stream layout": the operand
// fragments of v_mfma_f32_32x32x16_f16 stored in the order the lanes consume them, so that every load
// instruction of a wavefront is one contiguous KB and goes straight into the MFMA operand registers
// (no LDS staging, no transposition).  All loads of a wavefront's K range (up to DEPTH steps of 64) are
// issued before its first MFMA.
//
// Stream layout of W[N,K] (N % 64 == 0, K % 64 == 0), in 16-byte units of eight f16:
//   unit(T, t, j, s, h, x) = ((T * K/64 + t) * 8 + j * 4 + s) * 64 + h * 32 + x
//   holds W[64 T + 32 j + x][64 t + 32 h + 8 s .. + 7]
// (column tile T, K step t, 32-column block j, MFMA step s, lane = 32 h + x).  The MFMA wants from lane
// (x, h) eight consecutive k of column x; which eight is free as long as A and W agree, and A is read
// from LDS with the same assignment k = 64 t + 32 h + 8 s .. + 7.
//
// Work split: a workgroup owns 64 output columns and the K range of one split; its NW wavefronts take
// consecutive, equally long pieces of that range and each accumulates a full 32 x 64 partial product;
// the partial products are added through LDS in a fixed order (deterministic) by four wavefronts, a
// quarter of the block each, which apply the epilogue.  A (a few KB per wavefront, L2 resident) is staged in a wavefront-private LDS
// region with the same swizzled row layout as the big GEMM (gemm_core.h), so no workgroup barrier is
// needed before the reduction.
// Requirements: (K / 64) % (splits * NW) == 0, A and W 16-byte aligned, A smaller than 4 GiB.
#pragma once
#include "gemm_core16.h"

namespace ssd {

constexpr int STREAM_STEP_UNITS = 8 * 64;          // 16-byte units of one (column tile, K step) block of W

template <int NW, int DEPTH>
constexpr size_t gemm_stream_lds_bytes() {
    return (size_t)NW * (DEPTH * 4096 > 8192 ? DEPTH * 4096 : 8192);
}

// The end of a workgroup whose wavefronts hold partial products of the same 32 x 64 block: each stores its own to LDS as
// [j][r / 4][lane] float4 (512 of them), then the quarters r / 4 are summed in wavefront order and finished by different
// wavefronts.  (One wavefront doing all of it was up to 2 us of a launch: 16 greedy steps at 27 rows 23.8 -> 22.3 ms,
// verification of 116 rows 1.86 -> 1.76 ms.)
template <int QUARTERS = 4>
__device__ __forceinline__ void store_partial(float4* dst, const f32x16_t (&acc)[2], int lane) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int g = 0; g < QUARTERS; ++g)
            dst[(j * 4 + g) * 64 + lane] = make_float4(acc[j][4 * g], acc[j][4 * g + 1], acc[j][4 * g + 2], acc[j][4 * g + 3]);
}
template <int NW, class Epi>
__device__ __forceinline__ void finish_quarter(const float4* red, int stride, int q, int row0, int col0, int M, int lane, int split, const Epi& epi) {
    f32x4_t out[1][2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        float4 v[NW];
#pragma unroll
        for (int o = 0; o < NW; ++o) v[o] = red[o * stride + (j * 4 + q) * 64 + lane];
        out[0][j] = (f32x4_t){v[0].x, v[0].y, v[0].z, v[0].w};
#pragma unroll
        for (int o = 1; o < NW; ++o) out[0][j] += (f32x4_t){v[o].x, v[o].y, v[o].z, v[o].w};
    }
    if constexpr (Epi::WANTS_SPLIT)
        epi.template operator()<1, 2, Layout32Quarter>(out, row0 + 8 * q, col0, M, lane, split);
    else
        epi.template operator()<1, 2, Layout32Quarter>(out, row0 + 8 * q, col0, M, lane);
}

// AQ: pieces of eight rows that are loaded, summed and finished (M <= 8 AQ).  What LDS holds in the place of the others only reaches
// accumulator rows that nobody reads.
template <int NW, int DEPTH, int AQ, bool BF, class Epi>
__global__ void __launch_bounds__(64 * NW)
gemm_stream_kernel(const f16_t* __restrict__ A, const u32x4_t* __restrict__ Ws, int M, int N, int K, int splits, Epi epi) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    constexpr int WAVE_LDS = DEPTH * 4096 > 8192 ? DEPTH * 4096 : 8192;
    const int lane = threadIdx.x % 64;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int x = lane % 32, h = lane / 32;
    const int tile = blockIdx.x / splits, split = blockIdx.x % splits;
    const int KT = K / 64;
    const int steps = KT / (splits * NW);                    // K steps of this wavefront
    const int t_first = (split * NW + wave) * steps;
    unsigned char* my_lds = smem_raw + wave * WAVE_LDS;

    // A: global -> LDS, 1 KB instructions, AQ per K step (eight rows of 128 bytes each)
    const __amdgpu_buffer_rsrc_t a_rsrc = make_rsrc(A);
    const int lrow = lane / 8, lslot = lane % 8;
    unsigned a_off[4];                                       // (an array of AQ makes the host compiler drop the kernel's stub without a word)
#pragma unroll
    for (int q = 0; q < AQ; ++q) {
        const int r = q * 8 + lrow;
        a_off[q] = (unsigned)min(r, M - 1) * (unsigned)K * 2u + (unsigned)((lslot ^ ((r >> 1) & 7)) * 16);
    }
    int a_rd[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) a_rd[s] = x * GEMM_ROW_BYTES + (((4 * h + s) ^ ((x >> 1) & 7)) * 16);
    const u32x4_t* w_base = Ws + ((int64_t)tile * KT + t_first) * STREAM_STEP_UNITS + lane;

    f32x16_t acc[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;

    for (int t0 = 0; t0 < steps; t0 += DEPTH) {
        if (t0 > 0) {                                        // fragment reads of the previous batch are done
            __builtin_amdgcn_s_waitcnt(0xC07F);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int d = 0; d < DEPTH; ++d)
#pragma unroll
            for (int q = 0; q < AQ; ++q)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, (lds_void_t*)(my_lds + d * 4096 + q * 1024), 16, a_off[q],
                                                         (t_first + t0 + d) * GEMM_ROW_BYTES, 0, 0);
        // keep the issue order A, then W: the wait below counts on it
        __builtin_amdgcn_sched_barrier(0);
        u32x4_t w[DEPTH][2][4];
#pragma unroll
        for (int d = 0; d < DEPTH; ++d)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    w[d][j][s] = __builtin_nontemporal_load(w_base + (int64_t)(t0 + d) * STREAM_STEP_UNITS + (j * 4 + s) * 64);
        // the A loads are the oldest: wait for them only (8 DEPTH weight loads may stay in flight)
        __builtin_amdgcn_s_waitcnt(0x0F70 | ((8 * DEPTH) & 15) | (((8 * DEPTH) >> 4) << 14));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int d = 0; d < DEPTH; ++d)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const f16x8_t a = as_f16x8(*reinterpret_cast<const uint4*>(my_lds + d * 4096 + a_rd[s]));
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[j] = mfma_32x32x16<BF>(a, __builtin_bit_cast(f16x8_t, w[d][j][s]), acc[j]);
            }
    }

    // ---- add the NW partial products in wavefront order
    __syncthreads();                                         // every wavefront is done with its A region
    store_partial<AQ>(reinterpret_cast<float4*>(smem_raw) + wave * 512, acc, lane);
    __syncthreads();
    for (int q = wave; q < AQ; q += NW) finish_quarter<NW>(reinterpret_cast<const float4*>(smem_raw), 512, q, 0, tile * 64, M, lane, split, epi);
}

// The same product for more rows (33..128 and beyond): a workgroup owns 64 columns, 32 R rows and one K split; its NW
// wavefronts take consecutive pieces of that K range.  W comes from the stream layout straight into the operand
// registers, A through a wavefront-private ring of D LDS stages (one stage: 32 R rows of one 64-wide K step), and the
// loads of D steps are in flight per wavefront.  No wavefront waits for another before the partial products are added.
// The K range need not divide evenly: beyond its end a wavefront issues loads through an empty buffer descriptor
// (they fetch nothing), so that the number of loads in flight, which the waits count, is the same in every step.
// Workgroup order: the row tiles of one (column tile, split) read the same weights and get ids 8 apart, i.e. one XCD.
// buffer descriptor over p, or an empty one (every access out of range: loads return zero and fetch nothing)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc_if(const void* p, bool have) {
    const int bytes = __builtin_amdgcn_readfirstlane(have ? -1 : 0);
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}
__device__ __forceinline__ u32x4_t buffer_load_16(__amdgpu_buffer_rsrc_t rsrc, int off, int soff) {
    return __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, soff, 0);
}
template <int R, int NW, int D>
constexpr size_t gemm_stream_rows_lds_bytes() { return (size_t)NW * R * (D * 4096 > 8192 ? D * 4096 : 8192); }

template <int R, int NW, int D, bool BF, class Epi>
__device__ __forceinline__ void gemm_stream_rows(const f16_t* __restrict__ A, const u32x4_t* __restrict__ Ws, int M, int N, int K, int splits,
                                                 int row_tiles, const Epi& epi, unsigned char* smem_raw) {
    constexpr int STAGE = R * 4096;
    constexpr int WAVE_LDS = D * STAGE;
    constexpr int LOADS = 4 * R + 8;                         // per step
    static_assert((D - 1) * LOADS <= 63, "vmcnt range");
    const int lane = threadIdx.x % 64;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int x = lane % 32, h = lane / 32;
    const int units = (N / 64) * splits;
    int unit, rt;
    if (units % 8 == 0) {
        const int chunk = blockIdx.x / (8 * row_tiles), in = blockIdx.x % (8 * row_tiles);
        unit = chunk * 8 + in % 8;
        rt = in / 8;
    } else {
        unit = blockIdx.x / row_tiles;
        rt = blockIdx.x % row_tiles;
    }
    const int tile = unit / splits, split = unit % splits;
    const int row0 = rt * 32 * R;
    const int KT = K / 64, pieces = splits * NW, piece = split * NW + wave;
    // (said to be uniform: a descriptor or offset in vector registers would turn every load into a loop over the lanes)
    const int t_first = __builtin_amdgcn_readfirstlane(KT * piece / pieces);
    const int steps = __builtin_amdgcn_readfirstlane(KT * (piece + 1) / pieces) - t_first;
    const int w_first = __builtin_amdgcn_readfirstlane((tile * KT + t_first) * (STREAM_STEP_UNITS * 16));
    unsigned char* my_lds = smem_raw + wave * WAVE_LDS;

    const int lrow = lane / 8, lslot = lane % 8;
    unsigned a_off[4 * R];
#pragma unroll
    for (int q = 0; q < 4 * R; ++q) {
        const int r = q * 8 + lrow;
        a_off[q] = (unsigned)min(row0 + r, M - 1) * (unsigned)K * 2u + (unsigned)((lslot ^ ((r >> 1) & 7)) * 16);
    }
    int a_rd[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) a_rd[s] = x * GEMM_ROW_BYTES + (((4 * h + s) ^ ((x >> 1) & 7)) * 16);

    f32x16_t acc[R][2];
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    u32x4_t w[D][2][4];
    auto issue = [&](auto dc, int i) {                       // step i of this wavefront into stage d
        constexpr int d = decltype(dc)::value;
        const __amdgpu_buffer_rsrc_t a_rsrc = make_rsrc_if(A, i < steps), w_rsrc = make_rsrc_if(Ws, i < steps);
#pragma unroll
        for (int q = 0; q < 4 * R; ++q)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, (lds_void_t*)(my_lds + d * STAGE + q * 1024), 16, a_off[q], (t_first + i) * GEMM_ROW_BYTES, 0, 0);
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int s = 0; s < 4; ++s)
                w[d][j][s] = buffer_load_16(w_rsrc, lane * 16 + (j * 4 + s) * 1024, w_first + i * (STREAM_STEP_UNITS * 16));
        __builtin_amdgcn_sched_barrier(0);
    };
    auto compute = [&](auto dc) {
        constexpr int d = decltype(dc)::value;
        f16x8_t a[2][R];
        auto read = [&](int s) {
#pragma unroll
            for (int i = 0; i < R; ++i) a[s % 2][i] = as_f16x8(*reinterpret_cast<const uint4*>(my_lds + d * STAGE + i * 4096 + a_rd[s]));
        };
        read(0);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            __builtin_amdgcn_sched_barrier(0);
            if (s < 3) read(s + 1);
#pragma unroll
            for (int i = 0; i < R; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = mfma_32x32x16<BF>(a[s % 2][i], __builtin_bit_cast(f16x8_t, w[d][j][s]), acc[i][j]);
        }
    };
    constexpr int KEEP = (D - 1) * LOADS;
    auto step = [&](auto dc, int i) {
        __builtin_amdgcn_s_waitcnt(0x0F70 | (KEEP & 15) | ((KEEP >> 4) << 14));      // step i has landed, the D - 1 younger ones may be out
        __builtin_amdgcn_sched_barrier(0);
        if (i < steps) compute(dc);
        __builtin_amdgcn_s_waitcnt(0xC07F);                  // the fragment reads of this stage are done
        __builtin_amdgcn_sched_barrier(0);
        issue(dc, i + D);
    };
    auto for_stages = [&](auto f) {
        f(std::integral_constant<int, 0>());
        if constexpr (D > 1) f(std::integral_constant<int, 1>());
        if constexpr (D > 2) f(std::integral_constant<int, 2>());
        if constexpr (D > 3) f(std::integral_constant<int, 3>());
        static_assert(D <= 4, "stages");
    };
    for_stages([&](auto dc) { issue(dc, decltype(dc)::value); });
    int i0 = 0;
    do {                                                     // (a branch here would let the W loads sink below the A loads of later steps)
        for_stages([&](auto dc) { step(dc, i0 + decltype(dc)::value); });
        i0 += D;
    } while (i0 < steps);

    // ---- add the NW partial products in wavefront order; the wavefronts share the quarters of the row blocks
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < R; ++i) store_partial(reinterpret_cast<float4*>(smem_raw) + (wave * R + i) * 512, acc[i], lane);
    __syncthreads();
    for (int q = wave; q < 4 * R; q += NW) {
        if (row0 + q * 8 >= M) break;
        finish_quarter<NW>(reinterpret_cast<const float4*>(smem_raw) + (q / 4) * 512, R * 512, q % 4, row0 + (q / 4) * 32, tile * 64, M, lane, split, epi);
    }
}
template <int R, int NW, int D, bool BF, class Epi>
__global__ void __launch_bounds__(64 * NW)
gemm_stream_rows_kernel(const f16_t* __restrict__ A, const u32x4_t* __restrict__ Ws, int M, int N, int K, int splits, int row_tiles, Epi epi) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    gemm_stream_rows<R, NW, D, BF>(A, Ws, M, N, K, splits, row_tiles, epi, smem_raw);
}

// Row-major W[N,K] (f16) -> stream layout; one thread per 16-byte unit.
__global__ void __launch_bounds__(256) stream_layout_kernel(const u32x4_t* __restrict__ w, u32x4_t* __restrict__ out, int N, int K) {
    const int64_t n_units = (int64_t)N * K / 8;
    const int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (u >= n_units) return;
    const int KT = K / 64;
    const int xx = (int)(u % 32), hh = (int)((u / 32) % 2), ss = (int)((u / 64) % 4), jj = (int)((u / 256) % 2);
    const int64_t blk = u / STREAM_STEP_UNITS;
    const int t = (int)(blk % KT);
    const int64_t T = blk / KT;
    const int64_t row = T * 64 + jj * 32 + xx;
    out[u] = w[row * (K / 8) + 8 * t + 4 * hh + ss];
}

}  // namespace ssd
