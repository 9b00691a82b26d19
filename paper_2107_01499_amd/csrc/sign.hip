// 1-bit sign codec kernels: worker-side compress with error feedback, server-side
// decompress-average-recompress, and decompress (C_LP_S with the compression of "1-bit Adam",
// Sections 3.2 and 4.1 of the paper).
//
// Lane l of a wave owns elements 4l..4l+3 of every 256-element row, so the group of four that the
// fixed |v| summation order is defined on is exactly one lane's 128-bit load, accumulator m mod 64
// is lane m mod 64, and the final xor butterfly is a reduction over the wave.
#include <type_traits>

#include "batch.hpp"
#include "launchers.hpp"
#include "sign_device.hpp"

#pragma clang fp contract(off)

namespace bagua {

// ------------------------------------------------------------------------------------------
// MOM: the compressed tensor is the local momentum beta1*m + omb1*x of the compression stage of
// 1-bit Adam (x is then the gradient; m is read only), loaded without the nontemporal hint where the workgroup says `keep`, or
// streamed throughout where a wave has tail tests.
constexpr int kMomNone = 0, kMomKeep = 1, kMomStream = 2;
template <int RPW, bool EF, int MOM, bool FULL>
__device__ __forceinline__ void sign_compress_rows(const float* __restrict__ x, float* __restrict__ residual, int len, uint32_t chunk,
                                                   uint32_t* __restrict__ bits, float* __restrict__ scale_c,
                                                   const float* __restrict__ mom, float beta1, float omb1, float* s_q, int pace, int keep)
{
    const int wave = wave_index(), lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;
    f4 v[RPW];
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        const int off = static_cast<int>(wave * RPW + i) * kRow;
        const int remain = row_remain<FULL>(len, off);
        v[i] = f4{0.f, 0.f, 0.f, 0.f};
        if (remain > 0) v[i] = load_row(x + off, lane, remain, 0.0f);
        if (!FULL && pace) pace_loads();
    }
    if (MOM != kMomNone) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int off = static_cast<int>(wave * RPW + i) * kRow;
            const int remain = row_remain<FULL>(len, off);
            if (remain > 0) {
                const f4 m = FULL || (MOM == kMomKeep && keep) ? load_row_keep(mom + off, lane, remain, 0.0f) : load_row(mom + off, lane, remain, 0.0f);
                v[i].x = beta1 * m.x + omb1 * v[i].x;
                v[i].y = beta1 * m.y + omb1 * v[i].y;
                v[i].z = beta1 * m.z + omb1 * v[i].z;
                v[i].w = beta1 * m.w + omb1 * v[i].w;
            }
        }
    }
    if (EF) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int off = static_cast<int>(wave * RPW + i) * kRow;
            const int remain = row_remain<FULL>(len, off);
            if (remain > 0) {
                const f4 d = load_row(residual + off, lane, remain, 0.0f);
                if (!FULL && pace) pace_loads();
                v[i].x = v[i].x + d.x;
                v[i].y = v[i].y + d.y;
                v[i].z = v[i].z + d.z;
                v[i].w = v[i].w + d.w;
            }
        }
    }
    sign_encode_chunk<RPW, EF, false, FULL>(v, len, chunk, wave, lane, nwaves, residual, bits, scale_c, nullptr, s_q);
}

// The chunk that is cut short, without tests (see row_at).  With -> without, us per launch: C = 4096, 64 K 2.9 -> 2.7, 1 M 4.6 -> 3.9, with the
// momentum 5.2 -> 4.2, 3 M 10.4 -> 9.8; five buckets, C = 2048, 1 M 5.2 -> 4.0; above 6 M +-0.  (Chunks that are held in one row per wave: -0.1 .. 0 us.)
template <int RPW, bool EF, int MOM>
__device__ __forceinline__ void sign_compress_cut(const float* __restrict__ x, float* __restrict__ residual, int len, uint32_t chunk,
                                                  uint32_t* __restrict__ bits, float* __restrict__ scale_c, const float* __restrict__ mom,
                                                  float beta1, float omb1, float* s_q)
{
    const int wave = wave_index(), lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;
    f4 v[RPW], m[RPW], d[RPW];
    RowAt at[RPW];
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        at[i] = row_at<false>((wave * RPW + i) * kRow, len, lane);
        v[i] = load_at<false>(x, at[i]);
        if (MOM != kMomNone) m[i] = load_at<false, true>(mom, at[i]);
        if (EF) d[i] = load_at<false>(residual, at[i]);
    }
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        v[i] = settle<false>(v[i], at[i]);
        if (MOM != kMomNone) {
            const f4 mi = settle<false>(m[i], at[i]);
            v[i].x = beta1 * mi.x + omb1 * v[i].x;
            v[i].y = beta1 * mi.y + omb1 * v[i].y;
            v[i].z = beta1 * mi.z + omb1 * v[i].z;
            v[i].w = beta1 * mi.w + omb1 * v[i].w;
        }
        if (EF) {
            const f4 e = settle<false>(d[i], at[i]);
            v[i].x = v[i].x + e.x;
            v[i].y = v[i].y + e.y;
            v[i].z = v[i].z + e.z;
            v[i].w = v[i].w + e.w;
        }
        clear_absent(v[i], (wave * RPW + i) * kRow + lane * 4, len);
    }
    sign_encode_chunk<RPW, EF, false, false>(v, len, chunk, wave, lane, nwaves, residual, bits, scale_c, nullptr, s_q);
}

template <int RPW, bool EF, int MOM, bool SHORT>
__device__ __forceinline__ void sign_compress_chunk(const float* __restrict__ x, float* __restrict__ residual, size_t n,
                                                    uint32_t chunk, uint32_t* __restrict__ bits,
                                                    float* __restrict__ scale, const float* __restrict__ mom,
                                                    float beta1, float omb1, size_t c, float* s_q, int pace, int keep)
{
    const size_t base = c * static_cast<size_t>(chunk);
    const int len = static_cast<int>((n - base < chunk) ? (n - base) : chunk);
    float* res_c = EF ? residual + base : nullptr;
    const float* mom_c = MOM != kMomNone ? mom + base : nullptr;
    uint32_t* bits_c = bits + (base >> 5);
    if (SHORT && chunk_full<RPW>(len, blockDim.x >> 6))
        sign_compress_rows<RPW, EF, MOM, true>(x + base, res_c, len, chunk, bits_c, scale + c, mom_c, beta1, omb1, s_q, 0, 1);
    else if (SHORT && RPW > 1 && len < static_cast<int>(chunk) && base + len >= 4)
        sign_compress_cut<RPW, EF, MOM>(x + base, res_c, len, chunk, bits_c, scale + c, mom_c, beta1, omb1, s_q);
    else sign_compress_rows<RPW, EF, MOM, false>(x + base, res_c, len, chunk, bits_c, scale + c, mom_c, beta1, omb1, s_q, pace, keep);
}

// The local momentum is the one input that all workers of a GPU read, one call after the other, so what of it the Infinity Cache
// holds comes from there for all but the first.  Up to 2^26 elements (256 MB) all of it is kept and the tail tests are folded
// away; in longer launches the first 3 * 2^24 elements are, and the tests stay (without them -4 .. -8 %).  Whole rounds, streamed
// with the tests -> this: 8 workers x 36 M, C = 4096, 881 -> 799 us, x 50 M, C = 16384, 1314 -> 1179, 16 x 60 M, C = 2048, 2636 ->
// 2377, 3 x 60 M, C = 1536, 679 -> 646, 2 x 66 M, C = 4096, 590 -> 584, 8 x 67 M, C = 2048, 1592 -> 1523; beyond, 4 x 100 M, C = 2048,
// 1385 -> 1345, 8 x 134 M 3209 -> 3133, 2 x 134 M, C = 4096, 1186 -> 1177.  With 2^26 of them kept 16 x 100 M gains 1.7 % more, 2 x 134 M
// loses; with all, -0.3 .. -0.9 % against none.
// Eight waves of one row (chunks of 2048) stream it above 7 * 2^24 elements: the choice of the hint at run time costs them more than the
// hint gives.  Chosen -> streamed: 4 x 250 M 3563 -> 3399 us, 8 x 200 M 4816 -> 4615, 4 x 200 M 2778 -> 2687, 8 x 134 M 3147 -> 3091, 2 x 134 M 1156 ->
// 1142; below the line 4 x 100 M 1350 -> 1346, 16 x 100 M 4231 -> 4283, 8 x 80 M 1814 -> 1845.  Other chunks: C = 1536, 8 x 200 M, 4664 -> 4808, C =
// 4096, 8 x 134 M, 3171 -> 3215, 4 x 250 M 3537 -> 3526, C = 8192, 3501 -> 3422.
inline bool mom_fold(size_t n) { return n <= (static_cast<size_t>(1) << 26); }
inline uint32_t mom_keep(size_t chunk) { return static_cast<uint32_t>((static_cast<size_t>(3) << 24) / chunk); }

template <int RPW, bool EF, int MOM, bool SHORT>
__global__ void __launch_bounds__(wg_threads_max(RPW))
k_sign_compress(const float* __restrict__ x, float* __restrict__ residual, size_t n, uint32_t chunk,
                uint32_t* __restrict__ bits, float* __restrict__ scale, const float* __restrict__ mom, float beta1,
                float omb1, int pace, uint32_t keep, ChunkOrder order)
{
    extern __shared__ float s_q[];
    sign_compress_chunk<RPW, EF, MOM, SHORT>(x, residual, n, chunk, bits, scale, mom, beta1, omb1, order(blockIdx.x), s_q, pace,
                                             blockIdx.x < keep);
}

// Batched: entry = [x, residual, bits, scale, n]; unit = chunk.
template <int RPW, bool EF, bool SHORT, typename TABLE>
__global__ void __launch_bounds__(wg_threads_max(RPW))
k_sign_compress_batched(TABLE table, uint32_t chunk, int pace, ChunkOrder order)
{
    extern __shared__ float s_q[];
    const BatchView bv = table.view();
    const uint32_t unit = order(blockIdx.x), b = batch_find(bv, unit);
    const uint64_t* e = bv.entries + static_cast<size_t>(b) * bv.entry_words;
    sign_compress_chunk<RPW, EF, kMomNone, SHORT>(table_ptr<const float>(e[0]), table_ptr<float>(e[1]), e[4], chunk,
                                        table_ptr<uint32_t>(e[2]), table_ptr<float>(e[3]), nullptr, 0.0f,
                                        0.0f, unit - bv.first_unit[b], s_q, pace, 0);
}

// Server side with the sign codec: a = (sum_j +-scale_j) * inv_k in ascending j; w = a (+ eps).
// SRC names the workers' inputs: code(j) -> sign words of worker j, meta(j) -> its per-chunk scales.
struct SignTableSrc {   // pointers in the kernel arguments
    const PtrTable& bits;
    const PtrTable& scales;
    __device__ __forceinline__ const void* code(int j) const { return bits.p[j]; }
    __device__ __forceinline__ const float* meta(int j) const { return static_cast<const float*>(scales.p[j]); }
};
struct SignEntrySrc {   // pointers in a batch entry: [eps, bits_out, scale_out, out, n, bits[0..k), scale[0..k)]
    const uint64_t* e;
    int k;
    __device__ __forceinline__ const void* code(int j) const { return table_ptr<const void>(e[5 + j]); }
    __device__ __forceinline__ const float* meta(int j) const { return table_ptr<const float>(e[5 + k + j]); }
};

template <int RPW, bool EF, bool OUT, int REST, typename SRC>
__device__ __forceinline__ void drr_sign_chunk(const SRC& src, int k, float inv_k, float* __restrict__ eps, size_t n,
                                               uint32_t chunk, uint32_t* __restrict__ bits_out,
                                               float* __restrict__ scale_out, float* __restrict__ out, size_t c,
                                               float* s_q)
{
    const size_t base = c * static_cast<size_t>(chunk);
    const int len = static_cast<int>((n - base < chunk) ? (n - base) : chunk);
    const int wave = wave_index(), lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;
    const int sh = 4 * (lane & 7);

    // Scales of this chunk: lane j fetches worker j's (one memory round trip for all workers instead of a chain
    // of k dependent ones), broadcast below with readlane.
    float lane_scale = 0.0f;
    if (lane < k) lane_scale = src.meta(lane)[c];

    f4 v[RPW];
    constexpr int NJ = BAGUA_DRR_SIGN_NJ;   // workers whose sign words are fetched together
    // Workers are summed in ascending order; worker 0 starts the sum (s = d_0, not 0 + d_0).
    // The one row of a bucket's last chunk that is cut short (if any) is the only one that needs per-element tail
    // tests; a wave that does not own it sees complete rows and, past the chunk's end, absent ones.
    const int rows = static_cast<int>(len / kRow);   // complete rows of this chunk
    const int ragged_row = (len % kRow) ? rows : -1;
    if (rows > 0 && (ragged_row < wave * RPW || ragged_row >= wave * RPW + RPW)) {
        // ---- complete (or absent) rows only, wave-uniform: no tail tests, uniform row addresses, one shift + one
        // three-input bit operation + one add per element and worker.  An absent row re-reads row 0 of the chunk
        // (complete, since rows > 0) and is cleared afterwards.
        int row_of[RPW];
#pragma unroll
        for (int i = 0; i < RPW; ++i) row_of[i] = (wave * RPW + i < rows) ? wave * RPW + i : 0;
        f4 e[RPW];
        if (EF) {
#pragma unroll
            for (int i = 0; i < RPW; ++i)
                e[i] = ld_stream(reinterpret_cast<const f4*>(eps + base + static_cast<size_t>(row_of[i]) * kRow) + lane);
        }
        const uint32_t word = static_cast<uint32_t>(lane >> 3);
        const uint32_t s0 = 31u - sh, s1 = 30u - sh, s2 = 29u - sh, s3 = 28u - sh;   // element's bit -> bit 31
        auto fetch = [&](int j, uint32_t (&w)[RPW]) {
            const uint32_t* bj = static_cast<const uint32_t*>(src.code(j)) + (base >> 5);
#pragma unroll
            for (int i = 0; i < RPW; ++i) w[i] = bj[row_of[i] * (kRow / 32) + word];
        };
        auto decode = [&](int j, const uint32_t (&w)[RPW], bool first) {
            const uint32_t sc = __builtin_amdgcn_readlane(__float_as_uint(lane_scale), j);
            const uint32_t neg = sc ^ 0x80000000u;
#pragma unroll
            for (int i = 0; i < RPW; ++i) {
                f4 d;
                d.x = sign_select(w[i] << s0, sc, neg);
                d.y = sign_select(w[i] << s1, sc, neg);
                d.z = sign_select(w[i] << s2, sc, neg);
                d.w = sign_select(w[i] << s3, sc, neg);
                if (first) {
                    v[i] = d;
                } else {
                    v[i].x = v[i].x + d.x;
                    v[i].y = v[i].y + d.y;
                    v[i].z = v[i].z + d.z;
                    v[i].w = v[i].w + d.w;
                }
            }
        };
        // As many workers' words as there are left, up to NJ, are requested together, unless sign_rest() says otherwise.  Those of k mod NJ one after
        // the other -> together, us of the step: k = 2, C = 2048, 16 M 25.3 -> 24.2, 134 M 173 -> 170; k = 4, 1 M 4.1 -> 4.0, 16 M 28.3 -> 24.9, 134 M 203 -> 183; k = 7, 65 K 4.1 -> 3.8,
        // 8 M 18.4 -> 16.2, 33 M 61.7 -> 49.7, 134 M 255 -> 196; k = 5, C = 4096, 33 M 57.1 -> 49.2, C = 16384, 134 M 298 -> 257; k = 12, C = 8192, 134 M 298 ->
        // 255; k = 3, C = 1024, 8 M 15.2 -> 14.8.  (Where k is a multiple of NJ the bodies of the rest would cost 1-2 %.)
        auto group = [&](auto count, int j, bool first) {
            constexpr int N = decltype(count)::value;
            uint32_t w[N][RPW];
#pragma unroll
            for (int u = 0; u < N; ++u) fetch(j + u, w[u]);
#pragma unroll
            for (int u = 0; u < N; ++u) decode(j + u, w[u], first && u == 0);
        };
        for_worker_groups<NJ, REST>(k, group);
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            v[i].x = v[i].x * inv_k;
            v[i].y = v[i].y * inv_k;
            v[i].z = v[i].z * inv_k;
            v[i].w = v[i].w * inv_k;
            if (EF) {
                v[i].x = v[i].x + e[i].x;
                v[i].y = v[i].y + e[i].y;
                v[i].z = v[i].z + e[i].z;
                v[i].w = v[i].w + e[i].w;
            }
            if (wave * RPW + i >= rows) v[i] = f4{0.f, 0.f, 0.f, 0.f};   // absent row: +0 in the |v| sum, nothing stored
        }
    } else {
        // ---- the wave that owns the ragged row of a bucket's last chunk
        auto accumulate = [&](int j, uint32_t (&w)[RPW]) {
            const float sc = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(lane_scale), j));
            const float neg = -sc;
#pragma unroll
            for (int i = 0; i < RPW; ++i) {
                const uint32_t nib = w[i] >> sh;
                f4 d;
                d.x = (nib & 1u) ? sc : neg;
                d.y = (nib & 2u) ? sc : neg;
                d.z = (nib & 4u) ? sc : neg;
                d.w = (nib & 8u) ? sc : neg;
                if (j == 0) {
                    v[i] = d;
                } else {
                    v[i].x = v[i].x + d.x;
                    v[i].y = v[i].y + d.y;
                    v[i].z = v[i].z + d.z;
                    v[i].w = v[i].w + d.w;
                }
            }
        };
        for (int j = 0; j < k; ++j) {
            const uint32_t* bj = static_cast<const uint32_t*>(src.code(j)) + (base >> 5);
            uint32_t w[RPW];
#pragma unroll
            for (int i = 0; i < RPW; ++i) {
                const int off = static_cast<int>(wave * RPW + i) * kRow;
                const int remain = len - off;
                w[i] = 0;
                if (static_cast<int>(lane >> 3) * 32 < remain) w[i] = bj[(off >> 5) + (lane >> 3)];
            }
            accumulate(j, w);
        }
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int off = static_cast<int>(wave * RPW + i) * kRow;
            const int remain = len - off;
            const int e = lane * 4;
            // elements beyond the chunk must enter the |v| sum as +0.0f
            v[i].x = (e + 0 < remain) ? v[i].x * inv_k : 0.0f;
            v[i].y = (e + 1 < remain) ? v[i].y * inv_k : 0.0f;
            v[i].z = (e + 2 < remain) ? v[i].z * inv_k : 0.0f;
            v[i].w = (e + 3 < remain) ? v[i].w * inv_k : 0.0f;
        }
        if (EF) {
#pragma unroll
            for (int i = 0; i < RPW; ++i) {
                const int off = static_cast<int>(wave * RPW + i) * kRow;
                const int remain = len - off;
                if (remain > 0) {
                    const f4 d = load_row(eps + base + off, lane, remain, 0.0f);
                    v[i].x = v[i].x + d.x;
                    v[i].y = v[i].y + d.y;
                    v[i].z = v[i].z + d.z;
                    v[i].w = v[i].w + d.w;
                }
            }
        }
    }
    sign_encode_chunk<RPW, EF, OUT>(v, len, chunk, wave, lane, nwaves, EF ? eps + base : nullptr,
                                    bits_out + (base >> 5), scale_out + c, OUT ? out + base : nullptr, s_q);
}

template <int RPW, bool EF, bool OUT, int REST>
__global__ void __launch_bounds__(wg_threads_max(RPW))
k_drr_sign(PtrTable bits_in, PtrTable scale_in, int k, float inv_k, float* __restrict__ eps, size_t n,
           uint32_t chunk, uint32_t* __restrict__ bits_out, float* __restrict__ scale_out,
           float* __restrict__ out)
{
    extern __shared__ float s_q[];
    drr_sign_chunk<RPW, EF, OUT, REST>(SignTableSrc{bits_in, scale_in}, k, inv_k, eps, n, chunk, bits_out, scale_out, out,
                                 blockIdx.x, s_q);
}

template <int RPW, bool EF, bool OUT, int REST, typename TABLE>
__global__ void __launch_bounds__(wg_threads_max(RPW))
k_drr_sign_batched(TABLE table, int k, float inv_k, uint32_t chunk)
{
    extern __shared__ float s_q[];
    const BatchView bv = table.view();
    const uint32_t b = batch_find(bv, blockIdx.x);
    const uint64_t* e = bv.entries + static_cast<size_t>(b) * bv.entry_words;
    drr_sign_chunk<RPW, EF, OUT, REST>(SignEntrySrc{e, k}, k, inv_k, table_ptr<float>(e[0]), e[4], chunk,
                                 table_ptr<uint32_t>(e[1]), table_ptr<float>(e[2]),
                                 table_ptr<float>(e[3]), blockIdx.x - bv.first_unit[b], s_q);
}

__global__ void __launch_bounds__(kWave * kRowWaves)
k_decompress_sign(const uint32_t* __restrict__ bits, const float* __restrict__ scale, size_t n, uint32_t chunk,
                  float* __restrict__ out)
{
    const size_t row = static_cast<size_t>(blockIdx.x) * kRowWaves + wave_index();
    const int lane = threadIdx.x & 63;
    const size_t e0 = row * kRow;
    if (e0 >= n) return;
    const float sc = scale[e0 / chunk];
    const float neg = -sc;
    const int remain = static_cast<int>((n - e0 < static_cast<size_t>(kRow)) ? (n - e0) : kRow);
    uint32_t w = 0;
    if (static_cast<int>(lane >> 3) * 32 < remain) w = bits[(e0 >> 5) + (lane >> 3)];
    const uint32_t nib = w >> (4 * (lane & 7));
    f4 d;
    d.x = (nib & 1u) ? sc : neg;
    d.y = (nib & 2u) ? sc : neg;
    d.z = (nib & 4u) ? sc : neg;
    d.w = (nib & 8u) ? sc : neg;
    store_row(out + e0, lane, remain, d);
}

// ------------------------------------------------------------------------------------------ host
struct SignGeometry {
    dim3 grid, block;
    size_t lds;
    int rpw;
};
static SignGeometry sign_geometry(size_t n, size_t chunk, int preferred, bool worker_side)
{
    SignGeometry g;
    const int rows = static_cast<int>(chunk / kRow);
    g.rpw = worker_side ? pick_rpw_worker(rows, preferred) : pick_rpw(rows, preferred);
    const int waves = (rows + g.rpw - 1) / g.rpw;
    g.grid = dim3(static_cast<unsigned>(num_chunks(n, chunk)));
    g.block = dim3(64 * waves);
    g.lds = waves > 1 ? static_cast<size_t>(rows) * kWave * sizeof(float) : 0;
    return g;
}

int launch_sign_compress(const float* x, float* residual, size_t n, size_t chunk, uint32_t* bits, float* scale,
                         hipStream_t stream)
{
    const SignGeometry g = sign_geometry(n, chunk, BAGUA_RPW_SIGN, true);
    const uint32_t ch = static_cast<uint32_t>(chunk);
    if (residual) {
        BAGUA_DISPATCH_RPW_WORKER(g.rpw, BAGUA_DISPATCH_SHORT(short_launch(n), launch_kernel((k_sign_compress<RPW, true, kMomNone, SHORT>), g.grid, g.block,
                                                     g.lds, stream, x, residual, n, ch, bits, scale, nullptr, 0.0f, 0.0f, pace_for(n), 0u, chunk_order(g.grid.x, chunk, order_pays(n, chunk)))))
    } else {
        BAGUA_DISPATCH_RPW_WORKER(g.rpw, BAGUA_DISPATCH_SHORT(short_launch(n), launch_kernel((k_sign_compress<RPW, false, kMomNone, SHORT>), g.grid, g.block,
                                                     g.lds, stream, x, residual, n, ch, bits, scale, nullptr, 0.0f, 0.0f, pace_for(n), 0u, chunk_order(g.grid.x, chunk, order_pays(n, chunk)))))
    }
    return launch_status();
}

// How the workers beyond the last group of NJ are taken.  One by one where the launch is one go that more than half fills the chip: there the waves that
// request everything together only meet in the memory, and the longer chain of loads spreads them.  Together -> one by one, us of the step: C = 512, k =
// 3, 2.4 M 6.8 -> 5.9, 3 M 7.7 -> 6.5, 4 M 9.2 -> 8.2, 4.3 M 9.9 -> 10.0; C = 1024, k = 2, 3.9 M 8.3 -> 7.5, k = 5, 4 M 9.2 -> 8.0, k = 7, 3.5 M 9.0 -> 8.5, k = 11, 4 M
// 10.9 -> 10.2; from 1536 elements on later and for less than six: C = 2048, k = 3, 2.5 M 5.5 -> 5.6, 3 M 6.7 -> 6.1, 3.5 M 7.7 -> 6.9, 4 M 8.2 -> 8.1, k = 7, 3.9 M 9.2 ->
// 9.6; C = 4096, k = 2, 3.5 M 7.5 -> 6.4, k = 5, 2.7 M 7.2 -> 7.5, 3.9 M 8.5 -> 8.3, k = 7, 3.9 M 8.8 -> 9.1; C = 8192 nothing.  A single worker has nothing to be taken
// together with, and half the code is 2 to 5 % less time (C = 256, 3 M 8.3 -> 8.0).
static int sign_rest(int k, size_t groups, size_t waves)
{
    const int left = k % BAGUA_DRR_SIGN_NJ;
    if (left == 0) return kRestNone;
    if (k == 1 || BAGUA_DRR_SIGN_NJ > 8) return kRestOneByOne;
    const size_t at_once = kCus * (kWavesPerCu / waves) * waves, all = groups * waves;
    if (waves > 8 || all > at_once) return kRestTogether;
    if (waves <= 2) return all > at_once / 2 ? kRestOneByOne : kRestTogether;
    return left < 6 && all > at_once / 16 * 11 ? kRestOneByOne : kRestTogether;
}

// Expands `stmt` with a constexpr REST equal to the runtime value.
#define BAGUA_DISPATCH_REST(rest, stmt)                                                                                                          \
    switch (rest) {                                                                                                                              \
        case kRestNone: { constexpr int REST = kRestNone; stmt; } break;                                                                         \
        case kRestTogether: { constexpr int REST = BAGUA_DRR_SIGN_NJ <= 8 ? kRestTogether : kRestOneByOne; stmt; } break;   /* as sign_rest() */ \
        default: { constexpr int REST = kRestOneByOne; stmt; } break;                                                                            \
    }

int launch_drr_sign(const void* const* bits_in, const float* const* scale_in, int k, float* eps, size_t n,
                    size_t chunk, uint32_t* bits_out, float* scale_out, float* out, hipStream_t stream)
{
    PtrTable bt{}, st{};
    for (int j = 0; j < k; ++j) {
        bt.p[j] = bits_in[j];
        st.p[j] = scale_in[j];
    }
    const SignGeometry g = sign_geometry(n, chunk, BAGUA_RPW_DRR_SIGN, false);
    const int rest = sign_rest(k, g.grid.x, g.block.x / kWave);
    const float inv_k = 1.0f / static_cast<float>(k);
    const uint32_t ch = static_cast<uint32_t>(chunk);
#define BAGUA_DRR(EFv, OUTv)                                                                                      \
    BAGUA_DISPATCH_RPW(g.rpw, BAGUA_DISPATCH_REST(rest, launch_kernel((k_drr_sign<RPW, EFv, OUTv, REST>), g.grid, g.block, g.lds, stream, bt, \
                                                 st, k, inv_k, eps, n, ch, bits_out, scale_out, out)))
    if (eps && out) { BAGUA_DRR(true, true) }
    else if (eps) { BAGUA_DRR(true, false) }
    else if (out) { BAGUA_DRR(false, true) }
    else { BAGUA_DRR(false, false) }
#undef BAGUA_DRR
    return launch_status();
}

int launch_drr_sign_batched(const std::vector<uint64_t>& table, void* workspace, size_t B, int k, size_t chunk, bool ef,
                            bool with_out, hipStream_t stream)
{
    SignGeometry g = sign_geometry(chunk, chunk, BAGUA_RPW_DRR_SIGN, false);
    g.grid = dim3(static_cast<unsigned>(table[B]));
    const float inv_k = 1.0f / static_cast<float>(k);
    const uint32_t ch = static_cast<uint32_t>(chunk);
    const int rest = sign_rest(k, g.grid.x, g.block.x / kWave);
    return batch_launch(table, B, 5 + 2 * static_cast<size_t>(k), workspace, stream, [&](const auto& tab) {
        using TABLE = std::decay_t<decltype(tab)>;
#define BAGUA_DRR(EFv, OUTv)                                                                                       \
    BAGUA_DISPATCH_RPW(g.rpw, BAGUA_DISPATCH_REST(rest, launch_kernel((k_drr_sign_batched<RPW, EFv, OUTv, REST, TABLE>), g.grid, g.block, g.lds, stream, \
                                                 tab, k, inv_k, ch)))
        if (ef && with_out) { BAGUA_DRR(true, true) }
        else if (ef) { BAGUA_DRR(true, false) }
        else if (with_out) { BAGUA_DRR(false, true) }
        else { BAGUA_DRR(false, false) }
#undef BAGUA_DRR
    });
}

int launch_decompress_sign(const uint32_t* bits, const float* scale, size_t n, size_t chunk, float* out,
                           hipStream_t stream)
{
    const size_t rows = (n + kRow - 1) / kRow;
    dim3 grid(static_cast<unsigned>((rows + kRowWaves - 1) / kRowWaves)), block(kWave * kRowWaves);
    launch_kernel(k_decompress_sign, grid, block, 0, stream, bits, scale, n, static_cast<uint32_t>(chunk), out);
    return launch_status();
}

}  // namespace bagua

using namespace bagua;

extern "C" int bagua_sign_compress_ef(const float* x, float* residual, size_t n, size_t chunk, uint32_t* bits,
                                      float* scale, void* stream)
{
    if (!x || !bits || !scale || n == 0 || !chunk_ok(chunk)) return BAGUA_ERR_INVALID_ARG;
    RangeCheck rc;
    rc.reads(x, n * sizeof(float));
    rc.writes(residual, n * sizeof(float));
    rc.writes(bits, ((n + 31) / 32) * sizeof(uint32_t));
    rc.writes(scale, num_chunks(n, chunk) * sizeof(float));
    if (!rc.disjoint()) return BAGUA_ERR_INVALID_ARG;
    if (num_chunks(n, chunk) > kMaxGrid) return BAGUA_ERR_UNSUPPORTED;
    if (!aligned16(x) || !aligned16(residual) || !aligned16(bits) || !aligned4(scale)) return BAGUA_ERR_ALIGNMENT;
    return launch_sign_compress(x, residual, n, chunk, bits, scale, static_cast<hipStream_t>(stream));
}

extern "C" int bagua_momentum_sign_compress_ef(const float* g, const float* m, float beta1, float* residual, size_t n,
                                               size_t chunk, uint32_t* bits, float* scale, void* stream)
{
    if (!g || !m || !bits || !scale || n == 0 || !chunk_ok(chunk)) return BAGUA_ERR_INVALID_ARG;
    if (num_chunks(n, chunk) > kMaxGrid) return BAGUA_ERR_UNSUPPORTED;
    RangeCheck rc;
    rc.reads(g, n * sizeof(float));
    rc.reads(m, n * sizeof(float));
    rc.writes(residual, n * sizeof(float));
    rc.writes(bits, ((n + 31) / 32) * sizeof(uint32_t));
    rc.writes(scale, num_chunks(n, chunk) * sizeof(float));
    if (!rc.disjoint()) return BAGUA_ERR_INVALID_ARG;
    if (!aligned16(g) || !aligned16(m) || !aligned16(residual) || !aligned16(bits) || !aligned4(scale))
        return BAGUA_ERR_ALIGNMENT;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const SignGeometry geo = sign_geometry(n, chunk, BAGUA_RPW_SIGN, true);
    const uint32_t ch = static_cast<uint32_t>(chunk);
    const float omb1 = 1.0f - beta1;
    const ChunkOrder order = chunk_order(geo.grid.x, chunk, order_pays(n, chunk));
#define BAGUA_MOM(RPWv, EFv, MOMv, SHORTv)                                                                                      \
    launch_kernel((k_sign_compress<RPWv, EFv, MOMv, SHORTv>), geo.grid, geo.block, geo.lds, s, g, residual, n, ch, bits, scale, \
                       m, beta1, omb1, pace_for(n), mom_keep(chunk), order)
    if (mom_streams(n, geo.rpw, geo.block.x / kWave)) {
        if (residual) BAGUA_MOM(1, true, kMomStream, false);
        else BAGUA_MOM(1, false, kMomStream, false);
    } else if (residual) {
        BAGUA_DISPATCH_RPW_WORKER(geo.rpw, BAGUA_DISPATCH_SHORT(mom_fold(n), BAGUA_MOM(RPW, true, kMomKeep, SHORT)))
    } else {
        BAGUA_DISPATCH_RPW_WORKER(geo.rpw, BAGUA_DISPATCH_SHORT(mom_fold(n), BAGUA_MOM(RPW, false, kMomKeep, SHORT)))
    }
#undef BAGUA_MOM
    return launch_status();
}

extern "C" int bagua_sign_compress_ef_batched(const float* const* x, float* const* residual, const size_t* n, size_t B,
                                              size_t chunk, uint32_t* const* bits, float* const* scale, void* workspace,
                                              size_t workspace_bytes, void* stream)
{
    if (!x || !n || !bits || !scale || !workspace || B == 0 || B > 0xffffffffu || !chunk_ok(chunk))
        return BAGUA_ERR_INVALID_ARG;
    if (workspace_bytes < bagua_batch_workspace_bytes(B, 0)) return BAGUA_ERR_INVALID_ARG;
    if (!aligned16(workspace)) return BAGUA_ERR_ALIGNMENT;
    const bool ef = residual != nullptr;
    const size_t ew = 5;   // <= batch_entry_words_for(0)
    std::vector<uint64_t> table(batch_table_words(B, ew), 0);
    uint64_t* entries = table.data() + batch_first_words(B);
    RangeList rl;
    size_t total = 0;
    for (size_t b = 0; b < B; ++b) {
        if (!x[b] || !bits[b] || !scale[b] || n[b] == 0 || (ef && !residual[b])) return BAGUA_ERR_INVALID_ARG;
        float* r = ef ? residual[b] : nullptr;
        if (!aligned16(x[b]) || !aligned16(r) || !aligned16(bits[b]) || !aligned4(scale[b])) return BAGUA_ERR_ALIGNMENT;
        const size_t nc = num_chunks(n[b], chunk);
        rl.reads(x[b], n[b] * sizeof(float));
        rl.writes(r, n[b] * sizeof(float));
        rl.writes(bits[b], ((n[b] + 31) / 32) * sizeof(uint32_t));
        rl.writes(scale[b], nc * sizeof(float));
        table[b] = total;
        uint64_t* e = entries + b * ew;
        e[0] = reinterpret_cast<uintptr_t>(x[b]);
        e[1] = reinterpret_cast<uintptr_t>(r);
        e[2] = reinterpret_cast<uintptr_t>(bits[b]);
        e[3] = reinterpret_cast<uintptr_t>(scale[b]);
        e[4] = n[b];
        total += nc;
    }
    table[B] = total;
    batch_fill_lut(table.data(), B, ew);
    rl.writes(workspace, table.size() * sizeof(uint64_t));
    if (!rl.disjoint()) return BAGUA_ERR_INVALID_ARG;
    if (total > kMaxGrid) return BAGUA_ERR_UNSUPPORTED;
    hipStream_t s = static_cast<hipStream_t>(stream);
    SignGeometry g = sign_geometry(chunk, chunk, BAGUA_RPW_SIGN, false);
    g.grid = dim3(static_cast<unsigned>(total));
    const int groups = batched_groups(total * chunk, chunk, g.block.x);
    if (groups > 0) g.lds = lds_for_residency(groups);   // far more than the statistics need
    const uint32_t ch = static_cast<uint32_t>(chunk);
    return batch_launch(table, B, ew, workspace, s, [&](const auto& tab) {
        using TABLE = std::decay_t<decltype(tab)>;
        if (ef) {
            BAGUA_DISPATCH_RPW(g.rpw, BAGUA_DISPATCH_SHORT(groups > 0 || short_launch(total * chunk, true), launch_kernel(
                                          (k_sign_compress_batched<RPW, true, SHORT, TABLE>), g.grid, g.block, g.lds, s, tab, ch, pace_for(total * chunk), chunk_order(total, chunk, order_pays(total * chunk, chunk)))))
        } else {
            BAGUA_DISPATCH_RPW(g.rpw, BAGUA_DISPATCH_SHORT(groups > 0 || short_launch(total * chunk, true), launch_kernel(
                                          (k_sign_compress_batched<RPW, false, SHORT, TABLE>), g.grid, g.block, g.lds, s, tab, ch, pace_for(total * chunk), chunk_order(total, chunk, order_pays(total * chunk, chunk)))))
        }
    });
}
