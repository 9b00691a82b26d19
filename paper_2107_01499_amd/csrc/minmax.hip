// MinMax-u8 codec kernels: worker-side compress with error feedback, server-side
// decompress-average-recompress, and plain decompress (C_LP_S, Section 3.2 of the paper).
//
// All three are single-pass streaming kernels bound by HBM bandwidth: a chunk lives in
// registers between the statistics phase and the quantisation phase.
#include <type_traits>

#include "batch.hpp"
#include "launchers.hpp"
#include "minmax_device.hpp"

#pragma clang fp contract(off)

namespace bagua {

// ------------------------------------------------------------------------------------------
// Worker side: v = x (+ residual); codes = Q(v); residual <- v - decode.
// One workgroup per chunk, block = 64 * ceil(rows / RPW); c = index of the chunk in its bucket.
template <int RPW, bool EF, bool FULL>
__device__ __forceinline__ void compress_minmax_rows(const float* __restrict__ x, float* __restrict__ residual, int len,
                                                     uint8_t* __restrict__ codes, float* __restrict__ minmax_c, float* s_red, int pace, int keep)
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
    minmax_encode_chunk<RPW, EF, false, false, FULL>(v, len, wave, lane, nwaves, residual, codes, minmax_c, nullptr, s_red, keep);
}

// The chunk that is cut short, without tests (see row_at).  With -> without, us per launch: C = 4096, 64 K 3.1 -> 3.0, 1 M 4.8 -> 4.1, 3 M 8.4 -> 8.1;
// C = 16384, 1 M 7.0 -> 6.0; five buckets, 1 M 4.9 -> 4.6; above 6 M +-0.  (Chunks that are held in one row per wave gain nothing by it.)
template <int RPW, bool EF>
__device__ __forceinline__ void compress_minmax_cut(const float* __restrict__ x, float* __restrict__ residual, int len, uint8_t* __restrict__ codes,
                                                    float* __restrict__ minmax_c, float* s_red, int keep)
{
    const int wave = wave_index(), lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;
    f4 v[RPW], d[RPW];
    RowAt at[RPW];
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        at[i] = row_at<false>((wave * RPW + i) * kRow, len, lane);
        v[i] = load_at<false>(x, at[i]);
        if (EF) d[i] = load_at<false>(residual, at[i]);
    }
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        v[i] = settle<false>(v[i], at[i]);
        if (EF) {
            const f4 e = settle<false>(d[i], at[i]);
            v[i].x = v[i].x + e.x;
            v[i].y = v[i].y + e.y;
            v[i].z = v[i].z + e.z;
            v[i].w = v[i].w + e.w;
        }
    }
    minmax_encode_chunk<RPW, EF, false, false, false>(v, len, wave, lane, nwaves, residual, codes, minmax_c, nullptr, s_red, keep);
}

template <int RPW, bool EF, bool SHORT>
__device__ __forceinline__ void compress_minmax_chunk(const float* __restrict__ x, float* __restrict__ residual, size_t n,
                                                      uint32_t chunk, uint8_t* __restrict__ codes,
                                                      float* __restrict__ minmax, size_t c, float* s_red, int pace, int keep)
{
    const size_t base = c * static_cast<size_t>(chunk);
    const int len = static_cast<int>((n - base < chunk) ? (n - base) : chunk);
    float* res_c = EF ? residual + base : nullptr;
    if (SHORT && chunk_full<RPW>(len, blockDim.x >> 6))
        compress_minmax_rows<RPW, EF, true>(x + base, res_c, len, codes + base, minmax + 2 * c, s_red, 0, keep);
    else if (SHORT && RPW > 1 && len < static_cast<int>(chunk) && base + len >= 4)
        compress_minmax_cut<RPW, EF>(x + base, res_c, len, codes + base, minmax + 2 * c, s_red, keep);
    else compress_minmax_rows<RPW, EF, false>(x + base, res_c, len, codes + base, minmax + 2 * c, s_red, pace, keep);
}

template <int RPW, bool EF, bool SHORT>
__global__ void __launch_bounds__(wg_threads_max(RPW))
k_compress_minmax(const float* __restrict__ x, float* __restrict__ residual, size_t n, uint32_t chunk,
                  uint8_t* __restrict__ codes, float* __restrict__ minmax, int pace, uint32_t keep, ChunkOrder order)
{
    __shared__ float s_red[2 * kMaxWaves];
    compress_minmax_chunk<RPW, EF, SHORT>(x, residual, n, chunk, codes, minmax, order(blockIdx.x), s_red, pace, blockIdx.x < keep);
}

// Batched: entry = [x, residual, codes, minmax, n]; unit = chunk.
template <int RPW, bool EF, bool SHORT, typename TABLE>
__global__ void __launch_bounds__(wg_threads_max(RPW))
k_compress_minmax_batched(TABLE table, uint32_t chunk, int pace, uint32_t keep, ChunkOrder order)
{
    __shared__ float s_red[2 * kMaxWaves];
    const BatchView bv = table.view();
    const uint32_t unit = order(blockIdx.x), b = batch_find(bv, unit);
    const uint64_t* e = bv.entries + static_cast<size_t>(b) * bv.entry_words;
    compress_minmax_chunk<RPW, EF, SHORT>(table_ptr<const float>(e[0]), table_ptr<float>(e[1]), e[4], chunk,
                                   table_ptr<uint8_t>(e[2]), table_ptr<float>(e[3]),
                                   unit - bv.first_unit[b], s_red, pace, blockIdx.x < keep);
}

// ------------------------------------------------------------------------------------------
// Server side: a = (sum_j decode_j) * inv_k in ascending j; w = a (+ epsilon); then as above.
// SRC names the workers' inputs: code(j) -> u8 codes of worker j, meta(j) -> its (min, max) pairs.
struct DrrTableSrc {   // pointers in the kernel arguments
    const PtrTable& codes;
    const PtrTable& metas;
    __device__ __forceinline__ const void* code(int j) const { return codes.p[j]; }
    __device__ __forceinline__ const float* meta(int j) const { return static_cast<const float*>(metas.p[j]); }
};
struct DrrEntrySrc {   // pointers in a batch entry: [eps, codes_out, meta_out, out, n, code[0..k), meta[0..k)]
    const uint64_t* e;
    int k;
    __device__ __forceinline__ const void* code(int j) const { return table_ptr<const void>(e[5 + j]); }
    __device__ __forceinline__ const float* meta(int j) const { return table_ptr<const float>(e[5 + k + j]); }
};

// `base`, `len`: the chunk's first element and its length.  CUT: a chunk that is cut short, read without tests (row_at).
template <int RPW, bool EF, bool OUT, bool FULL, bool CUT, typename SRC>
__device__ __forceinline__ void drr_minmax_rows(const SRC& src, int k, float inv_k, float* __restrict__ eps, size_t base, int len,
                                                size_t c, uint8_t* __restrict__ codes_out, float* __restrict__ minmax_out,
                                                float* __restrict__ out, float* s_red, float* s_mn, float* s_step, int keep)
{
    const int wave = wave_index(), lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;

    // per-worker (min, step) of this chunk: one lane per worker, so the k divisions run side by side
    if (static_cast<int>(threadIdx.x) < k) {
        const float* m = src.meta(threadIdx.x);
        const float mn = m[2 * c], mx = m[2 * c + 1];
        s_mn[threadIdx.x] = mn;
        s_step[threadIdx.x] = minmax_step(mn, mx);
    }
    __syncthreads();

    f4 v[RPW];
    // workers are summed in ascending order
    for (int j = 0; j < k; ++j) {
        const uint8_t* cj = static_cast<const uint8_t*>(src.code(j)) + base;
        uint32_t w[RPW];
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int off = static_cast<int>(wave * RPW + i) * kRow;
            const int remain = row_remain<FULL>(len, off);
            w[i] = 0;
            if (CUT) w[i] = load_codes_at<false>(cj, row_at<false>(off, len, lane));
            else if (remain > 0) w[i] = load_codes_row(cj + off, lane, remain);
        }
        const float mn = s_mn[j], step = s_step[j];
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            if (CUT) w[i] = settle<false>(w[i], row_at<false>((wave * RPW + i) * kRow, len, lane));
            f4 d;
            d.x = mn + byte_to_float(w[i], 0) * step;
            d.y = mn + byte_to_float(w[i], 1) * step;
            d.z = mn + byte_to_float(w[i], 2) * step;
            d.w = mn + byte_to_float(w[i], 3) * step;
            if (j == 0) {
                v[i] = d;
            } else {
                v[i].x = v[i].x + d.x;
                v[i].y = v[i].y + d.y;
                v[i].z = v[i].z + d.z;
                v[i].w = v[i].w + d.w;
            }
        }
    }
    f4 e[RPW];
    if (EF) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int off = static_cast<int>(wave * RPW + i) * kRow;
            const int remain = row_remain<FULL>(len, off);
            e[i] = f4{0.f, 0.f, 0.f, 0.f};
            if (CUT) e[i] = load_at<false>(eps + base, row_at<false>(off, len, lane));
            else if (remain > 0) e[i] = load_row(eps + base + off, lane, remain, 0.0f);
        }
    }
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        if (EF && CUT) e[i] = settle<false>(e[i], row_at<false>((wave * RPW + i) * kRow, len, lane));
        v[i].x = v[i].x * inv_k;
        v[i].y = v[i].y * inv_k;
        v[i].z = v[i].z * inv_k;
        v[i].w = v[i].w * inv_k;
        if (EF && row_remain<FULL>(len, static_cast<int>(wave * RPW + i) * kRow) > 0) {
            v[i].x = v[i].x + e[i].x;
            v[i].y = v[i].y + e[i].y;
            v[i].z = v[i].z + e[i].z;
            v[i].w = v[i].w + e[i].w;
        }
    }
    minmax_encode_chunk<RPW, EF, OUT, false, FULL>(v, len, wave, lane, nwaves, EF ? eps + base : nullptr, codes_out + base,
                                                   minmax_out + 2 * c, OUT ? out + base : nullptr, s_red, keep);
}

// The same in a launch whose time is a workgroup's latency and not the memory's rate: the codes of the first F workers and the error
// state are requested before the workers' statistics are waited for, and then always F workers ahead.
template <int RPW, bool EF, bool OUT, bool FULL, typename SRC>
__device__ __forceinline__ void drr_minmax_rows_ahead(const SRC& src, int k, float inv_k, float* __restrict__ eps, size_t base, int len,
                                                      size_t c, uint8_t* __restrict__ codes_out, float* __restrict__ minmax_out,
                                                      float* __restrict__ out, float* s_red, float* s_mn, float* s_step, int keep)
{
    constexpr int F = 8 / RPW;
    const int wave = wave_index(), lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;
    RowAt at[RPW];
#pragma unroll
    for (int i = 0; i < RPW; ++i) at[i] = row_at<FULL>((wave * RPW + i) * kRow, len, lane);
    uint32_t w[F][RPW];
    auto fetch = [&](int g, int j) {
        const uint8_t* cj = static_cast<const uint8_t*>(src.code(j)) + base;
#pragma unroll
        for (int i = 0; i < RPW; ++i) w[g][i] = load_codes_at<FULL>(cj, at[i]);
    };
    float mn = 0.0f, mx = 0.0f;
    if (static_cast<int>(threadIdx.x) < k) {
        const float* m = src.meta(threadIdx.x);
        mn = m[2 * c];
        mx = m[2 * c + 1];
    }
#pragma unroll
    for (int g = 0; g < F; ++g)
        if (g < k) fetch(g, g);
    f4 e[RPW];
    if (EF) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) e[i] = load_at<FULL>(eps + base, at[i]);
    }
    if (static_cast<int>(threadIdx.x) < k) {
        s_mn[threadIdx.x] = mn;
        s_step[threadIdx.x] = minmax_step(mn, mx);
    }
    __syncthreads();

    f4 v[RPW];
    for (int j0 = 0; j0 < k; j0 += F) {
#pragma unroll
        for (int g = 0; g < F; ++g) {
            const int j = j0 + g;
            if (j >= k) break;
            const float mnj = s_mn[j], step = s_step[j];
#pragma unroll
            for (int i = 0; i < RPW; ++i) {
                const uint32_t wi = settle<FULL>(w[g][i], at[i]);
                f4 d;
                d.x = mnj + byte_to_float(wi, 0) * step;
                d.y = mnj + byte_to_float(wi, 1) * step;
                d.z = mnj + byte_to_float(wi, 2) * step;
                d.w = mnj + byte_to_float(wi, 3) * step;
                if (j == 0) {
                    v[i] = d;
                } else {
                    v[i].x = v[i].x + d.x;
                    v[i].y = v[i].y + d.y;
                    v[i].z = v[i].z + d.z;
                    v[i].w = v[i].w + d.w;
                }
            }
            if (j + F < k) fetch(g, j + F);
        }
    }
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        v[i].x = v[i].x * inv_k;
        v[i].y = v[i].y * inv_k;
        v[i].z = v[i].z * inv_k;
        v[i].w = v[i].w * inv_k;
        if (EF) {
            const f4 ei = settle<FULL>(e[i], at[i]);
            v[i].x = v[i].x + ei.x;
            v[i].y = v[i].y + ei.y;
            v[i].z = v[i].z + ei.z;
            v[i].w = v[i].w + ei.w;
        }
    }
    minmax_encode_chunk<RPW, EF, OUT, false, FULL>(v, len, wave, lane, nwaves, EF ? eps + base : nullptr, codes_out + base,
                                                   minmax_out + 2 * c, OUT ? out + base : nullptr, s_red, keep);
}

// How a complete chunk is read: row after row (kDrrTests), its rows at once (kDrrFold), the same with a body of its own for the chunk
// that is cut short (kDrrFoldCut), or workers ahead (kDrrAhead).
enum DrrForm { kDrrTests, kDrrFold, kDrrFoldCut, kDrrAhead };

template <int RPW, bool EF, bool OUT, int FORM, typename SRC>
__device__ __forceinline__ void drr_minmax_chunk(const SRC& src, int k, float inv_k, float* __restrict__ eps, size_t n,
                                                 uint32_t chunk, uint8_t* __restrict__ codes_out,
                                                 float* __restrict__ minmax_out, float* __restrict__ out, size_t c,
                                                 float* s_red, float* s_mn, float* s_step, int keep)
{
    const size_t base = c * static_cast<size_t>(chunk);
    const int len = static_cast<int>((n - base < chunk) ? (n - base) : chunk);
    const bool full = chunk_full<RPW>(len, blockDim.x >> 6), cut = len < static_cast<int>(chunk) && base + len >= 4;
    if (FORM == kDrrAhead && full)
        drr_minmax_rows_ahead<RPW, EF, OUT, true>(src, k, inv_k, eps, base, len, c, codes_out, minmax_out, out, s_red, s_mn, s_step, keep);
    else if (FORM == kDrrAhead)
        drr_minmax_rows_ahead<RPW, EF, OUT, false>(src, k, inv_k, eps, base, len, c, codes_out, minmax_out, out, s_red, s_mn, s_step, keep);
    else if ((FORM == kDrrFold || FORM == kDrrFoldCut) && full)
        drr_minmax_rows<RPW, EF, OUT, true, false>(src, k, inv_k, eps, base, len, c, codes_out, minmax_out, out, s_red, s_mn, s_step, keep);
    else if (FORM == kDrrFoldCut && cut)
        drr_minmax_rows<RPW, EF, OUT, false, true>(src, k, inv_k, eps, base, len, c, codes_out, minmax_out, out, s_red, s_mn, s_step, keep);
    else drr_minmax_rows<RPW, EF, OUT, false, false>(src, k, inv_k, eps, base, len, c, codes_out, minmax_out, out, s_red, s_mn, s_step, keep);
}

// Whether the server step folds the tail tests of complete chunks away.  With the tests a wave waits for one row's
// codes before it requests the next; four rows per wave make that a long chain.  Folded away against kept:
//   chunks above 4096 (8 or 16 waves): 16 workers x 335 M, C = 8192, 1443 -> 1341 us; 25.7 M 118 -> 105 us; 3 x 16.8 M,
//   C = 16384, 48 -> 38 us;
//   chunks up to 4096: 8 workers x 25.7 M, C = 4096, 92.5 -> 87.8 us, 2 workers, C = 2048, 52.6 -> 47.5 us, 16 x 33 M
//   137 -> 135 us; but with many code streams and more elements the slower chain streams better: 16 x 50 M 199 -> 206 us,
//   8 x 134 M 361 -> 369 us, against 242 -> 233 us with two workers.
inline bool drr_minmax_fold(size_t elements, size_t chunk, int k)
{
    return chunk > 4096 || k <= 4 || elements < (static_cast<size_t>(1) << 25);
}
// Whether the workers' codes are requested ahead: up to 2^22 elements of chunks up to 8192, where the launch is too short to be bound by HBM
// (14 bytes an element with k = 4), and up to 2^26 where four rows per wave leave a wave with two; an odd number of rows fills its waves
// with one row each only, up to 2^20 elements and 11 rows.  Four rows per wave and one worker at a time -> this, us of one launch (from a
// graph, four sets of buffers in turn):
//   k = 4, C = 4096: 64 K 4.2 -> 3.3, 1 M 6.3 -> 4.4, 2 M 7.8 -> 6.2, 4 M 11.2 -> 11.0;   k = 8, C = 2048: 64 K 5.0 -> 3.4, 1 M 9.1 -> 5.4, 2 M
//   10.9 -> 7.8, 4 M 14.8 -> 14.6;   k = 16, C = 8192: 64 K 7.4 -> 6.3, 1 M 14.2 -> 8.5, 2 M 16.5 -> 10.5, 4 M 20.9 -> 20.7;
//   outside: k = 16, C = 8192, 8 M 40.0 -> 41.4; k = 8, C = 3072, 6 M 20.9 -> 23.3; k = 8, C = 2048, 16 M 48.8 -> 49.8.  Chunks above 8192 take
//   four rows either way: C = 16384, k = 8, 64 K 6.7 -> 6.9, 400 K 9.0 -> 7.9, 1 M 10.7 -> 8.8, 2 M 11.6 -> 9.6, 3 M 13.6 -> 14.2; k = 16, 2 M 17.7 -> 13.3.
//   C = 1536, k = 5: 12 M 35.2 -> 31.8, 33 M 82.4 -> 73.7, 67 M 155.4 -> 150.9, 134 M 310.8 -> 324.7; C = 2560, k = 8: 12 M 43.0 -> 38.6, 67 M
//   189.0 -> 182.1, 134 M 377.8 -> 396.5.
inline bool drr_minmax_ahead(size_t n, size_t chunk, size_t least)
{
    const size_t rows = chunk / kRow;
    if (least < 4) return false;   // row_at
    if (rows % 2 != 0) return rows <= 12 && n <= (static_cast<size_t>(1) << 20);
    if (chunk > 8192) return rows % 4 == 0 && n > (static_cast<size_t>(1) << 18) && n <= (static_cast<size_t>(1) << 21);
    return n <= (static_cast<size_t>(1) << (rows % 4 == 2 ? 26 : 22));
}
// Rows per wave then: one in the shortest launches of chunks up to 3072 (two -> one: k = 16, C = 1536, 64 K 6.7 -> 5.6, 512 K 10.7 -> 9.9; k = 8,
// C = 2048, 1 M 5.7 -> 5.4, 2 M 7.8 -> 7.9), which is also how an odd number of rows fills its waves.
inline int drr_minmax_ahead_rpw(size_t n, size_t chunk)
{
    return chunk > 8192 ? 4 : chunk <= 12 * kRow && n <= (static_cast<size_t>(1) << 20) ? 1 : 2;
}

// The body of its own for the chunk cut short, which a workgroup otherwise spends 8 us on at the very end: up to 2^26 elements.  k = 8, C = 2048, 5 M
// 20.9 -> 16.8 us, 9 M 31.2 -> 29.6; k = 16, C = 8192, 5 M 30.7 -> 23.5, 9 M 46.1 -> 41.9, 20 M 86.4 -> 84.7; five buckets of 1.8 M, k = 8, C =
// 16384, 47.2 -> 41.2.  In longer launches, and in those with tests, the third body's registers cost more than it gives (k = 12, C = 1536,
// five buckets, 625.8 -> 659.1: 97 scalar registers instead of 86, seven waves per SIMD).
inline bool drr_minmax_cut(size_t elements) { return elements <= (static_cast<size_t>(1) << 26); }

template <int V>
using Const = std::integral_constant<int, V>;
// launch(rows per wave, form, workgroup) for n elements, the first two as types; least: of the shortest bucket.
template <typename F>
inline void drr_minmax_shape(size_t n, size_t least, size_t chunk, int k, const F& launch)
{
    const int rows = static_cast<int>(chunk / kRow);
    const bool ahead = drr_minmax_ahead(n, chunk, least), fold = drr_minmax_fold(n, chunk, k);
    const int rpw = ahead ? drr_minmax_ahead_rpw(n, chunk) : pick_rpw(rows, BAGUA_RPW_DRR);
    const dim3 block(kWave * ((rows + rpw - 1) / rpw));
    if (ahead && rpw == 1) launch(Const<1>{}, Const<kDrrAhead>{}, block);
    else if (ahead && rpw == 2) launch(Const<2>{}, Const<kDrrAhead>{}, block);
    else if (ahead) launch(Const<4>{}, Const<kDrrAhead>{}, block);
    else if (rpw == 2) launch(Const<2>{}, Const<kDrrTests>{}, block);
    else if (fold && drr_minmax_cut(n)) launch(Const<4>{}, Const<kDrrFoldCut>{}, block);
    else if (fold) launch(Const<4>{}, Const<kDrrFold>{}, block);
    else launch(Const<4>{}, Const<kDrrTests>{}, block);
}

template <int RPW, bool EF, bool OUT, int FORM>
__global__ void __launch_bounds__(wg_threads_max(RPW))
k_drr_minmax(PtrTable codes_in, PtrTable meta_in, int k, float inv_k, float* __restrict__ eps, size_t n,
             uint32_t chunk, uint8_t* __restrict__ codes_out, float* __restrict__ minmax_out,
             float* __restrict__ out, int keep)
{
    __shared__ float s_red[2 * kMaxWaves];
    __shared__ float s_mn[BAGUA_MAX_WORKERS], s_step[BAGUA_MAX_WORKERS];
    drr_minmax_chunk<RPW, EF, OUT, FORM>(DrrTableSrc{codes_in, meta_in}, k, inv_k, eps, n, chunk, codes_out, minmax_out, out,
                                   blockIdx.x, s_red, s_mn, s_step, keep);
}

template <int RPW, bool EF, bool OUT, int FORM, typename TABLE>
__global__ void __launch_bounds__(wg_threads_max(RPW))
k_drr_minmax_batched(TABLE table, int k, float inv_k, uint32_t chunk, int keep)
{
    __shared__ float s_red[2 * kMaxWaves];
    __shared__ float s_mn[BAGUA_MAX_WORKERS], s_step[BAGUA_MAX_WORKERS];
    const BatchView bv = table.view();
    const uint32_t b = batch_find(bv, blockIdx.x);
    const uint64_t* e = bv.entries + static_cast<size_t>(b) * bv.entry_words;
    drr_minmax_chunk<RPW, EF, OUT, FORM>(DrrEntrySrc{e, k}, k, inv_k, table_ptr<float>(e[0]), e[4], chunk,
                                   table_ptr<uint8_t>(e[1]), table_ptr<float>(e[2]),
                                   table_ptr<float>(e[3]), blockIdx.x - bv.first_unit[b], s_red, s_mn, s_step, keep);
}

// ------------------------------------------------------------------------------------------
// Decode: out = mn + code * step.  One wave per row, 4 rows per workgroup.
__global__ void __launch_bounds__(kWave * kRowWaves)
k_decompress_minmax(const uint8_t* __restrict__ codes, const float* __restrict__ minmax, size_t n,
                    uint32_t chunk, float* __restrict__ out)
{
    const size_t row = static_cast<size_t>(blockIdx.x) * kRowWaves + wave_index();
    const int lane = threadIdx.x & 63;
    const size_t e0 = row * kRow;
    if (e0 >= n) return;
    const size_t c = e0 / chunk;
    const float mn = minmax[2 * c], step = minmax_step(mn, minmax[2 * c + 1]);
    const int remain = static_cast<int>((n - e0 < static_cast<size_t>(kRow)) ? (n - e0) : kRow);
    const uint32_t w = load_codes_row(codes + e0, lane, remain);
    f4 d;
    d.x = mn + byte_to_float(w, 0) * step;
    d.y = mn + byte_to_float(w, 1) * step;
    d.z = mn + byte_to_float(w, 2) * step;
    d.w = mn + byte_to_float(w, 3) * step;
    store_row(out + e0, lane, remain, d);
}

// ------------------------------------------------------------------------------------------ host
int launch_compress_minmax(const float* x, float* residual, size_t n, size_t chunk, uint8_t* codes,
                           float* minmax, hipStream_t stream)
{
    const int rows = static_cast<int>(chunk / kRow);
    const int rpw = pick_rpw_worker(rows, BAGUA_RPW_COMPRESS);
    dim3 grid(static_cast<unsigned>(num_chunks(n, chunk))), block(64 * ((rows + rpw - 1) / rpw));
    const uint32_t ch = static_cast<uint32_t>(chunk);
    if (residual) {
        BAGUA_DISPATCH_RPW_WORKER(rpw, BAGUA_DISPATCH_SHORT(short_launch(n), launch_kernel((k_compress_minmax<RPW, true, SHORT>), grid, block, 0,
                                                                                 stream, x, residual, n, ch, codes, minmax, pace_for(n), keep_chunks(n, chunk), chunk_order(grid.x, chunk, order_pays(n, chunk)))))
    } else {
        BAGUA_DISPATCH_RPW_WORKER(rpw, BAGUA_DISPATCH_SHORT(short_launch(n), launch_kernel((k_compress_minmax<RPW, false, SHORT>), grid, block, 0,
                                                                                 stream, x, residual, n, ch, codes, minmax, pace_for(n), keep_chunks(n, chunk), chunk_order(grid.x, chunk, order_pays(n, chunk)))))
    }
    return launch_status();
}

int launch_drr_minmax(const void* const* codes_in, const float* const* meta_in, int k, float* eps, size_t n,
                      size_t chunk, uint8_t* codes_out, float* minmax_out, float* out, hipStream_t stream)
{
    PtrTable ct{}, mt{};
    for (int j = 0; j < k; ++j) {
        ct.p[j] = codes_in[j];
        mt.p[j] = meta_in[j];
    }
    const dim3 grid(static_cast<unsigned>(num_chunks(n, chunk)));
    const float inv_k = 1.0f / static_cast<float>(k);
    const uint32_t ch = static_cast<uint32_t>(chunk);
    drr_minmax_shape(n, n, chunk, k, [&](auto rpw, auto form, dim3 block) {
        constexpr int RPW = decltype(rpw)::value, FORM = decltype(form)::value;
#define BAGUA_DRR(EFv, OUTv)                                                                                     \
    launch_kernel((k_drr_minmax<RPW, EFv, OUTv, FORM>), grid, block, 0, stream, ct, mt, k, inv_k, eps, n, ch, \
                       codes_out, minmax_out, out, keep_server_codes(n))
        if (eps && out) BAGUA_DRR(true, true);
        else if (eps) BAGUA_DRR(true, false);
        else if (out) BAGUA_DRR(false, true);
        else BAGUA_DRR(false, false);
#undef BAGUA_DRR
    });
    return launch_status();
}

int launch_drr_minmax_batched(const std::vector<uint64_t>& table, void* workspace, size_t B, int k, size_t chunk, bool ef,
                              bool with_out, hipStream_t stream)
{
    const dim3 grid(static_cast<unsigned>(table[B]));
    const float inv_k = 1.0f / static_cast<float>(k);
    const uint32_t ch = static_cast<uint32_t>(chunk);
    const size_t n = table[B] * chunk;
    size_t least = n;
    for (size_t b = 0; b < B; ++b) least = std::min<size_t>(least, table[batch_first_words(B) + b * (5 + 2 * static_cast<size_t>(k)) + 4]);
    return batch_launch(table, B, 5 + 2 * static_cast<size_t>(k), workspace, stream, [&](const auto& tab) {
        using TABLE = std::decay_t<decltype(tab)>;
        drr_minmax_shape(n, least, chunk, k, [&](auto rpw, auto form, dim3 block) {
            constexpr int RPW = decltype(rpw)::value, FORM = decltype(form)::value;
#define BAGUA_DRR(EFv, OUTv)                                                                                              \
    launch_kernel((k_drr_minmax_batched<RPW, EFv, OUTv, FORM, TABLE>), grid, block, 0, stream, tab, k, inv_k, ch, \
                       keep_server_codes(n))
            if (ef && with_out) BAGUA_DRR(true, true);
            else if (ef) BAGUA_DRR(true, false);
            else if (with_out) BAGUA_DRR(false, true);
            else BAGUA_DRR(false, false);
#undef BAGUA_DRR
        });
    });
}

int launch_decompress_minmax(const uint8_t* codes, const float* minmax, size_t n, size_t chunk, float* out,
                             hipStream_t stream)
{
    const size_t rows = (n + kRow - 1) / kRow;
    dim3 grid(static_cast<unsigned>((rows + kRowWaves - 1) / kRowWaves)), block(kWave * kRowWaves);
    launch_kernel(k_decompress_minmax, grid, block, 0, stream, codes, minmax, n,
                       static_cast<uint32_t>(chunk), out);
    return launch_status();
}

}  // namespace bagua

using namespace bagua;

extern "C" int bagua_compress_minmax_u8(const float* x, float* residual, size_t n, size_t chunk,
                                        uint8_t* codes, float* minmax, void* stream)
{
    if (!x || !codes || !minmax || n == 0 || !chunk_ok(chunk)) return BAGUA_ERR_INVALID_ARG;
    RangeCheck rc;
    rc.reads(x, n * sizeof(float));
    rc.writes(residual, n * sizeof(float));
    rc.writes(codes, n);
    rc.writes(minmax, 2 * num_chunks(n, chunk) * sizeof(float));
    if (!rc.disjoint()) return BAGUA_ERR_INVALID_ARG;
    if (num_chunks(n, chunk) > kMaxGrid) return BAGUA_ERR_UNSUPPORTED;
    if (!aligned16(x) || !aligned16(residual) || !aligned16(codes) || !aligned4(minmax)) return BAGUA_ERR_ALIGNMENT;
    return launch_compress_minmax(x, residual, n, chunk, codes, minmax, static_cast<hipStream_t>(stream));
}

extern "C" int bagua_compress_minmax_u8_batched(const float* const* x, float* const* residual, const size_t* n, size_t B,
                                                size_t chunk, uint8_t* const* codes, float* const* minmax,
                                                void* workspace, size_t workspace_bytes, void* stream)
{
    if (!x || !n || !codes || !minmax || !workspace || B == 0 || B > 0xffffffffu || !chunk_ok(chunk))
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
        if (!x[b] || !codes[b] || !minmax[b] || n[b] == 0 || (ef && !residual[b])) return BAGUA_ERR_INVALID_ARG;
        float* r = ef ? residual[b] : nullptr;
        if (!aligned16(x[b]) || !aligned16(r) || !aligned16(codes[b]) || !aligned4(minmax[b])) return BAGUA_ERR_ALIGNMENT;
        const size_t nc = num_chunks(n[b], chunk);
        rl.reads(x[b], n[b] * sizeof(float));
        rl.writes(r, n[b] * sizeof(float));
        rl.writes(codes[b], n[b]);
        rl.writes(minmax[b], 2 * nc * sizeof(float));
        table[b] = total;
        uint64_t* e = entries + b * ew;
        e[0] = reinterpret_cast<uintptr_t>(x[b]);
        e[1] = reinterpret_cast<uintptr_t>(r);
        e[2] = reinterpret_cast<uintptr_t>(codes[b]);
        e[3] = reinterpret_cast<uintptr_t>(minmax[b]);
        e[4] = n[b];
        total += nc;
    }
    table[B] = total;
    batch_fill_lut(table.data(), B, ew);
    rl.writes(workspace, table.size() * sizeof(uint64_t));
    if (!rl.disjoint()) return BAGUA_ERR_INVALID_ARG;
    if (total > kMaxGrid) return BAGUA_ERR_UNSUPPORTED;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int rows = static_cast<int>(chunk / kRow);
    const int rpw = pick_rpw(rows, BAGUA_RPW_COMPRESS);
    dim3 grid(static_cast<unsigned>(total)), block(64 * ((rows + rpw - 1) / rpw));
    const uint32_t ch = static_cast<uint32_t>(chunk);
    const int groups = batched_groups(total * chunk, chunk, block.x);
    const size_t lds = groups > 0 ? lds_for_residency(groups, 2 * kMaxWaves * sizeof(float)) : 0;
    const bool is_short = short_launch(total * chunk, true);
    const uint32_t keep = is_short ? static_cast<uint32_t>(total) : keep_chunks(total * chunk, chunk);   // a short launch keeps all its codes
    return batch_launch(table, B, ew, workspace, s, [&](const auto& tab) {
        using TABLE = std::decay_t<decltype(tab)>;
        if (ef) {
            BAGUA_DISPATCH_RPW(rpw, BAGUA_DISPATCH_SHORT(groups > 0 || is_short, launch_kernel(
                                        (k_compress_minmax_batched<RPW, true, SHORT, TABLE>), grid, block, lds, s, tab, ch, pace_for(total * chunk), keep, chunk_order(total, chunk, order_pays(total * chunk, chunk)))))
        } else {
            BAGUA_DISPATCH_RPW(rpw, BAGUA_DISPATCH_SHORT(groups > 0 || is_short, launch_kernel(
                                        (k_compress_minmax_batched<RPW, false, SHORT, TABLE>), grid, block, lds, s, tab, ch, pace_for(total * chunk), keep, chunk_order(total, chunk, order_pays(total * chunk, chunk)))))
        }
    });
}
