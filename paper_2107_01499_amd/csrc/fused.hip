// Flatten fused into the worker-side MinMax-u8 compression: the rows of a chunk are gathered
// straight from the layer tensors (through the planned tensor table), so the flattened bucket is
// never written to and re-read from HBM.  Result = bagua_bucket_flatten followed by
// bagua_compress_minmax_u8, bit for bit; traffic = that of the compression alone.
#include <type_traits>

#include "flatten_device.hpp"
#include "launchers.hpp"
#include "minmax_device.hpp"
#include "sign_device.hpp"

#pragma clang fp contract(off)

namespace bagua {

// Rows per wave of the gathers: one up to 2^21 elements of chunks up to 4096, because a wave walks through the tensor table row after row.  Two -> one,
// us per launch: MinMax, C = 4096, 64 K 4.3 -> 4.1, 1 M 5.8 -> 5.0, 2 M 7.4 -> 6.6, 4 M 11.2 -> 12.3; C = 1024, 64 K 4.2 -> 3.7, 1 M 5.6 -> 4.8, 2 M 7.2
// -> 6.2; sign codec, C = 4096, 64 K 4.3 -> 4.0, 1 M 5.9 -> 4.7, 2 M 7.1 -> 5.8, 4 M 10.2 -> 11.0.  Workgroups that do not fill a CU's 32 waves up to
// 2^20: C = 3072, MinMax, 1 M 5.6 -> 5.0, 1.6 M 6.4 -> 6.7, sign codec, 1 M 5.7 -> 4.8, 1.6 M 6.4 -> 6.2 but 0.5 % of a round of 12 x 1.6 M more.
// A build that prefers four rows gets them at any size.
inline int pick_rpw_gather(int rows, size_t n, int preferred)
{
    const size_t most = static_cast<size_t>(1) << (kWavesPerCu % rows == 0 ? 21 : 20);
    return preferred == 2 && rows <= kMaxWaves && n <= most ? 1 : pick_rpw_worker(rows, preferred);
}

template <int RPW, bool EF, bool WB>
__global__ void __launch_bounds__(wg_threads_max(RPW))
k_flatten_compress_minmax(const TensorDesc* __restrict__ desc, const uint32_t* __restrict__ tile_first, uint32_t T,
                          float* __restrict__ residual, size_t n, uint32_t chunk, uint8_t* __restrict__ codes,
                          float* __restrict__ minmax, float* __restrict__ bucket_out, uint32_t keep, ChunkOrder order)
{
    __shared__ float s_red[2 * kMaxWaves];
    const size_t c = order(blockIdx.x);
    const size_t base = c * static_cast<size_t>(chunk);
    const int len = static_cast<int>((n - base < chunk) ? (n - base) : chunk);
    const int wave = wave_index(), lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;

    // the error state does not depend on the table lookups: get its loads going first
    f4 d[RPW];
    if (EF) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int off = static_cast<int>(wave * RPW + i) * kRow;
            const int remain = len - off;
            d[i] = f4{0.f, 0.f, 0.f, 0.f};
            if (remain > 0) d[i] = load_row(residual + base + off, lane, remain, 0.0f);
        }
    }
    f4 v[RPW];
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        const int off = static_cast<int>(wave * RPW + i) * kRow;
        const int remain = len - off;
        v[i] = f4{0.f, 0.f, 0.f, 0.f};
        if (remain > 0) {
            v[i] = gather_row(desc, tile_first, T, base + off, lane, remain);
            if (WB) store_row(bucket_out + base + off, lane, remain, v[i]);
        }
    }
    if (EF) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            v[i].x = v[i].x + d[i].x;
            v[i].y = v[i].y + d[i].y;
            v[i].z = v[i].z + d[i].z;
            v[i].w = v[i].w + d[i].w;
        }
    }
    minmax_encode_chunk<RPW, EF, false>(v, len, wave, lane, nwaves, EF ? residual + base : nullptr,
                                        codes + base, minmax + 2 * c, nullptr, s_red, blockIdx.x < keep);
}

// The same gather in front of the 1-bit sign codec: bagua_bucket_flatten followed by bagua_sign_compress_ef.
template <int RPW, bool EF, bool WB>
__global__ void __launch_bounds__(wg_threads_max(RPW))
k_flatten_sign_compress(const TensorDesc* __restrict__ desc, const uint32_t* __restrict__ tile_first, uint32_t T,
                        float* __restrict__ residual, size_t n, uint32_t chunk, uint32_t* __restrict__ bits,
                        float* __restrict__ scale, float* __restrict__ bucket_out, ChunkOrder order)
{
    extern __shared__ float s_q[];
    const size_t c = order(blockIdx.x);
    const size_t base = c * static_cast<size_t>(chunk);
    const int len = static_cast<int>((n - base < chunk) ? (n - base) : chunk);
    const int wave = wave_index(), lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;

    f4 d[RPW];
    if (EF) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int off = static_cast<int>(wave * RPW + i) * kRow;
            const int remain = len - off;
            d[i] = f4{0.f, 0.f, 0.f, 0.f};
            if (remain > 0) d[i] = load_row(residual + base + off, lane, remain, 0.0f);
        }
    }
    f4 v[RPW];
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        const int off = static_cast<int>(wave * RPW + i) * kRow;
        const int remain = len - off;
        v[i] = f4{0.f, 0.f, 0.f, 0.f};
        if (remain > 0) {
            v[i] = gather_row(desc, tile_first, T, base + off, lane, remain);
            if (WB) store_row(bucket_out + base + off, lane, remain, v[i]);
        }
    }
    if (EF) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            v[i].x = v[i].x + d[i].x;
            v[i].y = v[i].y + d[i].y;
            v[i].z = v[i].z + d[i].z;
            v[i].w = v[i].w + d[i].w;
        }
    }
    sign_encode_chunk<RPW, EF, false>(v, len, chunk, wave, lane, nwaves, EF ? residual + base : nullptr,
                                      bits + (base >> 5), scale + c, nullptr, s_q);
}

// The average of the k_local workers' rows and the error state on top, in a short launch: eight rows of the workers (what fits 32
// registers) and the error state are on their way at any time, without tests, and so is the chunk that is cut short.  What a lane holds
// beyond the end of the chunk means nothing.
template <int RPW, bool EF, bool FULL>
__device__ __forceinline__ void average_rows_ahead(const PtrTable& xs, int k_local, float inv_k, const float* residual_c, size_t base, int len, int wave,
                                                   int lane, f4 (&v)[RPW])
{
    constexpr int U = 8 / RPW;
    RowAt at[RPW];
#pragma unroll
    for (int i = 0; i < RPW; ++i) at[i] = row_at<FULL>((wave * RPW + i) * kRow, len, lane);
    f4 w[U][RPW];
    auto fetch = [&](int u, int j) {
        const float* xj = static_cast<const float*>(xs.p[j]) + base;
#pragma unroll
        for (int i = 0; i < RPW; ++i) w[u][i] = load_at<FULL>(xj, at[i]);
    };
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (u < k_local) fetch(u, u);
    f4 d[RPW];
    if (EF) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) d[i] = load_at<FULL>(residual_c, at[i]);
    }
    for (int j0 = 0; j0 < k_local; j0 += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = j0 + u;
            if (j >= k_local) break;
#pragma unroll
            for (int i = 0; i < RPW; ++i) {
                const f4 a = settle<FULL>(w[u][i], at[i]);
                if (j == 0) {
                    v[i] = a;
                } else {
                    v[i].x = v[i].x + a.x;
                    v[i].y = v[i].y + a.y;
                    v[i].z = v[i].z + a.z;
                    v[i].w = v[i].w + a.w;
                }
            }
            if (j + U < k_local) fetch(u, j + U);
        }
    }
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        v[i].x = v[i].x * inv_k;
        v[i].y = v[i].y * inv_k;
        v[i].z = v[i].z * inv_k;
        v[i].w = v[i].w * inv_k;
        if (EF) {
            const f4 e = settle<FULL>(d[i], at[i]);
            v[i].x = v[i].x + e.x;
            v[i].y = v[i].y + e.y;
            v[i].z = v[i].z + e.z;
            v[i].w = v[i].w + e.w;
        }
    }
}

// Up to 2^20 elements of chunks up to 8192.  Worker after worker -> this, us per launch: MinMax, 8 workers, C = 4096, 64 K 4.7 -> 4.1 (cut chunk
// 7.4 -> 5.2), 256 K 8.5 -> 5.8, 1 M 10.2 -> 8.7, 2 M 14.7 -> 16.0; 4 workers, C = 8192, 1 M 7.9 -> 7.2, 2 M 9.9 -> 12.7; sign codec, 4 workers, C =
// 2048, 64 K 3.3 -> 2.9, 256 K 4.6 -> 3.5, 1 M 5.9 -> 5.5, 2 M 9.2 -> 9.4.  C = 16384 (four rows per wave, 128 registers): 64 K 12.8 -> 16.5.
inline bool short_average(size_t n, size_t chunk) { return n >= 4 && n <= (static_cast<size_t>(1) << 20) && chunk <= 8192; }
// launch(rows per wave, whether it is a short launch), both as types.  Short chunks take one row per wave then.  There is no short form for a build
// that prefers four rows.
template <typename F>
inline void average_shape(size_t n, size_t chunk, int preferred, const F& launch)
{
    const int rows = static_cast<int>(chunk / kRow);
    if (preferred != 2 || !short_average(n, chunk)) {
        BAGUA_DISPATCH_RPW_WORKER(pick_rpw_worker(rows, preferred), (launch(std::integral_constant<int, RPW>{}, std::false_type{})))
    } else if (rows <= kMaxWaves) {
        launch(std::integral_constant<int, 1>{}, std::true_type{});
    } else {
        launch(std::integral_constant<int, 2>{}, std::true_type{});
    }
}

// Intra-node stage of hierarchical C_LP_S (Section 3.5): the k_local workers' uncompressed buckets are
// averaged (ascending order, one multiply by inv_k) and the leader compresses the average with its
// error state.  4*k_local + 9 bytes per element, one pass.
template <int RPW, bool EF, bool SHORT>
__global__ void __launch_bounds__(wg_threads_max(RPW))
k_reduce_compress_minmax(PtrTable xs, int k_local, float inv_k, float* __restrict__ residual, size_t n, uint32_t chunk,
                         uint8_t* __restrict__ codes, float* __restrict__ minmax, uint32_t keep, ChunkOrder order)
{
    __shared__ float s_red[2 * kMaxWaves];
    const size_t c = order(blockIdx.x);
    const size_t base = c * static_cast<size_t>(chunk);
    const int len = static_cast<int>((n - base < chunk) ? (n - base) : chunk);
    const int wave = wave_index(), lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;

    f4 v[RPW];
    if constexpr (SHORT) {
        float* res_c = EF ? residual + base : nullptr;
        if (chunk_full<RPW>(len, nwaves)) {
            average_rows_ahead<RPW, EF, true>(xs, k_local, inv_k, res_c, base, len, wave, lane, v);
            minmax_encode_chunk<RPW, EF, false, false, true>(v, len, wave, lane, nwaves, res_c, codes + base, minmax + 2 * c, nullptr, s_red, blockIdx.x < keep);
        } else {
            average_rows_ahead<RPW, EF, false>(xs, k_local, inv_k, res_c, base, len, wave, lane, v);
            minmax_encode_chunk<RPW, EF, false>(v, len, wave, lane, nwaves, res_c, codes + base, minmax + 2 * c, nullptr, s_red, blockIdx.x < keep);
        }
        return;
    }
    for (int j = 0; j < k_local; ++j) {
        const float* xj = static_cast<const float*>(xs.p[j]) + base;
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int off = static_cast<int>(wave * RPW + i) * kRow;
            const int remain = len - off;
            f4 d = f4{0.f, 0.f, 0.f, 0.f};
            if (remain > 0) d = load_row(xj + off, lane, remain, 0.0f);
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
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        v[i].x = v[i].x * inv_k;
        v[i].y = v[i].y * inv_k;
        v[i].z = v[i].z * inv_k;
        v[i].w = v[i].w * inv_k;
    }
    if (EF) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int off = static_cast<int>(wave * RPW + i) * kRow;
            const int remain = len - off;
            if (remain > 0) {
                const f4 d = load_row(residual + base + off, lane, remain, 0.0f);
                v[i].x = v[i].x + d.x;
                v[i].y = v[i].y + d.y;
                v[i].z = v[i].z + d.z;
                v[i].w = v[i].w + d.w;
            }
        }
    }
    minmax_encode_chunk<RPW, EF, false>(v, len, wave, lane, nwaves, EF ? residual + base : nullptr,
                                        codes + base, minmax + 2 * c, nullptr, s_red, blockIdx.x < keep);
}

// The same intra-node stage in front of the 1-bit sign codec.
template <int RPW, bool EF, bool SHORT>
__global__ void __launch_bounds__(wg_threads_max(RPW))
k_reduce_compress_sign(PtrTable xs, int k_local, float inv_k, float* __restrict__ residual, size_t n, uint32_t chunk,
                       uint32_t* __restrict__ bits, float* __restrict__ scale, ChunkOrder order)
{
    extern __shared__ float s_q[];
    const size_t c = order(blockIdx.x);
    const size_t base = c * static_cast<size_t>(chunk);
    const int len = static_cast<int>((n - base < chunk) ? (n - base) : chunk);
    const int wave = wave_index(), lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;

    f4 v[RPW];
    if constexpr (SHORT) {
        float* res_c = EF ? residual + base : nullptr;
        if (chunk_full<RPW>(len, nwaves)) {
            average_rows_ahead<RPW, EF, true>(xs, k_local, inv_k, res_c, base, len, wave, lane, v);
            sign_encode_chunk<RPW, EF, false, true>(v, len, chunk, wave, lane, nwaves, res_c, bits + (base >> 5), scale + c, nullptr, s_q);
        } else {
            average_rows_ahead<RPW, EF, false>(xs, k_local, inv_k, res_c, base, len, wave, lane, v);
#pragma unroll
            for (int i = 0; i < RPW; ++i) clear_absent(v[i], (wave * RPW + i) * kRow + lane * 4, len);
            sign_encode_chunk<RPW, EF, false>(v, len, chunk, wave, lane, nwaves, res_c, bits + (base >> 5), scale + c, nullptr, s_q);
        }
        return;
    }
    for (int j = 0; j < k_local; ++j) {
        const float* xj = static_cast<const float*>(xs.p[j]) + base;
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int off = static_cast<int>(wave * RPW + i) * kRow;
            const int remain = len - off;
            f4 d = f4{0.f, 0.f, 0.f, 0.f};
            if (remain > 0) d = load_row(xj + off, lane, remain, 0.0f);
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
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        v[i].x = v[i].x * inv_k;
        v[i].y = v[i].y * inv_k;
        v[i].z = v[i].z * inv_k;
        v[i].w = v[i].w * inv_k;
    }
    if (EF) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int off = static_cast<int>(wave * RPW + i) * kRow;
            const int remain = len - off;
            if (remain > 0) {
                const f4 d = load_row(residual + base + off, lane, remain, 0.0f);
                v[i].x = v[i].x + d.x;
                v[i].y = v[i].y + d.y;
                v[i].z = v[i].z + d.z;
                v[i].w = v[i].w + d.w;
            }
        }
    }
    sign_encode_chunk<RPW, EF, false>(v, len, chunk, wave, lane, nwaves, EF ? residual + base : nullptr,
                                      bits + (base >> 5), scale + c, nullptr, s_q);
}

}  // namespace bagua

using namespace bagua;

extern "C" int bagua_flatten_compress_minmax_u8(const void* workspace, size_t T, float* residual, size_t bucket_numel,
                                                size_t chunk, uint8_t* codes, float* minmax, float* bucket_out,
                                                void* stream)
{
    if (!workspace || !codes || !minmax || bucket_numel == 0 || !chunk_ok(chunk)) return BAGUA_ERR_INVALID_ARG;
    RangeCheck rc;
    rc.writes(residual, bucket_numel * sizeof(float));
    rc.writes(codes, bucket_numel);
    rc.writes(minmax, 2 * num_chunks(bucket_numel, chunk) * sizeof(float));
    rc.writes(bucket_out, bucket_numel * sizeof(float));
    if (!rc.disjoint()) return BAGUA_ERR_INVALID_ARG;
    if (T > 0xfffffff0u || num_chunks(bucket_numel, chunk) > kMaxGrid) return BAGUA_ERR_UNSUPPORTED;
    if (!aligned16(workspace) || !aligned16(residual) || !aligned16(codes) || !aligned4(minmax) ||
        !aligned16(bucket_out))
        return BAGUA_ERR_ALIGNMENT;
    const FlattenPlanView pv = plan_view(workspace, T);
    const int rows = static_cast<int>(chunk / kRow);
    const int rpw = pick_rpw_gather(rows, bucket_numel, BAGUA_RPW_COMPRESS);
    dim3 grid(static_cast<unsigned>(num_chunks(bucket_numel, chunk))), block(64 * ((rows + rpw - 1) / rpw));
    const uint32_t ch = static_cast<uint32_t>(chunk), t32 = static_cast<uint32_t>(T);
    hipStream_t s = static_cast<hipStream_t>(stream);
    // Short gathers stream their codes.  Streamed -> kept, gathered rounds: 8 workers x 2.5 M, C = 2048, 83.7 -> 86.8 us, C =
    // 16384 109 -> 114 us; 8 x 3.2 M, C = 8192, 101 -> 104 us, C = 2048 101 -> 99 us; 8 x 5 M, C = 4096, 131 -> 127 us, C = 8192
    // 132 -> 134 us; from 7 M on kept is faster or equal at any chunk length.  (A flat bucket's compression gains from 2 M on.)
    const uint32_t keep = bucket_numel < (static_cast<size_t>(1) << 22) ? 0 : keep_chunks(bucket_numel, chunk);
#define BAGUA_FC(EFv, WBv)                                                                                       \
    BAGUA_DISPATCH_RPW_WORKER(rpw, launch_kernel((k_flatten_compress_minmax<RPW, EFv, WBv>), grid, block, 0, s,    \
                                               pv.desc, pv.tile_first, t32, residual, bucket_numel, ch, codes,  \
                                               minmax, bucket_out, keep,                   \
                                               chunk_order(grid.x, chunk, order_pays_gather_minmax(bucket_numel, chunk))))
    if (residual && bucket_out) { BAGUA_FC(true, true) }
    else if (residual) { BAGUA_FC(true, false) }
    else if (bucket_out) { BAGUA_FC(false, true) }
    else { BAGUA_FC(false, false) }
#undef BAGUA_FC
    return launch_status();
}

extern "C" int bagua_flatten_sign_compress_ef(const void* workspace, size_t T, float* residual, size_t bucket_numel,
                                              size_t chunk, uint32_t* bits, float* scale, float* bucket_out,
                                              void* stream)
{
    if (!workspace || !bits || !scale || bucket_numel == 0 || !chunk_ok(chunk)) return BAGUA_ERR_INVALID_ARG;
    RangeCheck rc;
    rc.writes(residual, bucket_numel * sizeof(float));
    rc.writes(bits, ((bucket_numel + 31) / 32) * sizeof(uint32_t));
    rc.writes(scale, num_chunks(bucket_numel, chunk) * sizeof(float));
    rc.writes(bucket_out, bucket_numel * sizeof(float));
    if (!rc.disjoint()) return BAGUA_ERR_INVALID_ARG;
    if (T > 0xfffffff0u || num_chunks(bucket_numel, chunk) > kMaxGrid) return BAGUA_ERR_UNSUPPORTED;
    if (!aligned16(workspace) || !aligned16(residual) || !aligned16(bits) || !aligned4(scale) || !aligned16(bucket_out))
        return BAGUA_ERR_ALIGNMENT;
    const FlattenPlanView pv = plan_view(workspace, T);
    const int rows = static_cast<int>(chunk / kRow);
    const int rpw = pick_rpw_gather(rows, bucket_numel, BAGUA_RPW_SIGN);
    const int waves = (rows + rpw - 1) / rpw;
    dim3 grid(static_cast<unsigned>(num_chunks(bucket_numel, chunk))), block(64 * waves);
    const size_t lds = waves > 1 ? static_cast<size_t>(rows) * kWave * sizeof(float) : 0;
    const uint32_t ch = static_cast<uint32_t>(chunk), t32 = static_cast<uint32_t>(T);
    hipStream_t s = static_cast<hipStream_t>(stream);
#define BAGUA_FS(EFv, WBv)                                                                                       \
    BAGUA_DISPATCH_RPW_WORKER(rpw, launch_kernel((k_flatten_sign_compress<RPW, EFv, WBv>), grid, block, lds, s,    \
                                               pv.desc, pv.tile_first, t32, residual, bucket_numel, ch, bits,   \
                                               scale, bucket_out, chunk_order(grid.x, chunk)))
    if (residual && bucket_out) { BAGUA_FS(true, true) }
    else if (residual) { BAGUA_FS(true, false) }
    else if (bucket_out) { BAGUA_FS(false, true) }
    else { BAGUA_FS(false, false) }
#undef BAGUA_FS
    return launch_status();
}

extern "C" int bagua_reduce_compress_minmax_u8(const float* const* x, int k_local, float* residual, size_t n,
                                               size_t chunk, uint8_t* codes, float* minmax, void* stream)
{
    if (!x || k_local < 1 || k_local > BAGUA_MAX_WORKERS || !codes || !minmax || n == 0 || !chunk_ok(chunk))
        return BAGUA_ERR_INVALID_ARG;
    RangeCheck rc;
    for (int j = 0; j < k_local; ++j) {
        if (!x[j]) return BAGUA_ERR_INVALID_ARG;
        rc.reads(x[j], n * sizeof(float));
    }
    rc.writes(residual, n * sizeof(float));
    rc.writes(codes, n);
    rc.writes(minmax, 2 * num_chunks(n, chunk) * sizeof(float));
    if (!rc.disjoint()) return BAGUA_ERR_INVALID_ARG;
    if (num_chunks(n, chunk) > kMaxGrid) return BAGUA_ERR_UNSUPPORTED;
    for (int j = 0; j < k_local; ++j)
        if (!aligned16(x[j])) return BAGUA_ERR_ALIGNMENT;
    if (!aligned16(residual) || !aligned16(codes) || !aligned4(minmax)) return BAGUA_ERR_ALIGNMENT;
    PtrTable xt{};
    for (int j = 0; j < k_local; ++j) xt.p[j] = x[j];
    const dim3 grid(static_cast<unsigned>(num_chunks(n, chunk)));
    const float inv_k = 1.0f / static_cast<float>(k_local);
    const uint32_t ch = static_cast<uint32_t>(chunk), keep = keep_chunks(n, chunk);
    const ChunkOrder order = chunk_order(grid.x, chunk, order_pays_average(n, chunk, k_local));
    hipStream_t s = static_cast<hipStream_t>(stream);
    average_shape(n, chunk, BAGUA_RPW_COMPRESS, [&](auto rpw, auto is_short) {
        constexpr int RPW = decltype(rpw)::value;
        constexpr bool SHORT = decltype(is_short)::value;
        const dim3 block(kWave * ((chunk / kRow + RPW - 1) / RPW));
        if (residual) launch_kernel((k_reduce_compress_minmax<RPW, true, SHORT>), grid, block, 0, s, xt, k_local, inv_k, residual, n, ch, codes, minmax, keep, order);
        else launch_kernel((k_reduce_compress_minmax<RPW, false, SHORT>), grid, block, 0, s, xt, k_local, inv_k, residual, n, ch, codes, minmax, keep, order);
    });
    return launch_status();
}

extern "C" int bagua_reduce_compress_sign_ef(const float* const* x, int k_local, float* residual, size_t n, size_t chunk,
                                             uint32_t* bits, float* scale, void* stream)
{
    if (!x || k_local < 1 || k_local > BAGUA_MAX_WORKERS || !bits || !scale || n == 0 || !chunk_ok(chunk))
        return BAGUA_ERR_INVALID_ARG;
    RangeCheck rc;
    for (int j = 0; j < k_local; ++j) {
        if (!x[j]) return BAGUA_ERR_INVALID_ARG;
        rc.reads(x[j], n * sizeof(float));
    }
    rc.writes(residual, n * sizeof(float));
    rc.writes(bits, ((n + 31) / 32) * sizeof(uint32_t));
    rc.writes(scale, num_chunks(n, chunk) * sizeof(float));
    if (!rc.disjoint()) return BAGUA_ERR_INVALID_ARG;
    if (num_chunks(n, chunk) > kMaxGrid) return BAGUA_ERR_UNSUPPORTED;
    for (int j = 0; j < k_local; ++j)
        if (!aligned16(x[j])) return BAGUA_ERR_ALIGNMENT;
    if (!aligned16(residual) || !aligned16(bits) || !aligned4(scale)) return BAGUA_ERR_ALIGNMENT;
    PtrTable xt{};
    for (int j = 0; j < k_local; ++j) xt.p[j] = x[j];
    const dim3 grid(static_cast<unsigned>(num_chunks(n, chunk)));
    const float inv_k = 1.0f / static_cast<float>(k_local);
    const uint32_t ch = static_cast<uint32_t>(chunk);
    const ChunkOrder order = chunk_order(grid.x, chunk, order_pays_average(n, chunk, k_local));
    hipStream_t s = static_cast<hipStream_t>(stream);
    average_shape(n, chunk, BAGUA_RPW_SIGN, [&](auto rpw, auto is_short) {
        constexpr int RPW = decltype(rpw)::value;
        constexpr bool SHORT = decltype(is_short)::value;
        const dim3 block(kWave * ((chunk / kRow + RPW - 1) / RPW));
        const size_t lds = block.x > kWave ? chunk / kRow * kWave * sizeof(float) : 0;
        if (residual) launch_kernel((k_reduce_compress_sign<RPW, true, SHORT>), grid, block, lds, s, xt, k_local, inv_k, residual, n, ch, bits, scale, order);
        else launch_kernel((k_reduce_compress_sign<RPW, false, SHORT>), grid, block, lds, s, xt, k_local, inv_k, residual, n, ch, bits, scale, order);
    });
    return launch_status();
}
