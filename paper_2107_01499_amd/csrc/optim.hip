// Decode fused into the bucket-level optimizer step: the last step of C_LP_S on every worker
// (decode the tensor the server sent back) and the update of the flattened bucket (Section 3.5 of
// the paper) in one pass.  The decoded tensor is never written to memory.  SGD: 1 (or 1/8) + 8
// (+ 8 with momentum) bytes per element; Adam: 1 + 24 (full), 1/8 + 16 (frozen variance).
#include <cmath>

#include "launchers.hpp"

#pragma clang fp contract(off)

namespace bagua {

// Decoded values of the row starting at element e0 (chunk c): four per lane.
template <int CODEC>
__device__ __forceinline__ f4 decode_row(const void* __restrict__ codes, const float* __restrict__ meta, size_t e0,
                                         size_t c, int lane, int remain)
{
    f4 g;
    if (CODEC == BAGUA_CODEC_MINMAX_U8) {
        const float mn = meta[2 * c], step = minmax_step(mn, meta[2 * c + 1]);
        const uint32_t w = load_codes_row(static_cast<const uint8_t*>(codes) + e0, lane, remain);
        g.x = mn + byte_to_float(w, 0) * step;
        g.y = mn + byte_to_float(w, 1) * step;
        g.z = mn + byte_to_float(w, 2) * step;
        g.w = mn + byte_to_float(w, 3) * step;
    } else {
        const float sc = meta[c];
        const float neg = -sc;
        uint32_t w = 0;
        if (static_cast<int>(lane >> 3) * 32 < remain) w = static_cast<const uint32_t*>(codes)[(e0 >> 5) + (lane >> 3)];
        const uint32_t nib = w >> (4 * (lane & 7));
        g.x = (nib & 1u) ? sc : neg;
        g.y = (nib & 2u) ? sc : neg;
        g.z = (nib & 4u) ? sc : neg;
        g.w = (nib & 8u) ? sc : neg;
    }
    return g;
}

// One wave per 256-element row, kRowWaves rows per workgroup.
template <int CODEC, bool MOM, bool WD>
__global__ void __launch_bounds__(kWave * kRowWaves)
k_decompress_sgd(const void* __restrict__ codes, const float* __restrict__ meta, size_t n, uint32_t rows_per_chunk,
                 float* __restrict__ param, float* __restrict__ mbuf, float lr, float mu, float wd, ChunkOrder order)
{
    const uint32_t row = order(blockIdx.x) * kRowWaves + wave_index();
    const int lane = threadIdx.x & 63;
    const size_t e0 = static_cast<size_t>(row) * kRow;
    if (e0 >= n) return;
    const size_t c = row / rows_per_chunk;
    const int remain = static_cast<int>((n - e0 < static_cast<size_t>(kRow)) ? (n - e0) : kRow);

    f4 p = load_row(param + e0, lane, remain, 0.0f);
    f4 m = f4{0.f, 0.f, 0.f, 0.f};
    if (MOM) m = load_row(mbuf + e0, lane, remain, 0.0f);

    f4 g = decode_row<CODEC>(codes, meta, e0, c, lane, remain);
    if (WD) {
        g.x = g.x + wd * p.x;
        g.y = g.y + wd * p.y;
        g.z = g.z + wd * p.z;
        g.w = g.w + wd * p.w;
    }
    f4 u = g;
    if (MOM) {
        m.x = mu * m.x + g.x;
        m.y = mu * m.y + g.y;
        m.z = mu * m.z + g.z;
        m.w = mu * m.w + g.w;
        store_row(mbuf + e0, lane, remain, m);
        u = m;
    }
    p.x = p.x - lr * u.x;
    p.y = p.y - lr * u.y;
    p.z = p.z - lr * u.z;
    p.w = p.w - lr * u.w;
    store_row(param + e0, lane, remain, p);
}

// Adam-type update (no bias correction).  FROZEN: the decoded tensor is the averaged momentum of the
// compression stage of 1-bit Adam: it replaces m, and v is only read.
template <int CODEC, bool FROZEN, bool WD>
__global__ void __launch_bounds__(kWave * kRowWaves)
k_decompress_adam(const void* __restrict__ codes, const float* __restrict__ meta, size_t n, uint32_t rows_per_chunk,
                  float* __restrict__ param, float* __restrict__ mbuf, float* __restrict__ vbuf, float lr, float beta1,
                  float omb1, float beta2, float omb2, float eps, float wd, ChunkOrder order)
{
    const uint32_t row = order(blockIdx.x) * kRowWaves + wave_index();
    const int lane = threadIdx.x & 63;
    const size_t e0 = static_cast<size_t>(row) * kRow;
    if (e0 >= n) return;
    const size_t c = row / rows_per_chunk;
    const int remain = static_cast<int>((n - e0 < static_cast<size_t>(kRow)) ? (n - e0) : kRow);

    f4 p = load_row(param + e0, lane, remain, 0.0f);
    f4 v = load_row(vbuf + e0, lane, remain, 1.0f);
    const f4 d = decode_row<CODEC>(codes, meta, e0, c, lane, remain);
    f4 m = d;
    if (!FROZEN) {
        const f4 mo = load_row(mbuf + e0, lane, remain, 0.0f);
        m.x = beta1 * mo.x + omb1 * d.x;
        m.y = beta1 * mo.y + omb1 * d.y;
        m.z = beta1 * mo.z + omb1 * d.z;
        m.w = beta1 * mo.w + omb1 * d.w;
        v.x = beta2 * v.x + omb2 * (d.x * d.x);
        v.y = beta2 * v.y + omb2 * (d.y * d.y);
        v.z = beta2 * v.z + omb2 * (d.z * d.z);
        v.w = beta2 * v.w + omb2 * (d.w * d.w);
        store_row(vbuf + e0, lane, remain, v);
    }
    store_row(mbuf + e0, lane, remain, m);
    f4 u;
    u.x = m.x / (sqrtf(v.x) + eps);
    u.y = m.y / (sqrtf(v.y) + eps);
    u.z = m.z / (sqrtf(v.z) + eps);
    u.w = m.w / (sqrtf(v.w) + eps);
    if (WD) {
        u.x = u.x + wd * p.x;
        u.y = u.y + wd * p.y;
        u.z = u.z + wd * p.z;
        u.w = u.w + wd * p.w;
    }
    p.x = p.x - lr * u.x;
    p.y = p.y - lr * u.y;
    p.z = p.z - lr * u.z;
    p.w = p.w - lr * u.w;
    store_row(param + e0, lane, remain, p);
}

// ------------------------------------------------------------------------------------------ top-K codec
// Without momentum and weight decay (and lr >= +0, finite) only the kept entries change: p - fl(lr * +0) = p bit for
// bit.  One thread per (chunk, slot) entry.
__global__ void __launch_bounds__(256)
k_sgd_topk_sparse(const uint16_t* __restrict__ idx, const float* __restrict__ val, size_t entries, uint32_t chunk,
                  uint32_t keep, size_t n, float* __restrict__ param, float lr)
{
    const size_t e = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
    if (e >= entries) return;
    const uint32_t q = idx[e];
    if (q == 0xFFFFu) return;
    const size_t i = (e / keep) * chunk + q;
    if (i < n) param[i] = param[i] - lr * val[e];
}

// The entries of a sparse chunk, into its dense copy in LDS.  EARLY: one per thread is requested before anything else, so that the scatter
// waits for these two loads alone, and not for the index, then for the value, behind everything that the kernel reads.
// U: how many of a long list a thread requests at a time.  SINGLE: a list that gives no thread more than one is taken without looking for more,
// us of the step, SGD with late entries: C = 256, keep = 32, 1.1 M 4.80 -> 4.57, 4 M 13.8 -> 13.3; C = 2048, keep = 256, 2 M 6.27 -> 6.08, 4.9 M 15.5 -> 15.1;
// C = 1024, keep = 512 (no such list) 2 M 7.05 -> 6.87.  Adam loses by it from 3 M to 4 M (C = 4096, 4 M 16.4 -> 16.9, C = 7168, 3 M 13.3 -> 15.5), where a
// longer chain of loads spreads the waves.
template <bool EARLY, int U, bool SINGLE>
struct SparseEntries {
    const uint16_t* idx;
    const float* val;
    uint32_t keep, q = 0xFFFFu;
    float a = 0.0f;
    __device__ __forceinline__ SparseEntries(const uint16_t* __restrict__ idx_c, const float* __restrict__ val_c, uint32_t kept)
        : idx(idx_c), val(val_c), keep(kept)
    {
        if (EARLY && threadIdx.x < keep) {
            q = idx[threadIdx.x];
            a = val[threadIdx.x];
        }
    }
    // Those that lie in [from, from + size) of the chunk (unused slots are 0xFFFF, beyond any chunk).
    __device__ __forceinline__ void scatter(uint32_t from, uint32_t size, float* dense)
    {
        if (EARLY && q - from < size) dense[q - from] = a;
        if (!EARLY && (U == 1 || (SINGLE && keep <= blockDim.x))) {
            for (uint32_t s = threadIdx.x; s < keep; s += blockDim.x) {
                const uint32_t at = idx[s];
                if (at - from < size) dense[at - from] = val[s];
            }
            return;
        }
        for (uint32_t s = threadIdx.x + (EARLY ? blockDim.x : 0); s < keep; s += U * blockDim.x) {
            uint32_t at[U];
            float v[U];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                at[u] = 0xFFFFu;
                if (u == 0 || s + u * blockDim.x < keep) at[u] = idx[s + u * blockDim.x];
            }
#pragma unroll
            for (uint32_t u = 0; u < U; ++u)
                if (at[u] - from < size) v[u] = val[s + u * blockDim.x];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u)
                if (at[u] - from < size) dense[at[u] - from] = v[u];
        }
    }
};
// Late -> early, us of the step (four sets of buffers in turn): SGD, C = 4096, keep = 128, 64 K 2.7 -> 2.5, 1 M 4.1 -> 4.0, 3 M 7.9 -> 9.0, 4 M 11.0 ->
// 12.2, 8 M +-0, 12 M 33.8 -> 32.4, 25.7 M 69.0 -> 66.7, 100 M 265 -> 256; C = 1024, keep = 32, 25.7 M 72.9 -> 66.6; C = 16384, keep = 512, 8 M 22.9 ->
// 23.7, 100 M 264 -> 257; Adam, C = 4096, 25.7 M 106.3 -> 103.6.  From 2 M to 5 M, where the state fits the caches, all waves at once lose what the
// longer chain of loads spreads; chunks of several parts up to 10 M.
inline bool entries_early(size_t n, size_t chunk)
{
    return n <= (static_cast<size_t>(1) << 20) || n > (static_cast<size_t>(chunk <= 4096 ? 5 : 10) << 20);
}

// How a chunk is cut into the parts that a workgroup takes: up to kTopkPart elements, eight waves of two rows and 16 KB of LDS.  Each looks through
// all entries of its chunk.  One workgroup per chunk (16 waves of two rows or more) -> this, us of the step: Adam, C = 16384, keep = 512, 64 K 7.0 -> 3.5,
// 1 M 9.9 -> 5.5, 25.7 M 119 -> 103, 100 M 442 -> 409; SGD 64 K 3.9 -> 2.7, 1 M 6.1 -> 4.2, 25.7 M 76.3 -> 67.7; C = 8192, keep = 256, 1 M 4.8 -> 4.3, 25.7 M
// 69.8 -> 66.9, 100 M 284 -> 266; C = 6144 0 .. -5 %; C = 16384, keep = 2048, 64 K 4.2 -> 2.9, 40 M 118 -> 108.  Where that loses: topk_step_whole().
constexpr int kTopkPart = 4096;
// A whole chunk by one workgroup: up to MOST elements, 16 waves of two or of four rows, late entries.  So many parts that no grid holds them are taken so
// as well.
constexpr int kTopkWhole = 8192, kTopkWholeLong = 16384;
constexpr int topk_step_rpw(int most) { return most <= kTopkWhole ? 2 : 4; }
constexpr int topk_step_threads(int most) { return most / topk_step_rpw(most) / kRow * kWave; }
// Where the whole chunks all run at once and their parts, of which a CU holds no more elements, need a second, nearly empty go; up to 8192 elements also as
// long as there is a CU for every chunk and the entries come late.  Parts -> whole, us of the step: C = 8192, keep = 256, Adam 1.1 M 7.6 -> 6.7, 1.5 M 8.4 ->
// 7.4, 2 M 8.8 -> 8.7, 2.5 M 11.7 -> 13.6, SGD 1.1 M 4.9 -> 4.8; C = 9216 (three chunks on a CU), keep = 288, SGD 3.6 M 10.2 -> 10.4, 4.1 M 13.5 -> 11.8, 6 M 18.8
// -> 16.9, 6.8 M 21.6 -> 22.1, Adam 4.1 M 20.5 -> 18.8, 4.6 M 22.6 -> 25.2, 6 M 28.7 -> 27.4; C = 12288 (two), keep = 1536, SGD 4.6 M 15.8 -> 13.6, 6 M 19.5 -> 16.9, 6.8 M
// 21.5 -> 22.1, Adam 4.6 M 23.6 -> 21.3, 6 M 28.7 -> 26.7; C = 16384, keep = 2048, SGD 4.6 M 16.3 -> 16.6, 5.2 M 18.0 -> 17.4, 6 M 19.8 -> 17.6, 8 M 24.5 -> 22.6, 8.5 M
// 27.1 -> 27.8, Adam 5.2 M 26.2 -> 28.4, 6 M 29.3 -> 28.3, 8 M 37.1 -> 35.8, 8.5 M 40.7 -> 45; keep = 8192, of which every part reads all, SGD 4.6 M 20.6 -> 17.0, 8 M
// 29.3 -> 24.3, Adam 4.6 M 27.4 -> 27.4, 6 M 33.2 -> 27.5.
inline bool topk_step_whole(size_t chunks, size_t chunk, size_t keep)
{
    if (chunk <= kTopkWhole) return chunks * chunk > (static_cast<size_t>(1) << 20) && chunks <= kCus;
    if (chunk <= 9 * 4 * kRow) return chunks > 5 * kCus / 3 && chunks <= 3 * kCus;
    const size_t least = chunk <= 3 * kTopkPart ? 4 * kCus / 3 : keep > chunk / 4 ? 9 * kCus / 8 : 11 * kCus / 8;
    return chunks > least && chunks <= 2 * kCus;
}
struct TopkParts {
    uint32_t most, part, parts;   // most: elements that the kernel's workgroup can take
    dim3 grid, block;
    size_t lds;
    TopkParts(size_t chunks, size_t chunk, size_t keep)
    {
        const uint32_t rows = static_cast<uint32_t>(chunk / kRow);
        parts = static_cast<uint32_t>((chunk + kTopkPart - 1) / kTopkPart);
        most = kTopkPart;
        if (parts > 1 && (chunks > kMaxGrid / parts || topk_step_whole(chunks, chunk, keep))) {
            parts = 1;
            most = chunk <= kTopkWhole ? kTopkWhole : kTopkWholeLong;
        }
        part = (rows + parts - 1) / parts * kRow;
        const uint32_t rpw = static_cast<uint32_t>(topk_step_rpw(most));
        grid = dim3(static_cast<unsigned>(chunks * parts));
        block = dim3(kWave * ((part / kRow + rpw - 1) / rpw));
        lds = part * sizeof(float);
    }
};

// General case: the decoded gradient of a part of a chunk is built in LDS (+0 everywhere, then the kept entries), and every
// element is updated as in k_decompress_sgd.
template <bool MOM, bool WD, int MOST, bool EARLY, bool PARTS>
__global__ void __launch_bounds__(topk_step_threads(MOST))
k_decompress_sgd_topk(const uint16_t* __restrict__ idx, const float* __restrict__ val, size_t n, uint32_t chunk, uint32_t part, uint32_t parts,
                      uint32_t keep, float* __restrict__ param, float* __restrict__ mbuf, float lr, float mu, float wd)
{
    extern __shared__ float s_g[];   // part floats
    const uint32_t c = PARTS ? blockIdx.x / parts : blockIdx.x, from = PARTS ? (blockIdx.x - c * parts) * part : 0;   // part of chunk c: from element `from` on
    const size_t base = static_cast<size_t>(c) * chunk + from;
    if (PARTS && base >= n) return;
    const uint32_t size = PARTS && chunk - from > part ? part : chunk - from;
    const int len = static_cast<int>(n - base < size ? n - base : size);
    const int wave = wave_index(), lane = threadIdx.x & 63;

    SparseEntries<EARLY, 4, MOST != kTopkWholeLong> entries(idx + static_cast<size_t>(c) * keep, val + static_cast<size_t>(c) * keep, keep);
    // parameters (and momentum) do not depend on the decode: request them next
    constexpr int RPW = topk_step_rpw(MOST);
    f4 p[RPW], m[RPW];
    auto load = [&](auto full) {
        constexpr bool FULL = decltype(full)::value;
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int off = static_cast<int>(wave * RPW + i) * kRow;
            const int remain = row_remain<FULL>(len, off);
            p[i] = f4{0.f, 0.f, 0.f, 0.f};
            m[i] = p[i];
            if (remain > 0) {
                p[i] = load_row(param + base + off, lane, remain, 0.0f);
                if (MOM) m[i] = load_row(mbuf + base + off, lane, remain, 0.0f);
            }
        }
    };
    if (wave_full<RPW>(len, wave)) load(std::true_type{});   // no tail tests: all loads in flight together
    else load(std::false_type{});
    for (uint32_t e = threadIdx.x * 4; e < size; e += blockDim.x * 4)
        *reinterpret_cast<f4*>(s_g + e) = f4{0.f, 0.f, 0.f, 0.f};
    __syncthreads();
    entries.scatter(from, size, s_g);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        const int off = static_cast<int>(wave * RPW + i) * kRow;
        const int remain = len - off;
        if (remain <= 0) continue;
        f4 g = *reinterpret_cast<const f4*>(s_g + off + lane * 4);
        if (WD) {
            g.x = g.x + wd * p[i].x;
            g.y = g.y + wd * p[i].y;
            g.z = g.z + wd * p[i].z;
            g.w = g.w + wd * p[i].w;
        }
        f4 u = g;
        if (MOM) {
            m[i].x = mu * m[i].x + g.x;
            m[i].y = mu * m[i].y + g.y;
            m[i].z = mu * m[i].z + g.z;
            m[i].w = mu * m[i].w + g.w;
            store_row(mbuf + base + off, lane, remain, m[i]);
            u = m[i];
        }
        p[i].x = p[i].x - lr * u.x;
        p[i].y = p[i].y - lr * u.y;
        p[i].z = p[i].z - lr * u.z;
        p[i].w = p[i].w - lr * u.w;
        store_row(param + base + off, lane, remain, p[i]);
    }
}

// Adam-type update after a top-K round: the chunk's decoded tensor is built in LDS as above, then every element is
// updated as in k_decompress_adam.
template <bool FROZEN, bool WD, int MOST, bool EARLY, bool PARTS>
__global__ void __launch_bounds__(topk_step_threads(MOST))
k_decompress_adam_topk(const uint16_t* __restrict__ idx, const float* __restrict__ val, size_t n, uint32_t chunk, uint32_t part, uint32_t parts,
                       uint32_t keep, float* __restrict__ param, float* __restrict__ mbuf, float* __restrict__ vbuf,
                       float lr, float beta1, float omb1, float beta2, float omb2, float eps, float wd)
{
    extern __shared__ float s_g[];   // part floats
    const uint32_t c = PARTS ? blockIdx.x / parts : blockIdx.x, from = PARTS ? (blockIdx.x - c * parts) * part : 0;   // part of chunk c: from element `from` on
    const size_t base = static_cast<size_t>(c) * chunk + from;
    if (PARTS && base >= n) return;
    const uint32_t size = PARTS && chunk - from > part ? part : chunk - from;
    const int len = static_cast<int>(n - base < size ? n - base : size);
    const int wave = wave_index(), lane = threadIdx.x & 63;

    SparseEntries<EARLY, (MOST == kTopkPart ? 4 : 1), false> entries(idx + static_cast<size_t>(c) * keep, val + static_cast<size_t>(c) * keep, keep);
    // parameters and optimizer state do not depend on the decode: request them next
    constexpr int RPW = topk_step_rpw(MOST);
    f4 p[RPW], m[RPW], v[RPW];
    auto load = [&](auto full) {
        constexpr bool FULL = decltype(full)::value;
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int off = static_cast<int>(wave * RPW + i) * kRow;
            const int remain = row_remain<FULL>(len, off);
            p[i] = f4{0.f, 0.f, 0.f, 0.f};
            m[i] = p[i];
            v[i] = f4{1.f, 1.f, 1.f, 1.f};
            if (remain > 0) {
                p[i] = load_row(param + base + off, lane, remain, 0.0f);
                v[i] = load_row(vbuf + base + off, lane, remain, 1.0f);
                if (!FROZEN) m[i] = load_row(mbuf + base + off, lane, remain, 0.0f);
            }
        }
    };
    if (wave_full<RPW>(len, wave)) load(std::true_type{});
    else load(std::false_type{});
    for (uint32_t e = threadIdx.x * 4; e < size; e += blockDim.x * 4)
        *reinterpret_cast<f4*>(s_g + e) = f4{0.f, 0.f, 0.f, 0.f};
    __syncthreads();
    entries.scatter(from, size, s_g);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        const int off = static_cast<int>(wave * RPW + i) * kRow;
        const int remain = len - off;
        if (remain <= 0) continue;
        const f4 d = *reinterpret_cast<const f4*>(s_g + off + lane * 4);
        f4 mi = d;
        if (!FROZEN) {
            mi.x = beta1 * m[i].x + omb1 * d.x;
            mi.y = beta1 * m[i].y + omb1 * d.y;
            mi.z = beta1 * m[i].z + omb1 * d.z;
            mi.w = beta1 * m[i].w + omb1 * d.w;
            v[i].x = beta2 * v[i].x + omb2 * (d.x * d.x);
            v[i].y = beta2 * v[i].y + omb2 * (d.y * d.y);
            v[i].z = beta2 * v[i].z + omb2 * (d.z * d.z);
            v[i].w = beta2 * v[i].w + omb2 * (d.w * d.w);
            store_row(vbuf + base + off, lane, remain, v[i]);
        }
        store_row(mbuf + base + off, lane, remain, mi);
        f4 u;
        u.x = mi.x / (sqrtf(v[i].x) + eps);
        u.y = mi.y / (sqrtf(v[i].y) + eps);
        u.z = mi.z / (sqrtf(v[i].z) + eps);
        u.w = mi.w / (sqrtf(v[i].w) + eps);
        if (WD) {
            u.x = u.x + wd * p[i].x;
            u.y = u.y + wd * p[i].y;
            u.z = u.z + wd * p[i].z;
            u.w = u.w + wd * p[i].w;
        }
        p[i].x = p[i].x - lr * u.x;
        p[i].y = p[i].y - lr * u.y;
        p[i].z = p[i].z - lr * u.z;
        p[i].w = p[i].w - lr * u.w;
        store_row(param + base + off, lane, remain, p[i]);
    }
}

}  // namespace bagua

using namespace bagua;

extern "C" int bagua_decompress_sgd_step(int codec, const void* codes, const float* meta, size_t n, size_t chunk,
                                         float* param, float* momentum_buf, float lr, float momentum,
                                         float weight_decay, void* stream)
{
    if (codec != BAGUA_CODEC_MINMAX_U8 && codec != BAGUA_CODEC_SIGN1) return BAGUA_ERR_INVALID_ARG;
    if (!codes || !meta || !param || n == 0 || !chunk_ok(chunk)) return BAGUA_ERR_INVALID_ARG;
    {
        const size_t nc = num_chunks(n, chunk);
        RangeCheck rc;
        rc.reads(codes, codec == BAGUA_CODEC_MINMAX_U8 ? n : ((n + 31) / 32) * sizeof(uint32_t));
        rc.reads(meta, (codec == BAGUA_CODEC_MINMAX_U8 ? 2 * nc : nc) * sizeof(float));
        rc.writes(param, n * sizeof(float));
        rc.writes(momentum_buf, n * sizeof(float));
        if (!rc.disjoint()) return BAGUA_ERR_INVALID_ARG;
    }
    const size_t rows = (n + kRow - 1) / kRow;
    if ((rows + kRowWaves - 1) / kRowWaves > kMaxGrid) return BAGUA_ERR_UNSUPPORTED;
    if (!aligned16(codes) || !aligned4(meta) || !aligned16(param) || !aligned16(momentum_buf)) return BAGUA_ERR_ALIGNMENT;
    dim3 grid(static_cast<unsigned>((rows + kRowWaves - 1) / kRowWaves)), block(kWave * kRowWaves);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint32_t rpc = static_cast<uint32_t>(chunk / kRow);
    const ChunkOrder order = n <= (static_cast<size_t>(1) << 24) ? row_order(grid.x, rpc) : ChunkOrder{0, 0};
    const bool mom = momentum_buf != nullptr, wd = weight_decay != 0.0f;
#define BAGUA_SGD(CODEC, MOMv, WDv)                                                                          \
    launch_kernel((k_decompress_sgd<CODEC, MOMv, WDv>), grid, block, 0, s, codes, meta, n, rpc, param, \
                       momentum_buf, lr, momentum, weight_decay, order)
#define BAGUA_SGD_CODEC(CODEC)                       \
    if (mom && wd) BAGUA_SGD(CODEC, true, true);     \
    else if (mom) BAGUA_SGD(CODEC, true, false);     \
    else if (wd) BAGUA_SGD(CODEC, false, true);      \
    else BAGUA_SGD(CODEC, false, false);
    if (codec == BAGUA_CODEC_MINMAX_U8) { BAGUA_SGD_CODEC(BAGUA_CODEC_MINMAX_U8) }
    else { BAGUA_SGD_CODEC(BAGUA_CODEC_SIGN1) }
#undef BAGUA_SGD_CODEC
#undef BAGUA_SGD
    return launch_status();
}

extern "C" int bagua_decompress_adam_step(int codec, const void* codes, const float* meta, size_t n, size_t chunk,
                                          float* param, float* m, float* v, float lr, float beta1, float beta2,
                                          float eps, float weight_decay, int variance_frozen, void* stream)
{
    if (codec != BAGUA_CODEC_MINMAX_U8 && codec != BAGUA_CODEC_SIGN1) return BAGUA_ERR_INVALID_ARG;
    if (!codes || !meta || !param || !m || !v || n == 0 || !chunk_ok(chunk)) return BAGUA_ERR_INVALID_ARG;
    {
        const size_t nc = num_chunks(n, chunk);
        RangeCheck rc;
        rc.reads(codes, codec == BAGUA_CODEC_MINMAX_U8 ? n : ((n + 31) / 32) * sizeof(uint32_t));
        rc.reads(meta, (codec == BAGUA_CODEC_MINMAX_U8 ? 2 * nc : nc) * sizeof(float));
        rc.writes(param, n * sizeof(float));
        rc.writes(m, n * sizeof(float));
        rc.writes(v, n * sizeof(float));
        if (!rc.disjoint()) return BAGUA_ERR_INVALID_ARG;
    }
    const size_t rows = (n + kRow - 1) / kRow;
    if ((rows + kRowWaves - 1) / kRowWaves > kMaxGrid) return BAGUA_ERR_UNSUPPORTED;
    if (!aligned16(codes) || !aligned4(meta) || !aligned16(param) || !aligned16(m) || !aligned16(v))
        return BAGUA_ERR_ALIGNMENT;
    dim3 grid(static_cast<unsigned>((rows + kRowWaves - 1) / kRowWaves)), block(kWave * kRowWaves);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint32_t rpc = static_cast<uint32_t>(chunk / kRow);
    const ChunkOrder order = n <= (static_cast<size_t>(1) << 24) ? row_order(grid.x, rpc) : ChunkOrder{0, 0};
    const float omb1 = 1.0f - beta1, omb2 = 1.0f - beta2;
    const bool frozen = variance_frozen != 0, wd = weight_decay != 0.0f;
#define BAGUA_ADAM(CODEC, FRv, WDv)                                                                            \
    launch_kernel((k_decompress_adam<CODEC, FRv, WDv>), grid, block, 0, s, codes, meta, n, rpc, param, m, \
                       v, lr, beta1, omb1, beta2, omb2, eps, weight_decay, order)
#define BAGUA_ADAM_CODEC(CODEC)                        \
    if (frozen && wd) BAGUA_ADAM(CODEC, true, true);   \
    else if (frozen) BAGUA_ADAM(CODEC, true, false);   \
    else if (wd) BAGUA_ADAM(CODEC, false, true);       \
    else BAGUA_ADAM(CODEC, false, false);
    if (codec == BAGUA_CODEC_MINMAX_U8) { BAGUA_ADAM_CODEC(BAGUA_CODEC_MINMAX_U8) }
    else { BAGUA_ADAM_CODEC(BAGUA_CODEC_SIGN1) }
#undef BAGUA_ADAM_CODEC
#undef BAGUA_ADAM
    return launch_status();
}

// Expands `stmt` with constexpr MOST, EARLY and PARTS (whether a chunk has more than one).
#define BAGUA_DISPATCH_TOPK_STEP(tp, stmt)                                                                                 \
    if (tp.most == kTopkWholeLong) { constexpr int MOST = kTopkWholeLong; constexpr bool PARTS = false, EARLY = false; stmt; } \
    else if (tp.most == kTopkWhole) { constexpr int MOST = kTopkWhole; constexpr bool PARTS = false, EARLY = false; stmt; }    \
    else {                                                                                                                 \
        constexpr int MOST = kTopkPart;                                                                                    \
        if (tp.parts > 1 && entries_early(n, chunk)) { constexpr bool PARTS = true, EARLY = true; stmt; }                  \
        else if (tp.parts > 1) { constexpr bool PARTS = true, EARLY = false; stmt; }                                       \
        else if (entries_early(n, chunk)) { constexpr bool PARTS = false, EARLY = true; stmt; }                            \
        else { constexpr bool PARTS = false, EARLY = false; stmt; }                                                        \
    }

extern "C" int bagua_decompress_sgd_step_topk(const uint16_t* idx, const float* val, size_t n, size_t chunk, size_t keep,
                                              float* param, float* momentum_buf, float lr, float momentum,
                                              float weight_decay, void* stream)
{
    if (!idx || !val || !param || n == 0 || !chunk_ok(chunk) || keep < 1 || keep > chunk) return BAGUA_ERR_INVALID_ARG;
    const size_t nc = num_chunks(n, chunk);
    {
        RangeCheck rc;
        rc.reads(idx, nc * keep * sizeof(uint16_t));
        rc.reads(val, nc * keep * sizeof(float));
        rc.writes(param, n * sizeof(float));
        rc.writes(momentum_buf, n * sizeof(float));
        if (!rc.disjoint()) return BAGUA_ERR_INVALID_ARG;
    }
    if (nc > kMaxGrid || (nc * keep + 255) / 256 > kMaxGrid) return BAGUA_ERR_UNSUPPORTED;
    if (!aligned2(idx) || !aligned4(val) || !aligned16(param) || !aligned16(momentum_buf)) return BAGUA_ERR_ALIGNMENT;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint32_t ch = static_cast<uint32_t>(chunk), kp = static_cast<uint32_t>(keep);
    const bool mom = momentum_buf != nullptr, wd = weight_decay != 0.0f;
    // lr * (+0) must be +0 for the sparse form to equal the dense update: lr finite with a clear sign bit
    if (!mom && !wd && std::isfinite(lr) && !std::signbit(lr)) {
        const size_t entries = nc * keep;
        launch_kernel(k_sgd_topk_sparse, dim3(static_cast<unsigned>((entries + 255) / 256)), dim3(256), 0, s, idx, val,
                           entries, ch, kp, n, param, lr);
        return launch_status();
    }
    const TopkParts tp(nc, chunk, keep);
#define BAGUA_TS(MOMv, WDv)                                                                                               \
    BAGUA_DISPATCH_TOPK_STEP(tp, launch_kernel((k_decompress_sgd_topk<MOMv, WDv, MOST, EARLY, PARTS>), tp.grid, tp.block, tp.lds, s, idx, val, n, ch, \
                                       tp.part, tp.parts, kp, param, momentum_buf, lr, momentum, weight_decay))
    if (mom && wd) { BAGUA_TS(true, true) }
    else if (mom) { BAGUA_TS(true, false) }
    else if (wd) { BAGUA_TS(false, true) }
    else { BAGUA_TS(false, false) }
#undef BAGUA_TS
    return launch_status();
}

extern "C" int bagua_decompress_adam_step_topk(const uint16_t* idx, const float* val, size_t n, size_t chunk, size_t keep,
                                               float* param, float* m, float* v, float lr, float beta1, float beta2,
                                               float eps, float weight_decay, int variance_frozen, void* stream)
{
    if (!idx || !val || !param || !m || !v || n == 0 || !chunk_ok(chunk) || keep < 1 || keep > chunk)
        return BAGUA_ERR_INVALID_ARG;
    const size_t nc = num_chunks(n, chunk);
    {
        RangeCheck rc;
        rc.reads(idx, nc * keep * sizeof(uint16_t));
        rc.reads(val, nc * keep * sizeof(float));
        rc.writes(param, n * sizeof(float));
        rc.writes(m, n * sizeof(float));
        rc.writes(v, n * sizeof(float));
        if (!rc.disjoint()) return BAGUA_ERR_INVALID_ARG;
    }
    if (nc > kMaxGrid) return BAGUA_ERR_UNSUPPORTED;
    if (!aligned2(idx) || !aligned4(val) || !aligned16(param) || !aligned16(m) || !aligned16(v)) return BAGUA_ERR_ALIGNMENT;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint32_t ch = static_cast<uint32_t>(chunk), kp = static_cast<uint32_t>(keep);
    const float omb1 = 1.0f - beta1, omb2 = 1.0f - beta2;
    const bool frozen = variance_frozen != 0, wd = weight_decay != 0.0f;
    const TopkParts tp(nc, chunk, keep);
#define BAGUA_TA(FRv, WDv)                                                                                                 \
    BAGUA_DISPATCH_TOPK_STEP(tp, launch_kernel((k_decompress_adam_topk<FRv, WDv, MOST, EARLY, PARTS>), tp.grid, tp.block, tp.lds, s, idx, val, n, ch, \
                                       tp.part, tp.parts, kp, param, m, v, lr, beta1, omb1, beta2, omb2, eps, weight_decay))
    if (frozen && wd) { BAGUA_TA(true, true) }
    else if (frozen) { BAGUA_TA(true, false) }
    else if (wd) { BAGUA_TA(false, true) }
    else { BAGUA_TA(false, false) }
#undef BAGUA_TA
    return launch_status();
}
