// Decentralised averaging on a ring (D_FP_S / D_LP_S, Section 3.2; ring peers, Section 3.4).
//
// Full precision: one thread owns the same four elements of all k replicas, so every replica is
// read once and written once (8 bytes per element per peer) although each output has three inputs.
// Low precision: one workgroup owns one chunk of all k peers.  The per-peer difference is
// quantised, the public copies xhat are advanced and the three-neighbour mix is formed while x and
// the new xhat of every peer are still in registers: 17 bytes per element per peer, one pass, for any
// number of peers and any chunk length.
#include "launchers.hpp"
#include "minmax_device.hpp"

#pragma clang fp contract(off)

namespace bagua {

constexpr int kNarrowRows = 16;   // rows of a chunk of 4096 elements

__device__ __forceinline__ f4 add4(f4 a, f4 b) { return f4{a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w}; }
__device__ __forceinline__ f4 sub4(f4 a, f4 b) { return f4{a.x - b.x, a.y - b.y, a.z - b.z, a.w - b.w}; }
__device__ __forceinline__ f4 mul4(f4 a, float s) { return f4{a.x * s, a.y * s, a.z * s, a.w * s}; }

// ------------------------------------------------------------------------------------------ FP
// One wave per 256-element row and workgroup; K replicas held in registers.  Bound by how well the memory system copes with
// 2 K streams, which depends on how much of them is in flight on a CU: see ring_fp_waves.
template <int K>
__global__ void __launch_bounds__(kWave)
k_ring_avg_fp(PtrTable xin, MutPtrTable xout, size_t n, float third)
{
    const int lane = threadIdx.x;
    const size_t e0 = static_cast<size_t>(blockIdx.x) * kRow;
    const int remain = static_cast<int>((n - e0 < static_cast<size_t>(kRow)) ? (n - e0) : kRow);
    f4 x[K];
#pragma unroll
    for (int i = 0; i < K; ++i) x[i] = load_row(static_cast<const float*>(xin.p[i]) + e0, lane, remain, 0.0f);
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const f4 s = add4(add4(x[(i + K - 1) % K], x[i]), x[(i + 1) % K]);
        store_row(static_cast<float*>(xout.p[i]) + e0, lane, remain, mul4(s, third));
    }
}

// Any k: rolling window over the peers (fewer loads in flight; used above the templated range).
__global__ void __launch_bounds__(kWave * kRowWaves)
k_ring_avg_fp_any(PtrTable xin, MutPtrTable xout, int k, size_t n, float third)
{
    const size_t row = static_cast<size_t>(blockIdx.x) * kRowWaves + wave_index();
    const int lane = threadIdx.x & 63;
    const size_t e0 = row * kRow;
    if (e0 >= n) return;
    const int remain = static_cast<int>((n - e0 < static_cast<size_t>(kRow)) ? (n - e0) : kRow);
    const f4 first = load_row(static_cast<const float*>(xin.p[0]) + e0, lane, remain, 0.0f);
    f4 prev = load_row(static_cast<const float*>(xin.p[k - 1]) + e0, lane, remain, 0.0f);
    f4 cur = first;
    for (int i = 0; i < k; ++i) {
        const f4 next = (i + 1 < k) ? load_row(static_cast<const float*>(xin.p[i + 1]) + e0, lane, remain, 0.0f) : first;
        const f4 s = add4(add4(prev, cur), next);
        store_row(static_cast<float*>(xout.p[i]) + e0, lane, remain, mul4(s, third));
        prev = cur;
        cur = next;
    }
}

// ------------------------------------------------------------------------------------------ LP, fused
// Workgroup = one chunk of all K peers; wave w holds rows [w*RPW, (w+1)*RPW) of every peer.
// Peers are processed in order; peer p's output is formed as soon as the new public copies of
// p-1, p, p+1 exist, so only a short window of peers is live in registers at any time.
// Bound by the memory system's rate for 5 K interleaved streams.  Unrolled over the peers (the compiler moves the
// next peer's loads up) for K <= 16 and up to 32 rows, i.e. 16 waves of two rows.  16 peers x 25.6 M elements, C = 8192:
// 1.22 ms (5.7 TB/s); encode per peer + a mixing pass over the public copies, 25 bytes per element per peer, took 1.81 ms.
//
// The unrolled body stands here once, in the kernel itself.  Two of them (with and without tail tests) do not fit the
// instruction cache, which short launches pay for, and a body called through a lambda is scheduled differently.  Before
// -> now: 8 peers x 1 M, C = 1024, 34.0 -> 26.2 us, C = 4096, 31.0 -> 28.4 us; 16 x 1 M, C = 2048, 64 -> 47 us; 7 x
// 3.2 M, C = 3072, 83 -> 73 us; 2 x 4.2 M, 26.6 -> 24.7 us (66 VGPRs were one workgroup per CU too few, 64 are not).
//   FULL: no tail tests, so that a wave's loads are in flight together; a chunk that is cut short takes the loop over
//         the peers below instead.
//   WIDE: chunks above 4096 elements, more than eight waves.
template <int RPW, bool FULL>
__device__ __forceinline__ void ring_lp_chunk_any(const PtrTable& xin, const MutPtrTable& xout, const MutPtrTable& xhat,
                                                  const MutPtrTable& codes, const MutPtrTable& minmax, int k, size_t base, size_t c,
                                                  int len, float third, int keep, float (*s_red)[2 * kMaxWaves]);

template <int K, int RPW, int KEEP, bool FULL, bool WIDE>
__global__ void __launch_bounds__(WIDE ? wg_threads_max(RPW) : kWave * (kNarrowRows / RPW), K <= 2 ? 8 : 1)
k_ring_avg_lp(PtrTable xin, MutPtrTable xout, MutPtrTable xhat, MutPtrTable codes, MutPtrTable minmax, size_t n,
              uint32_t chunk, float third, ChunkOrder order)
{
    static_assert(!FULL || K >= 2, "the loop needs two entries of s_red");
    __shared__ float s_red[K][2 * kMaxWaves];
    const size_t c = order(blockIdx.x);
    const size_t base = c * static_cast<size_t>(chunk);
    const int len = static_cast<int>((n - base < chunk) ? (n - base) : chunk);
    const int wave = wave_index(), lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;

    if constexpr (FULL) {
        if (!chunk_full<RPW>(len, nwaves)) {
            ring_lp_chunk_any<RPW, false>(xin, xout, xhat, codes, minmax, K, base, c, len, third, KEEP, s_red);
            return;
        }
    }
    f4 h[K][RPW];    // new public copy xhat' of every peer
    f4 own[K][RPW];  // x - xhat' of every peer
    auto finalize = [&](int p) {
#pragma unroll
        for (int r = 0; r < RPW; ++r) {
            const int off = static_cast<int>(wave * RPW + r) * kRow;
            const int remain = row_remain<FULL>(len, off);
            const f4 s = add4(add4(h[(p + K - 1) % K][r], h[p][r]), h[(p + 1) % K][r]);
            const f4 o = add4(mul4(s, third), own[p][r]);
            if (remain > 0) store_row(static_cast<float*>(xout.p[p]) + base + off, lane, remain, o);
        }
    };
    // Peers are taken in groups of G: the statistics of a whole group sit behind one barrier.
    constexpr int G = BAGUA_LP_GROUP;
#pragma unroll
    for (int g0 = 0; g0 < K; g0 += G) {
        f4 x[G][RPW], d[G][RPW];
        float mn[G], mx[G];
#pragma unroll
        for (int gi = 0; gi < G; ++gi) {
            const int i = g0 + gi;
            if (i >= K) continue;
#pragma unroll
            for (int r = 0; r < RPW; ++r) {
                const int off = static_cast<int>(wave * RPW + r) * kRow;
                const int remain = row_remain<FULL>(len, off);
                x[gi][r] = f4{0.f, 0.f, 0.f, 0.f};
                h[i][r] = f4{0.f, 0.f, 0.f, 0.f};
                if (remain > 0) {
                    x[gi][r] = load_row(static_cast<const float*>(xin.p[i]) + base + off, lane, remain, 0.0f);
                    h[i][r] = load_row(static_cast<const float*>(xhat.p[i]) + base + off, lane, remain, 0.0f);
                }
                d[gi][r] = sub4(x[gi][r], h[i][r]);
            }
            chunk_minmax_partial<RPW, FULL>(d[gi], len, wave, lane, nwaves, s_red[i], mn[gi], mx[gi]);
        }
        if (nwaves > 1) __syncthreads();
#pragma unroll
        for (int gi = 0; gi < G; ++gi) {
            const int i = g0 + gi;
            if (i >= K) continue;
            chunk_minmax_finish(nwaves, s_red[i], mn[gi], mx[gi]);
            // d <- decode(Q(d)); codes and (min,max) of peer i are written on the way
            minmax_quantise_chunk<RPW, false, false, true, FULL>(d[gi], mn[gi], mx[gi], len, wave, lane, nullptr,
                                                                 static_cast<uint8_t*>(codes.p[i]) + base,
                                                                 static_cast<float*>(minmax.p[i]) + 2 * c, nullptr, KEEP);
#pragma unroll
            for (int r = 0; r < RPW; ++r) {
                const int off = static_cast<int>(wave * RPW + r) * kRow;
                const int remain = row_remain<FULL>(len, off);
                h[i][r] = add4(h[i][r], d[gi][r]);
                own[i][r] = sub4(x[gi][r], h[i][r]);
                if (remain > 0) store_row(static_cast<float*>(xhat.p[i]) + base + off, lane, remain, h[i][r]);
            }
            if (i >= 2) finalize(i - 1);
        }
    }
    finalize(K - 1);
    if (K > 1) finalize(0);
}

// ------------------------------------------------------------------------------------------ LP, any number of peers
// One peer's rows of a chunk: x and the public copy, as they are before the round.  READ_AGAIN: without the streaming
// hint, because the caller's next launch reads x and the new public copy, which is stored over the old one.
template <int RPW, bool READ_AGAIN = false>
__device__ __forceinline__ void lp_load(const float* x_c, const float* hat_c, int len, int wave, int lane, f4 (&x)[RPW], f4 (&h)[RPW])
{
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
        const int off = static_cast<int>(wave * RPW + r) * kRow;
        const int remain = len - off;
        x[r] = f4{0.f, 0.f, 0.f, 0.f};
        h[r] = f4{0.f, 0.f, 0.f, 0.f};
        if (remain > 0) {
            x[r] = READ_AGAIN ? load_row_keep(x_c + off, lane, remain, 0.0f) : load_row(x_c + off, lane, remain, 0.0f);
            h[r] = READ_AGAIN ? load_row_keep(hat_c + off, lane, remain, 0.0f) : load_row(hat_c + off, lane, remain, 0.0f);
        }
    }
}

// The same without a test, for a complete chunk (FULL) or one that is cut short: all of a wave's loads are in flight together.
template <int RPW, bool FULL, bool READ_AGAIN>
__device__ __forceinline__ void lp_load_at(const float* x_c, const float* hat_c, int len, int wave, int lane, f4 (&x)[RPW], f4 (&h)[RPW])
{
    RowAt at[RPW];
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
        at[r] = row_at<FULL>((wave * RPW + r) * kRow, len, lane);
        x[r] = load_at<FULL, READ_AGAIN>(x_c, at[r]);
        h[r] = load_at<FULL, READ_AGAIN>(hat_c, at[r]);
    }
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
        x[r] = settle<FULL>(x[r], at[r]);
        h[r] = settle<FULL>(h[r], at[r]);
    }
}

// Publish Q(x - h) of the rows just loaded and advance the public copy.  On return h = the new public copy (also
// stored), x = x - h, what the peer adds to the mix.  One barrier.
template <int RPW, bool FULL = false>
__device__ __forceinline__ void lp_publish(f4 (&x)[RPW], f4 (&h)[RPW], float* hat_c, uint8_t* codes_c, float* minmax_c, int len,
                                           int wave, int lane, int nwaves, float* s_red, int keep)
{
    f4 d[RPW];
#pragma unroll
    for (int r = 0; r < RPW; ++r) d[r] = sub4(x[r], h[r]);
    minmax_encode_chunk<RPW, false, false, true, FULL>(d, len, wave, lane, nwaves, nullptr, codes_c, minmax_c, nullptr, s_red, keep);
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
        const int off = static_cast<int>(wave * RPW + r) * kRow;
        const int remain = row_remain<FULL>(len, off);
        h[r] = add4(h[r], d[r]);
        x[r] = sub4(x[r], h[r]);
        if (remain > 0) store_row(hat_c + off, lane, remain, h[r]);
    }
}

template <int RPW>
__device__ __forceinline__ void copy_rows(f4 (&to)[RPW], const f4 (&from)[RPW])
{
#pragma unroll
    for (int r = 0; r < RPW; ++r) to[r] = from[r];
}

template <int RPW>
__device__ __forceinline__ void ring_mix(const f4 (&left)[RPW], const f4 (&mid)[RPW], const f4 (&right)[RPW], const f4 (&own)[RPW],
                                         float third, float* out_c, int len, int wave, int lane)
{
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
        const int off = static_cast<int>(wave * RPW + r) * kRow;
        const int remain = len - off;
        const f4 s = add4(add4(left[r], mid[r]), right[r]);
        if (remain > 0) store_row(out_c + off, lane, remain, add4(mul4(s, third), own[r]));
    }
}

// The same with the peers in a loop, for what the unrolled kernel cannot hold: the first peer's new copy is not kept
// for the wrap-around but read again at the end (12 bytes per element of a round, mostly from cache), which keeps four
// rows per wave within 128 VGPRs.  8 peers x 25.6 M elements, C = 16384: 0.71 ms against 0.98 ms in two passes.  Up to
// 32 rows it is 1-10 % slower than the unrolled kernel (8 peers x 109 M: 3.03 against 2.84 ms), except for chunks whose
// last wave has one row only (see launch_lp_k).  Requesting the next peer's rows ahead was slower in every launch of
// more than one workgroup per CU.
template <int RPW, bool FULL>
__device__ __forceinline__ void ring_lp_chunk_any(const PtrTable& xin, const MutPtrTable& xout, const MutPtrTable& xhat,
                                                  const MutPtrTable& codes, const MutPtrTable& minmax, int k, size_t base, size_t c,
                                                  int len, float third, int keep, float (*s_red)[2 * kMaxWaves])
{
    const int wave = wave_index(), lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;
    auto x_of = [&](int i) { return static_cast<const float*>(xin.p[i]) + base; };
    auto hat_of = [&](int i) { return static_cast<float*>(xhat.p[i]) + base; };
    auto out_of = [&](int i) { return static_cast<float*>(xout.p[i]) + base; };

    f4 left[RPW], mid[RPW], own[RPW];   // public copies of peers i - 2 and i - 1, and what the latter adds to its mix
    f4 x[RPW], h[RPW];
    for (int i = 0; i < k; ++i) {
        if constexpr (FULL) lp_load_at<RPW, true, false>(x_of(i), hat_of(i), len, wave, lane, x, h);
        else lp_load<RPW>(x_of(i), hat_of(i), len, wave, lane, x, h);
        lp_publish<RPW, FULL>(x, h, hat_of(i), static_cast<uint8_t*>(codes.p[i]) + base, static_cast<float*>(minmax.p[i]) + 2 * c, len,
                        wave, lane, nwaves, s_red[i & 1], keep);
        if (i >= 2) ring_mix<RPW>(left, mid, h, own, third, out_of(i - 1), len, wave, lane);
        copy_rows<RPW>(left, mid);
        copy_rows<RPW>(mid, h);
        copy_rows<RPW>(own, x);
    }
    // the wrap-around: peers k - 1 and 0 need the new copies of peers 0 and 1 again, which this lane has stored
    if (k == 1) {
        ring_mix<RPW>(mid, mid, mid, own, third, out_of(0), len, wave, lane);
        return;
    }
    f4 right[RPW];
    lp_load<RPW>(x_of(0), hat_of(0), len, wave, lane, x, h);
    lp_load<RPW>(hat_of(1), hat_of(1), len, wave, lane, right, right);
    ring_mix<RPW>(left, mid, h, own, third, out_of(k - 1), len, wave, lane);
#pragma unroll
    for (int r = 0; r < RPW; ++r) x[r] = sub4(x[r], h[r]);
    ring_mix<RPW>(mid, h, right, x, third, out_of(0), len, wave, lane);
}

// FOLD: complete chunks without tail tests on their loads.  In the longest launches of chunks of more than 32 rows, and in the shortest of a ring of one
// (two peers and more take two launches there); with the tests -> without, us: C = 16384, K = 3, 33 M 365 -> 353, 134 M 1476 -> 1412; K = 2, 8 M 67.8 -> 70.3, 33 M
// 248 -> 250, 134 M 1040 -> 1014; C = 12288, K = 5, 16 M 296 -> 288, 134 M 2321 -> 2249; K = 1, C = 16384, 64 K 6.7 -> 6.2, 256 K 7.1 -> 6.4, 1 M +-0, C = 8448, 64 K
// 4.7 -> 4.8.
static bool ring_lp_any_fold(int k, size_t n)
{
    return (k == 1 && n <= (static_cast<size_t>(1) << 18)) || k * n >= (static_cast<size_t>(5) << 24);
}

template <int RPW, bool FOLD>
__global__ void __launch_bounds__(wg_threads_max(RPW))
k_ring_avg_lp_any(PtrTable xin, MutPtrTable xout, MutPtrTable xhat, MutPtrTable codes, MutPtrTable minmax, int k, size_t n,
                  uint32_t chunk, float third, int keep, ChunkOrder order)
{
    __shared__ float s_red[2][2 * kMaxWaves];
    const size_t c = order(blockIdx.x);
    const size_t base = c * static_cast<size_t>(chunk);
    const int len = static_cast<int>((n - base < chunk) ? (n - base) : chunk);
    if (FOLD && chunk_full<RPW>(len, blockDim.x >> 6)) ring_lp_chunk_any<RPW, true>(xin, xout, xhat, codes, minmax, k, base, c, len, third, keep, s_red);
    else ring_lp_chunk_any<RPW, false>(xin, xout, xhat, codes, minmax, k, base, c, len, third, keep, s_red);
}

// Load and publish of a chunk in a launch short enough that its latency counts: neither a complete chunk nor one that is cut short has
// tail tests on its loads.
template <int RPW, bool READ_AGAIN>
__device__ __forceinline__ void lp_encode_folded(const float* x_c, float* hat_c, uint8_t* codes_c, float* minmax_c, int len, int wave, int lane,
                                                 int nwaves, f4 (&x)[RPW], f4 (&h)[RPW], float* s_red, int keep)
{
    if (chunk_full<RPW>(len, nwaves)) {
        lp_load_at<RPW, true, READ_AGAIN>(x_c, hat_c, len, wave, lane, x, h);
        lp_publish<RPW, true>(x, h, hat_c, codes_c, minmax_c, len, wave, lane, nwaves, s_red, keep);
    } else {
        lp_load_at<RPW, false, READ_AGAIN>(x_c, hat_c, len, wave, lane, x, h);
        lp_publish<RPW, false>(x, h, hat_c, codes_c, minmax_c, len, wave, lane, nwaves, s_red, keep);
    }
}

// ------------------------------------------------------------------------------------------ LP, in two launches
// Every chunk of every peer by a workgroup of its own, then the mix row by row: 25 bytes per element of a peer instead of 17, but no
// workgroup goes through the peers one after the other, which takes 1.6 to 5.6 us each (the unrolled kernel's instructions come from
// memory in every launch, and each peer waits for its statistics).  One launch -> two, us (from graphs, four sets of buffers in turn):
//   K = 8: C = 4096, 64 K elements per peer 13.3 -> 7.1, 256 K 19.1 -> 12.9, 1 M 27.3 -> 43.6; C = 8192, 64 K 17.1 -> 7.7, 256 K 27.7 -> 14.0, 1 M 35.5 -> 44.4;
//   K = 16: C = 4096, 64 K 32.0 -> 9.0, 256 K 37.3 -> 22.8, 1 M 51.8 -> 79.9; C = 8192, 64 K 47.4 -> 9.0, 256 K 55.7 -> 23.8, 1 M 70.7 -> 80.9;
//   C = 16384: K = 2, 64 K 10.0 -> 6.9, 1 M 19.7 -> 13.7, 1.25 M 20.8 -> 15.8; K = 3, 64 K 13.0 -> 7.4, 1 M 26.5 -> 18.1; K = 5, 64 K 25.6 -> 8.4, 1 M 39.3 -> 29.7,
//   2 M 46.5 -> 54.1; K = 8, 1 M 57.9 -> 42.4; K = 16, 64 K 90.0 -> 12.1, 1 M 107.6 -> 82.7, 2 M 127.1 -> 168.9;   C = 8192: K = 3, 64 K 8.0 -> 6.1, K = 4, 200 K
//   12.4 -> 9.1, K = 8, 400 K 30.0 -> 20.0;   C = 12288, K = 4, 1 M 26.9 -> 25.4, 1.25 M 29.0 -> 29.3.
// With chunks up to 4096 elements fewer peers gain less than a second launch costs the host (K = 4, C = 2048, 64 K 7.3 -> 5.6, K = 3 6.2 -> 5.5).
// One workgroup for all peers takes 2 to 3.5 us a peer, longer chunks more, at nearly any length; two launches take what the bytes take, so that the line
// does not rise with the peers for good.  K = 32: C = 1024, 393 K 70.2 -> 51.5, 500 K 73.6 -> 76.9, 786 K 80.6 -> 105.8; C = 2048, 500 K 79.2 -> 79.2, 600 K 80.8
// -> 85.0; C = 3072, 590 K 80.9 -> 79.2; C = 4096, 590 K 91.9 -> 78.5, 786 K 98.7 -> 105.9; C = 4352, 600 K 95.5 -> 85.6, 786 K 102.4 -> 106.2; C = 6144, 786 K 110.4 ->
// 106.8; K = 24: C = 1024, 500 K 56.6 -> 59.1; C = 4352, 786 K 79.3 -> 79.6.
static bool ring_lp_two_launches(int k, size_t n, size_t chunk)
{
    if (n < 4) return false;   // row_at
    if (chunk > 8192) return k >= 2 && n <= 5 * (static_cast<size_t>(1) << 18);
    if (chunk > 4096) return k >= 3 && n <= std::min<size_t>(static_cast<size_t>(k) << 16, k > 24 && chunk < 6144 ? 5 << 17 : 3 << 18);
    return k >= 5 && n <= static_cast<size_t>(std::min(k, chunk > 2048 ? 24 : 16)) * 24 * 1024;
}

template <int RPW>
__global__ void __launch_bounds__(wg_threads_max(RPW))
k_ring_publish(PtrTable xin, MutPtrTable xhat, MutPtrTable codes, MutPtrTable minmax, size_t n, uint32_t chunk)
{
    __shared__ float s_red[2 * kMaxWaves];
    const size_t c = blockIdx.x;
    const int i = blockIdx.y;
    const size_t base = c * static_cast<size_t>(chunk);
    const int len = static_cast<int>((n - base < chunk) ? (n - base) : chunk);
    const int wave = wave_index(), lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;
    f4 x[RPW], h[RPW];
    lp_encode_folded<RPW, true>(static_cast<const float*>(xin.p[i]) + base, static_cast<float*>(xhat.p[i]) + base,
                                static_cast<uint8_t*>(codes.p[i]) + base, static_cast<float*>(minmax.p[i]) + 2 * c, len, wave, lane, nwaves, x,
                                h, s_red, 0);
}

__global__ void __launch_bounds__(kWave * kRowWaves)
k_ring_mix(PtrTable xin, MutPtrTable xout, MutPtrTable xhat, int k, size_t n, float third, ChunkOrder order)
{
    const uint32_t row = order(blockIdx.x) * kRowWaves + wave_index();
    const int lane = threadIdx.x & 63, i = blockIdx.y, l = i == 0 ? k - 1 : i - 1, r = i == k - 1 ? 0 : i + 1;
    const size_t e0 = static_cast<size_t>(row) * kRow;
    if (e0 >= n) return;
    const int remain = static_cast<int>((n - e0 < static_cast<size_t>(kRow)) ? (n - e0) : kRow);
    const f4 x = load_row(static_cast<const float*>(xin.p[i]) + e0, lane, remain, 0.0f);
    const f4 h = load_row(static_cast<const float*>(xhat.p[i]) + e0, lane, remain, 0.0f);
    const f4 hl = load_row_keep(static_cast<const float*>(xhat.p[l]) + e0, lane, remain, 0.0f);
    const f4 hr = load_row_keep(static_cast<const float*>(xhat.p[r]) + e0, lane, remain, 0.0f);
    store_row(static_cast<float*>(xout.p[i]) + e0, lane, remain, add4(mul4(add4(add4(hl, h), hr), third), sub4(x, h)));
}

// ------------------------------------------------------------------------------------------ LP, one peer
// d = x - xhat; codes, minmax = Q(d); xhat <- xhat + decode.  The codes are for other peers, nothing here reads them
// next: they are streamed past the caches (kept there, encode + mix of 50 M elements takes 320 us instead of 315 us).
template <int RPW, bool READ_AGAIN, bool SHORT>
__global__ void __launch_bounds__(wg_threads_max(RPW))
k_lp_encode(const float* __restrict__ x_in, float* __restrict__ xhat, size_t n, uint32_t chunk,
            uint8_t* __restrict__ codes, float* __restrict__ minmax)
{
    __shared__ float s_red[2 * kMaxWaves];
    const size_t c = blockIdx.x;
    const size_t base = c * static_cast<size_t>(chunk);
    const int len = static_cast<int>((n - base < chunk) ? (n - base) : chunk);
    const int wave = wave_index(), lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;
    f4 x[RPW], h[RPW];
    if constexpr (SHORT) {
        lp_encode_folded<RPW, READ_AGAIN>(x_in + base, xhat + base, codes + base, minmax + 2 * c, len, wave, lane, nwaves, x, h, s_red, 0);
    } else {
        lp_load<RPW, READ_AGAIN>(x_in + base, xhat + base, len, wave, lane, x, h);
        lp_publish<RPW>(x, h, xhat + base, codes + base, minmax + 2 * c, len, wave, lane, nwaves, s_red, 0);
    }
}

// Up to 2^23 elements the encode has no tail tests on its loads: encode + mix, 64 K, C = 4096, 5.4 -> 5.2 us, C = 16384 7.3 -> 7.0, 2 M, C =
// 16384, 17.7 -> 17.2, 8 M 55.8 -> 55.2 (C = 8192); at 33 M +-0.2 %, C = 16384 +1 %.
inline bool lp_encode_short(size_t n) { return n >= 4 && n <= (static_cast<size_t>(1) << 23); }

// `elements`: of all peers that are encoded before the first mix.  READ_AGAIN pays up to 2^27 of them; without -> with it,
// encode + mix of one peer: 6.5 M 50.0 -> 46.6 us, 25.6 M 174 -> 158 us, 50 M 332 -> 315 us, 134 M 949 -> 936 us, 300 M 2169 ->
// 2185 us; 8 workers that all choose one way: 8 x 4 M 173 -> 163 us, 8 x 16 M 633 -> 624 us, 8 x 25 M 959 -> 960 us, 8 x 50 M
// 1888 -> 1963 us, 32 x 5 M 852 -> 881 us, 32 x 8 M 1307 -> 1361 us (without tail tests as well, for which there is no form that streams).
static void launch_lp_encode(const float* x, float* xhat, size_t n, size_t chunk, uint8_t* codes, float* minmax, size_t elements,
                             hipStream_t stream)
{
    const int rows = static_cast<int>(chunk / kRow);
    const int rpw = pick_rpw(rows, BAGUA_RPW_LP);
    const dim3 grid(static_cast<unsigned>(num_chunks(n, chunk))), block(64 * ((rows + rpw - 1) / rpw));
    const uint32_t ch = static_cast<uint32_t>(chunk);
    const bool again = elements <= (static_cast<size_t>(1) << 27);
    if (again && lp_encode_short(n)) {
        BAGUA_DISPATCH_RPW(rpw, launch_kernel((k_lp_encode<RPW, true, true>), grid, block, 0, stream, x, xhat, n, ch, codes, minmax))
    } else if (again) {
        BAGUA_DISPATCH_RPW(rpw, launch_kernel((k_lp_encode<RPW, true, false>), grid, block, 0, stream, x, xhat, n, ch, codes, minmax))
    } else {
        BAGUA_DISPATCH_RPW(rpw, launch_kernel((k_lp_encode<RPW, false, false>), grid, block, 0, stream, x, xhat, n, ch, codes, minmax))
    }
}

// ------------------------------------------------------------------------------------------ host
static size_t ring_fp_groups(int k, size_t n)
{
    const size_t rows = (n + kRow - 1) / kRow, per = static_cast<size_t>(ring_fp_rows(k));
    return (rows + per - 1) / per;
}

template <int K>
static void launch_fp_k(const PtrTable& in, const MutPtrTable& out, size_t n, float third, hipStream_t s)
{
    const dim3 grid(static_cast<unsigned>(ring_fp_groups(K, n)));
    const size_t lds = K >= 2 && ring_fp_long(K, n) ? lds_for_residency(ring_fp_waves(K)) : 0;   // one replica is a copy
    launch_kernel((k_ring_avg_fp<K>), grid, dim3(kWave), lds, s, in, out, n, third);
}

static int launch_ring_fp(const float* const* x_in, float* const* x_out, int k, size_t n, hipStream_t stream)
{
    PtrTable in{};
    MutPtrTable out{};
    for (int i = 0; i < k; ++i) {
        in.p[i] = x_in[i];
        out.p[i] = x_out[i];
    }
    const float third = 1.0f / 3.0f;
    switch (k) {
#define BAGUA_FP_CASE(K) case K: launch_fp_k<K>(in, out, n, third, stream); break;
        BAGUA_FP_CASE(1) BAGUA_FP_CASE(2) BAGUA_FP_CASE(3) BAGUA_FP_CASE(4) BAGUA_FP_CASE(5) BAGUA_FP_CASE(6)
        BAGUA_FP_CASE(7) BAGUA_FP_CASE(8) BAGUA_FP_CASE(9) BAGUA_FP_CASE(10) BAGUA_FP_CASE(11) BAGUA_FP_CASE(12)
        BAGUA_FP_CASE(13) BAGUA_FP_CASE(14) BAGUA_FP_CASE(15) BAGUA_FP_CASE(16)
#undef BAGUA_FP_CASE
        default:
            launch_kernel(k_ring_avg_fp_any, dim3(static_cast<unsigned>(ring_fp_groups(k, n))), dim3(kWave * kRowWaves), 0, stream, in,
                               out, k, n, third);
    }
    return launch_status();
}

// Which instance runs (K peers, chunks of at most 32 rows), all figures by this rule against the other instance:
//   no tail tests (FULL) in wide chunks: 16 peers x 25.6 M, C = 8192, 1258 -> 1209 us, 8 x 100 M 2578 -> 2500 us, 8 x 2 M
//     55 -> 49 us; C = 6144, 8 x 100 M, 2672 -> 2501 us; only 4 and 5 peers x 34-134 M at C = 8192 lose 1-3 %;
//   and in short launches: below 2^21 elements, 8 x 1 M, C = 2048, 30.3 -> 25.5 us, 4 x 1 M, C = 4096, 16.8 -> 15.1 us.
//     In longer ones chunks up to 4096 elements stream better with the tests, which keep a wave's rows apart: 16 x 3.2 M,
//     C = 2048, 149 against 159 us, 16 x 25.6 M, C = 4096, 1307 against 1349 us;
//   two and three peers hold little enough without: 3 x 2 M, C = 6144, 23 against 26 us;
//   an odd number of rows never fills the last wave; from 8 peers on the loop is then faster than unrolled tail tests: 8 x
//     25.6 M, C = 5376, 761 -> 704 us, 16 x 25.6 M 1428 -> 1393 us, but 4 x 25.6 M 335 against 364 us.
template <int K>
static void launch_lp_k(const PtrTable& in, const MutPtrTable& out, const MutPtrTable& hat, const MutPtrTable& cd,
                        const MutPtrTable& mm, size_t n, uint32_t chunk, float third, dim3 grid, dim3 block,
                        hipStream_t s)
{
    const bool wide = chunk > kNarrowRows * kRow, odd = chunk % (BAGUA_RPW_LP * kRow) != 0;
    const int keep = keep_codes_of_round(K * n);
    const ChunkOrder order = chunk_order(grid.x, chunk);
#define BAGUA_RING_KEEP(KEEPv, FULLv, WIDEv)                                                                                  \
    launch_kernel((k_ring_avg_lp<K, BAGUA_RPW_LP, KEEPv, FULLv, WIDEv>), grid, block, 0, s, in, out, hat, cd, mm, n, chunk, third, order)
#define BAGUA_RING(FULLv, WIDEv)                   \
    {                                              \
        if (keep) BAGUA_RING_KEEP(1, FULLv, WIDEv); \
        else BAGUA_RING_KEEP(0, FULLv, WIDEv);      \
        return;                                    \
    }
    if constexpr (K >= 4) {
        if (!odd && (wide || n < (static_cast<size_t>(1) << 21))) BAGUA_RING(true, true)
    }
    if (!wide) BAGUA_RING(false, false)
    if constexpr (K < 8) BAGUA_RING(false, true)
    launch_kernel((k_ring_avg_lp_any<BAGUA_RPW_LP, false>), grid, block, 0, s, in, out, hat, cd, mm, K, n, chunk, third, keep, order);
#undef BAGUA_RING_KEEP
#undef BAGUA_RING
}

static int launch_ring_lp(const float* const* x_in, float* const* x_out, float* const* xhat, uint8_t* const* codes,
                          float* const* minmax, int k, size_t n, size_t chunk, hipStream_t stream)
{
    PtrTable in{};
    MutPtrTable out{}, hat{}, cd{}, mm{};
    for (int i = 0; i < k; ++i) {
        in.p[i] = x_in[i];
        out.p[i] = x_out[i];
        hat.p[i] = xhat[i];
        cd.p[i] = codes[i];
        mm.p[i] = minmax[i];
    }
    const float third = 1.0f / 3.0f;
    const size_t nc = num_chunks(n, chunk);
    const int rows = static_cast<int>(chunk / kRow);
    const int rpw = pick_rpw(rows, BAGUA_RPW_LP);
    dim3 grid(static_cast<unsigned>(nc)), block(64 * ((rows + rpw - 1) / rpw));
    const uint32_t ch = static_cast<uint32_t>(chunk);
    if (ring_lp_two_launches(k, n, chunk)) {
        const size_t nrows = (n + kRow - 1) / kRow;
        const dim3 all(static_cast<unsigned>(nc), k), mix(static_cast<unsigned>((nrows + kRowWaves - 1) / kRowWaves), k);
        BAGUA_DISPATCH_RPW(rpw, launch_kernel((k_ring_publish<RPW>), all, block, 0, stream, in, hat, cd, mm, n, ch))
        launch_kernel(k_ring_mix, mix, dim3(kWave * kRowWaves), 0, stream, in, out, hat, k, n, third,
                           row_order(mix.x, static_cast<uint32_t>(rows)));
        return launch_status();
    }
    if (rpw == BAGUA_RPW_LP) {   // at most kMaxWaves waves of that many rows
        switch (k) {
#define BAGUA_LP_CASE(K) case K: launch_lp_k<K>(in, out, hat, cd, mm, n, ch, third, grid, block, stream); return launch_status();
            BAGUA_LP_CASE(1) BAGUA_LP_CASE(2) BAGUA_LP_CASE(3) BAGUA_LP_CASE(4) BAGUA_LP_CASE(5) BAGUA_LP_CASE(6)
            BAGUA_LP_CASE(7) BAGUA_LP_CASE(8) BAGUA_LP_CASE(9) BAGUA_LP_CASE(10) BAGUA_LP_CASE(11) BAGUA_LP_CASE(12)
            BAGUA_LP_CASE(13) BAGUA_LP_CASE(14) BAGUA_LP_CASE(15) BAGUA_LP_CASE(16)
#undef BAGUA_LP_CASE
        }
    }
#define BAGUA_RING_ANY(RPWv, FOLDv)                                                                                    \
    launch_kernel((k_ring_avg_lp_any<RPWv, FOLDv>), grid, block, 0, stream, in, out, hat, cd, mm, k, n, ch, third, \
                  keep_codes_of_round(k * n), chunk_order(nc, chunk))
    if (rpw == 2) BAGUA_RING_ANY(2, false);
    else if (ring_lp_any_fold(k, n)) BAGUA_RING_ANY(4, true);
    else BAGUA_RING_ANY(4, false);
#undef BAGUA_RING_ANY
    return launch_status();
}

}  // namespace bagua

using namespace bagua;

extern "C" int bagua_decentralized_avg(int mode, const float* const* x_in, float* const* x_out, float* const* xhat,
                                       uint8_t* const* codes, float* const* minmax, int k, size_t n, size_t chunk,
                                       void* stream)
{
    if (mode != BAGUA_AVG_FP && mode != BAGUA_AVG_LP_MINMAX_U8) return BAGUA_ERR_INVALID_ARG;
    if (!x_in || !x_out || k < 1 || k > BAGUA_MAX_WORKERS || n == 0) return BAGUA_ERR_INVALID_ARG;
    const bool lp = mode == BAGUA_AVG_LP_MINMAX_U8;
    if (lp && (!xhat || !codes || !minmax || !chunk_ok(chunk))) return BAGUA_ERR_INVALID_ARG;
    for (int i = 0; i < k; ++i) {
        if (!x_in[i] || !x_out[i]) return BAGUA_ERR_INVALID_ARG;
        if (lp && (!xhat[i] || !codes[i] || !minmax[i])) return BAGUA_ERR_INVALID_ARG;
    }
    {
        const size_t bytes = n * sizeof(float);
        RangeCheck rc;
        for (int i = 0; i < k; ++i) {
            rc.reads(x_in[i], bytes);
            rc.writes(x_out[i], bytes);
            if (lp) {
                rc.writes(xhat[i], bytes);
                rc.writes(codes[i], n);
                rc.writes(minmax[i], 2 * num_chunks(n, chunk) * sizeof(float));
            }
        }
        if (!rc.disjoint()) return BAGUA_ERR_INVALID_ARG;
    }
    for (int i = 0; i < k; ++i) {
        if (!aligned16(x_in[i]) || !aligned16(x_out[i])) return BAGUA_ERR_ALIGNMENT;
        if (lp && (!aligned16(xhat[i]) || !aligned16(codes[i]) || !aligned4(minmax[i]))) return BAGUA_ERR_ALIGNMENT;
    }
    if ((lp ? num_chunks(n, chunk) : ring_fp_groups(k, n)) > kMaxGrid) return BAGUA_ERR_UNSUPPORTED;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (!lp) return launch_ring_fp(x_in, x_out, k, n, s);
    return launch_ring_lp(x_in, x_out, xhat, codes, minmax, k, n, chunk, s);
}

// ------------------------------------------------------------------------------------------ chosen peers
// x_out[i] = (x_in[i] + x_in[peer[i]]) * 0.5.  The host turns the peer map into "jobs": a matched
// pair (a, b) is one job that reads both replicas once and writes the same bits to both outputs
// (8 bytes per element per peer); any other worker is a job of its own that reads its two inputs.
namespace bagua {

struct PeerJobs {
    const float* a[BAGUA_MAX_WORKERS];
    const float* b[BAGUA_MAX_WORKERS];
    float* out_a[BAGUA_MAX_WORKERS];
    float* out_b[BAGUA_MAX_WORKERS];  // nullptr for a single-output job
};

__global__ void __launch_bounds__(kWave * kRowWaves)
k_peer_avg_fp(PeerJobs jobs, size_t n)
{
    const int job = blockIdx.y;
    const size_t row = static_cast<size_t>(blockIdx.x) * kRowWaves + wave_index();
    const int lane = threadIdx.x & 63;
    const size_t e0 = row * kRow;
    if (e0 >= n) return;
    const int remain = static_cast<int>((n - e0 < static_cast<size_t>(kRow)) ? (n - e0) : kRow);
    const f4 xa = load_row(jobs.a[job] + e0, lane, remain, 0.0f);
    const f4 xb = load_row(jobs.b[job] + e0, lane, remain, 0.0f);
    const f4 o = mul4(add4(xa, xb), 0.5f);
    store_row(jobs.out_a[job] + e0, lane, remain, o);
    if (jobs.out_b[job]) store_row(jobs.out_b[job] + e0, lane, remain, o);
}

}  // namespace bagua

extern "C" int bagua_decentralized_avg_peers(const float* const* x_in, float* const* x_out, const int* peer, int k,
                                             size_t n, void* stream)
{
    if (!x_in || !x_out || !peer || k < 1 || k > BAGUA_MAX_WORKERS || n == 0) return BAGUA_ERR_INVALID_ARG;
    for (int i = 0; i < k; ++i)
        if (!x_in[i] || !x_out[i] || peer[i] < 0 || peer[i] >= k) return BAGUA_ERR_INVALID_ARG;
    {
        RangeCheck rc;
        for (int i = 0; i < k; ++i) {
            rc.reads(x_in[i], n * sizeof(float));
            rc.writes(x_out[i], n * sizeof(float));
        }
        if (!rc.disjoint()) return BAGUA_ERR_INVALID_ARG;
    }
    for (int i = 0; i < k; ++i)
        if (!aligned16(x_in[i]) || !aligned16(x_out[i])) return BAGUA_ERR_ALIGNMENT;
    const size_t rows = (n + kRow - 1) / kRow;
    if ((rows + kRowWaves - 1) / kRowWaves > kMaxGrid) return BAGUA_ERR_UNSUPPORTED;
    PeerJobs jobs{};
    int nj = 0;
    for (int i = 0; i < k; ++i) {
        const int p = peer[i];
        const bool matched = p != i && peer[p] == i;
        if (matched && p < i) continue;  // written by the partner's job
        jobs.a[nj] = x_in[i];
        jobs.b[nj] = x_in[p];
        jobs.out_a[nj] = x_out[i];
        jobs.out_b[nj] = matched ? x_out[p] : nullptr;
        ++nj;
    }
    launch_kernel(k_peer_avg_fp, dim3(static_cast<unsigned>((rows + kRowWaves - 1) / kRowWaves), nj), dim3(kWave * kRowWaves), 0,
                       static_cast<hipStream_t>(stream), jobs, n);
    return launch_status();
}

// ------------------------------------------------------------------------------------------ C_FP_S
// Centralised full-precision average of k replicas: out = (x_0 + x_1 + ...) * inv_k, ascending order.
// One wave per row; the loads of four workers are in flight together.
namespace bagua {

__global__ void __launch_bounds__(kWave * kRowWaves)
k_centralized_avg_fp(PtrTable xs, int k, float inv_k, size_t n, float* __restrict__ out)
{
    const size_t row = static_cast<size_t>(blockIdx.x) * kRowWaves + wave_index();
    const int lane = threadIdx.x & 63;
    const size_t e0 = row * kRow;
    if (e0 >= n) return;
    const int remain = static_cast<int>((n - e0 < static_cast<size_t>(kRow)) ? (n - e0) : kRow);
    f4 s = load_row(static_cast<const float*>(xs.p[0]) + e0, lane, remain, 0.0f);
    int j = 1;
    for (; j + 4 <= k; j += 4) {
        f4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = load_row(static_cast<const float*>(xs.p[j + u]) + e0, lane, remain, 0.0f);
#pragma unroll
        for (int u = 0; u < 4; ++u) s = add4(s, v[u]);
    }
    for (; j < k; ++j) s = add4(s, load_row(static_cast<const float*>(xs.p[j]) + e0, lane, remain, 0.0f));
    store_row(out + e0, lane, remain, mul4(s, inv_k));
}

}  // namespace bagua

extern "C" int bagua_centralized_avg_fp(const float* const* x, int k, size_t n, float* out, void* stream)
{
    if (!x || k < 1 || k > BAGUA_MAX_WORKERS || n == 0 || !out) return BAGUA_ERR_INVALID_ARG;
    {
        RangeCheck rc;
        for (int j = 0; j < k; ++j) {
            if (!x[j]) return BAGUA_ERR_INVALID_ARG;
            rc.reads(x[j], n * sizeof(float));
        }
        rc.writes(out, n * sizeof(float));
        if (!rc.disjoint()) return BAGUA_ERR_INVALID_ARG;
    }
    for (int j = 0; j < k; ++j)
        if (!aligned16(x[j])) return BAGUA_ERR_ALIGNMENT;
    if (!aligned16(out)) return BAGUA_ERR_ALIGNMENT;
    const size_t rows = (n + kRow - 1) / kRow;
    if ((rows + kRowWaves - 1) / kRowWaves > kMaxGrid) return BAGUA_ERR_UNSUPPORTED;
    PtrTable xt{};
    for (int j = 0; j < k; ++j) xt.p[j] = x[j];
    launch_kernel(k_centralized_avg_fp, dim3(static_cast<unsigned>((rows + kRowWaves - 1) / kRowWaves)), dim3(kWave * kRowWaves), 0,
                       static_cast<hipStream_t>(stream), xt, k, 1.0f / static_cast<float>(k), n, out);
    return launch_status();
}

// ------------------------------------------------------------------------------------------ chosen peers, LP
// D_LP_S with one chosen peer per worker (Sections 3.2 and 3.4): every worker publishes Q(x - xhat),
// all holders advance xhat, then x_out[i] = (xhat[i] + xhat[peer[i]]) * 0.5 + (x[i] - xhat[i]).
// A matched pair is one fused job: a workgroup owns one chunk of both partners, so x and xhat of
// each are read once and out, xhat, codes written once (17 bytes per element per peer).  A worker
// that is its own peer (the odd one out of a random matching) is a job with one side.  Only a worker
// whose peer chose somebody else takes two passes: k_lp_encode, then a mix over the advanced public copies.
namespace bagua {

struct PeerLpJobs {
    const float* x[2][BAGUA_MAX_WORKERS];   // side 1 is unused where a worker is its own peer
    float* out[2][BAGUA_MAX_WORKERS];
    float* hat[2][BAGUA_MAX_WORKERS];
    uint8_t* codes[2][BAGUA_MAX_WORKERS];
    float* minmax[2][BAGUA_MAX_WORKERS];
};

// Job after job over blockIdx.y, so that only one pair's ten streams are interleaved.  7 workers x 25.6 M elements
// (three pairs and a single), C = 4096: 0.50 ms; encode + mix in two passes 0.83 ms.
// Two rows per wave are held in 64 VGPRs, eight waves per SIMD; the compiler would take 70.  Up to C = 6144 that is +-1 %.  At
// C = 8192 it is two workgroups per CU instead of one: 8 x 1 M 27.9 -> 24.4 us, 2 x 6.5 M 45.3 -> 41.3 us, 4 x 12 M +-0, but
// 4 x 25.6 M 303 -> 314 us and 8 x 100 M 2477 -> 2569 us.
// SHORT: no tail tests on the loads, and the workers that sit out are jobs from `npairs` on in the pairs' launch.  Two launches with tests
// -> one without, us: three pairs and a single, C = 4096, 64 K 8.7 -> 5.2, 256 K 12.0 -> 7.6, 1 M 23.6 -> 22.5, 8 M 163.3 -> 159.2, 16 M 338.8 ->
// 345.2; C = 16384, 64 K 18.0 -> 10.6, 1 M 29.1 -> 22.2, 8 M 177.9 -> 172.8, 16 M 368.2 -> 374.6; one pair, C = 4096, 256 K 6.3 -> 5.6, 1 M 8.7 ->
// 8.1, 2 M +-0, 8 M 47.9 -> 48.5; C = 16384, 2 M 17.0 -> 15.3, 4 M 27.7 -> 29.4.
inline bool gossip_short(size_t n, int singles) { return n >= 4 && n <= (static_cast<size_t>(1) << (singles ? 23 : 21)); }

// Chunks above 8192 elements in two launches, as in the ring, where all workers together have little to do.  A pair at a time -> this, us: one pair,
// C = 16384, 64 K 9.5 -> 6.7, 200 K 9.2 -> 7.6, 700 K +-0; three pairs and a single 64 K 10.5 -> 7.6, 200 K 12.5 -> 12.8; eight pairs 64 K 11.8 -> 11.4.
inline bool gossip_wide_short(size_t chunk, int k, size_t n) { return chunk > 8192 && n >= 4 && k * n <= (static_cast<size_t>(1) << 19); }

template <int RPW, bool PAIR, bool SHORT>
__global__ void __launch_bounds__(wg_threads_max(RPW), RPW <= 2 ? 8 : 1)
k_peer_avg_lp(PeerLpJobs jobs, int npairs, size_t n, uint32_t chunk, int keep, ChunkOrder order)
{
    __shared__ float s_red[2][2 * kMaxWaves];
    const int job = blockIdx.y;
    const size_t c = order(blockIdx.x);
    const size_t base = c * static_cast<size_t>(chunk);
    const int len = static_cast<int>((n - base < chunk) ? (n - base) : chunk);
    const int wave = wave_index(), lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;

    f4 h[2][RPW], own[2][RPW];
    auto publish = [&](int sd) {
        const float* x_c = jobs.x[sd][job] + base;
        float *hat_c = jobs.hat[sd][job] + base, *minmax_c = jobs.minmax[sd][job] + 2 * c;
        uint8_t* codes_c = jobs.codes[sd][job] + base;
        if constexpr (SHORT) {
            lp_encode_folded<RPW, false>(x_c, hat_c, codes_c, minmax_c, len, wave, lane, nwaves, own[sd], h[sd], s_red[sd], keep);
        } else {
            lp_load<RPW>(x_c, hat_c, len, wave, lane, own[sd], h[sd]);
            lp_publish<RPW>(own[sd], h[sd], hat_c, codes_c, minmax_c, len, wave, lane, nwaves, s_red[sd], keep);
        }
    };
    auto mix = [&](int sd, int second) {   // the sum of a pair is the same one for both sides
#pragma unroll
        for (int r = 0; r < RPW; ++r) {
            const int off = static_cast<int>(wave * RPW + r) * kRow;
            const int remain = len - off;
            const f4 avg = mul4(add4(h[0][r], h[second][r]), 0.5f);
            if (remain > 0) store_row(jobs.out[sd][job] + base + off, lane, remain, add4(avg, own[sd][r]));
        }
    };
    publish(0);
    if (PAIR && (!SHORT || job < npairs)) {
        publish(1);
        mix(0, 1);
        mix(1, 1);
    } else {
        mix(0, 0);
    }
}

// Second pass of the general case: worker i = blockIdx.y reads the advanced xhat of itself and of its peer.
struct PeerMixJobs {
    const float* x[BAGUA_MAX_WORKERS];
    const float* hat_own[BAGUA_MAX_WORKERS];
    const float* hat_peer[BAGUA_MAX_WORKERS];
    float* out[BAGUA_MAX_WORKERS];
};

__global__ void __launch_bounds__(kWave * kRowWaves)
k_peer_mix_lp(PeerMixJobs jobs, size_t n)
{
    const int i = blockIdx.y;
    const size_t row = static_cast<size_t>(blockIdx.x) * kRowWaves + wave_index();
    const int lane = threadIdx.x & 63;
    const size_t e0 = row * kRow;
    if (e0 >= n) return;
    const int remain = static_cast<int>((n - e0 < static_cast<size_t>(kRow)) ? (n - e0) : kRow);
    const f4 a = load_row(jobs.hat_own[i] + e0, lane, remain, 0.0f);
    const f4 b = load_row(jobs.hat_peer[i] + e0, lane, remain, 0.0f);
    const f4 xi = load_row(jobs.x[i] + e0, lane, remain, 0.0f);
    store_row(jobs.out[i] + e0, lane, remain, add4(mul4(add4(a, b), 0.5f), sub4(xi, a)));
}

}  // namespace bagua

extern "C" int bagua_decentralized_avg_peers_lp(const float* const* x_in, float* const* x_out, float* const* xhat,
                                                uint8_t* const* codes, float* const* minmax, const int* peer, int k,
                                                size_t n, size_t chunk, void* stream)
{
    if (!x_in || !x_out || !xhat || !codes || !minmax || !peer || k < 1 || k > BAGUA_MAX_WORKERS || n == 0 ||
        !chunk_ok(chunk))
        return BAGUA_ERR_INVALID_ARG;
    for (int i = 0; i < k; ++i)
        if (!x_in[i] || !x_out[i] || !xhat[i] || !codes[i] || !minmax[i] || peer[i] < 0 || peer[i] >= k)
            return BAGUA_ERR_INVALID_ARG;
    {
        const size_t bytes = n * sizeof(float);
        RangeCheck rc;
        for (int i = 0; i < k; ++i) {
            rc.reads(x_in[i], bytes);
            rc.writes(x_out[i], bytes);
            rc.writes(xhat[i], bytes);
            rc.writes(codes[i], n);
            rc.writes(minmax[i], 2 * num_chunks(n, chunk) * sizeof(float));
        }
        if (!rc.disjoint()) return BAGUA_ERR_INVALID_ARG;
    }
    for (int i = 0; i < k; ++i)
        if (!aligned16(x_in[i]) || !aligned16(x_out[i]) || !aligned16(xhat[i]) || !aligned16(codes[i]) ||
            !aligned4(minmax[i]))
            return BAGUA_ERR_ALIGNMENT;
    const size_t nrows = (n + kRow - 1) / kRow;
    if ((nrows + 3) / 4 > kMaxGrid) return BAGUA_ERR_UNSUPPORTED;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const size_t nc = num_chunks(n, chunk);
    const int rows = static_cast<int>(chunk / kRow);
    const uint32_t ch = static_cast<uint32_t>(chunk);

    const int rpw = pick_rpw(rows, BAGUA_RPW_LP);
    dim3 grid(static_cast<unsigned>(nc)), block(64 * ((rows + rpw - 1) / rpw));
    const ChunkOrder order = chunk > 4096 ? chunk_order(nc, chunk) : ChunkOrder{0, 0};   // shorter chunks: -3 .. +1.5 %
    // matched pairs and workers that are their own peer: one pass
    PeerLpJobs pairs{}, singles{};
    PeerMixJobs mix{};
    int npairs = 0, nsingles = 0, nmix = 0;
    size_t encoded = 0;
    for (int i = 0; i < k; ++i) encoded += peer[peer[i]] != i;
    for (int i = 0; i < k; ++i) {
        const int p = peer[i];
        if (peer[p] != i) {                             // its choice chose somebody else: two passes
            launch_lp_encode(x_in[i], xhat[i], n, chunk, codes[i], minmax[i], encoded * n, s);
            mix.x[nmix] = x_in[i];
            mix.hat_own[nmix] = xhat[i];
            mix.hat_peer[nmix] = xhat[p];
            mix.out[nmix] = x_out[i];
            ++nmix;
        } else if (p >= i) {
            PeerLpJobs& jobs = p == i ? singles : pairs;
            const int j = p == i ? nsingles++ : npairs++;
            const int side[2] = {i, p};
            for (int sd = 0; sd < (p == i ? 1 : 2); ++sd) {
                jobs.x[sd][j] = x_in[side[sd]];
                jobs.out[sd][j] = x_out[side[sd]];
                jobs.hat[sd][j] = xhat[side[sd]];
                jobs.codes[sd][j] = codes[side[sd]];
                jobs.minmax[sd][j] = minmax[side[sd]];
            }
        }
    }
    if (nmix == 0 && gossip_wide_short(chunk, k, n)) {
        PtrTable in{};
        MutPtrTable hat{}, cd{}, mm{};
        PeerMixJobs all{};
        for (int i = 0; i < k; ++i) {
            in.p[i] = x_in[i];
            hat.p[i] = xhat[i];
            cd.p[i] = codes[i];
            mm.p[i] = minmax[i];
            all.x[i] = x_in[i];
            all.hat_own[i] = xhat[i];
            all.hat_peer[i] = xhat[peer[i]];
            all.out[i] = x_out[i];
        }
        BAGUA_DISPATCH_RPW(rpw, launch_kernel((k_ring_publish<RPW>), dim3(grid.x, k), block, 0, s, in, hat, cd, mm, n, ch))
        launch_kernel(k_peer_mix_lp, dim3(static_cast<unsigned>((nrows + kRowWaves - 1) / kRowWaves), k), dim3(kWave * kRowWaves), 0, s, all, n);
        return launch_status();
    }
    if (npairs && gossip_short(n, nsingles)) {
        for (int j = 0; j < nsingles; ++j) {
            pairs.x[0][npairs + j] = singles.x[0][j];
            pairs.out[0][npairs + j] = singles.out[0][j];
            pairs.hat[0][npairs + j] = singles.hat[0][j];
            pairs.codes[0][npairs + j] = singles.codes[0][j];
            pairs.minmax[0][npairs + j] = singles.minmax[0][j];
        }
        BAGUA_DISPATCH_RPW(rpw, launch_kernel((k_peer_avg_lp<RPW, true, true>), dim3(grid.x, npairs + nsingles), block, 0, s, pairs, npairs, n, ch,
                                                   keep_codes_of_round(k * n), order))
        nsingles = 0;
    } else if (npairs) {
        BAGUA_DISPATCH_RPW(rpw, launch_kernel((k_peer_avg_lp<RPW, true, false>), dim3(grid.x, npairs), block, gossip_pairs_lds(chunk, npairs * n), s, pairs, npairs,
                                                   n, ch, keep_codes_of_round(k * n), order))
    }
    if (nsingles) {
        BAGUA_DISPATCH_RPW(rpw, launch_kernel((k_peer_avg_lp<RPW, false, false>), dim3(grid.x, nsingles), block, 0, s, singles, 0, n, ch,
                                                   keep_codes_of_round(k * n), order))
    }
    if (nmix) {                                         // all public copies are advanced by now
        launch_kernel(k_peer_mix_lp, dim3(static_cast<unsigned>((nrows + kRowWaves - 1) / kRowWaves), nmix),
                           dim3(kWave * kRowWaves), 0, s, mix, n);
    }
    return launch_status();
}

// ------------------------------------------------------------------------------------------ one peer's share of D_LP_S
// What a single GPU does in a sharded run of the low-precision ring (Sections 3.2 and 3.4): it encodes
// its own difference and advances its own public copy (k_lp_encode, 13 bytes per element), receives the
// two neighbours' codes, advances its copies of their public replicas and forms its own new replica
// (k_lp_apply_mix, 30 bytes per element).  The arithmetic is that of the all-peers kernel above.
namespace bagua {

// APPLY_L / APPLY_R: that neighbour's codes are decoded into its copy (otherwise the copy is current).
// SAME: both neighbours are one peer (ring of two): one copy, advanced once, counted twice.
template <bool APPLY_L, bool APPLY_R, bool SAME>
__global__ void __launch_bounds__(kWave * kRowWaves)
k_lp_apply_mix(const float* __restrict__ x, const float* __restrict__ h_own, float* h_left, float* h_right,
               const uint8_t* __restrict__ c_left, const float* __restrict__ m_left,
               const uint8_t* __restrict__ c_right, const float* __restrict__ m_right, size_t n, uint32_t rows_per_chunk,
               float third, float* __restrict__ x_out, ChunkOrder order)
{
    const uint32_t row = order(blockIdx.x) * kRowWaves + wave_index();
    const int lane = threadIdx.x & 63;
    const size_t e0 = static_cast<size_t>(row) * kRow;
    if (e0 >= n) return;
    const size_t c = row / rows_per_chunk;
    const int remain = static_cast<int>((n - e0 < static_cast<size_t>(kRow)) ? (n - e0) : kRow);
    const f4 xi = load_row(x + e0, lane, remain, 0.0f);
    const f4 ho = load_row(h_own + e0, lane, remain, 0.0f);
    auto advanced = [&](float* h, const uint8_t* codes, const float* mm, bool apply) {
        f4 v = load_row(h + e0, lane, remain, 0.0f);
        if (apply) {
            const float mn = mm[2 * c], step = minmax_step(mn, mm[2 * c + 1]);
            const uint32_t w = load_codes_row(codes + e0, lane, remain);
            v.x = v.x + (mn + byte_to_float(w, 0) * step);
            v.y = v.y + (mn + byte_to_float(w, 1) * step);
            v.z = v.z + (mn + byte_to_float(w, 2) * step);
            v.w = v.w + (mn + byte_to_float(w, 3) * step);
            store_row(h + e0, lane, remain, v);
        }
        return v;
    };
    const f4 hl = advanced(h_left, c_left, m_left, APPLY_L);
    const f4 hr = SAME ? hl : advanced(h_right, c_right, m_right, APPLY_R);
    const f4 s = add4(add4(hl, ho), hr);
    store_row(x_out + e0, lane, remain, add4(mul4(s, third), sub4(xi, ho)));
}

}  // namespace bagua

extern "C" int bagua_lp_encode(const float* x, float* xhat, size_t n, size_t chunk, uint8_t* codes, float* minmax,
                               void* stream)
{
    if (!x || !xhat || !codes || !minmax || n == 0 || !chunk_ok(chunk)) return BAGUA_ERR_INVALID_ARG;
    RangeCheck rc;
    rc.reads(x, n * sizeof(float));
    rc.writes(xhat, n * sizeof(float));
    rc.writes(codes, n);
    rc.writes(minmax, 2 * num_chunks(n, chunk) * sizeof(float));
    if (!rc.disjoint()) return BAGUA_ERR_INVALID_ARG;
    if (num_chunks(n, chunk) > kMaxGrid) return BAGUA_ERR_UNSUPPORTED;
    if (!aligned16(x) || !aligned16(xhat) || !aligned16(codes) || !aligned4(minmax)) return BAGUA_ERR_ALIGNMENT;
    launch_lp_encode(x, xhat, n, chunk, codes, minmax, n, static_cast<hipStream_t>(stream));
    return launch_status();
}

extern "C" int bagua_lp_apply_mix(const float* x, const float* xhat_own, float* xhat_left, float* xhat_right,
                                  const uint8_t* codes_left, const float* minmax_left, const uint8_t* codes_right,
                                  const float* minmax_right, size_t n, size_t chunk, float* x_out, void* stream)
{
    if (!x || !xhat_own || !xhat_left || !xhat_right || !x_out || n == 0 || !chunk_ok(chunk)) return BAGUA_ERR_INVALID_ARG;
    if ((codes_left == nullptr) != (minmax_left == nullptr) || (codes_right == nullptr) != (minmax_right == nullptr))
        return BAGUA_ERR_INVALID_ARG;
    const bool same = xhat_left == xhat_right;
    if (same && codes_right) return BAGUA_ERR_INVALID_ARG;  // one copy is advanced once, through codes_left
    const size_t bytes = n * sizeof(float), mbytes = 2 * num_chunks(n, chunk) * sizeof(float);
    RangeCheck rc;
    rc.reads(x, bytes);
    rc.reads(codes_left, n);
    rc.reads(minmax_left, mbytes);
    rc.reads(codes_right, n);
    rc.reads(minmax_right, mbytes);
    rc.writes(x_out, bytes);
    // a neighbour copy that is not advanced is only read (on a ring of one it is the peer's own copy)
    if (codes_left) rc.writes(xhat_left, bytes); else rc.reads(xhat_left, bytes);
    if (!same) { if (codes_right) rc.writes(xhat_right, bytes); else rc.reads(xhat_right, bytes); }
    rc.reads(xhat_own, bytes);
    if (!rc.disjoint()) return BAGUA_ERR_INVALID_ARG;
    const size_t rows = (n + kRow - 1) / kRow;
    if ((rows + kRowWaves - 1) / kRowWaves > kMaxGrid) return BAGUA_ERR_UNSUPPORTED;
    if (!aligned16(x) || !aligned16(xhat_own) || !aligned16(xhat_left) || !aligned16(xhat_right) || !aligned16(codes_left) ||
        !aligned16(codes_right) || !aligned4(minmax_left) || !aligned4(minmax_right) || !aligned16(x_out))
        return BAGUA_ERR_ALIGNMENT;
    dim3 grid(static_cast<unsigned>((rows + kRowWaves - 1) / kRowWaves)), block(kWave * kRowWaves);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint32_t rpc = static_cast<uint32_t>(chunk / kRow);
    const ChunkOrder order = n <= (static_cast<size_t>(1) << 25) ? row_order(grid.x, rpc) : ChunkOrder{0, 0};
    const float third = 1.0f / 3.0f;
#define BAGUA_MIX(L, R, S)                                                                                            \
    launch_kernel((k_lp_apply_mix<L, R, S>), grid, block, 0, s, x, xhat_own, xhat_left, xhat_right, codes_left, \
                       minmax_left, codes_right, minmax_right, n, rpc, third, x_out, order)
    const bool al = codes_left != nullptr, ar = codes_right != nullptr;
    if (same) { if (al) BAGUA_MIX(true, false, true); else BAGUA_MIX(false, false, true); }
    else if (al && ar) BAGUA_MIX(true, true, false);
    else if (al) BAGUA_MIX(true, false, false);
    else if (ar) BAGUA_MIX(false, true, false);
    else BAGUA_MIX(false, false, false);
#undef BAGUA_MIX
    return launch_status();
}
