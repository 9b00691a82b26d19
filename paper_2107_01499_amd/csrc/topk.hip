// Per-chunk top-K sparsification as a third compression function Q of C_LP_S (the aggressive
// compression the paper names when it motivates error compensation, Section 3.2): worker-side
// compress with error feedback, server-side decompress-average-recompress, and decompress.
//
// Selection of the K largest |v| of a chunk (ties: lower index) without sorting: the chunk stays in registers and is
// counted by the distance of each magnitude (as an integer: the bit pattern of |v|) below the chunk's largest one.  A
// first histogram of 64 bins per binade finds the bin with the K-th largest magnitude; if it does not reach that far
// down (an outlier, layers of different scale, fewer than K values that are not zero), one of a bin per binade follows.
// As long as the bin found holds more elements than are still needed, it alone is counted again, eight bits finer.
// Integer atomics in LDS only, so the result does not depend on execution order.  The kept
// elements' output slots come from ballots and bit counts.
#include "launchers.hpp"

#pragma clang fp contract(off)

namespace bagua {

// Bins of the first histogram: distances in units of 2^17 = 64 bins per binade, the four binades below the largest
// magnitude; what lies below is not counted, and looked at only if the bins do not reach the K-th.  Counted in a last
// bin instead, where many lanes of a wave meet in one counter, a short launch (1 M elements, one workgroup per CU) took
// 8.9 us instead of 7.2; two or four copies of the bins gained nothing.
constexpr int kBinBits = 8, kBins = 1 << kBinBits;
constexpr uint32_t kFirstShift = 17, kFirstBits = kFirstShift + kBinBits;
// The binades below: one lane sums one binade, so 64 of them (the last one takes what lies farther down as well), in eight
// copies, because a chunk's values share a handful of binades.
constexpr uint32_t kBinadeShift = 23, kBinadeCopies = 8;
// 0: the first histogram, 1 and 2: the binades.  Refinements take 1, 2 and 3, or 3, 0 and 1 behind the binades.  4.2 KB: 32
// workgroups of one wave still fit a CU.
constexpr int kHists = 4, kHistWords = kHists * kBins;
constexpr int kTopkLdsWords = kHistWords + 2 * kMaxWaves;
static_assert(kWave * kBinadeCopies == 2 * kBins, "the binades' counters take two histograms");

__device__ __forceinline__ uint32_t mag_key(float v) { return __float_as_uint(v) & 0x7fffffffu; }

struct OpMaxU { __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return a > b ? a : b; } };
struct OpAddU { __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return a + b; } };

// Inclusive prefix sum over the 64 lanes.
__device__ __forceinline__ uint32_t wave_prefix_incl(uint32_t x)
{
    x += dpp<kShr1>(x);
    x += dpp<kShr2>(x);
    x += dpp<kShr4>(x);
    x += dpp<kShr8>(x);
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), kBcast15, 0xa, 0xf, false));   // rows 1 and 3
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), kBcast31, 0xc, 0xf, false));   // rows 2 and 3
    return x;
}

// All lanes of a wave: bin = first of the 256 bins up to which the counts reach `need`, before = their sum below it,
// in_bin = its count.  If all of them together do not reach `need`, bin = 256, before = their sum and in_bin = 0.
__device__ __forceinline__ void find_bin(const uint32_t* h, int lane, uint32_t need, uint32_t& bin, uint32_t& before, uint32_t& in_bin)
{
    const uint4 b = reinterpret_cast<const uint4*>(h)[lane];
    const uint32_t c = b.x + b.y + b.z + b.w;
    const uint32_t pre = wave_prefix_incl(c);
    const unsigned long long reached = __ballot(pre >= need);
    if (reached == 0) {
        bin = 4 * kWave;
        before = __builtin_amdgcn_readlane(static_cast<int>(pre), 63);
        in_bin = 0;
        return;
    }
    const int L = __builtin_ctzll(reached);   // the lane whose four bins hold it
    const uint32_t below = __builtin_amdgcn_readlane(static_cast<int>(pre - c), L);
    const uint32_t own = h[4 * L + (lane & 3)];
    uint32_t run = own;   // inclusive sums over lanes 0..3; the others are not looked at
    run += dpp<kShr1>(run);
    run += dpp<kShr2>(run);
    const int q = __builtin_ctzll(__ballot(below + run >= need));
    bin = static_cast<uint32_t>(4 * L + q);
    in_bin = __builtin_amdgcn_readlane(static_cast<int>(own), q);
    before = below + __builtin_amdgcn_readlane(static_cast<int>(run), q) - in_bin;
}

__device__ __forceinline__ void topk_clear(uint32_t* hist, int words)
{
    for (int t = threadIdx.x; t < words / 4; t += blockDim.x) reinterpret_cast<uint4*>(hist)[t] = uint4{0u, 0u, 0u, 0u};
}

// Adds the wave's elements with distances in [lo, lo + 2^bits) to h, one bin per 2^shift.  Lanes that meet in one counter are
// served one after another; where many share a bin (`crowded`), all lanes that are in the bin of the first one that has
// any are added at once.
template <int RPW>
__device__ __forceinline__ void count_bins(const uint32_t (&dist)[RPW][4], uint32_t lo, uint32_t bits, uint32_t shift, bool crowded, int lane, uint32_t* h)
{
    if (__builtin_expect(!crowded, 1)) {
#pragma unroll
        for (int i = 0; i < RPW; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t r = dist[i][e] - lo;
                if ((r >> bits) == 0) atomicAdd(&h[r >> shift], 1u);
            }
        return;
    }
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t r = dist[i][e] - lo, bin = r >> shift;
            const unsigned long long in = __ballot((r >> bits) == 0);
            const int first = in != 0 ? __builtin_ctzll(in) : 0;
            const unsigned long long same = in & __ballot(bin == static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(bin), first)));
            const unsigned long long adds = (in & ~same) | (same & (0ull - same));   // same's first lane for all of them
            if (adds >> lane & 1) atomicAdd(&h[bin], lane == first ? static_cast<uint32_t>(__builtin_popcountll(same)) : 1u);
        }
    }
}

// The wave's elements with distances from lo on, one bin per binade, zeros left out.
template <int RPW>
__device__ __forceinline__ void count_binades(const uint32_t (&dist)[RPW][4], uint32_t lo, uint32_t top, int lane, uint32_t* h)
{
    constexpr uint32_t kFar = (static_cast<uint32_t>(kWave) << kBinadeShift) - 1;   // in the last of the 64
#pragma unroll
    for (int i = 0; i < RPW; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t r = dist[i][e] - lo;
            if (r < top - lo) atomicAdd(&h[((r < kFar ? r : kFar) >> kBinadeShift) * kBinadeCopies + (lane & (kBinadeCopies - 1))], 1u);
        }
}

// Number of lanes below this one with their bit set, added to acc.
__device__ __forceinline__ uint32_t lanes_below(unsigned long long mask, uint32_t acc)
{
    return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), acc));
}

// What bounds it: HBM from 2048-element chunks on if the magnitudes spread like a normal distribution's (12.2 bytes per element at
// 5.9 TB/s for 25.7 M elements), below that the waves per CU.  Before (four radix passes from the exponent down, its histogram in
// 16 copies: 20 KB of LDS per chunk, seven barriers, 122 vector instructions per element of a lane against 52) -> now, whole
// rounds: 3 workers x 33 M, C = 1024, 582 -> 398 us, 12 x 2.6 M, C = 2048, 144 -> 116 us, 8 x 25.7 M, C = 4096, 543 -> 530 us,
// 4 x 25.6 M, C = 16384, 574 -> 409 us.
// Other data, 25.7 M elements without error state that fit the caches, compression / server step of 4 workers; the radix passes -> this
// selection without count_binades and without the crowded form of count_bins -> with both:
//                                          C = 4096, K = 128                    C = 1024, K = 32
//   normal distribution                    33 / 39 -> 30.3 / 25 -> 30.7 / 25    74 / 89 -> 26.7 / 24 -> 27.1 / 24 us
//   the same and one outlier per chunk     32 / 39 -> 52 / 98 -> 39 / 28        75 / 90 -> 43 / 95 -> 35 / 27 us
//   all zero                               275 / 282 -> 355 / 360 -> 123 / 120  286 / 298 -> 348 / 356 -> 108 / 114 us
//   99 % zero                              272 / 280 -> 360 / 360 -> 33 / 32    284 / 296 -> 348 / 353 -> 30 / 31 us
//   all magnitudes equal                   274 / 39 -> 354 / 23 -> 123 / 23     286 / 90 -> 347 / 23 -> 108 / 23 us
// What is left of the equal magnitudes is the first histogram: a test for them before it costs normal data 2 %.
//
// Encode the chunk held in v (absent elements must be +0.0f).  idx_c/val_c point at the chunk's `keep` output slots,
// residual/out at the chunk's first element (nullptr = not wanted).
// smem: kTopkLdsWords words of LDS, the first kHistWords of them cleared (no barrier needed in between).
// JOINT: how the kept entries are stored, see the end.
template <int RPW, bool JOINT = false>
__device__ __forceinline__ void topk_encode_chunk(const f4 (&v)[RPW], int len, uint32_t keep, int wave, int lane, int nwaves,
                                                  float* __restrict__ residual, uint16_t* __restrict__ idx_c,
                                                  float* __restrict__ val_c, float* __restrict__ out, uint32_t* smem)
{
    uint32_t* s_top = smem + kHistWords;
    uint32_t* s_count = s_top + kMaxWaves;
    const uint32_t keff = (static_cast<int>(keep) < len) ? keep : static_cast<uint32_t>(len);

    // ---- the largest magnitude of the chunk, and every element's distance below it (absent elements: beyond all others)
    uint32_t top = 0;
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        top = OpMaxU{}(OpMaxU{}(top, mag_key(v[i].x)), mag_key(v[i].y));
        top = OpMaxU{}(OpMaxU{}(top, mag_key(v[i].z)), mag_key(v[i].w));
    }
    top = wave_reduce(top, OpMaxU{});
    if (lane == 0) s_top[wave] = top;
    __syncthreads();
    if (nwaves > 1) {
        if ((lane & (kMaxWaves - 1)) < nwaves) top = s_top[lane & (kMaxWaves - 1)];
        top = __builtin_amdgcn_readfirstlane(static_cast<int>(row16_reduce(top, OpMaxU{})));
    }
    uint32_t dist[RPW][4];
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        const float el[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) dist[i][e] = top - mag_key(el[e]);
    }
    if (!wave_full<RPW>(len, wave)) {
#pragma unroll
        for (int i = 0; i < RPW; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if ((wave * RPW + i) * kRow + lane * 4 + e >= len) dist[i][e] = 0xffffffffu;
    }

    // ---- threshold: the `need` first of the `in_bin` elements with distances in [lo, lo + 2^bits) are kept, and all below lo
    count_bins<RPW>(dist, 0, kFirstBits, kFirstShift, false, lane, smem);
    __syncthreads();
    uint32_t need = keff, bin, before, in_bin;
    find_bin(smem, lane, need, bin, before, in_bin);
    need -= before;
    uint32_t lo = bin << kFirstShift, bits = kFirstShift;
    auto refine = [&](uint32_t* h, bool crowded) {
        const uint32_t shift = bits > kBinBits ? bits - kBinBits : 0;
        count_bins<RPW>(dist, lo, bits, shift, crowded, lane, h);
        __syncthreads();
        find_bin(h, lane, need, bin, before, in_bin);
        need -= before;
        lo += bin << shift;
        bits = shift;
    };
    // An eighth of a chunk in a 64th of a binade: values that are equal, or nearly so, and go on sharing their bins.
    if (__builtin_expect(bin != kBins && in_bin <= static_cast<uint32_t>(len) / 8, 1)) {
        uint32_t* h = smem;
        while (in_bin != need && bits != 0) refine(h += kBins, false);   // at most three times
    } else {
        const bool far = bin == kBins;
        if (far) {
            uint32_t* h = smem + kBins;
            count_binades<RPW>(dist, lo, top, lane, h);
            __syncthreads();
            const uint4 p = reinterpret_cast<const uint4*>(h)[2 * lane], q = reinterpret_cast<const uint4*>(h)[2 * lane + 1];
            const uint32_t c = ((p.x + p.y) + (p.z + p.w)) + ((q.x + q.y) + (q.z + q.w));
            const uint32_t pre = wave_prefix_incl(c);
            const unsigned long long reached = __ballot(pre >= need);
            if (reached == 0) {   // all of them are kept, and zeros
                need -= __builtin_amdgcn_readlane(static_cast<int>(pre), kWave - 1);
                lo = top;
                bits = 0;
            } else {
                const int L = __builtin_ctzll(reached);
                in_bin = L < kWave - 1 ? __builtin_amdgcn_readlane(static_cast<int>(c), L) : 0;   // the last one's range has the zeros in it
                need -= __builtin_amdgcn_readlane(static_cast<int>(pre - c), L);
                lo += static_cast<uint32_t>(L) << kBinadeShift;
                bits = L < kWave - 1 ? kBinadeShift : 31;
            }
        }
        int next = far ? 3 : 1;
        bool crowded = !far;   // a binade's elements spread over the bins again
        while (in_bin != need && bits != 0) {
            // Behind the binades up to four refinements: the next one's histogram is cleared here, where every wave is past the
            // barrier before which the waves read it last.
            if (far) topk_clear(smem + ((next + 1) & (kHists - 1)) * kBins, kBins);
            refine(smem + (next & (kHists - 1)) * kBins, crowded);
            crowded = in_bin > static_cast<uint32_t>(len) / 8;
            ++next;
        }
    }
    // Either all of the last bin is kept, or it is one magnitude of which the first `need` in index order are kept.
    const bool ties = in_bin != need;
    const uint32_t limit = ties ? lo : lo + (1u << bits);   // kept: dist < limit (and some of the ties)

    // ---- counts of the waves before this one: low half = dist < limit, high half = ties
    uint32_t count = 0;
#pragma unroll
    for (int i = 0; i < RPW; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            count += __builtin_popcountll(__ballot(dist[i][e] < limit));
            if (ties) count += static_cast<uint32_t>(__builtin_popcountll(__ballot(dist[i][e] == limit))) << 16;
        }
    uint32_t pos = 0;   // output slots used by the waves before this one
    if (nwaves > 1) {
        if (lane == 0) s_count[wave] = count;
        __syncthreads();
        const int w = lane & (kMaxWaves - 1);
        pos = __builtin_amdgcn_readfirstlane(static_cast<int>(row16_reduce(w < wave ? s_count[w] : 0u, OpAddU{})));
    }
    uint32_t bound = limit;
    if (ties) {   // those of the ties that are not kept move beyond the bound
        uint32_t tie = pos >> 16;
        pos = (pos & 0xffffu) + (tie < need ? tie : need);
        bound = limit + 1;
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            uint32_t mine = tie;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const unsigned long long m = __ballot(dist[i][e] == limit);
                mine = lanes_below(m, mine);
                tie += __builtin_popcountll(m);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (dist[i][e] == limit) {
                    if (mine >= need) dist[i][e] = 0xffffffffu;
                    ++mine;
                }
            }
        }
    }

    // ---- emit
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        const int off = static_cast<int>(wave * RPW + i) * kRow;
        const int remain = len - off;
        if (remain <= 0) continue;
        uint32_t mine = pos;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const unsigned long long m = __ballot(dist[i][e] < bound);
            mine = lanes_below(m, mine);
            pos += __builtin_popcountll(m);
        }
        const float el[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
        float res[4], dec[4];
        uint32_t left = 0;   // which of the lane's four are kept and still to be stored
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool sel = dist[i][e] < bound;
            const float stored = el[e] + 0.0f;  // -0 is stored as +0
            if (JOINT) {
                left |= sel ? 1u << e : 0u;
            } else if (sel) {
                idx_c[mine] = static_cast<uint16_t>(off + lane * 4 + e);
                val_c[mine] = stored;
                ++mine;
            }
            res[e] = sel ? 0.0f : el[e];
            dec[e] = sel ? stored : 0.0f;
        }
        // A store takes the memory pipeline as long for one lane as for 64, and few lanes keep more than one of their four: all store their
        // first one together, then those that have another.
        if (JOINT) {
            while (__ballot(left != 0)) {
                if (left != 0) {
                    idx_c[mine] = static_cast<uint16_t>(off + lane * 4 + __builtin_ctz(left));
                    val_c[mine] = (left & 1u) ? dec[0] : (left & 2u) ? dec[1] : (left & 4u) ? dec[2] : dec[3];
                    ++mine;
                    left &= left - 1;
                }
            }
        }
        if (residual) store_row(residual + off, lane, remain, f4{res[0], res[1], res[2], res[3]});
        if (out) store_row(out + off, lane, remain, f4{dec[0], dec[1], dec[2], dec[3]});
    }
    for (uint32_t t = keff + threadIdx.x; t < keep; t += blockDim.x) {  // unused slots of a short last chunk
        idx_c[t] = 0xFFFFu;
        val_c[t] = 0.0f;
    }
}

// ------------------------------------------------------------------------------------------ worker side
// Long launches of chunks of 512 to 1536 elements, where the many small workgroups wait for their stores.  One element of the lane at a time -> joint, us:
// C = 1024, keep = 32, 2 M 6.8 -> 7.1, 8 M +-0, 25.7 M 52.8 -> 51.1, 60 M 116.4 -> 113.7, 134 M 259.0 -> 252.1, keep = 128, 134 M 286.3 -> 278.4, keep = 10, 134 M
// 255.4 -> 251.2; C = 1536, keep = 192, 60 M 118.5 -> 114.3; C = 768, 134 M 250.4 -> 244.1.  Longer chunks +0.2 us in short launches, -0.5 .. +0.4 % in long ones.
// C = 256, a single wave of one row, loses: keep = 32, 25 M 56.7 -> 58.8, 60 M 130.6 -> 134.3, keep = 2, 10 M 23.4 -> 24.4.
// Only two rows per wave are built that way: a build with another BAGUA_RPW_TOPK stores one element at a time throughout.
static bool topk_stores_joint(size_t n, size_t chunk, int rpw) { return rpw == 2 && chunk > kRow && chunk <= 1536 && n > (static_cast<size_t>(1) << 23); }

template <int RPW, bool EF, bool JOINT>
__global__ void __launch_bounds__(wg_threads_max(RPW))
k_compress_topk(const float* __restrict__ x, float* __restrict__ residual, size_t n, uint32_t chunk, uint32_t keep,
                uint16_t* __restrict__ idx, float* __restrict__ val, ChunkOrder order)
{
    __shared__ __align__(16) uint32_t smem[kTopkLdsWords];
    const size_t c = order(blockIdx.x);
    const size_t base = c * static_cast<size_t>(chunk);
    const int len = static_cast<int>((n - base < chunk) ? (n - base) : chunk);
    const int wave = wave_index(), lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;
    f4 v[RPW], d[RPW];
    auto load = [&](auto full) {
        constexpr bool FULL = decltype(full)::value;
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int off = static_cast<int>(wave * RPW + i) * kRow;
            const int remain = row_remain<FULL>(len, off);
            v[i] = f4{0.f, 0.f, 0.f, 0.f};
            d[i] = v[i];
            if (remain > 0) {
                v[i] = load_row(x + base + off, lane, remain, 0.0f);
                if (EF) d[i] = load_row(residual + base + off, lane, remain, 0.0f);
            }
        }
    };
    // No tail tests where all rows of the wave are complete: its eight loads are in flight together instead of one row after
    // the other.  With the same in the server and optimizer steps, whole rounds: 4 workers x 25.7 M, C = 2048, 384 -> 355 us;
    // 8 x 25.7 M, C = 4096, 551 -> 543 us; 3 x 100 M, C = 8192, 1057 -> 1029 us.  Asked of the wave and not of the chunk, whose
    // rows need not fill its last wave: 4 x 112 M, C = 1536, 1972 -> 1834 us, C = 768, 3199 -> 3034 us.
    if (wave_full<RPW>(len, wave)) load(std::true_type{});
    else load(std::false_type{});
    topk_clear(smem, kHistWords);   // while the loads are in flight
    if (EF) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            v[i].x = v[i].x + d[i].x;
            v[i].y = v[i].y + d[i].y;
            v[i].z = v[i].z + d[i].z;
            v[i].w = v[i].w + d[i].w;
        }
    }
    topk_encode_chunk<RPW, JOINT>(v, len, keep, wave, lane, nwaves, EF ? residual + base : nullptr, idx + c * keep,
                           val + c * keep, nullptr, smem);
}

// ------------------------------------------------------------------------------------------ server side
// The k sparse chunks are summed into a dense LDS copy of the chunk, one worker after the other
// (ascending order; a worker's indices are unique, so its adds never collide), then averaged,
// the server error state is added and the result is sparsified again.

// dense[index] += value, worker after worker.  E entries per thread and pass over a worker's list; as many workers' passes
// as make eight entries are fetched together, so the chain of k dependent steps pays one memory latency per group.
template <int E>
__device__ __forceinline__ void sum_entries(const PtrTable& idx_in, const PtrTable& val_in, int k, size_t entry0, uint32_t keep,
                                            int len, float* dense)
{
    constexpr int G = 8 / E;
    const uint32_t passes = E < 8 ? 1 : (keep + E * blockDim.x - 1) / (E * blockDim.x);
    for (int j0 = 0; j0 < k; j0 += G) {
        for (uint32_t pass = 0; pass < passes; ++pass) {
            uint32_t p[G][E];
            float a[G][E];
#pragma unroll
            for (int g = 0; g < G; ++g) {
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const uint32_t t = (pass * E + e) * blockDim.x + threadIdx.x;
                    p[g][e] = 0xFFFFu;
                    a[g][e] = 0.0f;
                    if (j0 + g < k && t < keep) {
                        p[g][e] = static_cast<const uint16_t*>(idx_in.p[j0 + g])[entry0 + t];
                        a[g][e] = static_cast<const float*>(val_in.p[j0 + g])[entry0 + t];
                    }
                }
            }
#pragma unroll
            for (int g = 0; g < G; ++g) {
                if (j0 + g >= k) break;
                if (pass == 0) __syncthreads();  // the previous worker's sums (or the clear) are complete
#pragma unroll
                for (int e = 0; e < E; ++e)
                    if (static_cast<int>(p[g][e]) < len) dense[p[g][e]] = dense[p[g][e]] + a[g][e];
            }
        }
    }
    __syncthreads();
}

template <int RPW, bool EF, bool OUT>
__global__ void __launch_bounds__(wg_threads_max(RPW))
k_drr_topk(PtrTable idx_in, PtrTable val_in, int k, float inv_k, uint32_t keep, float* __restrict__ eps, size_t n,
           uint32_t chunk, uint16_t* __restrict__ idx_out, float* __restrict__ val_out, float* __restrict__ out)
{
    extern __shared__ uint32_t smem[];
    float* dense = reinterpret_cast<float*>(smem);
    const size_t c = blockIdx.x;
    const size_t base = c * static_cast<size_t>(chunk);
    const int len = static_cast<int>((n - base < chunk) ? (n - base) : chunk);
    const int wave = wave_index(), lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;

    // The error state of this wave's rows is requested first: it is not needed before the sparse sums are done.
    f4 e[RPW];
    auto load = [&](auto full) {
        constexpr bool FULL = decltype(full)::value;
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int off = static_cast<int>(wave * RPW + i) * kRow;
            const int remain = row_remain<FULL>(len, off);
            e[i] = f4{0.f, 0.f, 0.f, 0.f};
            if (remain > 0) e[i] = load_row(eps + base + off, lane, remain, 0.0f);
        }
    };
    if (EF) {
        if (wave_full<RPW>(len, wave)) load(std::true_type{});
        else load(std::false_type{});
    }
    for (uint32_t t = threadIdx.x; t < chunk / 4; t += blockDim.x) reinterpret_cast<f4*>(dense)[t] = f4{0.f, 0.f, 0.f, 0.f};
    const size_t entry0 = c * keep;
    if (keep <= blockDim.x) sum_entries<1>(idx_in, val_in, k, entry0, keep, len, dense);
    else if (keep <= 2 * blockDim.x) sum_entries<2>(idx_in, val_in, k, entry0, keep, len, dense);
    else if (keep <= 4 * blockDim.x) sum_entries<4>(idx_in, val_in, k, entry0, keep, len, dense);
    else sum_entries<8>(idx_in, val_in, k, entry0, keep, len, dense);
    f4 v[RPW];
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        const int off = static_cast<int>(wave * RPW + i) * kRow;
        const int remain = len - off;
        v[i] = f4{0.f, 0.f, 0.f, 0.f};
        if (remain > 0) {
            const f4 a = *reinterpret_cast<const f4*>(dense + off + lane * 4);
            v[i].x = a.x * inv_k;
            v[i].y = a.y * inv_k;
            v[i].z = a.z * inv_k;
            v[i].w = a.w * inv_k;
            if (EF) {
                v[i].x = v[i].x + e[i].x;
                v[i].y = v[i].y + e[i].y;
                v[i].z = v[i].z + e[i].z;
                v[i].w = v[i].w + e[i].w;
            }
        }
    }
    __syncthreads();  // the dense copy is dead: its LDS is reused by the selection
    topk_clear(smem, kHistWords);
    topk_encode_chunk<RPW>(v, len, keep, wave, lane, nwaves, EF ? eps + base : nullptr, idx_out + c * keep,
                           val_out + c * keep, OUT ? out + base : nullptr, smem);
}

// ------------------------------------------------------------------------------------------ decode
// Dense chunk assembled in LDS, written out with coalesced 128-bit stores.
__global__ void __launch_bounds__(256)
k_decompress_topk(const uint16_t* __restrict__ idx, const float* __restrict__ val, size_t n, uint32_t chunk,
                  uint32_t keep, float* __restrict__ out)
{
    extern __shared__ uint32_t smem[];
    float* dense = reinterpret_cast<float*>(smem);
    const size_t c = blockIdx.x;
    const size_t base = c * static_cast<size_t>(chunk);
    const int len = static_cast<int>((n - base < chunk) ? (n - base) : chunk);
    for (uint32_t t = threadIdx.x; t < chunk; t += blockDim.x) dense[t] = 0.0f;
    __syncthreads();
    for (uint32_t t = threadIdx.x; t < keep; t += blockDim.x) {
        const uint32_t p = idx[c * keep + t];
        if (static_cast<int>(p) < len) dense[p] = val[c * keep + t];
    }
    __syncthreads();
    const int wave = wave_index(), lane = threadIdx.x & 63;
    for (int off = static_cast<int>(wave) * kRow; off < len; off += 4 * kRow)
        store_row(out + base + off, lane, len - off, *reinterpret_cast<const f4*>(dense + off + lane * 4));
}

}  // namespace bagua

using namespace bagua;

static bool topk_args_ok(size_t n, size_t chunk, size_t keep) { return n != 0 && chunk_ok(chunk) && keep >= 1 && keep <= chunk; }

extern "C" int bagua_compress_topk_ef(const float* x, float* residual, size_t n, size_t chunk, size_t keep,
                                      uint16_t* idx, float* val, void* stream)
{
    if (!x || !idx || !val || !topk_args_ok(n, chunk, keep)) return BAGUA_ERR_INVALID_ARG;
    {
        const size_t slots = num_chunks(n, chunk) * keep;
        RangeCheck rc;
        rc.reads(x, n * sizeof(float));
        rc.writes(residual, n * sizeof(float));
        rc.writes(idx, slots * sizeof(uint16_t));
        rc.writes(val, slots * sizeof(float));
        if (!rc.disjoint()) return BAGUA_ERR_INVALID_ARG;
    }
    if (num_chunks(n, chunk) > kMaxGrid) return BAGUA_ERR_UNSUPPORTED;
    if (!aligned16(x) || !aligned16(residual) || !aligned2(idx) || !aligned4(val)) return BAGUA_ERR_ALIGNMENT;
    const int rows = static_cast<int>(chunk / kRow);
    const int rpw = pick_rpw_topk(rows, num_chunks(n, chunk));
    dim3 grid(static_cast<unsigned>(num_chunks(n, chunk))), block(64 * ((rows + rpw - 1) / rpw));
    const uint32_t ch = static_cast<uint32_t>(chunk), kp = static_cast<uint32_t>(keep);
    hipStream_t s = static_cast<hipStream_t>(stream);
#define BAGUA_TOPK(RPWv, EFv, JOINTv)                                                                                \
    launch_kernel((k_compress_topk<RPWv, EFv, JOINTv>), grid, block, 0, s, x, residual, n, ch, kp, idx, val, chunk_order(grid.x, chunk))
    if (topk_stores_joint(n, chunk, rpw)) {
        if (residual) BAGUA_TOPK(2, true, true);
        else BAGUA_TOPK(2, false, true);
    } else if (residual) {
        BAGUA_DISPATCH_RPW(rpw, BAGUA_TOPK(RPW, true, false))
    } else {
        BAGUA_DISPATCH_RPW(rpw, BAGUA_TOPK(RPW, false, false))
    }
#undef BAGUA_TOPK
    return launch_status();
}

extern "C" int bagua_decompress_reduce_recompress_topk(const uint16_t* const* idx_in, const float* const* val_in, int k,
                                                       size_t keep, float* server_residual, size_t n, size_t chunk,
                                                       uint16_t* idx_out, float* val_out, float* out_fp32, void* stream)
{
    if (!idx_in || !val_in || k < 1 || k > BAGUA_MAX_WORKERS || !idx_out || !val_out || !topk_args_ok(n, chunk, keep))
        return BAGUA_ERR_INVALID_ARG;
    {
        const size_t slots = num_chunks(n, chunk) * keep;
        RangeCheck rc;
        for (int j = 0; j < k; ++j) {
            if (!idx_in[j] || !val_in[j]) return BAGUA_ERR_INVALID_ARG;
            rc.reads(idx_in[j], slots * sizeof(uint16_t));
            rc.reads(val_in[j], slots * sizeof(float));
        }
        rc.writes(server_residual, n * sizeof(float));
        rc.writes(idx_out, slots * sizeof(uint16_t));
        rc.writes(val_out, slots * sizeof(float));
        rc.writes(out_fp32, n * sizeof(float));
        if (!rc.disjoint()) return BAGUA_ERR_INVALID_ARG;
    }
    if (num_chunks(n, chunk) > kMaxGrid) return BAGUA_ERR_UNSUPPORTED;
    for (int j = 0; j < k; ++j)
        if (!aligned2(idx_in[j]) || !aligned4(val_in[j])) return BAGUA_ERR_ALIGNMENT;
    if (!aligned16(server_residual) || !aligned2(idx_out) || !aligned4(val_out) || !aligned16(out_fp32))
        return BAGUA_ERR_ALIGNMENT;
    PtrTable it{}, vt{};
    for (int j = 0; j < k; ++j) {
        it.p[j] = idx_in[j];
        vt.p[j] = val_in[j];
    }
    const int rows = static_cast<int>(chunk / kRow);
    const int rpw = pick_rpw(rows, BAGUA_RPW_DRR_TOPK);
    dim3 grid(static_cast<unsigned>(num_chunks(n, chunk))), block(64 * ((rows + rpw - 1) / rpw));
    size_t lds = chunk * sizeof(float);
    if (lds < kTopkLdsWords * sizeof(uint32_t)) lds = kTopkLdsWords * sizeof(uint32_t);
    const float inv_k = 1.0f / static_cast<float>(k);
    const uint32_t ch = static_cast<uint32_t>(chunk), kp = static_cast<uint32_t>(keep);
    hipStream_t s = static_cast<hipStream_t>(stream);
#define BAGUA_DRR(EFv, OUTv)                                                                                      \
    BAGUA_DISPATCH_RPW(rpw, launch_kernel((k_drr_topk<RPW, EFv, OUTv>), grid, block, lds, s, it, vt, k, inv_k, \
                                               kp, server_residual, n, ch, idx_out, val_out, out_fp32))
    if (server_residual && out_fp32) { BAGUA_DRR(true, true) }
    else if (server_residual) { BAGUA_DRR(true, false) }
    else if (out_fp32) { BAGUA_DRR(false, true) }
    else { BAGUA_DRR(false, false) }
#undef BAGUA_DRR
    return launch_status();
}

extern "C" int bagua_decompress_topk(const uint16_t* idx, const float* val, size_t n, size_t chunk, size_t keep,
                                     float* out, void* stream)
{
    if (!idx || !val || !out || !topk_args_ok(n, chunk, keep)) return BAGUA_ERR_INVALID_ARG;
    {
        const size_t slots = num_chunks(n, chunk) * keep;
        RangeCheck rc;
        rc.reads(idx, slots * sizeof(uint16_t));
        rc.reads(val, slots * sizeof(float));
        rc.writes(out, n * sizeof(float));
        if (!rc.disjoint()) return BAGUA_ERR_INVALID_ARG;
    }
    if (num_chunks(n, chunk) > kMaxGrid) return BAGUA_ERR_UNSUPPORTED;
    if (!aligned2(idx) || !aligned4(val) || !aligned16(out)) return BAGUA_ERR_ALIGNMENT;
    launch_kernel(k_decompress_topk, dim3(static_cast<unsigned>(num_chunks(n, chunk))), dim3(256),
                       chunk * sizeof(float), static_cast<hipStream_t>(stream), idx, val, n, static_cast<uint32_t>(chunk),
                       static_cast<uint32_t>(keep), out);
    return launch_status();
}
