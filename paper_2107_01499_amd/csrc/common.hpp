// Device-side building blocks shared by the gfx950 kernels of this library.
//
// Data layout used by every chunked kernel: a chunk of C elements (C a multiple of 256) is cut
// into "rows" of 256 consecutive elements.  One 64-lane wavefront reads or writes a row with a
// single 128-bit access per lane (lane l owns elements 4l..4l+3 of the row), which is the widest
// coalesced access the memory pipeline offers.  A wavefront keeps ROWS_PER_WAVE rows in registers,
// so a chunk is read from HBM exactly once: statistics and quantisation both work on registers.
// A workgroup is the ceil(rows / ROWS_PER_WAVE) wavefronts of one chunk; their partial statistics
// meet in LDS behind a single barrier.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>
#include <stddef.h>
#include <stdint.h>

#include "bagua_hip.h"

namespace bagua {

// 128-bit lane payload as a native clang vector (the nontemporal builtins need one).
typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint8_t b4 __attribute__((ext_vector_type(4)));

// Streaming accesses: every bucket byte is touched once per kernel, so loads and stores carry the
// nontemporal hint and do not displace each other in L2 / Infinity Cache.
#ifndef BAGUA_NT
#define BAGUA_NT 1
#endif
template <typename T>
__device__ __forceinline__ T ld_stream(const T* p)
{
#if BAGUA_NT
    return __builtin_nontemporal_load(p);
#else
    return *p;
#endif
}
template <typename T>
__device__ __forceinline__ void st_stream(T* p, T v)
{
#if BAGUA_NT
    __builtin_nontemporal_store(v, p);
#else
    *p = v;
#endif
}

// Except for what the next call of the round reads again, as long as the 256 MB Infinity Cache makes that faster; such data
// is stored, or loaded the first time, without the hint.  The lines below are measured crossovers of whole rounds; they are
// not the cache's capacity, a part of which helps too.
//
// The codes of one worker's call: the server step (or the network) reads them next, and the next round overwrites them.
// How many workers follow is not known here, so only the first 2^25 codes of a call are kept: whole MinMax rounds, C = 4096,
// all streamed -> this -> all kept: 2 workers x 100 M 846 -> 825 -> 806 us, 8 x 50 M 1099 -> 1058 -> 1064 us, 8 x 134 M 2922 ->
// 2873 -> 2961 us, 16 x 100 M 3949 -> 3937 -> 4034 us, 16 x 134 M 5290 -> 5290 -> 5442 us.  Above 2^27 elements it gains
// nothing: 2 x 335 M 2906 -> 2936 us.  The value: how many chunks of the launch, from the first on.
inline uint32_t keep_chunks(size_t n, size_t chunk)
{
    return n <= (static_cast<size_t>(1) << 27) ? static_cast<uint32_t>((static_cast<size_t>(1) << 25) / chunk) : 0;
}

// The server step's codes, which the decode reads next: 2 workers x 100 M 846 -> 833 us for the round, intra-node average and
// round of 2 x 4 x 134 M 1474 -> 1421 us, 16 x 134 M +-0.
inline int keep_server_codes(size_t n) { return n <= (static_cast<size_t>(1) << 27) ? 1 : 0; }

// The codes of a whole ring or gossip round, `elements` of all peers together.  Other work runs between two rounds, so the
// line is the one of rounds on buffers that the caches do not hold (three sets in turn).  With the hint -> without: ring of
// 8, C = 4096, by the codes of the round: 16 MB 47.9 -> 46.9 us, 48 MB 142 -> 135 us, 88 MB 269 -> 255 us, 96 MB 287 -> 284 us,
// 128 MB 388 -> 403 us, 192 MB 601 -> 619 us; rings of 2, 4 and 16 peers and gossip of 2 to 8 cross at 90 to 105 MB too.
// (The same round over and over on one set of buffers gains up to 205 MB.)
inline int keep_codes_of_round(size_t elements)
{
    return elements <= (static_cast<size_t>(11) << 23) ? 1 : 0;
}

// A flattened bucket of n floats, which the compression reads next: 8 workers x 25.6 M elements in 5 buckets 793 -> 766 us,
// 4 x 60 M 914 -> 869 us, 4 x 130 M 2153 -> 2115 us for the whole round; above the line 8 x 160 M 4768 -> 4921 us, 4 x 200 M
// 3227 -> 3307 us, 2 x 160 M +-0.  (The momentum that every worker's sign compression reads: see mom_keep; the replica that
// encode and mix both read: see k_lp_encode.)
inline bool keep_bucket(size_t n) { return n <= (static_cast<size_t>(1) << 27); }

// Preferred rows (of 256 elements) per wave for each chunked kernel (compile-time tuning knobs).
// Measured on MI355X: two rows per wave (512 elements, 8 waves for a 4096-element chunk) stream
// fastest in the worker-side kernels, the fused ring kernel and the sign codec's server kernel; the MinMax
// and the top-K server kernels prefer four.  Larger values are used only when a chunk would need more than 16 waves.
#ifndef BAGUA_RPW_COMPRESS
#define BAGUA_RPW_COMPRESS 2
#endif
#ifndef BAGUA_RPW_DRR
#define BAGUA_RPW_DRR 4
#endif
#ifndef BAGUA_RPW_SIGN
#define BAGUA_RPW_SIGN 2
#endif
#ifndef BAGUA_RPW_DRR_SIGN
#define BAGUA_RPW_DRR_SIGN 2
#endif
#ifndef BAGUA_RPW_TOPK
#define BAGUA_RPW_TOPK 2
#endif
#ifndef BAGUA_RPW_DRR_TOPK
#define BAGUA_RPW_DRR_TOPK 4
#endif
#ifndef BAGUA_RPW_LP
#define BAGUA_RPW_LP 2
#endif
// The rows per wave that every BAGUA_DISPATCH_RPW* below has an instance for; a launch with any other value would run the
// instance of four and leave rows out.
constexpr bool rpw_built(int rpw) { return rpw == 2 || rpw == 4; }
static_assert(rpw_built(BAGUA_RPW_COMPRESS) && rpw_built(BAGUA_RPW_DRR) && rpw_built(BAGUA_RPW_SIGN) && rpw_built(BAGUA_RPW_DRR_SIGN) &&
              rpw_built(BAGUA_RPW_TOPK) && rpw_built(BAGUA_RPW_DRR_TOPK) && rpw_built(BAGUA_RPW_LP), "no kernel instance for this many rows per wave");
// Peers whose statistics share one barrier in the fused ring kernel.
#ifndef BAGUA_LP_GROUP
#define BAGUA_LP_GROUP 1
#endif
// Workers whose sign words are fetched together in the sign codec's server-side kernel.
#ifndef BAGUA_DRR_SIGN_NJ
#define BAGUA_DRR_SIGN_NJ 8
#endif

constexpr int kWave = 64;
constexpr int kRow = 256;      // elements per wave-wide 128-bit access
constexpr int kMaxWaves = 16;  // waves per workgroup (1024 threads)
constexpr int kCus = 256, kWavesPerCu = 32;   // and the most waves that one holds
// Rows (one wavefront each) per workgroup of the kernels that stream row by row without a chunk statistic (decode,
// optimizer steps, peer averaging, the probes).  Measured: two waves per workgroup are 0.5-3 % faster than four and than one.
#ifndef BAGUA_ROW_WAVES
#define BAGUA_ROW_WAVES 2
#endif
constexpr int kRowWaves = BAGUA_ROW_WAVES;

// Upper bound on the workgroup size of a chunked kernel that keeps RPW rows per wave: chunks have at most
// 64 rows, and pick_rpw never asks for more than kMaxWaves waves.
constexpr int wg_threads_max(int rpw)
{
    return kWave * (((64 + rpw - 1) / rpw) < kMaxWaves ? ((64 + rpw - 1) / rpw) : kMaxWaves);
}
static_assert(wg_threads_max(1) <= 1024 && wg_threads_max(2) <= 1024 && 4 * kMaxWaves >= 64, "four rows per wave hold any chunk");

// A kernel that moves many streams at once is fastest with no more waves on a CU than keep the memory busy: what is in
// flight beyond that only spreads the accesses over more DRAM pages at a time (most of all where the streams lie close
// together in HBM).  Such a launch asks for LDS that it does not use, so that at most `groups` of its workgroups fit a
// CU: the largest multiple of the allocation's granule that leaves room for them.
constexpr size_t kLdsPerCu = 160 * 1024, kLdsGranule = 1280;
// `own`: what the kernel uses of it anyway, if the launch's figure comes on top of that.
constexpr size_t lds_for_residency(int groups, size_t own = 0)
{
    return (kLdsPerCu / kLdsGranule / static_cast<size_t>(groups) - (own + kLdsGranule - 1) / kLdsGranule) * kLdsGranule;
}
static_assert(lds_for_residency(4) <= 64 * 1024, "the most that a launch gets without asking the runtime for more");
// The least with which no more than two workgroups fit.
constexpr size_t kLdsForTwo = (kLdsPerCu / kLdsGranule / 3 + 1) * kLdsGranule;

// Gossip pairs of chunks of 2561 to 4096 elements: two workgroups of six to eight waves on a CU instead of as many as fit, `elements` of
// all pairs of the launch.  Unbounded -> two, buffers that lie far apart in HBM | back to back: one pair x 100 M 525.8 -> 525.1 | 541.5 ->
// 539.5 us, x 45 M 234.3 -> 233.3 | 240.0 -> 239.1, two x 25 M 278.3 -> 274.2 | 270.4 -> 269.6, x 33 M, C = 3072, 364.0 -> 357.9 | 359.2 -> 354.3,
// four x 17 M 370.6 -> 368.3 | 368.9 -> 367.0; below the line one pair x 33 M 171.3 -> 171.6 | 170.8 -> 172.3, x 25 M 132.7 -> 134.3 | 135.9
// -> 135.7, x 17 M 89.6 -> 93.2 | 90.9 -> 93.3, two x 17 M 185.2 -> 185.3 | 176.8 -> 178.3.  Shorter chunks lose 1-3 %, longer ones do not
// care.  Workers that sit out move half as many streams and lose 1-2 %: 25.6 M 68.8 -> 69.9 | 68.9 -> 70.1.
inline size_t gossip_pairs_lds(size_t chunk, size_t elements)
{
    return chunk > 2560 && chunk <= 4096 && elements >= (static_cast<size_t>(5) << 23) ? kLdsForTwo : 0;
}

// The full-precision ring of up to 16 peers: one wave per row of all peers and workgroup, and in launches that read and write 2^27 bytes
// or more no more waves on a CU than keep the memory busy.  In us, eight rows per workgroup and as many as fit -> this, sets of buffers in
// turn that lie far apart in HBM, as in a training process | back to back:
//   2 peers, 100 MB 18.0 -> 17.1 | 18.6 -> 17.5, 420 MB 66.0 -> 64.0 | 69.6 -> 64.3;   3 peers, 140 MB 24.3 -> 23.4 | 25.6 -> 24.3, 420 MB 66.5 ->
//   65.5 | 70.7 -> 65.8;   5 peers, 300 MB 49.5 -> 47.6 | 53.6 -> 49.9;   8 peers, 140 MB 25.9 -> 24.6 | 28.2 -> 26.6, 300 MB 49.3 -> 49.0 | 56.8 -> 54.5;
//   12 peers, 100 MB 17.9 -> 17.7 | 18.4 -> 18.4, 200 MB 33.8 -> 34.6 | 38.0 -> 36.3, 420 MB 70.0 -> 68.3 | 85.5 -> 73.8;   14 peers, 420 MB 72.0 -> 68.6
//   | 88.5 -> 73.9;   8 x 110 M 1087 .. 1125 -> 1080 .. 1105 | 1110 .. 1240 -> 1089 .. 1132;   16 x 55 M 1116 .. 1139 -> 1108 .. 1126 | 1127 -> 1126.
// The bench's own spread placement of 8 x 110 M, 1.103 .. 1.110 -> 1.119 ms, is the one large launch seen to lose more than 1 %.
// The waves are the least with which buffers far apart lose nothing in long launches; back to back one or two fewer are the
// fastest (8 x 110 M, far apart, 4, 5, 6, 7, 8, 10 waves: 1156, 1104, 1089, 1093, 1105, 1122 us; 8 peers, 300 MB, 5 -> 7 waves: 49.7 -> 49.0 | 52.7 ->
// 54.5).  One replica is a copy, which wants all the waves there are: 1 x 200 M 240 -> 269 us with 24 of them.
inline bool ring_fp_long(int peers, size_t n) { return 2 * static_cast<size_t>(peers) * n * sizeof(float) >= (static_cast<size_t>(1) << 27); }
constexpr int ring_fp_waves(int peers)
{
    return peers <= 2 ? 16 : peers == 3 ? 12 : peers <= 5 ? 9 : peers == 6 ? 8 : peers <= 8 ? 7 : peers <= 11 ? 6 : peers <= 14 ? 5 : 4;
}
constexpr int ring_fp_rows(int peers) { return peers > 16 ? kRowWaves : 1; }

// Which chunk a workgroup takes.  Workgroup b runs on die (XCD) b % 8; in the order of the workgroups neighbouring chunks lie on
// different dies, and a die's share of a stream is every eighth chunk.  Here a die takes 2^lg chunks in a row and the eight of
// them 8 * 2^lg together; what is left at the end keeps the plain order.  What it does to the memory system was measured, not
// derived: the dies then touch fewer, longer stretches of every stream.  Lengths from 2^0 to 2^8, 50 M elements per worker, the
// gain of a whole round in %, worker-side kernels of both codecs and the LP ring:
//   chunks up to 1024: 2^7 +0.6 .. +2.7, 2^5 -0.8 .. +2.2;
//   1536 to 4096: 2^5 +0.5 .. +3.8 except 4096 elements gathered or reduced, -0.2 .. +1.0; 2^2 down to -2;
//   longer: 2^2 +1.0 .. +5.6, 2^5 -1.4 .. +5.1, 2^7 negative.
// Top-K: 0 .. +3 (4 x 60 M, C = 1536, 831 -> 807 us); gossip pairs of chunks above 4096: -0.6 .. +5.7 (8 x 60 M, C = 8192, 1530 -> 1448).
// From 2048 chunks on; below, +1 .. -6 without a pattern.  The server steps, the decodes and the full-precision kernels gained
// nothing at any length (the ring of eight -1 .. -8 %).  From 2^28 elements on the longer chunks gain as much (batched MinMax, plain -> this:
// 600 M, C = 2048, 1215 -> 1179 us, 700 M, C = 4096, 1443 -> 1405, 1.5 G, C = 16384, 3325 -> 3152), and short ones lose: see order_pays_*.
struct ChunkOrder {
    uint32_t lg, end;   // chunks from `end` on: plain order
    __device__ __forceinline__ uint32_t operator()(uint32_t b) const
    {
        const uint32_t r = b & ((8u << lg) - 1u);
        return b < end ? b - r + ((r & 7u) << lg) + (r >> 3) : b;
    }
};
inline ChunkOrder chunk_order(size_t chunks, size_t chunk, bool pays = true)
{
    const uint32_t lg = !pays || chunks < 2048 ? 0 : chunk <= 1024 ? 7 : chunk <= 4096 ? 5 : 2;
    return ChunkOrder{lg, lg == 0 ? 0 : static_cast<uint32_t>(chunks) & ~((8u << lg) - 1u)};
}
// Where short chunks keep the plain order, plain -> runs of 128 in us.  Contiguous input, chunks of 1024: sign codec, 268 M 503 -> 496, 350 M
// 642 -> 647, 500 M 941 -> 953, 700 M 1284 -> 1292; MinMax, 268 M 554 -> 549, 350 M 700 -> 702, 500 M 997 -> 1007, 700 M 1381 -> 1392.  (C = 768
// +-0.4 % above the line; C = 512 from 2^28 on between -1.1 and +2 % from one set of buffers to the next, without a pattern.)
inline bool order_pays(size_t n, size_t chunk) { return chunk != 1024 || n <= (static_cast<size_t>(1) << 28); }
// Intra-node average of three and more, chunks up to 512: MinMax, whole rounds of two nodes of four, C = 512, 35 M 368 -> 367, 50 M 528 ->
// 534, 100 M 1062 -> 1105, C = 256, 25 M 290 -> 291, 35 M 397 -> 403; of eight, C = 256, 50 M 477 -> 491, sign codec 100 M 846 -> 867.  Two in a
// node gain (50 M 391 -> 389, 100 M 792 -> 793), longer chunks do (C = 768, 100 M, 1074 -> 1054).
inline bool order_pays_average(size_t n, size_t chunk, int k_local) { return chunk > 512 || k_local <= 2 || n <= (static_cast<size_t>(1) << 25); }
// Gather and MinMax, chunks up to 512: whole rounds, C = 512, 4 x 50 M 557 -> 554, 4 x 134 M 1492 -> 1515, 2 x 300 M 2070 -> 2098; C = 256 +-0.
// The sign codec gains (C = 512, 2 x 450 M 2637 -> 2623).
inline bool order_pays_gather_minmax(size_t n, size_t chunk) { return chunk > 512 || n <= (static_cast<size_t>(1) << 26); }

// Kernels that take row after row (`groups` workgroups of kRowWaves) behind one that takes chunk after chunk in plain order: the rows of a
// chunk on the die of its workgroup, in whose L2 they may still lie.  Chunks whose workgroups are not a power of two in number keep
// the plain order.  Measured in plain order -> this:
//   the mix of an LP ring share, which reads the x and the public copy that the encode has just read and written: up to 2^25 elements; encode
//   + mix, three sets of buffers in turn, 1.5 M 15.2 -> 13.7 us, 4 M, C = 8192, 32.2 -> 27.0, C = 1024, 31.0 -> 27.4, 6.5 M, C = 4096, 46.6 ->
//   44.1, 13 M 85.3 -> 83.0, 30 M 186.7 -> 183.4, C = 2048 187.8 -> 187.8; 45 M 283 -> 286;
//   the SGD and Adam steps, which read the server step's codes and the momentum: up to 2^24 elements; whole rounds, sign codec, 4 workers x 4 M,
//   C = 4096, 67.8 -> 65.9 us, 8 x 6.5 M, C = 2048, 158.0 -> 157.4, 2 x 8 M, C = 1024, +-0; MinMax, 2 x 4 M, C = 2048, 44.7 -> 44.3, 2 x 8 M, C =
//   8192, 81.0 -> 79.9; 16 M +-0, 40 M without the limit -0.4 .. -0.7 %.
inline ChunkOrder row_order(unsigned groups, uint32_t rows_per_chunk)
{
    const uint32_t per = rows_per_chunk / kRowWaves;
    if (per == 0 || per * kRowWaves != rows_per_chunk || (per & (per - 1)) != 0) return ChunkOrder{0, 0};
    const uint32_t lg = static_cast<uint32_t>(__builtin_ctz(per));
    return ChunkOrder{lg, groups & ~((8u << lg) - 1u)};
}

struct PtrTable {
    const void* p[BAGUA_MAX_WORKERS];
};
struct MutPtrTable {
    void* p[BAGUA_MAX_WORKERS];
};

// Pacing of a wave's streaming loads in the worker-side kernels.  In a very large launch the memory system is
// saturated and latency is mostly queueing: a wave that waits for each row before it requests the next keeps the
// queues shorter, which the DRAM scheduler rewards (+3 % for the batched sign compression over 229 buckets of
// 1.5 G elements, +0.5-1 % for the unbatched launches in an A/B on the same buffers); in a small launch the longer
// chain of dependent requests costs 3 %.  The launchers pace from 2^28 elements per launch on.
__device__ __forceinline__ void pace_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
inline int pace_for(size_t elements_per_launch) { return elements_per_launch >= (static_cast<size_t>(1) << 28) ? 1 : 0; }

// Index of this wavefront in its workgroup, as a scalar.  The compiler cannot tell that threadIdx.x >> 6 is the same
// in all 64 lanes and would carry every row offset and tail test derived from it through 64-bit vector arithmetic
// and exec-mask branches; read from the first lane it lives in scalar registers.
__device__ __forceinline__ int wave_index()
{
    return __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
}

// Worker-side launches short enough that a wave's latency shows: with the tail tests folded away (row_remain<true>) all
// loads of a wave are in flight together; with them the compiler waits for one row before it requests the next, which
// in a long launch is the better pattern (see pace_loads).  Measured with the tests kept and folded away: a momentum +
// sign compression round of 8 workers x 6.5 M elements 197 -> 183 us; 4 workers, MinMax: 6.5 M 106 -> 103 us, 25.6 M
// 347 -> 343 us, 50 M 672 -> 679 us, 100 M 1306 -> 1322 us, sign codec 300 M 4138 -> 4337 us.  A batched launch, whose
// waves first look up their bucket, gains up to twice that size (60 M in 9 buckets 697 -> 682 us, sign 604 -> 590 us;
// 120 M +-1 %).
inline bool short_launch(size_t elements_per_launch, bool batched = false)
{
    return elements_per_launch < (static_cast<size_t>(1) << (batched ? 26 : 25));
}

// A batched worker-side launch of 2^26 to 2^29 elements with chunks of 1536 or 2048 elements (three or four waves), to 2^28 with chunks of
// 1024 (two): tail tests folded away, and 16 waves on a CU at a time.  Each alone loses (without the bound up to -7 %, bounded to 24
// waves or with the tests -1 .. -30 %); tests and all waves -> this, whole rounds in buckets of 6.5 M, C = 1024 | 1536 | 2048:
//   sign codec, 4 workers x 134 M 1304 -> 1272 | 1290 -> 1239 | 1317 -> 1273 us, 4 x 200 M 1905 -> 1862 | 1947 -> 1868 | 1973 -> 1912, 2 x 268 M
//   1490 -> 1467 | 1555 -> 1490 | 1618 -> 1590, 4 x 374 M, 1536 | 2048, 3610 -> 3551 | 3581 -> 3533, 2 x 500 M 2841 -> 2829 | 2908 -> 2920;
//   MinMax, 4 x 134 M 1474 -> 1429 | 1494 -> 1444 | 1456 -> 1391, 2 x 268 M 1772 -> 1746 | 1873 -> 1763 | 1796 -> 1751, 4 x 374 M, 1536 | 2048,
//   4195 -> 4116 | 3980 -> 3992, 2 x 500 M 3333 -> 3316 | 3226 -> 3258.
// Above 2^28 chunks of 1024 keep the tests and the plain order: sign codec, that -> folded in runs of 128, 4 x 300 M 2818 -> 2839, 4 x 450 M
// 4267 -> 4346, 2 x 500 M 2875 -> 2922; MinMax 3269 -> 3292, 4964 -> 4998, 3335 -> 3366 (4 x 374 M +0.6, -0.8 %).  With 12 waves MinMax is up to
// 1.3 % faster at C = 1536 from 300 M on and up to 7 % slower at 70 M; at 1024 and 2048 elements 16 are as fast or faster.  Longer
// chunks lose 1-14 %, 768 elements never fill the last wave.  Unbatched launches of 1536 and 2048 elements run one row per wave
// and gained nothing; of the others MinMax would gain 2.0 .. 4.5 % at C = 512 and about 1 % at C = 1024, the sign codec nothing.  Beyond
// 2^29, in time: 8 x 700 M, C = 2048, sign codec -0.5 %, MinMax -1.1 .. +0.9 %, 8 x 1.5 G +-0.4 %.  The value: workgroups on a CU, or 0.
inline int batched_groups(size_t elements, size_t chunk, unsigned threads)
{
    const bool pays = chunk >= 1024 && chunk <= 2048 && chunk % (2 * kRow) == 0 && elements >= (static_cast<size_t>(1) << 26) &&
                      elements <= (static_cast<size_t>(1) << (chunk == 1024 ? 28 : 29));
    return pays ? 16 / static_cast<int>(threads / kWave) : 0;
}

// The momentum compression above which eight waves of one row stream the momentum (sign.hip: mom_fold).
inline bool mom_streams(size_t n, int rows_per_wave, unsigned waves)
{
    return rows_per_wave == 1 && waves == 8 && n > (static_cast<size_t>(7) << 24);
}

// f(0), ..., f(N - 1) written out.  A loop over the rows of a wave would do, but where N = 1 the compiler moves a store
// out of the one-trip loop before it unrolls it, and the store loses its nontemporal hint (-12 % at 100 M elements).
template <int N, typename F>
__device__ __forceinline__ void unrolled(const F& f)
{
    if constexpr (N > 0) {
        unrolled<N - 1>(f);
        f(N - 1);
    }
}

// ---------------------------------------------------------------- wave-level reductions
// Exchanges between lanes on the vector ALU (data-parallel primitives).  A chunk's statistic stands between its loads and its
// stores, so what it takes is time in which the workgroup moves nothing: through the LDS crossbar (ds_bpermute) a step of the
// butterfly is a round trip of some 100 cycles, here it is one instruction.  Sign codec, whole rounds, crossbar -> here: 8
// workers x 6.5 M 162.0 -> 158.4 us, 2 x 4 x 25.6 M 262.9 -> 261.0 us; MinMax within 0.5 % (its server step has no slack to give).
constexpr int kXor1 = 0xB1, kXor2 = 0x4E;              // quad_perm [1,0,3,2] and [2,3,0,1]: lane l reads l xor 1, l xor 2
constexpr int kHalfMirror = 0x141, kMirror = 0x140;    // 7 - l in each half row, 15 - l in each row of 16 lanes
constexpr int kShr1 = 0x111, kShr2 = 0x112, kShr4 = 0x114, kShr8 = 0x118;   // lane l reads l - 1, ... of its row, or 0
constexpr int kBcast15 = 0x142, kBcast31 = 0x143;      // lane 15 of the row before; lane 31 into rows 2 and 3
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v)
{
    return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ float dpp(float v)
{
    return __uint_as_float(dpp<CTRL>(__float_as_uint(v)));
}
// op over the lane's row of 16, in every lane of the row: with xor 1, 2 the four lanes of a quad hold the same value, so
// the half mirror reads what lane l xor 4 holds, and the mirror then what lane l xor 8 holds.
template <typename T, typename F>
__device__ __forceinline__ T row16_reduce(T v, const F& op)
{
    v = op(v, dpp<kXor1>(v));
    v = op(v, dpp<kXor2>(v));
    v = op(v, dpp<kHalfMirror>(v));
    return op(v, dpp<kMirror>(v));
}
// op over the wave: the butterfly of xor 1, 2, 4, 8, 16, 32, for a commutative op bit for bit.  Rows 1 and 3 add their
// neighbour, row 3 then rows 0 and 1 together; lane 63 has the result (the lanes that no row reaches read 0 and are not used).
template <typename T, typename F>
__device__ __forceinline__ T wave_reduce(T v, const F& op)
{
    v = row16_reduce(v, op);
    v = op(v, dpp<kBcast15>(v));
    v = op(v, dpp<kBcast31>(v));
    return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
struct OpMinF { __device__ __forceinline__ float operator()(float a, float b) const { return fminf(a, b); } };
struct OpMaxF { __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); } };
struct OpAddF { __device__ __forceinline__ float operator()(float a, float b) const { return a + b; } };

// ---------------------------------------------------------------- row accessors with ragged tails
// Valid elements of a chunk from element `off` on.  FULL: every row of every wave of the workgroup is complete, and the
// constant lets all tail tests fold away.
template <bool FULL>
__device__ __forceinline__ int row_remain(int len, int off)
{
    return FULL ? kRow : len - off;
}
template <int RPW>
__device__ __forceinline__ bool chunk_full(int len, int nwaves)
{
    return len == RPW * kRow * nwaves;
}
// The same for one wave's rows, where no barrier stands in between.
template <int RPW>
__device__ __forceinline__ bool wave_full(int len, int wave)
{
    return len >= (wave + 1) * RPW * kRow;
}
// `remain` = number of valid elements counted from the start of the row (wave-uniform, may be <= 0
// for an absent row or >= 256 for a full one).  Absent elements read as `fill`.
__device__ __forceinline__ f4 load_row(const float* __restrict__ row, int lane, int remain, float fill)
{
    f4 r;
    if (remain >= kRow) {
        r = ld_stream(reinterpret_cast<const f4*>(row) + lane);
    } else {
        const int e = lane * 4;
        r.x = (e + 0 < remain) ? row[e + 0] : fill;
        r.y = (e + 1 < remain) ? row[e + 1] : fill;
        r.z = (e + 2 < remain) ? row[e + 2] : fill;
        r.w = (e + 3 < remain) ? row[e + 3] : fill;
    }
    return r;
}
// A complete row that is read again soon: without the streaming hint (see keep_chunks).
__device__ __forceinline__ f4 load_row_keep(const float* __restrict__ row, int lane, int remain, float fill)
{
    if (remain >= kRow) return reinterpret_cast<const f4*>(row)[lane];
    return load_row(row, lane, remain, fill);
}
__device__ __forceinline__ void store_row(float* __restrict__ row, int lane, int remain, f4 v)
{
    if (remain >= kRow) {
        st_stream(reinterpret_cast<f4*>(row) + lane, v);
    } else {
        const int e = lane * 4;
        if (e + 0 < remain) row[e + 0] = v.x;
        if (e + 1 < remain) row[e + 1] = v.y;
        if (e + 2 < remain) row[e + 2] = v.z;
        if (e + 3 < remain) row[e + 3] = v.w;
    }
}
// Four u8 codes per lane, little-endian in one dword.
__device__ __forceinline__ uint32_t load_codes_row(const uint8_t* __restrict__ row, int lane, int remain)
{
    if (remain >= kRow) return ld_stream(reinterpret_cast<const uint32_t*>(row) + lane);
    uint32_t w = 0;
    const int e = lane * 4;
#pragma unroll
    for (int t = 0; t < 4; ++t)
        if (e + t < remain) w |= static_cast<uint32_t>(row[e + t]) << (8 * t);
    return w;
}
// keep (wave-uniform): without the streaming hint (see keep_chunks).
__device__ __forceinline__ void store_codes_row(uint8_t* __restrict__ row, int lane, int remain, uint32_t w, int keep)
{
    if (remain >= kRow) {
        // as four bytes: two stores of one type would be merged into one without the hint
        if (keep) reinterpret_cast<b4*>(row)[lane] = __builtin_bit_cast(b4, w);
        else st_stream(reinterpret_cast<uint32_t*>(row) + lane, w);
    } else {
        const int e = lane * 4;
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (e + t < remain) row[e + t] = static_cast<uint8_t>(w >> (8 * t));
    }
}

// A row of a chunk that may be cut short, read without a test: every lane makes one access and the lane on the edge the last one
// that ends inside the chunk, so that what it gets begins `skip` elements before its own; settle() shifts it.  What a lane
// beyond the end holds means nothing (in a chunk of fewer than four elements all of them reach back into the chunk before it, and
// settle() drops what they find there).  With the tests of load_row a wave waits for one row, and in load_codes_row for one byte,
// before it asks for the next, and the one chunk that is cut short decides how long a short launch takes.  The access and settle()
// are two steps because the compiler moves a load whose result is used under a condition behind the condition.  The buffer must hold
// four elements.
struct RowAt {
    int at, skip;   // in elements; at: from the beginning of the chunk
};
template <bool FULL>
__device__ __forceinline__ RowAt row_at(int off, int len, int lane)
{
    if (FULL) return RowAt{off + lane * 4, 0};
    off = off < len ? off : 0;   // a row that is not there: any address
    const int e = off + lane * 4, last = len - 4;
    const int at = e >= len ? last & ~3 : e < last ? e : last;
    return RowAt{at, e - at};
}
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32u __attribute__((aligned(1)));
template <bool FULL, bool READ_AGAIN = false>
__device__ __forceinline__ f4 load_at(const float* __restrict__ chunk, RowAt r)
{
    if (FULL && READ_AGAIN) return *reinterpret_cast<const f4*>(chunk + r.at);
    if (FULL) return ld_stream(reinterpret_cast<const f4*>(chunk + r.at));
    if (READ_AGAIN) return *reinterpret_cast<const f4u*>(chunk + r.at);
    return __builtin_nontemporal_load(reinterpret_cast<const f4u*>(chunk + r.at));
}
template <bool FULL>
__device__ __forceinline__ uint32_t load_codes_at(const uint8_t* __restrict__ chunk, RowAt r)
{
    if (FULL) return ld_stream(reinterpret_cast<const uint32_t*>(chunk + r.at));
    return __builtin_nontemporal_load(reinterpret_cast<const u32u*>(chunk + r.at));
}
template <bool FULL>
__device__ __forceinline__ f4 settle(f4 q, RowAt r)
{
    if (FULL) return q;
    const bool one = (r.skip & 1) != 0, two = (r.skip & 2) != 0;
    const f4 s = two ? f4{q.z, q.w, q.w, q.w} : q;
    return one ? f4{s.y, s.z, s.w, s.w} : s;
}
template <bool FULL>
__device__ __forceinline__ uint32_t settle(uint32_t w, RowAt r)
{
    return FULL ? w : w >> ((8 * r.skip) & 31);
}

// +0.0f in the elements from `len` on; e: the lane's first one.
__device__ __forceinline__ void clear_absent(f4& v, int e, int len)
{
    v.x = e + 0 < len ? v.x : 0.0f;
    v.y = e + 1 < len ? v.y : 0.0f;
    v.z = e + 2 < len ? v.z : 0.0f;
    v.w = e + 3 < len ? v.w : 0.0f;
}

__device__ __forceinline__ float byte_to_float(uint32_t w, int b) { return static_cast<float>((w >> (8 * b)) & 0xffu); }

// Quantisation step of a chunk from its stored statistics: fl(fl(mx - mn) / 255), 0 for a flat chunk.
__device__ __forceinline__ float minmax_step(float mn, float mx)
{
    const float r = mx - mn;
    return (r == 0.0f) ? 0.0f : r / 255.0f;
}

// ---------------------------------------------------------------- host-side argument checks
inline bool chunk_ok(size_t chunk) { return chunk >= 256 && chunk <= 16384 && chunk % 256 == 0; }
inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
// Per-chunk metadata and top-K entry arrays are accessed element by element: natural alignment suffices, so a
// partition's slice of them (any whole number of chunks) can be passed as it is.
inline bool aligned4(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 3u) == 0; }
inline bool aligned2(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 1u) == 0; }
inline size_t num_chunks(size_t n, size_t chunk) { return (n + chunk - 1) / chunk; }
constexpr size_t kMaxGrid = 0x7fffffffu;

// Aliasing rule of every entry point: a buffer the call writes must not overlap, by byte range, any
// other buffer of the same call (buffers that are only read may overlap each other).
struct RangeCheck {
    struct Item {
        uintptr_t lo, hi;  // [lo, hi)
        bool written;
    };
    Item item[6 * BAGUA_MAX_WORKERS + 12];
    int count = 0;
    void add(const void* p, size_t bytes, bool written)
    {
        if (!p || bytes == 0) return;
        const uintptr_t lo = reinterpret_cast<uintptr_t>(p);
        item[count++] = Item{lo, lo + bytes, written};
    }
    void writes(const void* p, size_t bytes) { add(p, bytes, true); }
    void reads(const void* p, size_t bytes) { add(p, bytes, false); }
    // Sweep over the ranges in address order: a written range must start at or after the end of every
    // earlier range, a read-only range at or after the end of every earlier written range.
    bool disjoint()
    {
        std::sort(item, item + count, [](const Item& a, const Item& b) { return a.lo < b.lo; });
        uintptr_t end_any = 0, end_written = 0;
        for (int i = 0; i < count; ++i) {
            const Item& r = item[i];
            if (r.lo < (r.written ? end_any : end_written)) return false;
            if (r.hi > end_any) end_any = r.hi;
            if (r.written && r.hi > end_written) end_written = r.hi;
        }
        return true;
    }
};

// Rows per wave actually used: the preferred value, doubled until the chunk fits kMaxWaves waves.
inline int pick_rpw(int rows, int preferred)
{
    int rpw = preferred;
    while (rpw < 4 && (rows + rpw - 1) / rpw > kMaxWaves) rpw *= 2;
    return rpw;
}

// Worker-side kernels (compress with error feedback, both codecs), one launch over one contiguous buffer: two rows
// per wave stream fastest, except for chunks of 6 to 8 rows (1536..2048 elements), where that gives a workgroup of
// three or four waves -- measured slowest at every chunk size -- and one row per wave (six to eight waves) is
// 1-4 % faster.  Not used by the batched launches: there every wave first looks up its bucket, and with half the
// bytes per wave that latency is no longer hidden (11 % slower).
inline int pick_rpw_worker(int rows, int preferred)
{
    return pick_rpw(rows, (preferred == 2 && rows >= 6 && rows <= 8) ? 1 : preferred);
}

// The top-K compression.  Two rows per wave, but four where a launch of chunks above 4096 elements then runs all at once instead of
// in two goes, the second of them nearly empty.  Whole rounds of 8 workers, two -> four: C = 8192, 4.2 M elements 139.8 -> 126.5 us,
// 6 M 171.8 -> 156.5, 8 M 210.4 -> 207.5; C = 6144, 4.2 M 137.8 -> 125.4, 6 M 170.2 -> 156.7; C = 4608, 4.2 M 130.0 -> 127.3.
// Outside: C = 8192, 3 M 107.1 -> 108.5, 25 M 537 -> 547; C = 6144, 3 M 95.7 -> 103.7, 8 M 217.6 -> 222.0; C = 4608, 3 M 98.4 -> 108.3, 6 M
// 170.9 -> 186.5; C = 4096 and below, 2 M to 15 M, +4 .. +12 %.
inline int pick_rpw_topk(int rows, size_t chunks)
{
    const int rpw = pick_rpw(rows, BAGUA_RPW_TOPK), waves = (rows + rpw - 1) / rpw;
    const size_t at_once = static_cast<size_t>(kCus * (kWavesPerCu / waves));
    return rpw == 2 && waves > 8 && chunks > at_once && chunks <= static_cast<size_t>(4 * kCus) ? 4 : rpw;
}

// Expands `stmt` with a constexpr RPW equal to the runtime value rpw (2 or 4; chunks have at most 64 rows).
#define BAGUA_DISPATCH_RPW(rpw, stmt)                    \
    switch (rpw) {                                        \
        case 2: { constexpr int RPW = 2; stmt; } break;  \
        default: { constexpr int RPW = 4; stmt; } break; \
    }

// The same for the worker-side kernels, which also come with one row per wave.
#define BAGUA_DISPATCH_RPW_WORKER(rpw, stmt)             \
    switch (rpw) {                                        \
        case 1: { constexpr int RPW = 1; stmt; } break;  \
        case 2: { constexpr int RPW = 2; stmt; } break;  \
        default: { constexpr int RPW = 4; stmt; } break; \
    }

// Expands `stmt` with a constexpr SHORT equal to the runtime value is_short (see short_launch).
#define BAGUA_DISPATCH_SHORT(is_short, stmt)            \
    if (is_short) { constexpr bool SHORT = true; stmt; } \
    else { constexpr bool SHORT = false; stmt; }

// A launch without the detour of <<< >>> over the runtime's call stack, 0.25 of 2.7 us of host time.
template <typename T>
struct SameType {
    using type = T;
};
template <typename... P>
inline void launch_kernel(void (*kernel)(P...), dim3 grid, dim3 block, size_t lds, hipStream_t stream, typename SameType<P>::type... args)
{
    void* at[] = {const_cast<void*>(static_cast<const void*>(&args))...};
    (void)hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, at, lds, stream);   // launch_status() tells
}

inline int launch_status()
{
    return hipGetLastError() == hipSuccess ? BAGUA_OK : BAGUA_ERR_LAUNCH;
}

}  // namespace bagua
