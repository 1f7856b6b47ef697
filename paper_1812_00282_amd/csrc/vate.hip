// VATE hot path for MI355X (gfx950): pool init, packet ingest (SetAT),
// pool census, per-host estimation, clock advance and two-block preservation,
// behind the C ABI declared in include/vate.h.
//
// Paper: Xu, Ding, Hu, "VATE: a trade-off between memory and preserving time
// for high accuracy cardinalities estimation under sliding time window",
// arXiv 1812.00282.  Algorithm 4 is the per-slice loop; Sec. 4.2 describes
// its three GPU phases (scan, estimate, maintain), which map to k_ingest,
// k_census + the estimate kernels and k_advance + k_preserve here.  An estimate
// gathers its VATs' bits one by one (k_estimate, k_gather), from LDS slice by
// slice (vate_sliced.h), one part of the bitmap per XCD (vate_parts.h), or
// sorted by pool slice (vate_part.h), by the sketch and the number of hosts.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <initializer_list>
#include <type_traits>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>

#include "vate.h"
#include "vate_core.h"
#include "vate_mlp.h"
#include "mlp_core.h"
#include "vate_batch.h"

namespace vate {

// ---------------------------------------------------------------------------
// Device state block (caller-owned, 256-byte aligned).
// ---------------------------------------------------------------------------
struct DevState {
    unsigned long long t;        // current slice
    uint32_t bact0;              // ACT of block 0 (Eq. 7)
    uint32_t pad0;
    uint32_t ticket;             // workgroups done (k_preserve), zero between kernels
    uint32_t pad1[3];
};
constexpr size_t kStateHeader = sizeof(DevState);
static_assert(kStateHeader == 32, "state header layout");

// k counters follow the header: pool ATs whose distance is d < k.
__host__ __device__ __forceinline__ unsigned long long *census_of(DevState *st)
{
    return reinterpret_cast<unsigned long long *>(st + 1);
}
__host__ __device__ __forceinline__ const unsigned long long *census_of(const DevState *st)
{
    return reinterpret_cast<const unsigned long long *>(st + 1);
}
constexpr int kMaxHistK = 256;              // largest k of vate_estimate's histograms
constexpr uint32_t kCensusLdsBins = 4096;   // census histogram bins kept in LDS

// State block layout: header, k census counters, then (256-byte aligned) the
// activity bitmap of N bits.
static size_t bitmap_offset(uint32_t k)
{
    size_t b = kStateHeader + 8ull * k;
    return (b + 255) & ~size_t(255);
}

static size_t bitmap_bytes(uint64_t N)
{
    size_t bm = (size_t)((N + 7) / 8);
    return bm < 16 ? 16 : bm;
}

// After the bitmap: kCensusCopies partial censuses (k counters each) that the
// workgroups of large censuses add into, so that no counter takes an atomic
// from every one of them; k_census_fold then adds them to the census and clears
// them (they are zero between censuses).
constexpr uint32_t kCensusCopies = 16;

static size_t copies_offset(uint32_t k, uint64_t N)
{
    return (bitmap_offset(k) + bitmap_bytes(N) + 255) & ~size_t(255);
}

static size_t state_bytes_for(uint32_t k, uint64_t N)
{
    return (copies_offset(k, N) + 8ull * kCensusCopies * k + 255) & ~size_t(255);
}

// ---------------------------------------------------------------------------
// Parameter validation / geometry.
// ---------------------------------------------------------------------------
int make_geo(const vate_params *p, Geo *G, const char **why)
{
    if (!p) { *why = "params is NULL"; return VATE_E_INVAL; }
    if (p->counter > 1) { *why = "counter must be 0 (AT) or 1 (DR)"; return VATE_E_INVAL; }
    if (p->log2_pool < 1 || p->log2_pool > 32) { *why = "log2_pool must be in [1, 32]"; return VATE_E_INVAL; }
    if (p->width < 1 || p->width > 16) { *why = "width must be in [1, 16]"; return VATE_E_INVAL; }
    if (p->k < 1) { *why = "k must be >= 1"; return VATE_E_INVAL; }
    if (p->counter == 0 && (1ull << p->width) < 2ull * p->k + 1) {
        *why = "width too small: an AT needs 2^width >= 2k+1";
        return VATE_E_INVAL;
    }
    if (p->counter == 1 && (1ull << p->width) < 1ull * p->k + 1) {
        *why = "width too small: a DR needs 2^width >= k+1";
        return VATE_E_INVAL;
    }
    if (p->g < 1 || p->g > 65535) { *why = "g must be in [1, 65535]"; return VATE_E_INVAL; }
    if (p->partition > 1) { *why = "partition must be 0 or 1"; return VATE_E_INVAL; }
    if (p->block_log2 > 10 || p->block_log2 > p->log2_pool) {
        *why = "block_log2 must be in [0, min(10, log2_pool)]";
        return VATE_E_INVAL;
    }
    uint64_t N = 1ull << p->log2_pool;
    if (N < 2ull * p->k) { *why = "pool smaller than 2k ATs"; return VATE_E_INVAL; }
    const bool exact = p->width != 4 && p->width != 8 && p->width != 16;
    if (!exact && N * p->width / 8 < 16) { *why = "pool smaller than 16 bytes"; return VATE_E_INVAL; }
    if (exact && N < 32) { *why = "widths other than 4, 8, 16 need a pool of >= 32 counters"; return VATE_E_INVAL; }
    Geo g{};
    g.N = N;
    g.c = p->log2_pool;
    g.shift = 32 - p->log2_pool;
    g.k = p->k;
    g.twok = 2 * p->k;
    g.g = p->g;
    g.seed_a = p->seed_a;
    g.seed_b = p->seed_b;
    g.partition = p->partition;
    g.dr = p->counter;
    g.wb = p->width;
    g.blog = p->block_log2;
    const uint64_t E = exact ? 32 : 128 / p->width;   // counters per 16-byte chunk / per word group
    if (p->partition == 0) {
        g.a = N / (g.twok - 1);
        g.thresh = 0;
        g.base1 = 0;
        g.div_a = make_div32(g.a);
        g.div_a1 = make_div32(1);
        g.fast_blocks = g.a >= E;
    } else {
        uint64_t ap = N / g.twok, bp = N % g.twok;
        g.a = ap;
        g.base1 = (uint32_t)(g.twok - bp);
        g.thresh = ap * (g.twok - bp);
        g.div_a = make_div32(ap);
        g.div_a1 = make_div32(ap + 1);
        g.fast_blocks = ap >= E;
    }
    *G = g;
    *why = "";
    return VATE_OK;
}

// ---------------------------------------------------------------------------
// Container access.  AT p sits at bits [p*W, p*W+W) of the pool, little-endian.
// ---------------------------------------------------------------------------
// A preservation of at most this many workgroups steps the clock itself, in the
// workgroup that finishes last, instead of in a kernel of its own: a launch
// costs the host 3 us and the GPU 2 to 5, a ticket about 12 ns per workgroup,
// one after the other.
constexpr uint32_t kTicketMax = 64;

// Whether this workgroup is the last of the launch to get here (every thread
// of it calls).
__device__ __forceinline__ bool last_workgroup(uint32_t *ticket)
{
    __shared__ uint32_t last;
    __syncthreads();
    if (threadIdx.x == 0) {
        last = atomicAdd(ticket, 1u) == gridDim.x - 1u;
        if (last) atomicExch(ticket, 0u);
    }
    __syncthreads();
    return last != 0;
}

// Whether the workgroups of a census add into the census itself: so few that the
// atomics, one per workgroup and counter and one after the other on a counter,
// cost less than the launch that folds the partial censuses (steady traffic, a
// slice of 2^20 7-bit ATs, k = 60: 27 us straight, 29 by copies; 2^22 32 and 32;
// 2^24 55 and 39; 2^24 2-bit ATs, k = 1: 68 and 58).  Folding in the workgroup
// that ends last takes as long as its k counters times kCensusCopies: 100 us at
// k = 4000, 18 straight.
static bool census_direct(unsigned blocks) { return blocks <= 256u; }

// Adds a census workgroup's LDS histogram to the census (`direct`) or to copy
// blockIdx mod kCensusCopies, from where k_census_fold adds it.
__device__ __forceinline__ void census_flush(const Geo &G, DevState *__restrict__ st, const uint32_t *hist,
                                             unsigned long long *__restrict__ copies, bool direct)
{
    unsigned long long *to = direct ? census_of(st) : copies + (size_t)(blockIdx.x % kCensusCopies) * G.k;
    for (uint32_t d = threadIdx.x; d < G.k; d += blockDim.x)
        if (hist[d]) atomicAdd(&to[d], (unsigned long long)hist[d]);
}

// ---------------------------------------------------------------------------
// Slice advance: BACT^0 = (BACT^0 + 1) mod 2k, t = t + 1 (Alg. 4 end of loop),
// census cleared for the new slice, by one workgroup: k_advance, the last one
// of a small k_preserve, or the first one of DR maintenance (whose kernels do
// not read the clock).
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t next_bact0(const Geo &G, uint32_t bact0) { return bact0 + 1 == G.twok ? 0 : bact0 + 1; }

__device__ __forceinline__ void advance_clock(const Geo &G, DevState *__restrict__ st)
{
    if (threadIdx.x == 0) {
        st->bact0 = next_bact0(G, st->bact0);
        st->t = st->t + 1;
    }
    for (uint32_t d = threadIdx.x; d < G.k; d += blockDim.x) census_of(st)[d] = 0;
}

__global__ void k_advance(Geo G, DevState *__restrict__ st) { advance_clock(G, st); }

#include "vate_exact.h"

// W = 0: the exact width wb (counters packed back to back in 32-bit words).
template <int W>
__device__ __forceinline__ uint32_t load_at(const uint8_t *__restrict__ pool, uint32_t pid, uint32_t wb)
{
    if constexpr (W == 0) {
        return load_x(reinterpret_cast<const uint32_t *>(pool), pid, wb);
    } else if constexpr (W == 8) {
        return pool[pid];
    } else if constexpr (W == 16) {
        return reinterpret_cast<const uint16_t *>(pool)[pid];
    } else {
        return (pool[pid >> 1] >> ((pid & 1u) << 2)) & 0xFu;
    }
}

// Value e (0 <= e < 128/W) of a 16-byte chunk.
template <int W>
__device__ __forceinline__ uint32_t chunk_get(const uint4 &v, uint32_t e)
{
    constexpr uint32_t per_word = 32 / W;
    uint32_t w = e / per_word, s = (e % per_word) * W;
    uint32_t word = w == 0 ? v.x : w == 1 ? v.y : w == 2 ? v.z : v.w;
    return (word >> s) & ((1u << W) - 1u);
}

template <int W>
__device__ __forceinline__ void chunk_set(uint4 &v, uint32_t e, uint32_t val)
{
    constexpr uint32_t per_word = 32 / W;
    uint32_t w = e / per_word, s = (e % per_word) * W;
    uint32_t mask = ((1u << W) - 1u) << s;
    uint32_t *word = w == 0 ? &v.x : w == 1 ? &v.y : w == 2 ? &v.z : &v.w;
    *word = (*word & ~mask) | (val << s);
}

template <int W>
__host__ __device__ __forceinline__ uint32_t replicate(uint32_t val)
{
    uint32_t r = 0;
    for (int s = 0; s < 32; s += W) r |= val << s;
    return r;
}

// ---------------------------------------------------------------------------
// k_init: InitAT on every AT (value 2k), t = 0, BACT^0 = 0, census cleared.
// ---------------------------------------------------------------------------
template <int W>
__global__ void __launch_bounds__(256) k_init(Geo G, uint4 *__restrict__ pool4, uint64_t nchunks,
                                              DevState *__restrict__ st, unsigned long long *__restrict__ copies)
{
    const uint32_t pat = replicate<W>(inactive_value(G));
    const uint4 v = make_uint4(pat, pat, pat, pat);
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i < nchunks; i += (uint64_t)gridDim.x * blockDim.x) pool4[i] = v;
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) {
            st->t = 0;
            st->bact0 = 0;
            st->ticket = 0;
        }
        for (uint32_t d = threadIdx.x; d < G.k; d += blockDim.x) census_of(st)[d] = 0;
        for (uint32_t d = threadIdx.x; d < kCensusCopies * G.k; d += blockDim.x) copies[d] = 0;
    }
}

// ---------------------------------------------------------------------------
// k_ingest: the scan phase.  Each thread takes 4 consecutive packets (two
// 16-byte loads, so a wavefront reads 2 x 1 KiB contiguous), hashes them in
// registers and stores the block ACT into the AT (SetAT).  Concurrent SetATs
// of one AT in a slice all write the same value, so plain byte/short stores
// are race-free; 4-bit ATs share a 32-bit word with their neighbours and are
// set like exact-width counters (set_bits).
// ---------------------------------------------------------------------------
template <int W>
__device__ __forceinline__ void set_at(uint8_t *__restrict__ pool, uint32_t pid, uint32_t act, bool crowded)
{
    if constexpr (W == 8) {
        pool[pid] = (uint8_t)act;
    } else if constexpr (W == 16) {
        reinterpret_cast<uint16_t *>(pool)[pid] = (uint16_t)act;
    } else {
        const uint32_t s = (pid & 7u) << 2;
        uint32_t *word = reinterpret_cast<uint32_t *>(pool) + (pid >> 3);
        if (crowded) put_bits(word, 0xFu << s, act << s);
        else set_bits(word, 0xFu << s, act << s);
    }
}

// A workgroup's filter of counters it has set already (widths set by
// compare-and-swap): slot s holds the last pid with pid mod kSeen == s.  A few
// hosts send most packets (Zipf), and swaps on one address take about 12 ns
// each one after the other, whoever sends them: 1M packets of 1M Zipf(1.1)
// hosts took 2.8 ms with every packet going to its word.  The exchange is an
// LDS atomic, so of the lanes that bring one pid together only one finds
// another pid in the slot and sets the counter.
constexpr uint32_t kSeen = 2048;

__device__ __forceinline__ void seen_clear(uint32_t *seen)
{
    for (uint32_t q = threadIdx.x; q < kSeen; q += blockDim.x) seen[q] = q ^ 1u;   // no pid of slot q
}

template <int W>
constexpr bool kUsesSeen = W == 0 || W == 4;

// Whether n packets crowd a small pool's words: several for each word (of up to
// 2^15), so that most swaps would fail, but not so many for each counter that
// most find it set.  Then counters are put without a look at them (2^16 nibbles,
// k = 2, a slice of 260,000 packets 87 us by swaps and 61 so, 1M 147 and 113, 4M
// 150 and 327; 2^16 3-bit ATs 260,000 78 and 47).  Beyond 2^15 words
// the few hosts that send most decide: 2^19 nibbles, 1M packets of evenly spread
// hosts 139 us by swaps and 114 without a look, of Zipf(1.3) hosts 97 and 136.
__host__ __device__ __forceinline__ bool crowded_words(const Geo &G, uint64_t n)
{
    const uint64_t words = G.N * G.wb / 32u;
    return words <= 32768u && n >= words && n < (G.wb <= 4 ? 32u : 4u) * G.N;
}

template <int W>
__device__ __forceinline__ void ingest_one(const Geo &G, uint8_t *__restrict__ pool, uint32_t bact0,
                                           uint32_t aip, uint32_t bip, uint32_t *seen, bool crowded)
{
    uint32_t vid = bh(G, bip);
    uint32_t pid = vat_pid(G, host_key(G, aip), vid);
    if constexpr (kUsesSeen<W>) {
        if (atomicExch(&seen[pid & (kSeen - 1u)], pid) == pid) return;
    }
    // SetAT stores the block's ACT; a DR is reset to 0
    uint32_t val = G.dr ? 0u : block_act(G, bact0, block_of(G, pid));
    if constexpr (W == 0)
        set_x(reinterpret_cast<uint32_t *>(pool), pid, G.wb, val, crowded);
    else
        set_at<W>(pool, pid, val, crowded);
}

template <int W, bool ALIGNED16>
__global__ void __launch_bounds__(256) k_ingest(Geo G, const uint32_t *__restrict__ pairs, uint64_t n,
                                                uint8_t *__restrict__ pool, const DevState *__restrict__ st,
                                                bool crowded)
{
    __shared__ uint32_t seen[kUsesSeen<W> ? kSeen : 1];
    if constexpr (kUsesSeen<W>) {
        seen_clear(seen);
        __syncthreads();
    }
    const uint32_t bact0 = st->bact0;
    for (uint64_t base = (uint64_t)blockIdx.x * 1024; base < n; base += (uint64_t)gridDim.x * 1024) {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const uint64_t j = base + (uint64_t)half * 512 + 2ull * threadIdx.x;   // first of 2 packets
            if (ALIGNED16 && j + 2 <= n) {
                uint4 v = reinterpret_cast<const uint4 *>(pairs)[j >> 1];
                ingest_one<W>(G, pool, bact0, v.x, v.y, seen, crowded);
                ingest_one<W>(G, pool, bact0, v.z, v.w, seen, crowded);
            } else {
                for (uint64_t q = j; q < j + 2 && q < n; ++q) {
                    uint2 v = reinterpret_cast<const uint2 *>(pairs)[q];
                    ingest_one<W>(G, pool, bact0, v.x, v.y, seen, crowded);
                }
            }
        }
    }
}

// Few packets of widths with a filter: a packet per thread at a time, whose two
// round trips (the word's read, the swap) are all there is to wait for, by one
// workgroup per CU (more of them swap slower: 130,000 packets on 2^24 nibbles 48
// us by 256 workgroups, 58 by 512).  4,000 packets of 10-bit ATs on 2^16, a
// slice: four per thread 37.6 us, 23.5 so.
constexpr uint64_t kFewPackets = 1u << 18;

template <int W>
__global__ void __launch_bounds__(256) k_ingest_few(Geo G, const uint32_t *__restrict__ pairs, uint64_t n,
                                                    uint8_t *__restrict__ pool, const DevState *__restrict__ st)
{
    __shared__ uint32_t seen[kSeen];
    seen_clear(seen);
    __syncthreads();
    const uint32_t bact0 = st->bact0;
    for (uint64_t j = (uint64_t)blockIdx.x * 256 + threadIdx.x; j < n; j += (uint64_t)gridDim.x * 256) {
        const uint2 v = reinterpret_cast<const uint2 *>(pairs)[j];
        ingest_one<W>(G, pool, bact0, v.x, v.y, seen, false);
    }
}

// ---------------------------------------------------------------------------
// k_census: one streaming pass over the pool at the end of a slice.  Builds
// the histogram of AT distances d < k (Eq. 5) with per-workgroup LDS counters
// flushed by 64-bit atomics; Z_p for any k' is then N minus a prefix sum.
// In steady state most ATs hold 2k, so 16-byte chunks that are entirely
// inactive are skipped after one compare.
// ---------------------------------------------------------------------------

// The same pass writes the activity bitmap: bit p is set iff AT p is active
// for the longest window k at the end of this slice (value != 2k and
// distance < k).  The bitmap (N bits; 32 MiB for 2^28 ATs) is small enough to
// stay resident in the MI355X's 256 MB Infinity Cache, so the per-host gather
// in k_estimate reads bits from it instead of AT bytes from HBM.
template <int W>
__device__ __forceinline__ void store_bits(uint8_t *__restrict__ bitmap, uint64_t ch, uint32_t bits)
{
    if constexpr (W == 8)
        reinterpret_cast<uint16_t *>(bitmap)[ch] = (uint16_t)bits;   // 16 ATs per chunk
    else if constexpr (W == 4)
        reinterpret_cast<uint32_t *>(bitmap)[ch] = bits;             // 32 ATs per chunk
    else
        bitmap[ch] = (uint8_t)bits;                                  // 8 ATs per chunk
}

// One 16-byte chunk of the census: returns the chunk's activity bits and adds
// each active AT's distance to hist (LDS counters) or, without LDS, directly
// to the sketch's census.
template <int W>
__device__ __forceinline__ uint32_t census_chunk(const Geo &G, const uint4 &v, uint64_t ch, uint32_t bact0,
                                                 uint32_t *hist, unsigned long long *census)
{
    constexpr uint32_t E = 128 / W;
    const uint32_t inact = inactive_value(G);
    const uint32_t pat = replicate<W>(inact);
    if (v.x == pat && v.y == pat && v.z == pat && v.w == pat) return 0;
    uint32_t bits = 0;
    const uint64_t p0 = ch * E;
    uint32_t bid0 = 0, act0 = 0;
    uint64_t next = 0;
    if (G.fast_blocks && !G.dr) {
        bid0 = block_of(G, (uint32_t)p0);
        act0 = block_act(G, bact0, bid0);
        next = block_start(G, bid0 + 1);
    }
    for (uint32_t e = 0; e < E; ++e) {
        uint32_t val = chunk_get<W>(v, e);
        if (val == inact) continue;
        uint32_t d;
        if (G.dr) {
            d = val;                         // a DR holds its distance
        } else {
            uint32_t act;
            if (G.fast_blocks)
                act = p0 + e < next ? act0 : block_act(G, bact0, bid0 + 1);
            else
                act = block_act(G, bact0, block_of(G, (uint32_t)(p0 + e)));
            d = at_dist(G, act, val);
        }
        if (d < G.k) {
            bits |= 1u << e;
            if (hist) atomicAdd(&hist[d], 1u);
            else atomicAdd(&census[d], 1ull);
        }
    }
    return bits;
}

// Byte ATs of a chunk inside one block: the activity test four ATs at a time
// in packed 16-bit lanes (each 32-bit word split into its even and odd
// bytes).  For ACT a and value v in [0, 2k]: u = a + 2k - v, the distance is
// (a - v) mod 2k = min(u, u - 2k) (the second wraps when u < 2k), raised to
// at least k when v = 2k (inactive), and the AT is active iff it is below k.
// A DR's value is its distance.  Only the active ATs (a few per cent) take
// the per-AT histogram step.
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t active_bits8(const Geo &G, const uint4 &v, uint32_t act)
{
    const u16x2 K = (u16x2)(unsigned short)G.k;
    const u16x2 A = (u16x2)(unsigned short)(act + G.twok);
    const u16x2 T = (u16x2)(unsigned short)G.twok;
    const u16x2 T1 = (u16x2)(unsigned short)(G.twok - 1u);
    const uint32_t w4[4] = {v.x, v.y, v.z, v.w};
    uint32_t bits = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        uint32_t f2[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const u16x2 x = __builtin_bit_cast(u16x2, (w4[j] >> (8 * h)) & 0x00FF00FFu);
            u16x2 d;
            if (G.dr) {
                d = x;
            } else {
                const u16x2 u = A - x;
                d = __builtin_elementwise_min(u, u - T);
                d = __builtin_elementwise_max(d, __builtin_elementwise_sub_sat(x, T1) * K);
            }
            f2[h] = __builtin_bit_cast(uint32_t, (u16x2)((d - K) >> (unsigned short)15));   // 1 iff d < k
        }
        // f2[0] holds bytes 0 and 2 of word j, f2[1] bytes 1 and 3
        const uint32_t x = f2[0] | (f2[1] << 1);
        bits |= ((x & 3u) | ((x >> 14) & 0xCu)) << (4 * j);
    }
    return bits;
}

// One chunk of the census with the fast paths: an all-inactive chunk (most
// of them in steady state) has no bits; byte ATs of a chunk inside one block
// (or any chunk of byte DRs) take the packed test when the histogram is in
// LDS; anything else goes through census_chunk.
template <int W>
__device__ __forceinline__ uint32_t census_chunk_fast(const Geo &G, const uint4 &v, uint64_t ch, uint32_t bact0,
                                                      uint32_t pat, uint32_t *hist, unsigned long long *census)
{
    if constexpr (W == 8) {
        if (v.x == pat && v.y == pat && v.z == pat && v.w == pat) return 0u;
        if (hist) {
            const uint32_t p0 = (uint32_t)(ch * 16u);
            uint32_t bid0 = 0, act = 0;
            bool one = G.dr != 0;
            if (!one && G.fast_blocks) {
                bid0 = block_of(G, p0);
                one = (uint64_t)p0 + 16u <= block_start(G, bid0 + 1);
                act = block_act(G, bact0, bid0);
            }
            if (one) {
                const uint32_t bits = active_bits8(G, v, act);
                uint32_t rest = bits;
                while (rest) {
                    const uint32_t e = __builtin_ctz(rest);
                    rest &= rest - 1u;
                    const uint32_t val = chunk_get<8>(v, e);
                    atomicAdd(&hist[G.dr ? val : at_dist(G, act, val)], 1u);
                }
                return bits;
            }
        }
    }
    return census_chunk<W>(G, v, ch, bact0, hist, census);
}

// Nibbles and 16-bit counters; byte counters take k_census8.
template <int W>
__global__ void __launch_bounds__(256) k_census(Geo G, const uint4 *__restrict__ pool4, uint64_t nchunks,
                                                DevState *__restrict__ st, uint8_t *__restrict__ bitmap,
                                                unsigned long long *__restrict__ copies, bool direct)
{
    __shared__ uint32_t hist[kCensusLdsBins];
    const bool lds = G.k <= kCensusLdsBins;
    if (lds)
        for (uint32_t d = threadIdx.x; d < G.k; d += blockDim.x) hist[d] = 0;
    __syncthreads();
    const uint32_t bact0 = st->bact0;
    const uint32_t pat = replicate<W>(inactive_value(G));
    constexpr int U = 4;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t c0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; c0 < nchunks; c0 += U * stride) {
        uint4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            uint64_t ch = c0 + u * stride;
            v[u] = ch < nchunks ? pool4[ch] : make_uint4(pat, pat, pat, pat);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t ch = c0 + u * stride;
            if (ch < nchunks)
                store_bits<W>(bitmap, ch,
                              census_chunk_fast<W>(G, v[u], ch, bact0, pat, lds ? hist : nullptr, census_of(st)));
        }
    }
    __syncthreads();
    if (lds) census_flush(G, st, hist, copies, direct);
}

// k_census8: the census of byte counters (k <= 255).  In steady
// state only a few per cent of the chunks hold an active AT, but nearly every
// wavefront has one among its 64, so a per-lane test would run the packed
// activity test on all of them.  Here each wavefront stages the busy chunks
// of a round in LDS (compacted, in lane order), its lanes test the staged
// chunks one each and leave each chunk's bits in its staging slot, and the
// chunk's own lane picks them up; all-inactive chunks have zero bits.
//
// A lane takes U consecutive chunks per round (64 contiguous bytes, a
// wavefront 4 KiB) and stores their 16-bit bitmap words as one 8-byte
// store.  The rounds in which every lane's chunks lie inside the pool are
// software pipelined: a round's loads are issued before the previous round
// is tested, and its bitmap store after, so the wait for the loads never
// covers a store that is still in flight.  The remaining round (at most
// one) is guarded.
constexpr uint32_t kCensus8Bins = 256;
constexpr int kCensus8U = 4;   // consecutive chunks per lane and round

struct Census8Lds {
    uint32_t hist[kCensus8Bins];
    uint4 v[4][64 * kCensus8U];       // staged chunks of each wavefront
    uint16_t c[4][64 * kCensus8U];    // staged chunk's (u * 64 + lane), then its bits
};

// One round: chunk u of this lane is c0 + u; bits[u] = its activity bits.
__device__ __forceinline__ void census8_round(const Geo &G, const uint4 (&v)[kCensus8U], uint64_t c0, uint32_t bact0,
                                              uint32_t pat, Census8Lds &L, uint32_t (&bits)[kCensus8U],
                                              unsigned long long *census)
{
    constexpr int U = kCensus8U;
    const uint32_t lane = threadIdx.x & 63u, wv = threadIdx.x >> 6;
    uint32_t n = 0;          // staged chunks of this wavefront (uniform)
    uint32_t pos[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const bool busy = v[u].x != pat || v[u].y != pat || v[u].z != pat || v[u].w != pat;
        const uint64_t m = __ballot(busy);
        pos[u] = busy ? n + (uint32_t)__popcll(m & ((1ull << lane) - 1ull)) : ~0u;
        if (busy) {
            L.v[wv][pos[u]] = v[u];
            L.c[wv][pos[u]] = (uint16_t)(u * 64 + lane);
        }
        n += (uint32_t)__popcll(m);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const uint64_t wbase = c0 - (uint64_t)U * lane;     // the wavefront's first chunk
    for (uint32_t i = lane; i < n; i += 64) {
        const uint32_t code = L.c[wv][i];
        const uint64_t ch = wbase + (uint64_t)U * (code & 63u) + (code >> 6);
        L.c[wv][i] = (uint16_t)census_chunk_fast<8>(G, L.v[wv][i], ch, bact0, pat, L.hist, census);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int u = 0; u < U; ++u) bits[u] = pos[u] != ~0u ? (uint32_t)L.c[wv][pos[u]] : 0u;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__global__ void __launch_bounds__(256) k_census8(Geo G, const uint4 *__restrict__ pool4, uint64_t nchunks,
                                                 DevState *__restrict__ st, uint8_t *__restrict__ bitmap,
                                                 unsigned long long *__restrict__ copies, bool direct)
{
    constexpr int U = kCensus8U;
    static_assert(U == 4, "one 8-byte bitmap store per lane and round");
    __shared__ Census8Lds L;
    for (uint32_t d = threadIdx.x; d < G.k; d += blockDim.x) L.hist[d] = 0;
    __syncthreads();
    const uint32_t bact0 = st->bact0;
    const uint32_t pat = replicate<8>(inactive_value(G));
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t step = (uint64_t)U * gridDim.x * blockDim.x;     // chunks per round
    uint16_t *bm16 = reinterpret_cast<uint16_t *>(bitmap);
    uint64_t c0 = (uint64_t)U * (blockIdx.x * blockDim.x + threadIdx.x);
    uint32_t bits[U];
    const uint64_t full = nchunks / step;      // rounds with every chunk inside the pool
    if (full > 0) {
        uint4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = pool4[c0 + u];
        // The first round's chunks are waited for here, so that the loop
        // entry leaves no load in flight that the loop head would wait for
        // (a wait there would also cover the previous round's store).
#pragma unroll
        for (int u = 0; u < U; ++u) asm volatile("" ::"v"(v[u].x), "v"(v[u].y), "v"(v[u].z), "v"(v[u].w));
        for (uint64_t r = 0; r < full; ++r, c0 += step) {
            // the next round's chunks (the last round reloads its own)
            const uint64_t nx = r + 1 < full ? c0 + step : c0;
            uint4 w[U];
#pragma unroll
            for (int u = 0; u < U; ++u) w[u] = pool4[nx + u];
            census8_round(G, v, c0, bact0, pat, L, bits, census_of(st));
            *reinterpret_cast<uint2 *>(bm16 + c0) = make_uint2(bits[0] | bits[1] << 16, bits[2] | bits[3] << 16);
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = w[u];
        }
    }
    if (c0 - (uint64_t)U * lane < nchunks) {   // the guarded last round (uniform per wavefront)
        uint4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = c0 + u < nchunks ? pool4[c0 + u] : make_uint4(pat, pat, pat, pat);
        census8_round(G, v, c0, bact0, pat, L, bits, census_of(st));
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (c0 + u < nchunks) bm16[c0 + u] = (uint16_t)bits[u];
    }
    __syncthreads();
    census_flush(G, st, L.hist, copies, direct);
}

__global__ void __launch_bounds__(256) k_census_fold(Geo G, DevState *__restrict__ st,
                                                     unsigned long long *__restrict__ copies)
{
    for (uint32_t d = blockIdx.x * blockDim.x + threadIdx.x; d < G.k; d += gridDim.x * blockDim.x) {
        unsigned long long sum = 0;
        for (uint32_t c = 0; c < kCensusCopies; ++c) {
            sum += copies[(size_t)c * G.k + d];
            copies[(size_t)c * G.k + d] = 0;
        }
        census_of(st)[d] += sum;
    }
}

// ---------------------------------------------------------------------------
// k_estimate: the closed form by a direct gather, L lanes per host.  The g
// VATs of a host are gathered in batches of U independent reads per lane,
// decoded with CheckAT (Alg. 1), counted and summed over the host's lanes, and
// the estimate of Eq. 11 is formed in FP32 from exact integer counts.  (With
// the distance histogram: k_gather.)  Bound by L2 once the chip is full: it
// serves about 2.5e11 of these reads a second.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float estimate_from_counts(uint64_t u_v, uint64_t u_p, uint32_t g, uint32_t c)
{
    if (u_v == 0) u_v = 1;
    if (u_p == 0) u_p = 1;
    const uint64_t N = 1ull << c;
    const long long D = (long long)(u_p * g) - (long long)(N * u_v);
    const float den = ldexpf((float)u_v, (int)c);          // N * u_v, exact
    const float x = (float)D / den;
    if (x >= -0.5f)
        return (float)g * log1pf(x);
    return (float)g * logf((float)(u_p * g) / den);
}

// Number of pool ATs active for k' (sum of census bins d < k'), per wavefront.
__device__ __forceinline__ uint64_t pool_active(const DevState *__restrict__ st, uint32_t kprime)
{
    const uint32_t lane = threadIdx.x & 63u;
    unsigned long long s = 0;
    for (uint32_t d = lane; d < kprime; d += 64) s += census_of(st)[d];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    return s;
}

// VATs sub, sub + L, ... of one host that are active for k', by U gathers in
// flight.  The activity bitmap answers CheckAT(., k) directly; the AT value
// (for its distance) is only read for VATs that are active at all, and only
// when a shorter window needs it, again with V of a batch in flight.
template <int W, int L, int U, int V = U>
__device__ __forceinline__ uint32_t lane_live(const Geo &G, const uint8_t *__restrict__ pool,
                                              const uint8_t *__restrict__ bitmap, uint32_t kprime, uint32_t key, bool valid, uint32_t bact0, uint32_t sub)
{
    const bool need_dist = kprime < G.k;
    uint32_t live = 0;
    for (uint32_t i0 = sub; i0 < G.g; i0 += L * U) {
        uint32_t pid[U], bit[U];
#pragma unroll
        for (int u = 0; u < U; ++u) pid[u] = vat_pid(G, key, i0 + u * L);
#pragma unroll
        for (int u = 0; u < U; ++u) bit[u] = (valid && i0 + u * L < G.g) ? (uint32_t)bitmap[pid[u] >> 3] : 0u;
#pragma unroll
        for (int u = 0; u < U; ++u) bit[u] = (bit[u] >> (pid[u] & 7u)) & 1u;
        if (!need_dist) {
#pragma unroll
            for (int u = 0; u < U; ++u) live += bit[u];
            continue;
        }
#pragma unroll
        for (int u0 = 0; u0 < U; u0 += V) {
            uint32_t val[V];
#pragma unroll
            for (int u = 0; u < V; ++u) val[u] = bit[u0 + u] ? load_at<W>(pool, pid[u0 + u], G.wb) : 0u;
#pragma unroll
            for (int u = 0; u < V; ++u)
                if (bit[u0 + u] && value_dist(G, bact0, pid[u0 + u], val[u]) < kprime) ++live;
            if constexpr (V < U) __builtin_amdgcn_sched_barrier(0);
        }
    }
    return live;
}

template <int L>
__device__ __forceinline__ uint32_t sum_lanes(uint32_t x)
{
#pragma unroll
    for (int off = 1; off < L; off <<= 1) x += __shfl_xor(x, off, 64);
    return x;
}

template <int W, int L, int U>
__global__ void __launch_bounds__(256) k_estimate(Geo G, const uint8_t *__restrict__ pool,
                                                  const DevState *__restrict__ st,
                                                  const uint8_t *__restrict__ bitmap,
                                                  const uint32_t *__restrict__ hosts, uint32_t n,
                                                  uint32_t kprime, float *__restrict__ est,
                                                  uint32_t *__restrict__ live_out)
{
    constexpr uint32_t per = 256 / L;
    const uint32_t sub = threadIdx.x % L;
    const uint32_t bact0 = st->bact0;
    const uint64_t active_pool = pool_active(st, kprime);
    for (uint64_t h0 = (uint64_t)blockIdx.x * per; h0 < n; h0 += (uint64_t)gridDim.x * per) {
        const uint64_t h = h0 + threadIdx.x / L;
        const bool valid = h < n;
        const uint32_t key = host_key(G, valid ? hosts[h] : 0u);
        const uint32_t live = sum_lanes<L>(lane_live<W, L, U>(G, pool, bitmap, kprime, key, valid, bact0, sub));
        if (valid && sub == 0) {
            est[h] = estimate_from_counts(G.g - live, G.N - active_pool, G.g, G.c);
            if (live_out) live_out[h] = live;
        }
    }
}

// ---------------------------------------------------------------------------
// k_estimate_blocked: the closed form for window k under the locality-blocked
// H with blocks of >= 32 VATs, where a block is whole 32-bit words of the
// activity bitmap.  L lanes per host (L = blocks per host rounded up to a
// power of two, at most 64), each counting the set bits of its blocks with
// popcount; the host's lanes are summed by shuffles.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_estimate_blocked(Geo G, const DevState *__restrict__ st,
                                                          const uint32_t *__restrict__ bitmap,
                                                          const uint32_t *__restrict__ hosts, uint32_t n,
                                                          uint32_t lanes_log2, float *__restrict__ est,
                                                          uint32_t *__restrict__ live_out)
{
    const uint64_t active_pool = pool_active(st, G.k);
    const uint32_t L = 1u << lanes_log2;
    const uint32_t gid = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t h = gid >> lanes_log2, sub = gid & (L - 1u);
    const bool valid = h < n;
    const uint32_t key = host_key(G, valid ? hosts[h] : 0u);
    const uint32_t beta = 1u << G.blog, words = beta >> 5;
    const uint32_t nb = (G.g + beta - 1u) >> G.blog;
    uint32_t live = 0;
    if (valid)
        for (uint32_t q = sub; q < nb; q += L) {
            const uint32_t base = vat_pid(G, key, q << G.blog);          // block-aligned first AT
            const uint32_t in_block = min(beta, G.g - (q << G.blog));      // VATs of this block
            const uint32_t *w = bitmap + (base >> 5);
            for (uint32_t x = 0; x < words; ++x) {
                const uint32_t lo = x << 5;
                if (lo >= in_block) break;
                uint32_t v = w[x];
                if (in_block - lo < 32) v &= (1u << (in_block - lo)) - 1u;
                live += __popc(v);
            }
        }
    for (uint32_t off = 1; off < L; off <<= 1) live += __shfl_xor(live, off, 64);
    if (valid && sub == 0) {
        est[h] = estimate_from_counts(G.g - live, G.N - active_pool, G.g, G.c);
        if (live_out) live_out[h] = live;
    }
}

static bool blocked_gather_ok(const Geo &G, uint32_t kprime) { return G.blog >= 5 && kprime == G.k; }

constexpr int kLearnMaxK = VATE_MLP_FEATURES - 3;

#include "vate_part.h"
#include "vate_sliced.h"
#include "vate_parts.h"

__global__ void k_set_clock(Geo G, DevState *__restrict__ st, unsigned long long t, uint32_t bact0)
{
    if (threadIdx.x == 0) {
        st->t = t;
        st->bact0 = bact0;
    }
    for (uint32_t d = threadIdx.x; d < G.k; d += blockDim.x) census_of(st)[d] = 0;
}

// ---------------------------------------------------------------------------
// k_preserve: PreserveAT (Alg. 3) over the two blocks whose ACT is now 0
// (block i0) or k (block i1), Cor. 1.  Block indices come from the device
// clock so a captured graph replays correctly.  Each 16-byte chunk that
// overlaps a due block is owned by exactly one thread (a chunk shared by both
// blocks belongs to the i0 pass), which rewrites it only if an AT changed.
// ---------------------------------------------------------------------------
template <int W>
__device__ __forceinline__ void preserve_chunk(const Geo &G, uint4 *__restrict__ pool4, uint32_t bact0, uint64_t j,
                                               uint64_t max_chunks)
{
    constexpr uint64_t E = 128 / W;
    const uint32_t i0 = bact0 == 0 ? 0 : G.twok - bact0;                        // (BACT^0 + i0) mod 2k == 0
    const uint32_t i1 = bact0 <= G.k ? G.k - bact0 : G.twok + G.k - bact0;      // == k
    const uint64_t s0 = block_start(G, i0), e0 = block_start(G, i0 + 1);
    const uint64_t s1 = block_start(G, i1), e1 = block_start(G, i1 + 1);
    const uint64_t c0lo = s0 / E, c0hi = s0 < e0 ? (e0 + E - 1) / E : c0lo;
    const uint64_t c1lo = s1 / E, c1hi = s1 < e1 ? (e1 + E - 1) / E : c1lo;
    const bool second = j >= max_chunks;
    const uint64_t ch = second ? c1lo + (j - max_chunks) : c0lo + j;
    if (j >= 2 * max_chunks) return;
    if (ch >= (second ? c1hi : c0hi)) return;
    if (second && ch >= c0lo && ch < c0hi) return;
    uint4 v = pool4[ch];
    const uint32_t pat = replicate<W>(G.twok);       // inactive ATs stay as they are (most chunks)
    if (v.x == pat && v.y == pat && v.z == pat && v.w == pat) return;
    bool changed = false;
    for (uint32_t e = 0; e < E; ++e) {
        const uint64_t p = ch * E + e;
        const bool in0 = p >= s0 && p < e0, in1 = p >= s1 && p < e1;
        if (!in0 && !in1) continue;
        const uint32_t val = chunk_get<W>(v, e);
        bool mark;
        if (in0)   // ACT == 0: 0 <= Value <= k
            mark = val <= G.k;
        else       // ACT == k: k <= Value <= 2k-1, or Value == 0
            mark = (val >= G.k && val <= G.twok - 1) || val == 0;
        if (mark && val != G.twok) {
            chunk_set<W>(v, e, G.twok);
            changed = true;
        }
    }
    if (changed) pool4[ch] = v;
}

// `ends`: the clock is still the old slice's, and the last workgroup moves it
// (each has read it by then).
template <int W>
__global__ void __launch_bounds__(256) k_preserve(Geo G, uint4 *__restrict__ pool4, DevState *st, uint64_t max_chunks,
                                                  bool ends)
{
    const uint32_t bact0 = ends ? next_bact0(G, st->bact0) : st->bact0;
    for (uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; j < 2 * max_chunks;
         j += (uint64_t)gridDim.x * blockDim.x)
        preserve_chunk<W>(G, pool4, bact0, j, max_chunks);
    if (ends && last_workgroup(&st->ticket)) advance_clock(G, st);
}

// ---------------------------------------------------------------------------
// DR maintenance (the VDRE baseline of Sec. 5): at every slide each counter of
// the pool grows by one, saturating at k (Sec. 1).  The whole pool is read;
// a 16-byte chunk is written back only if one of its counters changed.
// ---------------------------------------------------------------------------
template <int W>
__device__ __forceinline__ void dr_maintain_chunk(const Geo &G, uint4 *__restrict__ pool4, uint64_t ch)
{
    constexpr uint32_t E = 128 / W;
    uint4 v = pool4[ch];
    const uint32_t pat = replicate<W>(G.k);
    if (v.x == pat && v.y == pat && v.z == pat && v.w == pat) return;
    bool changed = false;
    for (uint32_t e = 0; e < E; ++e) {
        const uint32_t val = chunk_get<W>(v, e);
        if (val < G.k) {
            chunk_set<W>(v, e, val + 1);
            changed = true;
        }
    }
    if (changed) pool4[ch] = v;
}

template <int W>
__global__ void __launch_bounds__(256) k_dr_maintain(Geo G, uint4 *__restrict__ pool4, uint64_t nchunks,
                                                     DevState *__restrict__ st)
{
    if (blockIdx.x == 0) advance_clock(G, st);
    for (uint64_t ch = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; ch < nchunks;
         ch += (uint64_t)gridDim.x * blockDim.x)
        dr_maintain_chunk<W>(G, pool4, ch);
}

#include "vate_batch_kernels.h"

}  // namespace vate

// ===========================================================================
// C ABI
// ===========================================================================
using namespace vate;

struct vate_sketch {
    vate_params p;
    Geo G;
    uint8_t *pool;
    DevState *st;
    uint8_t *bitmap;             // activity bitmap inside the state block
    unsigned long long *copies;  // partial censuses inside the state block
    size_t pool_bytes, state_bytes;
    uint64_t max_block_chunks;   // chunks a due block can overlap
    int closed;                  // 1: slice ended, estimates allowed
    int dead;                    // sticky device error
    uint32_t lds_budget;         // dynamic LDS a partitioned-scatter workgroup may use (bytes)
    uint32_t n_cu;               // compute units of the device
    const void *plan_ws;         // workspace holding a host plan (vate_estimate_plan), or null
    uint64_t plan_n;             // its host count
    uint32_t plan_hosts;         // its hosts per subgroup; 0: the workspace holds the host list itself
    char err[256];
};

static int fail(vate_sketch *s, int code, const char *msg)
{
    if (s) {
        snprintf(s->err, sizeof(s->err), "%s", msg);
        if (code == VATE_E_DEVICE) s->dead = 1;
    }
    return code;
}

static int check_launch(vate_sketch *s, const char *what)
{
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        char buf[200];
        snprintf(buf, sizeof(buf), "%s: %s", what, hipGetErrorString(e));
        return fail(s, VATE_E_DEVICE, buf);
    }
    return VATE_OK;
}

static unsigned grid_for(uint64_t items, unsigned per_block, unsigned cap)
{
    uint64_t b = (items + per_block - 1) / per_block;
    if (b < 1) b = 1;
    return (unsigned)std::min<uint64_t>(b, cap);
}

// HIP refuses a grid of 2^32 threads and more: the most workgroups of 256.
constexpr unsigned kMaxGrid256 = (1u << 24) - 1u;

// Width dispatch: 4, 8 and 16 bits use their containers; any other width is
// the exact packing (template width 0).
template <class F>
static auto by_width(uint32_t w, F &&f)
{
    if (w == 4) return f(std::integral_constant<int, 4>{});
    if (w == 8) return f(std::integral_constant<int, 8>{});
    if (w == 16) return f(std::integral_constant<int, 16>{});
    return f(std::integral_constant<int, 0>{});
}

// Exact widths as a compile-time constant for the streaming kernels.
template <class F>
static void by_exact_width(uint32_t w, F &&f)
{
    using std::integral_constant;
    switch (w) {
    case 1: return f(integral_constant<int, 1>{});
    case 2: return f(integral_constant<int, 2>{});
    case 3: return f(integral_constant<int, 3>{});
    case 5: return f(integral_constant<int, 5>{});
    case 6: return f(integral_constant<int, 6>{});
    case 7: return f(integral_constant<int, 7>{});
    case 9: return f(integral_constant<int, 9>{});
    case 10: return f(integral_constant<int, 10>{});
    case 11: return f(integral_constant<int, 11>{});
    case 12: return f(integral_constant<int, 12>{});
    case 13: return f(integral_constant<int, 13>{});
    case 14: return f(integral_constant<int, 14>{});
    default: return f(integral_constant<int, 15>{});
    }
}

template <int W>
static void launch_init(vate_sketch *s, hipStream_t st)
{
    if constexpr (W == 0) {
        const uint64_t ng = s->G.N / 32;
        k_init_x<<<grid_for(ng, 256, 8192), 256, 0, st>>>(s->G, reinterpret_cast<uint32_t *>(s->pool), ng, s->st,
                                                            s->copies);
    } else {
        uint64_t nch = s->pool_bytes / 16;
        k_init<W><<<grid_for(nch, 256, 8192), 256, 0, st>>>(s->G, reinterpret_cast<uint4 *>(s->pool), nch, s->st,
                                                             s->copies);
    }
}

template <int W>
static void launch_census(vate_sketch *s, hipStream_t st)
{
    const bool lds = s->G.k <= kCensusLdsBins;      // longer windows are counted straight into the census
    const uint64_t units = W == 0 ? s->G.N / 32 : s->pool_bytes / 16;
    const unsigned blocks = W == 0 ? grid_for(units, 256, (s->G.c >= 27 ? 16u : 8u) * s->n_cu)
                          : W == 8 ? grid_for(units, 256 * kCensus8U, 4096) : grid_for(units, 256 * 4, 2048);
    const bool direct = census_direct(blocks);
    if constexpr (W == 0) {
        by_exact_width(s->p.width, [&](auto WB) {
            k_census_x<decltype(WB)::value><<<blocks, 256, 0, st>>>(s->G, reinterpret_cast<const uint32_t *>(s->pool),
                                                                    units, s->st, s->bitmap, s->copies, direct);
        });
    } else {
        const uint4 *pool4 = reinterpret_cast<const uint4 *>(s->pool);
        if constexpr (W == 8)           // k <= 255 (2^8 >= k + 1)
            k_census8<<<blocks, 256, 0, st>>>(s->G, pool4, units, s->st, s->bitmap, s->copies, direct);
        else
            k_census<W><<<blocks, 256, 0, st>>>(s->G, pool4, units, s->st, s->bitmap, s->copies, direct);
    }
    if (lds && !direct) k_census_fold<<<(s->G.k + 255) / 256, 256, 0, st>>>(s->G, s->st, s->copies);
}

// The slide of the window: the clock and Alg. 3.
template <int W>
static void launch_preserve(vate_sketch *s, hipStream_t st)
{
    const unsigned blocks = grid_for(2 * s->max_block_chunks, 256, 8u * s->n_cu);
    const bool ends = blocks <= kTicketMax;
    if (!ends) k_advance<<<1, 256, 0, st>>>(s->G, s->st);
    if constexpr (W == 0)
        by_exact_width(s->p.width, [&](auto WB) {
            k_preserve_x<decltype(WB)::value><<<blocks, 256, 0, st>>>(s->G, reinterpret_cast<uint32_t *>(s->pool), s->st,
                                                                      s->max_block_chunks, ends);
        });
    else
        k_preserve<W><<<blocks, 256, 0, st>>>(s->G, reinterpret_cast<uint4 *>(s->pool), s->st, s->max_block_chunks, ends);
}

template <int W>
static void launch_dr_maintain(vate_sketch *s, hipStream_t st)
{
    if constexpr (W == 0) {
        const uint64_t ng = s->G.N / 32;
        by_exact_width(s->p.width, [&](auto WB) {
            k_dr_maintain_x<decltype(WB)::value><<<grid_for(ng, 256, 8192), 256, 0, st>>>(
                s->G, reinterpret_cast<uint32_t *>(s->pool), ng, s->st);
        });
    } else {
        const uint64_t nch = s->pool_bytes / 16;
        k_dr_maintain<W><<<grid_for(nch, 256, 8192), 256, 0, st>>>(s->G, reinterpret_cast<uint4 *>(s->pool), nch, s->st);
    }
}

template <int W>
static void launch_ingest(vate_sketch *s, const uint32_t *pairs, uint64_t n, hipStream_t st)
{
    const bool crowded = kUsesSeen<W> && crowded_words(s->G, n);
    if constexpr (kUsesSeen<W>)
        if (n <= kFewPackets && !crowded) {
            k_ingest_few<W><<<grid_for(n, 256, s->n_cu), 256, 0, st>>>(s->G, pairs, n, s->pool, s->st);
            return;
        }
    // Widths with a filter: few enough workgroups that each sees several
    // thousand packets.  Others: one workgroup per 1024 packets.
    unsigned blocks = grid_for(n, 1024, kUsesSeen<W> ? 4u * s->n_cu : 1u << 30);
    if ((reinterpret_cast<uintptr_t>(pairs) & 15u) == 0)
        k_ingest<W, true><<<blocks, 256, 0, st>>>(s->G, pairs, n, s->pool, s->st, crowded);
    else
        k_ingest<W, false><<<blocks, 256, 0, st>>>(s->G, pairs, n, s->pool, s->st, crowded);
}

static void dispatch_init(vate_sketch *s, hipStream_t st)
{
    by_width(s->p.width, [&](auto W) { launch_init<decltype(W)::value>(s, st); });
}

static void dispatch_census(vate_sketch *s, hipStream_t st)
{
    by_width(s->p.width, [&](auto W) { launch_census<decltype(W)::value>(s, st); });
}

static int advance(vate_sketch *s, hipStream_t st)
{
    if (s->G.dr)
        by_width(s->p.width, [&](auto W) { launch_dr_maintain<decltype(W)::value>(s, st); });
    else
        by_width(s->p.width, [&](auto W) { launch_preserve<decltype(W)::value>(s, st); });
    s->closed = 0;
    return check_launch(s, "advance/preserve");
}

// Raises a kernel's dynamic-LDS limit to the device's: a per-device function
// attribute, set once per kernel and device (bit d of the mask).  A failure is
// reported by the check_launch after the launches.
template <auto Kernel>
static bool allow_lds(const vate_sketch *s)
{
    static std::atomic<uint64_t> done{0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) dev = 0;
    const uint64_t bit = 1ull << (dev & 63);
    if (done.load(std::memory_order_acquire) & bit) return true;
    const void *fn = reinterpret_cast<const void *>(Kernel);
    hipFuncAttributes a;
    if (hipFuncGetAttributes(&a, fn) != hipSuccess) return false;
    const size_t most = s->lds_budget + kRunLdsStatic - std::max<size_t>(kRunLdsStatic, a.sharedSizeBytes);
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)most) != hipSuccess) return false;
    done.fetch_or(bit, std::memory_order_release);
    return true;
}

// log2 of the lanes per host.  As many as hold a host's VATs, P each; with one
// slice, where going round again costs no copy, 16 at most (64 hosts per
// workgroup) while every CU has a workgroup.
static uint32_t sliced_lanes(const vate_sketch *s, uint32_t n, uint32_t P)
{
    uint32_t lg = 0;
    while (lg < 6 && (P << lg) < s->G.g) ++lg;
    if (s->G.c <= kSliceLog2)
        while (lg > 4 && (uint64_t)n << (lg - 1) >= (uint64_t)kSlicedThreads * s->n_cu) --lg;
    return lg;
}

// Whether, and in what shape, the lookups of n hosts go through LDS slice by
// slice.  A thread tests P VATs whether the host has that many or not, and every
// CU takes as long as the fullest, so what counts are slots: the threads of all
// CUs in all rounds, times P.  A gathered lookup costs as much as this many
// sixteenths of a slot (byte ATs, g = 1 to 4096, 2,000 to 3M hosts; by log2 of
// the pool): little where the CU's first-level cache holds the bitmap (2^18), most
// on the largest pool of one slice, and less again the more slices a slot is
// tested against.  (2280 closed forms timed both ways: 26 take more than 1.1 times
// the better way's time, none 1.35.)  g = 4, 3M hosts, 2^23 ATs: 59 us gathered, 303 by slices; g = 1024,
// 130,000 hosts, 2^20 ATs: 387 and 84.  Values that have to be read for every
// active VAT (k' < k, histograms) narrow the difference, and histogram rows leave
// fewer hosts to a workgroup.  The network runs on 64 hosts of a workgroup's 1024
// threads, so it goes through LDS only where lookups outweigh it (500,000 hosts,
// 2^21 ATs: g = 128 gathered 317 us, through LDS 400 to 640; g = 1024 1862 and
// 1367).
enum SlicedUse { SLICED_FORM, SLICED_SHORT, SLICED_HIST, SLICED_WINDOWS, SLICED_LEARNED };

struct SlicedShape {
    uint32_t P, lg;      // VATs per thread (0: gathered), log2 of the lanes per host
};

static SlicedShape sliced_shape(const vate_sketch *s, uint32_t n, SlicedUse use, uint32_t row_bytes = 0,
                                uint32_t room = 0)
{
    static const uint8_t gain[][12] = {      // up to 2^12, 2^13, ... 2^23 ATs
        {0, 17, 22, 22, 28, 28, 33, 37, 54, 44, 23, 14},
        {0, 0, 0, 0, 17, 21, 23, 37, 40, 37, 23, 14},
        {0, 0, 0, 0, 0, 0, 0, 29, 29, 29, 17, 0},
        {0, 0, 0, 0, 16, 17, 18, 35, 42, 42, 22, 0},
        {36, 36, 36, 36, 36, 36, 36, 36, 36, 36, 18, 0},
    };
    const Geo &G = s->G;
    SlicedShape best{0, 0};
    if (G.blog > 0 || G.c > kSlicedLog2 || (use == SLICED_LEARNED && G.g < 512)) return best;
    uint64_t least = 2ull * n * G.g * gain[use][std::max(G.c, 12u) - 12u];       // in 1/32 slots
    for (uint32_t P = 16; P <= (G.c > kSliceLog2 ? 32u : 16u); P *= 2) {
        uint32_t lg = sliced_lanes(s, n, P);
        if (use == SLICED_LEARNED && lg < 4) lg = 4;      // the network takes 64 hosts at a time
        while (lg < 6 && (row_bytes * kSlicedThreads >> lg) > room) ++lg;
        if ((row_bytes * kSlicedThreads >> lg) > room) continue;
        const uint64_t per_round = (uint64_t)s->n_cu * (kSlicedThreads >> lg), again = (G.g + (P << lg) - 1u) / (P << lg);
        const uint64_t slots = (n + per_round - 1u) / per_round * s->n_cu * kSlicedThreads * P * again;
        const uint64_t cost = slots * (P == 32 ? 23u : 32u);      // (of 32 VATs a thread each costs 0.72 as much)
        if (cost <= least) least = cost, best = {P, lg};
    }
    return best;
}

// Calls f with the kernel's VATs per thread and whether there is one slice.
template <class F>
static void by_slices(const vate_sketch *s, uint32_t P, F &&f)
{
    using std::integral_constant;
    if (s->G.c <= kSliceLog2) f(integral_constant<uint32_t, 16>{}, std::true_type{});
    else if (P == 32) f(integral_constant<uint32_t, 32>{}, std::false_type{});
    else f(integral_constant<uint32_t, 16>{}, std::false_type{});
}

// Workgroups of `lds` bytes that a CU holds.
static unsigned sliced_cap(const vate_sketch *s, uint32_t lds) { return s->n_cu * (s->G.c <= kSliceLog2 && lds <= s->lds_budget / 2 ? 2u : 1u); }

// Gathers per host of the closed form for window k: its VATs, or its locality
// blocks where those are whole words of the bitmap.
static uint32_t parts_gathers(const Geo &G)
{
    return blocked_gather_ok(G, G.k) ? (G.g + (1u << G.blog) - 1u) >> G.blog : G.g;
}

// Whether the closed form goes by parts of the bitmap (k_parts_count): window
// k, a bitmap larger than an XCD's L2, enough gathers (a block of 32 VATs or
// more is one) to pay for three launches and a pass over the bitmap, and enough
// of them per host: every part hashes a host's gathers by the batch whether the
// host has that many or not.  3M hosts with one gather each: 2^26 ATs 40 us
// gathered, 72 by parts, 2^28 58 and 216; with three 2^26 at par, 2^28 149 and
// 214; with five 2^28 at par (blocks with six: 500,000 hosts of five 46 and 50).
// Blocks of eight words and more, which the other gather reads word by word, pay
// with half as many (1M hosts, two blocks of 256 VATs, 2^27 ATs: 135 and 101).
// Smaller blocks share one line among their VATs, so a host takes as many lines
// as it has blocks, but is hashed VAT by VAT: 4M hosts with one block of eight on
// 2^26 ATs 87 and 121, and eight parts do not pay at all (150,000 hosts, 128 such
// blocks, 2^28 ATs: 515 and 666).
static bool parts_gather(const vate_sketch *s, uint32_t n, uint32_t kprime)
{
    const Geo &G = s->G;
    const uint32_t pl = parts_log2(G.c);
    if (pl == 0 || kprime != G.k) return false;
    const uint64_t gathers = parts_gathers(G);
    const bool words = blocked_gather_ok(G, kprime), shared = G.blog > 0 && !words;
    if (shared && pl == 3 && G.blog > 1) return false;
    const uint64_t lines = shared ? gathers >> G.blog : G.blog >= 8 ? 2u * gathers : gathers;
    return n * gathers >= kPartsMin && lines > std::max(2u, (1u << pl) / 2u + (words ? 1u : 0u));
}

static void launch_parts(vate_sketch *s, const uint32_t *hosts, uint32_t n, float *est, uint32_t *live, hipStream_t st)
{
    uint32_t *acc = live ? live : reinterpret_cast<uint32_t *>(est);
    const uint32_t *bitmap = reinterpret_cast<const uint32_t *>(s->bitmap);
    const Geo &G = s->G;
    const bool blocked = blocked_gather_ok(G, G.k);
    // lanes per host: one while the hosts alone fill the chip, and no more than
    // a host's gathers fill
    const uint32_t gathers = parts_gathers(G), batch = blocked ? kPartsBlockU : kPartsU;
    const uint64_t threads = 2048ull * s->n_cu >> (3u - parts_log2(G.c));
    uint32_t lg = 0;
    while (lg < 6 && ((uint64_t)n << lg) < threads && (batch << (lg + 1u)) <= gathers) ++lg;
    const unsigned grid = (std::max(1u, grid_for((uint64_t)n << lg, kPartsThreads, s->n_cu)) + 7u) & ~7u;
    k_parts_clear<<<grid_for(n, 256, 4u * s->n_cu), 256, 0, st>>>(n, acc);
    if (blocked) k_parts_count<true><<<grid * 8u, kPartsThreads, 0, st>>>(G, bitmap, hosts, n, lg, acc);
    else k_parts_count<false><<<grid * 8u, kPartsThreads, 0, st>>>(G, bitmap, hosts, n, lg, acc);
    k_parts_finish<<<grid_for(n, 256, 4u * s->n_cu), 256, 0, st>>>(G, s->st, n, acc, est);
}

// The closed form without histograms.  Lanes per host: as many as keep the
// chip's 2048 threads per CU busy, so that few hosts take few serial rounds; one
// where it alone holds most of a host's VATs and the hosts keep them busy (3M
// hosts, g = 1, 2^24 ATs: 35 us with one lane, 110 with four).
template <int W>
static void launch_estimate(vate_sketch *s, const uint32_t *hosts, uint32_t n, uint32_t kprime, float *est,
                            uint32_t *live, hipStream_t st)
{
    // (the parts' counts would overwrite a host list that is also their output)
    if (parts_gather(s, n, kprime) && hosts != (live ? live : reinterpret_cast<const uint32_t *>(est))) {
        launch_parts(s, hosts, n, est, live, st);
        return;
    }
    if (blocked_gather_ok(s->G, kprime)) {
        const uint32_t nb = (s->G.g + (1u << s->G.blog) - 1u) >> s->G.blog;
        uint32_t lg = 0;
        while ((1u << lg) < nb && lg < 6) ++lg;
        k_estimate_blocked<<<grid_for((uint64_t)n << lg, 256, 1u << 30), 256, 0, st>>>(
            s->G, s->st, reinterpret_cast<const uint32_t *>(s->bitmap), hosts, n, lg, est, live);
        return;
    }
    const uint64_t lanes = (uint64_t)s->n_cu * 2048u / n;       // lanes a host may take (n >= 1)
    using std::integral_constant;
    if (const SlicedShape sh = sliced_shape(s, n, kprime < s->G.k ? SLICED_SHORT : SLICED_FORM); sh.P) {
        by_slices(s, sh.P, [&](auto Pv, auto One) {
            constexpr uint32_t P = decltype(Pv)::value;
            constexpr bool one = decltype(One)::value;
            if (!allow_lds<k_sliced<W, P, one>>(s)) return;
            const uint32_t lds = 4u * sliced_words(s->G);
            k_sliced<W, P, one><<<grid_for(n, kSlicedThreads >> sh.lg, sliced_cap(s, lds)), kSlicedThreads, lds, st>>>(
                s->G, s->pool, s->st, s->bitmap, hosts, n, sh.lg, kprime, est, live);
        });
        return;
    }
    // Workgroups persist, which saves the shortest their start; one lane that goes
    // round again gets a workgroup per 256 hosts (4M hosts, g = 20 in blocks of 16,
    // 2^24 ATs: 165 us by 4096 persistent workgroups, 134 by 15625).
    const unsigned cap = 16u * s->n_cu;
    auto go = [&](auto L, auto U) {
        constexpr int l = decltype(L)::value, u = decltype(U)::value;
        k_estimate<W, l, u><<<grid_for(n, 256 / l, l == 1 && s->G.g > u ? kMaxGrid256 : cap), 256, 0, st>>>(
            s->G, s->pool, s->st, s->bitmap, hosts, n, kprime, est, live);
    };
    if (lanes >= 64 && s->G.g <= 256) go(integral_constant<int, 64>{}, integral_constant<int, 4>{});
    else if (lanes >= 64) go(integral_constant<int, 64>{}, integral_constant<int, 16>{});
    else if (lanes >= 16 || ((lanes > 5 || s->G.c >= 26) && s->G.g >= 256)) go(integral_constant<int, 16>{}, integral_constant<int, 16>{});
    else if (lanes > 5 || s->G.g >= 64) go(integral_constant<int, 4>{}, integral_constant<int, 16>{});
    else go(integral_constant<int, 1>{}, integral_constant<int, 16>{});
}

// The direct gather with per-host distance histograms (MODE as in
// finish_hosts).  Hosts per workgroup: 1 while the chip has room for a
// workgroup per host, up to 256, or 64 for windows and the network.  Lookups that
// fill the slots of k_sliced_hist on a small pool go there.
template <int W, int MODE>
static void launch_gather(vate_sketch *s, const uint32_t *hosts, uint32_t n, uint32_t kprime, float *est,
                          uint32_t *live, uint32_t *hist, const Windows &win, const void *weights, float *cf,
                          hipStream_t st)
{
    const uint32_t rowp = hist_row_words(s->G.k), row_bytes = rowp * 4u;
    const auto *net = static_cast<const mlp::Packed *>(weights);
    using std::integral_constant;
    constexpr uint32_t fixed = (MODE == kFinLearned ? 10u : 1u) * 1024u;
    const uint32_t bits = 4u * sliced_words(s->G);
    constexpr SlicedUse use = MODE == kFinLearned ? SLICED_LEARNED : MODE == kFinMulti ? SLICED_WINDOWS : SLICED_HIST;
    if (const SlicedShape sh = sliced_shape(s, n, use, row_bytes, s->lds_budget - bits - fixed); sh.P) {
        by_slices(s, sh.P, [&](auto Pv, auto One) {
            constexpr uint32_t P = decltype(Pv)::value;
            constexpr bool one = decltype(One)::value;
            if (!allow_lds<k_sliced_hist<W, MODE, P, one>>(s)) return;
            const uint32_t lds = bits + (row_bytes * kSlicedThreads >> sh.lg);
            k_sliced_hist<W, MODE, P, one><<<grid_for(n, kSlicedThreads >> sh.lg, sliced_cap(s, lds + fixed)),
                                             kSlicedThreads, lds, st>>>(s->G, s->pool, s->st, s->bitmap, hosts, n,
                                                                        sh.lg, rowp, kprime, est, live, hist, win,
                                                                        net, cf);
        });
        return;
    }
    // (the network takes 16 hosts a wavefront: a tile as soon as every CU has one, the
    // last two wavefronts' where each has four and the network outweighs the gathers:
    // 100,000 hosts, 2^28 ATs, k = 7, g = 1000 1731 us with 64 hosts, 1641 with 32)
    constexpr uint32_t room = MODE == kFinLearned ? 2u : 8u, kept = MODE == kFinLearned ? 6u : 4u;
    // More hosts per workgroup, while each CU has six, where a thread then takes no
    // more than two batches of gathers (four where the first-level cache holds the
    // bitmap), or an eighth fewer slots stay empty; and 32 where there are sixteen
    // such workgroups.  (300,000 histograms, k = 60, 2^20 ATs, 16 hosts per workgroup
    // and more: g = 1 65 us and, with 256, 25; g = 64 87 and, with 64, 73; g = 256
    // 245 and, with 32, 248, on 2^14 ATs 116 and 107.)
    constexpr uint32_t most = MODE == kFinClosedForm ? 8u : 6u;
    auto slots = [&](uint32_t lg) {
        const uint32_t batch = kGatherU * (kFinThreads >> lg);
        return (s->G.g + batch - 1u) / batch * batch;
    };
    auto more = [&](uint32_t lg) {
        if ((row_bytes << (lg + 1)) > 32u * 1024u) return false;
        const uint64_t groups = (uint64_t)n >> lg;
        if (lg < kept) return groups > (lg == 5 ? 4u : room) * s->n_cu && (lg < 5 || s->G.g < (s->G.c <= 18 ? 512u : 256u));
        const uint32_t batches = s->G.c <= 18 ? 4u : 2u;
        return (lg == 4 && groups > 16u * s->n_cu) ||
               (groups > 6u * s->n_cu && (batches * kGatherU * (kFinThreads >> (lg + 1)) >= s->G.g ||
                                          8u * slots(lg + 1) <= 7u * slots(lg)));
    };
    uint32_t lg = 0;
    while (lg < most && more(lg)) ++lg;
    if (!allow_lds<k_gather<W, MODE>>(s)) return;
    k_gather<W, MODE><<<grid_for(n, 1u << lg, kMaxGrid256), 256, row_bytes << lg, st>>>(
        s->G, s->pool, s->st, s->bitmap, hosts, n, lg, rowp, kprime, est, live, hist, win, net, cf);
}

// vate_estimate's gather, with or without histograms.
static void direct_estimate(vate_sketch *s, const uint32_t *hosts, uint32_t n, uint32_t kprime, float *est,
                            uint32_t *live, uint32_t *hist, hipStream_t st)
{
    by_width(s->p.width, [&](auto W) {
        constexpr int w = decltype(W)::value;
        if (hist)
            launch_gather<w, kFinClosedForm>(s, hosts, n, kprime, est, live, hist, Windows{}, nullptr, nullptr, st);
        else
            launch_estimate<w>(s, hosts, n, kprime, est, live, st);
    });
}

static void direct_learned(vate_sketch *s, const uint32_t *hosts, uint32_t n, const void *weights, float *est,
                           float *cf, hipStream_t st)
{
    by_width(s->p.width, [&](auto W) {
        launch_gather<decltype(W)::value, kFinLearned>(s, hosts, n, s->p.k, est, nullptr, nullptr, Windows{}, weights,
                                                       cf, st);
    });
}

// ---- partitioned estimate: geometry, workspace layout and launches ----

static uint64_t part_slices(const Geo &G) { return G.N >> std::min(G.c, kSliceLog2); }

// Padded entries of a subgroup, and the distance between subgroups' regions.
static uint64_t part_cap(const Geo &G, uint64_t hosts) { return (hosts * G.g + 3 * part_slices(G) + 3) & ~3ull; }
static uint64_t part_region(const Geo &G, uint64_t hosts) { return (part_cap(G, hosts) + 63) & ~63ull; }

// The scatter's LDS: counters, keys, 32-bit sort slots.
static uint64_t part_lds(const Geo &G, uint64_t hosts)
{
    return 4 * (((part_slices(G) + 3) & ~3ull) + ((hosts + 3) & ~3ull)) + 4 * part_cap(G, hosts);
}

// Hosts per subgroup at most: the largest count whose VATs' pids fit the
// scatter threads' registers (kRunPerThread each), whose padded sort of 32-bit
// entries (+ slice counters, keys) fits its LDS, and whose histograms fit the
// finalize's LDS.  0 where the partitioned path has no geometry for n hosts (g
// VATs of one host too many for one LDS sort, the locality-blocked H, whose
// direct gather already reads whole blocks, or entries past the lookup's 32-bit
// chunk index); the entry points then use the direct gather.
static uint32_t part_max_hosts(const vate_sketch *s, uint64_t n)
{
    const Geo &G = s->G;
    if (G.blog > 0 || part_slices(G) > kRunMaxSlices) return 0;
    uint64_t hosts = kRunMaxHosts;
    hosts = std::min<uint64_t>(hosts, (uint64_t)kRunPerThread * kRunThreads / G.g);
    hosts = std::min<uint64_t>(hosts, kFinHistBytes / (4ull * hist_row_words(G.k)));
    while (hosts > 0 && part_lds(G, hosts) > s->lds_budget) --hosts;
    if (hosts == 0) return 0;
    const uint64_t n_sub = (uint32_t)((n + hosts - 1) / hosts);
    if (n_sub * (part_region(G, hosts) / 4u) >= (1ull << 32)) return 0;
    return (uint32_t)hosts;
}

static size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

struct RunWs {
    uint32_t *entries;          // [n_sub][region] sorted entries
    uint32_t *hits;             // [n_sub][region] live results (host << 16 | distance), packed at the front of each run's slots
    uint32_t *table;            // [n_sub][n_slices + 1] run starts and live counts
    uint32_t *heads;            // [n_sub][n_slices][4] each run's first four live results
    size_t bytes;
};

static RunWs run_ws(const Geo &G, uint64_t n, uint64_t hosts, void *base)
{
    RunWs w;
    const uintptr_t p = reinterpret_cast<uintptr_t>(base);
    const uint64_t ns = part_slices(G), n_sub = (n + hosts - 1) / hosts;
    const size_t ents = (size_t)n_sub * part_region(G, hosts);
    size_t off = 0;
    w.entries = reinterpret_cast<uint32_t *>(p + off);
    off += align256(ents * 4);
    w.hits = reinterpret_cast<uint32_t *>(p + off);
    off += align256(ents * 4);
    w.table = reinterpret_cast<uint32_t *>(p + off);
    off += align256((size_t)n_sub * (ns + 1) * 4);
    w.heads = reinterpret_cast<uint32_t *>(p + off);
    off += align256((size_t)n_sub * ns * 16);
    off += align256((size_t)(G.k + 1) * 8);   // kept in the size, which callers may have stored
    w.bytes = off;
    return w;
}

// The workspace an estimate of n hosts has to be given: the layout with the
// most hosts per subgroup, whichever path is taken (256 bytes where there is no
// partitioned geometry).
static size_t workspace_need(const vate_sketch *s, uint64_t n)
{
    const uint32_t hosts = part_max_hosts(s, n);
    return hosts ? run_ws(s->G, n, hosts, nullptr).bytes : 256;
}

// Hosts per subgroup that leave no scatter workgroup without a subgroup in
// the last round: as many rounds of n_cu subgroups as the largest subgroups
// take, with the hosts spread over all of them.  (20,011 hosts, g = 1024: 742
// subgroups of 27 in three rounds instead of 527 of 38, of which the third
// round had 15.)  It takes a little more workspace (run padding), which a
// caller who kept an older size may not have given.
static uint32_t part_hosts(const vate_sketch *s, uint64_t n, size_t have)
{
    const uint32_t most = part_max_hosts(s, n);
    if (most == 0) return 0;
    const uint64_t n_sub = (n + most - 1) / most, rounds = (n_sub + s->n_cu - 1) / s->n_cu;
    const uint32_t even = (uint32_t)std::max<uint64_t>(1, (n + rounds * s->n_cu - 1) / (rounds * s->n_cu));
    return even < most && run_ws(s->G, n, even, nullptr).bytes <= have ? even : most;
}

// Whether the partitioned lookups answer n hosts.  A direct gather is a read
// through L2 per lookup, 2.5e11 a second while an XCD's 4 MiB L2 holds the
// bitmap (up to 2^25 ATs) and 6.5e10 on a 2^28 pool; partitioned lookups reach
// 3.5e11 and more but take three passes and 25 us at least.  Measured (byte
// ATs, g = 64 .. 1024) they break even at lookups x ATs of about 2^49: 2M
// lookups on 2^28 ATs (36 us each way), 16M on 2^25 (70), 64M on 2^23 (240);
// from 2^27 to 2^26 at half of that.  A plan's runs leave out the first pass:
// half the lookups.  Beyond 2^28 ATs a pass over the bitmap of a larger pool has
// to be earned (k' < k, gathered and partitioned: 2^30 ATs 2M lookups 44 and 77
// us, 6M 119 and 84; 2^32 2M 44 and 616, 64M 1,223 and 1,067), so the number
// doubles with the pool from there.  The closed form for window k, which from 2^26 ATs on is
// gathered by parts, breaks even at 6M to 10M there (8M on 2^28: 51 us by parts,
// 48 partitioned).  On 2^23 ATs it stays with k_sliced, below everything does
// (512M lookups on 2^22: 0.87 of the partitioned time by gathers).
enum PartUse { PART_FORM, PART_HIST, PART_PLANNED };   // the closed form for k; what needs distances; a plan
static bool partitioned(const vate_sketch *s, uint64_t n, PartUse use)
{
    static_assert(kPartLog2 >= kSliceLog2 + 3u, "the lookup gives each of 8 XCDs whole slices");
    if (s->G.c < (use == PART_FORM ? kPartLog2 + 1u : kPartLog2)) return false;
    uint64_t least = s->G.c <= 28 ? kPartMin >> s->G.c : (kPartMin >> 28) << (s->G.c - 28u);
    if (use == PART_FORM) least = std::max(least, kPartFormMin);
    if (use == PART_PLANNED) least /= 2;
    return n * s->G.g >= least && part_max_hosts(s, n) > 0;
}

// The workspace size reported to callers: enough for the even subgroups.
static size_t workspace_size(const vate_sketch *s, uint64_t n)
{
    size_t need = workspace_need(s, n);
    if (partitioned(s, n, PART_PLANNED)) need = std::max(need, run_ws(s->G, n, part_hosts(s, n, ~size_t(0)), nullptr).bytes);
    return need;
}

// The workspace that several windows have to be given (without a partitioned
// geometry, as much as full histograms).
static size_t multi_need(const vate_sketch *s, uint64_t n)
{
    if (part_max_hosts(s, n) > 0) return workspace_need(s, n);
    return align256((size_t)n * (s->p.k + 1) * 4) + align256(8ull * (s->p.k + 1));
}

// The calls with a workspace may put their outputs over the host list: the
// partitioned path writes them when all hosts have been read.  The gathers
// don't, so they get a copy of such a list, in the workspace (which holds 8 g
// bytes per host and more wherever there is a partitioned geometry; where there
// is none, every such call has always gathered).
struct Output {
    const void *p;
    size_t bytes;
};

static const uint32_t *hosts_to_gather(const vate_sketch *s, const uint32_t *hosts, uint32_t n, void *workspace,
                                       std::initializer_list<Output> outputs, hipStream_t st)
{
    const uintptr_t lo = reinterpret_cast<uintptr_t>(hosts), hi = lo + 4ull * n;
    bool over = false;
    for (const Output &o : outputs) {
        const uintptr_t p = reinterpret_cast<uintptr_t>(o.p);
        over |= p != 0 && p < hi && lo < p + o.bytes;
    }
    if (!over || part_max_hosts(s, n) == 0) return hosts;
    k_copy_hosts<<<grid_for(n, 256, 4096), 256, 0, st>>>(hosts, n, static_cast<uint32_t *>(workspace));
    return static_cast<const uint32_t *>(workspace);
}

// The geometry for n hosts, `hosts` per subgroup (from part_hosts); `network`: for
// the learned estimate.
static PartGeo part_geo(const vate_sketch *s, uint64_t n, uint32_t hosts, bool network)
{
    const Geo &G = s->G;
    const uint64_t ns = part_slices(G);
    PartGeo p{};
    p.n_slices = (uint32_t)ns;
    p.rowp = hist_row_words(G.k);
    p.hosts = hosts;
    p.n_sub = (uint32_t)((n + hosts - 1) / hosts);
    p.vats = hosts * G.g;
    p.cap = (uint32_t)part_cap(G, hosts);
    p.region = (uint32_t)part_region(G, hosts);
    p.dq = kRunThreads / G.g;
    p.dr = kRunThreads % G.g;
    p.fast = G.a >= (1ull << kSliceLog2) ? 1u : 0u;
    const uint32_t cus = std::max<uint32_t>(1u, s->n_cu);
    // Subgroups per finalize workgroup, as long as the histograms leave a CU room
    // for three workgroups.  The network takes hosts in tiles of 64, so the count
    // that leaves the fullest CU the fewest tiles (the fewest subgroups on a tie):
    // 300,000 hosts, k = 60, 147 per subgroup: three, 55 KB, take 119 us, two, 36
    // KB, 95; 600,000 hosts, k = 7, 768 subgroups of 782: two each 230 us for the
    // estimate, one 177.  Without it as many as have a thread per host, while
    // each CU has four workgroups (250,000 hosts, k = 16, 38 per subgroup, a slice:
    // 318 us with three, 310 with six).
    {
        uint64_t least = ~0ull;
        for (uint32_t f = 1; f <= 16; ++f) {
            const uint64_t fh = f * hosts, groups = (p.n_sub + f - 1u) / f;
            if (fh * 4ull * p.rowp > (f == 1 ? kFinHistBytes : kFinGroupBytes)) break;
            if (!network && f > 1 && (fh > kFinThreads || groups < 4u * cus)) break;
            const uint64_t tiles = (groups + cus - 1u) / cus * ((fh + 63) / 64);
            if (!network || tiles < least) least = tiles, p.fgroup = f;
        }
    }
    p.lds_scatter = (uint32_t)part_lds(G, hosts);
    {   // lookup LDS: bits, rank tables, run counters, then as many live ATs'
        // distances as fit
        constexpr uint32_t nblk = kBmWordsLds / 8u, nsup = (nblk + 7u) / 8u;
        constexpr uint32_t fixed = 4u * (kBmWordsLds + nsup + (nblk + 1u) / 2u + kRunThreads);
        p.dist16 = G.k > 256 ? 1u : 0u;
        const uint32_t room = s->lds_budget > fixed ? s->lds_budget - fixed : 0u;
        p.dist_cap = room >> p.dist16;
        p.lds_lookup = (fixed + (p.dist_cap << p.dist16) + 15u) & ~15u;
        if (p.lds_lookup > s->lds_budget) p.lds_lookup = s->lds_budget & ~15u, p.dist_cap = (p.lds_lookup - fixed) >> p.dist16;
    }
    p.lds_final = p.fgroup * p.hosts * p.rowp * 4u + 4u;
    // Each slice's walk over the subgroups is cut into ranges, one workgroup
    // each, so that the launch has at least one workgroup per CU (each builds
    // its slice's LDS tables once); a range holds at least one subgroup per
    // wavefront.  The subgroups of a wavefront's window are as many as leave
    // every wavefront of the range a window, 64 at most: with 64 always, the
    // 742 subgroups of 20,011 hosts kept 12 of a workgroup's 16 wavefronts.
    constexpr uint32_t waves = kRunThreads / 64u;
    const uint32_t want = std::max<uint32_t>(1u, std::min<uint32_t>((cus + p.n_slices - 1u) / p.n_slices,
                                                                    p.n_sub / waves));
    const uint32_t range = (p.n_sub + want - 1u) / want;
    p.win = 64;
    while (p.win > 1 && (range + p.win - 1) / p.win < waves) p.win /= 2;
    p.span = (range + p.win - 1u) & ~(p.win - 1u);
    p.split = (p.n_sub + p.span - 1u) / p.span;
    return p;
}

// PART_ALL: scatter, lookup, finalize; PART_PLAN: the scatter only (the
// host plan); PART_RUN: lookup and finalize from an existing plan.
enum PartSteps { PART_ALL = 0, PART_PLAN = 1, PART_RUN = 2 };

template <int W, int MODE>
static int launch_part(vate_sketch *s, const PartGeo &pg, void *ws, const uint32_t *hosts, uint32_t n,
                       uint32_t kprime, float *est, uint32_t *live, uint32_t *hist, const Windows &win,
                       const void *weights, float *cf, hipStream_t st, int steps = PART_ALL)
{
    if (!allow_lds<k_run_scatter>(s) || !allow_lds<k_run_lookup<W, true>>(s) || !allow_lds<k_run_lookup<W, false>>(s) ||
         !allow_lds<k_run_finalize<MODE>>(s))
        return check_launch(s, "dynamic LDS");
    const RunWs w = run_ws(s->G, n, pg.hosts, ws);
    if (steps != PART_RUN)
        k_run_scatter<<<std::min(pg.n_sub, s->n_cu), kRunThreads, pg.lds_scatter, st>>>(s->G, pg, hosts, n, w.entries,
                                                                                       w.table);
    if (steps == PART_PLAN) return VATE_OK;
    auto lookup = [&](auto dists) {
        k_run_lookup<W, decltype(dists)::value><<<pg.n_slices * pg.split, kRunThreads, pg.lds_lookup, st>>>(
            s->G, pg, s->pool, reinterpret_cast<const uint32_t *>(s->bitmap), s->st, w.entries, w.table, w.hits,
            w.heads);
    };
    if (MODE != kFinClosedForm || hist != nullptr || kprime < s->p.k) lookup(std::true_type{});
    else lookup(std::false_type{});
    k_run_finalize<MODE><<<(pg.n_sub + pg.fgroup - 1) / pg.fgroup, kFinThreads, pg.lds_final, st>>>(
        s->G, pg, s->st, n, kprime, w.hits, w.heads, w.table, est, live, hist, win,
        static_cast<const mlp::Packed *>(weights), cf);
    return VATE_OK;
}

template <int MODE>
static int launch_part_w(vate_sketch *s, const PartGeo &pg, void *ws, const uint32_t *hosts, uint32_t n,
                         uint32_t kprime, float *est, uint32_t *live, uint32_t *hist, const Windows &win,
                         const void *weights, float *cf, hipStream_t st, int steps = PART_ALL)
{
    return by_width(s->p.width, [&](auto W) {
        return launch_part<decltype(W)::value, MODE>(s, pg, ws, hosts, n, kprime, est, live, hist, win, weights, cf,
                                                     st, steps);
    });
}

extern "C" {
int vate_estimate_learned_workspace_bytes(const vate_sketch *s, size_t n_hosts, size_t *bytes);

int vate_state_bytes(const vate_params *p, size_t *pool_bytes, size_t *state_bytes)
{
    Geo G;
    const char *why;
    int rc = make_geo(p, &G, &why);
    if (rc != VATE_OK) return rc;
    if (pool_bytes) *pool_bytes = (size_t)(G.N * p->width / 8);
    if (state_bytes) *state_bytes = state_bytes_for(p->k, G.N);
    return VATE_OK;
}

int vate_create(const vate_params *p, void *pool_dev, void *state_dev, void *stream, vate_sketch **out)
{
    if (!out) return VATE_E_INVAL;
    *out = nullptr;
    Geo G;
    const char *why;
    int rc = make_geo(p, &G, &why);
    if (rc != VATE_OK) return rc;
    if (!pool_dev || !state_dev) return VATE_E_INVAL;
    if ((reinterpret_cast<uintptr_t>(pool_dev) & 255u) || (reinterpret_cast<uintptr_t>(state_dev) & 255u))
        return VATE_E_INVAL;
    vate_sketch *s = new (std::nothrow) vate_sketch();
    if (!s) return VATE_E_NOMEM;
    s->p = *p;
    s->G = G;
    s->pool = static_cast<uint8_t *>(pool_dev);
    s->st = static_cast<DevState *>(state_dev);
    s->pool_bytes = (size_t)(G.N * p->width / 8);
    s->state_bytes = state_bytes_for(p->k, G.N);
    s->bitmap = static_cast<uint8_t *>(state_dev) + bitmap_offset(p->k);
    s->copies = reinterpret_cast<unsigned long long *>(static_cast<uint8_t *>(state_dev) + copies_offset(p->k, G.N));
    uint64_t maxb = 0;
    for (uint32_t i = 0; i < G.twok; ++i)
        maxb = std::max<uint64_t>(maxb, block_start(G, i + 1) - block_start(G, i));
    const bool exact = p->width != 4 && p->width != 8 && p->width != 16;
    const uint64_t E = exact ? 32 : 128 / p->width;      // counters per word group / 16-byte chunk
    s->max_block_chunks = (maxb + E - 1) / E + 1;
    {   // LDS a workgroup may use: the largest the device reports (gfx950: 160 KiB)
        int dev = 0, lds = 64 * 1024;
        if (hipGetDevice(&dev) == hipSuccess)
            for (hipDeviceAttribute_t a : {hipDeviceAttributeMaxSharedMemoryPerBlock,
                                           hipDeviceAttributeSharedMemPerBlockOptin,
                                           hipDeviceAttributeMaxSharedMemoryPerMultiprocessor}) {
                int v = 0;
                if (hipDeviceGetAttribute(&v, a, dev) == hipSuccess && v > lds) lds = v;
            }
        s->lds_budget = std::min<uint32_t>((uint32_t)lds, kRunLdsMax) - kRunLdsStatic;
        int cus = 0;
        s->n_cu = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0
                      ? (uint32_t)cus
                      : 256u;
    }
    s->closed = 0;
    s->dead = 0;
    s->err[0] = 0;
    dispatch_init(s, static_cast<hipStream_t>(stream));
    rc = check_launch(s, "init");
    if (rc != VATE_OK) {
        delete s;
        return rc;
    }
    *out = s;
    return VATE_OK;
}

int vate_ingest(vate_sketch *s, const uint32_t *pairs_dev, size_t n, void *stream)
{
    if (!s) return VATE_E_INVAL;
    if (s->dead) return VATE_E_DEVICE;
    if (n > 0 && (!pairs_dev || (reinterpret_cast<uintptr_t>(pairs_dev) & 7u)))
        return fail(s, VATE_E_INVAL, "pairs must be non-NULL and 8-byte aligned");
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (s->closed) {
        int rc = advance(s, st);
        if (rc != VATE_OK) return rc;
    }
    if (n == 0) return VATE_OK;
    by_width(s->p.width, [&](auto W) { launch_ingest<decltype(W)::value>(s, pairs_dev, n, st); });
    return check_launch(s, "ingest");
}

int vate_close_slice(vate_sketch *s, void *stream)
{
    if (!s) return VATE_E_INVAL;
    if (s->dead) return VATE_E_DEVICE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (s->closed) {
        int rc = advance(s, st);
        if (rc != VATE_OK) return rc;
    }
    dispatch_census(s, st);
    int rc = check_launch(s, "census");
    if (rc != VATE_OK) return rc;
    s->closed = 1;
    return VATE_OK;
}

int vate_estimate(vate_sketch *s, const uint32_t *hosts_dev, size_t n_hosts, uint32_t kprime, float *est_dev,
                  uint32_t *live_dev, uint32_t *hist_dev, void *stream)
{
    if (!s) return VATE_E_INVAL;
    if (s->dead) return VATE_E_DEVICE;
    if (!s->closed) return fail(s, VATE_E_STATE, "estimate needs a closed slice (call vate_close_slice)");
    if (kprime < 1 || kprime > s->p.k) return fail(s, VATE_E_INVAL, "k' must be in [1, k]");
    if (n_hosts > 0xFFFFFFFFull - 1024) return fail(s, VATE_E_INVAL, "too many hosts");
    if (hist_dev && s->p.k > (uint32_t)kMaxHistK)
        return fail(s, VATE_E_UNSUPPORTED, "per-host histogram needs k <= 256");
    if (n_hosts == 0) return VATE_OK;
    if (!hosts_dev || !est_dev || (reinterpret_cast<uintptr_t>(hosts_dev) & 3u) ||
        (reinterpret_cast<uintptr_t>(est_dev) & 3u) || (reinterpret_cast<uintptr_t>(live_dev) & 3u) ||
        (reinterpret_cast<uintptr_t>(hist_dev) & 3u))
        return fail(s, VATE_E_INVAL, "hosts/est/live/hist must be non-NULL (live, hist may be NULL) and 4-byte aligned");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const uint32_t n = (uint32_t)n_hosts;
    direct_estimate(s, hosts_dev, n, kprime, est_dev, live_dev, hist_dev, st);
    return check_launch(s, "estimate");
}

int vate_estimate_workspace_bytes(const vate_sketch *s, size_t n_hosts, size_t *bytes)
{
    if (!s || !bytes) return VATE_E_INVAL;
    if (n_hosts > 0xFFFFFFFFull - 1024) return VATE_E_INVAL;
    *bytes = workspace_size(s, n_hosts);
    return VATE_OK;
}

}  // extern "C"

// vate_estimate_ws and vate_estimate_noalloc: the same checks and launches;
// `what` names the entry point in error messages.
static int estimate_ws_impl(vate_sketch *s, const uint32_t *hosts_dev, size_t n_hosts, uint32_t kprime,
                            float *est_dev, uint32_t *live_dev, uint32_t *hist_dev, void *workspace_dev,
                            size_t workspace_bytes, hipStream_t st, const char *what)
{
    if (s->dead) return VATE_E_DEVICE;
    if (!s->closed) return fail(s, VATE_E_STATE, "estimate needs a closed slice (call vate_close_slice)");
    if (kprime < 1 || kprime > s->p.k) return fail(s, VATE_E_INVAL, "k' must be in [1, k]");
    if (n_hosts > 0xFFFFFFFFull - 1024) return fail(s, VATE_E_INVAL, "too many hosts");
    if (n_hosts == 0) return VATE_OK;
    if (!workspace_dev || workspace_bytes < workspace_need(s, n_hosts) || (reinterpret_cast<uintptr_t>(workspace_dev) & 255u))
        return fail(s, VATE_E_INVAL, "workspace missing, too small or not 256-byte aligned");
    if (!hosts_dev || !est_dev || (reinterpret_cast<uintptr_t>(hosts_dev) & 3u) ||
        (reinterpret_cast<uintptr_t>(est_dev) & 3u) || (reinterpret_cast<uintptr_t>(live_dev) & 3u) ||
        (reinterpret_cast<uintptr_t>(hist_dev) & 3u))
        return fail(s, VATE_E_INVAL, "hosts/est/live/hist must be non-NULL (live, hist may be NULL) and 4-byte aligned");
    const uint32_t n = (uint32_t)n_hosts;
    if (workspace_dev == s->plan_ws) s->plan_ws = nullptr;   // the plan is overwritten
    if (hist_dev && s->p.k > (uint32_t)kMaxHistK && part_max_hosts(s, n) == 0)
        return fail(s, VATE_E_UNSUPPORTED, "per-host histogram of this geometry needs k <= 256");
    if (!partitioned(s, n, hist_dev || kprime < s->p.k ? PART_HIST : PART_FORM)) {
        const uint32_t *hosts = hosts_to_gather(s, hosts_dev, n, workspace_dev, {{est_dev, 4ull * n}, {live_dev, 4ull * n},
                                                {hist_dev, 4ull * n * (s->p.k + 1)}}, st);
        direct_estimate(s, hosts, n, kprime, est_dev, live_dev, hist_dev, st);
        return check_launch(s, what);
    }
    const PartGeo pg = part_geo(s, n, part_hosts(s, n, workspace_bytes), false);
    const int rc = launch_part_w<kFinClosedForm>(s, pg, workspace_dev, hosts_dev, n, kprime, est_dev, live_dev,
                                                 hist_dev, Windows{}, nullptr, nullptr, st);
    if (rc != VATE_OK) return rc;
    return check_launch(s, what);
}

// Workspace of vate_estimate_noalloc: a fixed array in device memory.  Each
// GPU the library runs on holds its own copy from module load until the
// process ends.  Host code never uses the array's name as a device address
// (on the host it names a stand-in): the address is looked up once per
// device with hipGetSymbolAddress, and that pointer is what the launches get.
static __device__ __align__(256) uint8_t scratch[VATE_NOALLOC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
static std::atomic<void *> g_scratch_dev[kMaxDevices];

// Device address of the current device's scratch array (looked up on the
// first call per device), or null with the HIP error in *err.
static void *scratch_address(hipError_t *err)
{
    int dev = 0;
    *err = hipGetDevice(&dev);
    if (*err != hipSuccess) return nullptr;
    if (dev < 0 || dev >= kMaxDevices) {
        *err = hipErrorInvalidDevice;
        return nullptr;
    }
    void *p = g_scratch_dev[dev].load(std::memory_order_acquire);
    if (p) return p;
    *err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (*err != hipSuccess) return nullptr;
    g_scratch_dev[dev].store(p, std::memory_order_release);
    return p;
}

extern "C" {
int vate_estimate_ws(vate_sketch *s, const uint32_t *hosts_dev, size_t n_hosts, uint32_t kprime, float *est_dev,
                     uint32_t *live_dev, uint32_t *hist_dev, void *workspace_dev, size_t workspace_bytes,
                     void *stream)
{
    if (!s) return VATE_E_INVAL;
    return estimate_ws_impl(s, hosts_dev, n_hosts, kprime, est_dev, live_dev, hist_dev, workspace_dev,
                            workspace_bytes, static_cast<hipStream_t>(stream), "estimate_ws");
}

int vate_estimate_noalloc(vate_sketch *s, const uint32_t *hosts_dev, size_t n_hosts, uint32_t kprime,
                          float *est_dev, uint32_t *live_dev, uint32_t *hist_dev, void *stream)
{
    if (!s) return VATE_E_INVAL;
    if (s->dead) return VATE_E_DEVICE;
    if (n_hosts > 0xFFFFFFFFull - 1024) return fail(s, VATE_E_INVAL, "too many hosts");
    const size_t need = workspace_need(s, n_hosts);
    if (need > VATE_NOALLOC_SCRATCH_BYTES) {
        char buf[200];
        snprintf(buf, sizeof(buf), "estimate_noalloc: %zu hosts need %zu bytes of workspace, more than the %u of the "
                 "fixed scratch (use vate_estimate_ws)", n_hosts, need, (unsigned)VATE_NOALLOC_SCRATCH_BYTES);
        return fail(s, VATE_E_INVAL, buf);
    }
    hipError_t e = hipSuccess;
    void *ws = scratch_address(&e);
    if (!ws) return fail(s, VATE_E_DEVICE, hipGetErrorString(e));
    return estimate_ws_impl(s, hosts_dev, n_hosts, kprime, est_dev, live_dev, hist_dev, ws,
                            VATE_NOALLOC_SCRATCH_BYTES, static_cast<hipStream_t>(stream), "estimate_noalloc");
}

int vate_estimate_plan(vate_sketch *s, const uint32_t *hosts_dev, size_t n_hosts, void *workspace_dev,
                       size_t workspace_bytes, void *stream)
{
    if (!s) return VATE_E_INVAL;
    if (s->dead) return VATE_E_DEVICE;
    if (n_hosts == 0 || n_hosts > 0xFFFFFFFFull - 1024) return fail(s, VATE_E_INVAL, "need 1 .. 2^32-1025 hosts");
    if (part_max_hosts(s, n_hosts) == 0)
        return fail(s, VATE_E_UNSUPPORTED, "no partitioned plan for this sketch (use vate_estimate)");
    if (!workspace_dev || workspace_bytes < workspace_need(s, n_hosts) ||
        (reinterpret_cast<uintptr_t>(workspace_dev) & 255u))
        return fail(s, VATE_E_INVAL, "workspace missing, too small or not 256-byte aligned");
    if (!hosts_dev || (reinterpret_cast<uintptr_t>(hosts_dev) & 3u))
        return fail(s, VATE_E_INVAL, "hosts must be non-NULL and 4-byte aligned");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const uint32_t n = (uint32_t)n_hosts;
    if (partitioned(s, n, PART_PLANNED)) {
        const PartGeo pg = part_geo(s, n, part_hosts(s, n, workspace_bytes), false);
        const int rc = launch_part_w<kFinClosedForm>(s, pg, workspace_dev, hosts_dev, n, s->p.k, nullptr, nullptr,
                                                     nullptr, Windows{}, nullptr, nullptr, st, PART_PLAN);
        if (rc != VATE_OK) return rc;
        s->plan_hosts = pg.hosts;
    } else {
        // the runs gather directly: they need the hosts alone (4 of the
        // workspace's 8 g or more bytes per host)
        k_copy_hosts<<<grid_for(n, 256, 4096), 256, 0, st>>>(hosts_dev, n, static_cast<uint32_t *>(workspace_dev));
        s->plan_hosts = 0;
    }
    s->plan_ws = workspace_dev;
    s->plan_n = n_hosts;
    return check_launch(s, "estimate_plan");
}

// A run needs a closed slice and the plan made for this workspace and host count.
static int check_plan(vate_sketch *s, size_t n_hosts, const void *workspace_dev, size_t workspace_bytes)
{
    if (s->dead) return VATE_E_DEVICE;
    if (!s->closed) return fail(s, VATE_E_STATE, "estimate needs a closed slice (call vate_close_slice)");
    if (!workspace_dev || workspace_dev != s->plan_ws || n_hosts != s->plan_n)
        return fail(s, VATE_E_STATE, "no plan for this workspace and host count (call vate_estimate_plan)");
    // (a plan of even subgroups takes more than the least that a plan may be given)
    const size_t need = s->plan_hosts ? run_ws(s->G, n_hosts, s->plan_hosts, nullptr).bytes : workspace_need(s, n_hosts);
    if (workspace_bytes < need) return fail(s, VATE_E_INVAL, "workspace too small");
    return VATE_OK;
}

int vate_estimate_run(vate_sketch *s, size_t n_hosts, uint32_t kprime, float *est_dev, uint32_t *live_dev,
                      uint32_t *hist_dev, void *workspace_dev, size_t workspace_bytes, void *stream)
{
    if (!s) return VATE_E_INVAL;
    if (kprime < 1 || kprime > s->p.k) return fail(s, VATE_E_INVAL, "k' must be in [1, k]");
    int rc = check_plan(s, n_hosts, workspace_dev, workspace_bytes);
    if (rc != VATE_OK) return rc;
    if (!est_dev || (reinterpret_cast<uintptr_t>(est_dev) & 3u) || (reinterpret_cast<uintptr_t>(live_dev) & 3u) ||
        (reinterpret_cast<uintptr_t>(hist_dev) & 3u))
        return fail(s, VATE_E_INVAL, "est/live/hist must be 4-byte aligned, est non-NULL");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const uint32_t n = (uint32_t)n_hosts;
    if (s->plan_hosts == 0) {
        direct_estimate(s, static_cast<const uint32_t *>(workspace_dev), n, kprime, est_dev, live_dev, hist_dev, st);
        return check_launch(s, "estimate_run");
    }
    rc = launch_part_w<kFinClosedForm>(s, part_geo(s, n, s->plan_hosts, false), workspace_dev, nullptr, n, kprime, est_dev,
                                       live_dev, hist_dev, Windows{}, nullptr, nullptr, st, PART_RUN);
    if (rc != VATE_OK) return rc;
    return check_launch(s, "estimate_run");
}

int vate_estimate_learned_run(vate_sketch *s, size_t n_hosts, const void *weights_dev, float *est_dev,
                              float *est_cf_dev, void *workspace_dev, size_t workspace_bytes, void *stream)
{
    if (!s) return VATE_E_INVAL;
    if (s->p.k > (uint32_t)kLearnMaxK) return fail(s, VATE_E_UNSUPPORTED, "learned estimator needs k + 3 <= 64");
    int rc = check_plan(s, n_hosts, workspace_dev, workspace_bytes);
    if (rc != VATE_OK) return rc;
    if (!est_dev || !est_cf_dev || !weights_dev || (reinterpret_cast<uintptr_t>(est_dev) & 3u) ||
        (reinterpret_cast<uintptr_t>(est_cf_dev) & 3u) || (reinterpret_cast<uintptr_t>(weights_dev) & 255u))
        return fail(s, VATE_E_INVAL, "est/est_cf must be 4-byte and weights 256-byte aligned, non-NULL");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const uint32_t n = (uint32_t)n_hosts;
    if (s->plan_hosts == 0) {
        direct_learned(s, static_cast<const uint32_t *>(workspace_dev), n, weights_dev, est_dev, est_cf_dev, st);
        return check_launch(s, "estimate_learned_run");
    }
    rc = launch_part_w<kFinLearned>(s, part_geo(s, n, s->plan_hosts, true), workspace_dev, nullptr, n, s->p.k, est_dev,
                                    nullptr, nullptr, Windows{}, weights_dev, est_cf_dev, st, PART_RUN);
    if (rc != VATE_OK) return rc;
    return check_launch(s, "estimate_learned_run");
}

int vate_estimate_learned_ws(vate_sketch *s, const uint32_t *hosts_dev, size_t n_hosts, const void *weights_dev,
                             float *est_dev, float *est_cf_dev, void *workspace_dev, size_t workspace_bytes,
                             void *stream)
{
    if (!s) return VATE_E_INVAL;
    if (s->dead) return VATE_E_DEVICE;
    if (!s->closed) return fail(s, VATE_E_STATE, "estimate needs a closed slice (call vate_close_slice)");
    if (s->p.k > (uint32_t)kLearnMaxK) return fail(s, VATE_E_UNSUPPORTED, "learned estimator needs k + 3 <= 64");
    if (n_hosts > 0xFFFFFFFFull - 1024) return fail(s, VATE_E_INVAL, "too many hosts");
    if (n_hosts == 0) return VATE_OK;
    if (!workspace_dev || workspace_bytes < workspace_need(s, n_hosts) || (reinterpret_cast<uintptr_t>(workspace_dev) & 255u))
        return fail(s, VATE_E_INVAL, "workspace missing, too small or not 256-byte aligned");
    if (!hosts_dev || !est_dev || !est_cf_dev || !weights_dev || (reinterpret_cast<uintptr_t>(hosts_dev) & 3u) ||
        (reinterpret_cast<uintptr_t>(est_dev) & 3u) || (reinterpret_cast<uintptr_t>(est_cf_dev) & 3u) ||
        (reinterpret_cast<uintptr_t>(weights_dev) & 255u))
        return fail(s, VATE_E_INVAL, "hosts/est/est_cf must be 4-byte and weights 256-byte aligned, non-NULL");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const uint32_t n = (uint32_t)n_hosts;
    if (workspace_dev == s->plan_ws) s->plan_ws = nullptr;   // the plan is overwritten
    if (!partitioned(s, n, PART_HIST)) {
        const uint32_t *hosts = hosts_to_gather(s, hosts_dev, n, workspace_dev,
                                                {{est_dev, 4ull * n}, {est_cf_dev, 4ull * n}}, st);
        direct_learned(s, hosts, n, weights_dev, est_dev, est_cf_dev, st);
        return check_launch(s, "estimate_learned_ws");
    }
    const PartGeo pg = part_geo(s, n, part_hosts(s, n, workspace_bytes), true);
    const int rc = launch_part_w<kFinLearned>(s, pg, workspace_dev, hosts_dev, n, s->p.k, est_dev, nullptr, nullptr,
                                              Windows{}, weights_dev, est_cf_dev, st);
    if (rc != VATE_OK) return rc;
    return check_launch(s, "estimate_learned_ws");
}

int vate_estimate_multi_workspace_bytes(const vate_sketch *s, size_t n_hosts, size_t *bytes)
{
    if (!s || !bytes) return VATE_E_INVAL;
    if (n_hosts > 0xFFFFFFFFull - 1024) return VATE_E_INVAL;
    *bytes = multi_need(s, n_hosts);
    if (partitioned(s, n_hosts, PART_PLANNED)) *bytes = std::max(*bytes, workspace_size(s, n_hosts));
    return VATE_OK;
}

int vate_estimate_multi_ws(vate_sketch *s, const uint32_t *hosts_dev, size_t n_hosts, const uint32_t *kprimes,
                           uint32_t m, float *est_dev, void *workspace_dev, size_t workspace_bytes, void *stream)
{
    if (!s) return VATE_E_INVAL;
    if (s->dead) return VATE_E_DEVICE;
    if (!s->closed) return fail(s, VATE_E_STATE, "estimate needs a closed slice (call vate_close_slice)");
    if (!kprimes || m < 1 || m > kMaxWindows) return fail(s, VATE_E_INVAL, "need 1..64 windows");
    Windows win;
    win.m = m;
    for (uint32_t j = 0; j < m; ++j) {
        if (kprimes[j] < 1 || kprimes[j] > s->p.k || (j > 0 && kprimes[j] <= kprimes[j - 1]))
            return fail(s, VATE_E_INVAL, "windows must be ascending, distinct and in [1, k]");
        win.kp[j] = kprimes[j];
    }
    if (n_hosts > 0xFFFFFFFFull - 1024) return fail(s, VATE_E_INVAL, "too many hosts");
    if (n_hosts == 0) return VATE_OK;
    if (!workspace_dev || workspace_bytes < multi_need(s, n_hosts) || (reinterpret_cast<uintptr_t>(workspace_dev) & 255u))
        return fail(s, VATE_E_INVAL, "workspace missing, too small or not 256-byte aligned");
    if (!hosts_dev || !est_dev || (reinterpret_cast<uintptr_t>(hosts_dev) & 3u) ||
        (reinterpret_cast<uintptr_t>(est_dev) & 3u))
        return fail(s, VATE_E_INVAL, "hosts/est must be non-NULL and 4-byte aligned");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const uint32_t n = (uint32_t)n_hosts;
    if (workspace_dev == s->plan_ws) s->plan_ws = nullptr;   // the plan is overwritten
    if (s->p.k > (uint32_t)kMaxHistK && part_max_hosts(s, n) == 0)
        return fail(s, VATE_E_UNSUPPORTED, "several windows for this geometry need k <= 256");
    if (partitioned(s, n, PART_HIST)) {
        const PartGeo pg = part_geo(s, n, part_hosts(s, n, workspace_bytes), false);
        const int rc = launch_part_w<kFinMulti>(s, pg, workspace_dev, hosts_dev, n, s->p.k, est_dev, nullptr,
                                                nullptr, win, nullptr, nullptr, st);
        if (rc != VATE_OK) return rc;
        return check_launch(s, "estimate_multi_ws");
    }
    const uint32_t *hosts = hosts_to_gather(s, hosts_dev, n, workspace_dev, {{est_dev, 4ull * n * m}}, st);
    by_width(s->p.width, [&](auto W) {
        launch_gather<decltype(W)::value, kFinMulti>(s, hosts, n, s->p.k, est_dev, nullptr, nullptr, win, nullptr,
                                                     nullptr, st);
    });
    return check_launch(s, "estimate_multi_ws");
}

int vate_estimate_learned_workspace_bytes(const vate_sketch *s, size_t n_hosts, size_t *bytes)
{
    if (!s || !bytes) return VATE_E_INVAL;
    if (n_hosts > 0xFFFFFFFFull - 1024) return VATE_E_INVAL;
    *bytes = workspace_size(s, n_hosts);
    return VATE_OK;
}

int vate_estimate_learned(vate_sketch *s, const uint32_t *hosts_dev, size_t n_hosts, const void *weights_dev,
                          float *est_dev, float *est_cf_dev, void *stream)
{
    if (!s) return VATE_E_INVAL;
    if (s->dead) return VATE_E_DEVICE;
    if (!s->closed) return fail(s, VATE_E_STATE, "estimate needs a closed slice (call vate_close_slice)");
    if (s->p.k > (uint32_t)kLearnMaxK) return fail(s, VATE_E_UNSUPPORTED, "learned estimator needs k + 3 <= 64");
    if (n_hosts > 0xFFFFFFFFull - 1024) return fail(s, VATE_E_INVAL, "too many hosts");
    if (n_hosts == 0) return VATE_OK;
    if (!hosts_dev || !est_dev || !est_cf_dev || !weights_dev || (reinterpret_cast<uintptr_t>(hosts_dev) & 3u) ||
        (reinterpret_cast<uintptr_t>(est_dev) & 3u) || (reinterpret_cast<uintptr_t>(est_cf_dev) & 3u) ||
        (reinterpret_cast<uintptr_t>(weights_dev) & 255u))
        return fail(s, VATE_E_INVAL, "hosts/est/est_cf must be 4-byte and weights 256-byte aligned, non-NULL");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const uint32_t n = (uint32_t)n_hosts;
    direct_learned(s, hosts_dev, n, weights_dev, est_dev, est_cf_dev, st);
    return check_launch(s, "estimate_learned");
}

int vate_read_census(vate_sketch *s, uint64_t *census_host, void *stream)
{
    if (!s || !census_host) return VATE_E_INVAL;
    if (s->dead) return VATE_E_DEVICE;
    if (!s->closed) return fail(s, VATE_E_STATE, "census needs a closed slice");
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipError_t e = hipStreamSynchronize(st);
    if (e == hipSuccess)
        e = hipMemcpy(census_host, census_of(s->st), 8ull * s->p.k, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return fail(s, VATE_E_DEVICE, hipGetErrorString(e));
    uint64_t act = 0;
    for (uint32_t d = 0; d < s->p.k; ++d) act += census_host[d];
    census_host[s->p.k] = s->G.N - act;
    return VATE_OK;
}

int vate_read_state(vate_sketch *s, void *pool_dst, uint64_t *t, uint32_t *bact0, int *closed, void *stream)
{
    if (!s) return VATE_E_INVAL;
    if (s->dead) return VATE_E_DEVICE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipError_t e = hipStreamSynchronize(st);
    DevState hdr;
    if (e == hipSuccess && pool_dst) e = hipMemcpy(pool_dst, s->pool, s->pool_bytes, hipMemcpyDefault);
    if (e == hipSuccess) e = hipMemcpy(&hdr, s->st, kStateHeader, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return fail(s, VATE_E_DEVICE, hipGetErrorString(e));
    if (t) *t = hdr.t;
    if (bact0) *bact0 = hdr.bact0;
    if (closed) *closed = s->closed;
    return VATE_OK;
}

int vate_load_state(vate_sketch *s, const void *pool_src, uint64_t t, uint32_t bact0, int closed, void *stream)
{
    if (!s || !pool_src) return VATE_E_INVAL;
    if (s->dead) return VATE_E_DEVICE;
    if (bact0 >= s->G.twok) return fail(s, VATE_E_INVAL, "bact0 must be < 2k");
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipError_t e = hipMemcpyAsync(s->pool, pool_src, s->pool_bytes, hipMemcpyDefault, st);
    if (e != hipSuccess) return fail(s, VATE_E_DEVICE, hipGetErrorString(e));
    k_set_clock<<<1, 256, 0, st>>>(s->G, s->st, (unsigned long long)t, bact0);
    int rc = check_launch(s, "load_state");
    if (rc != VATE_OK) return rc;
    s->closed = 0;
    if (closed) {
        dispatch_census(s, st);
        rc = check_launch(s, "census");
        if (rc != VATE_OK) return rc;
        s->closed = 1;
    }
    return VATE_OK;
}

const char *vate_last_error(const vate_sketch *s)
{
    return s ? s->err : "";
}

const char *vate_status_string(int code)
{
    switch (code) {
    case VATE_OK: return "ok";
    case VATE_E_INVAL: return "invalid argument";
    case VATE_E_STATE: return "call not allowed in the current slice phase";
    case VATE_E_DEVICE: return "HIP device error";
    case VATE_E_NOMEM: return "out of host memory";
    case VATE_E_UNSUPPORTED: return "unsupported request";
    default: return "unknown status";
    }
}

void vate_destroy(vate_sketch *s)
{
    delete s;
}

uint32_t vate_host_hash(const vate_params *p, uint32_t which, uint32_t x, uint32_t i)
{
    Geo G;
    const char *why;
    if (make_geo(p, &G, &why) != VATE_OK) return 0xFFFFFFFFu;
    if (which == 0) return bh(G, x);
    if (which == 1) return vat_pid(G, host_key(G, x), i);
    return 0xFFFFFFFFu;
}

uint32_t vate_host_block(const vate_params *p, uint64_t pid)
{
    Geo G;
    const char *why;
    if (make_geo(p, &G, &why) != VATE_OK || pid >= G.N) return 0xFFFFFFFFu;
    return block_of(G, (uint32_t)pid);
}

}  // extern "C"

#include "vate_batch_api.h"
