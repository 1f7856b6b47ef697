// Exact-width counters: an AT of ceil(log2(2k+1)) bits (a DR of
// ceil(log2(k+1)) bits) packed back to back, as the paper sizes its pool
// (Sec. 3: 2k+1 values per AT; Sec. 5: 10-bit ATs at k = 300).  Counter p
// sits at bits [p w, (p+1) w) of the pool read as little-endian 32-bit words,
// so a group of 32 counters fills exactly w words and starts on a word.
// Included into vate.hip inside namespace vate; single counters are read and
// set with the width w = G.wb at run time (template width 0 of the lookups).
//
// Streaming kernels (census, preservation, DR maintenance) give each thread
// whole groups, read and where counters change written back by kernels with
// the width at compile time; init and the batched kernels, which meet any mix
// of widths, go through a 64-bit bit buffer (template width 0).
// SetAT writes the w bits of one counter, which may straddle two words, with
// a compare-and-swap on each word that does not hold them yet: the bits of
// neighbouring counters are never changed, and every writer of a counter
// within a slice writes the same value, so the counter ends at that value
// under any interleaving.

__device__ __forceinline__ uint32_t low_mask(uint32_t w) { return w >= 32 ? ~0u : (1u << w) - 1u; }

// Value of counter pid from 32-bit words (global or LDS).
__device__ __forceinline__ uint32_t load_x(const uint32_t *__restrict__ words, uint64_t pid, uint32_t wb)
{
    const uint64_t o = pid * wb;
    const uint32_t *p = words + (o >> 5);
    const uint32_t sh = (uint32_t)o & 31u;
    uint32_t v = p[0] >> sh;
    if (sh + wb > 32) v |= p[1] << (32 - sh);
    return v & low_mask(wb);
}

// SetAT on the bits that one 32-bit word holds of a counter (mask m, value v
// in place).  Every writer of a slice writes the same value, so a word whose
// bits already equal it needs no write: the word is read first (a load that
// passes L1 by, so that a hot counter set by another CU is seen as set; a
// stale word only costs a needless exchange), and one compare-and-swap then
// sets it.  A failed swap returns the word as another writer left it; a
// counter changes once per slice, so at most as many swaps fail as the word
// holds counters.
__device__ __forceinline__ void set_bits(uint32_t *__restrict__ p, uint32_t m, uint32_t v)
{
    uint32_t old = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    while ((old & m) != v) {
        const uint32_t got = atomicCAS(p, old, (old & ~m) | v);
        if (got == old) break;
        old = got;
    }
}

// The same without a look at the word, by two atomics that nothing waits for:
// every interleaving of a slice's writers, who all bring v, ends at v.
__device__ __forceinline__ void put_bits(uint32_t *__restrict__ p, uint32_t m, uint32_t v)
{
    atomicOr(p, v);
    atomicAnd(p, ~m | v);
}

__device__ __forceinline__ void set_x(uint32_t *__restrict__ words, uint64_t pid, uint32_t wb, uint32_t val, bool crowded)
{
    const uint64_t o = pid * wb;
    uint32_t *p = words + (o >> 5);
    const uint32_t sh = (uint32_t)o & 31u;
    const uint32_t n0 = min(wb, 32u - sh);             // bits in the first word
    const uint32_t m0 = low_mask(n0);
    if (crowded) {
        put_bits(p, m0 << sh, (val & m0) << sh);
        if (n0 < wb) put_bits(p + 1, low_mask(wb - n0), val >> n0);
    } else {
        set_bits(p, m0 << sh, (val & m0) << sh);
        if (n0 < wb) set_bits(p + 1, low_mask(wb - n0), val >> n0);
    }
}

// The 32 counters of a group (its wb words in order).  WB: the width at
// compile time, so that every shift is a constant and the words are loaded up
// to 16 bytes at a time (4-byte aligned); WB = 0: any width, through a bit
// buffer.
template <int WB>
__device__ __forceinline__ void read_group(const uint32_t *__restrict__ src, uint32_t wb, uint32_t vals[32])
{
    if constexpr (WB > 0) {
        uint32_t w[WB];
        __builtin_memcpy(w, src, sizeof w);
        constexpr uint32_t m = (1u << WB) - 1u;
#pragma unroll
        for (int e = 0; e < 32; ++e) {
            const int o = e * WB, i = o >> 5, sh = o & 31;
            vals[e] = (sh + WB <= 32 ? w[i] >> sh : __builtin_amdgcn_alignbit(w[(i + 1) % WB], w[i], sh)) & m;
        }
    } else {
        uint64_t buf = 0;
        uint32_t have = 0;
        const uint32_t m = low_mask(wb);
#pragma unroll
        for (int e = 0; e < 32; ++e) {
            if (have < wb) {
                buf |= (uint64_t)(*src++) << have;
                have += 32;
            }
            vals[e] = (uint32_t)buf & m;
            buf >>= wb;
            have -= wb;
        }
    }
}

template <int WB>
__device__ __forceinline__ void write_group(uint32_t *__restrict__ dst, uint32_t wb, const uint32_t vals[32])
{
    if constexpr (WB > 0) {
        uint32_t w[WB] = {};
#pragma unroll
        for (int e = 0; e < 32; ++e) {
            const int o = e * WB, i = o >> 5, sh = o & 31;
            w[i] |= vals[e] << sh;
            if (sh + WB > 32) w[(i + 1) % WB] |= vals[e] >> ((32 - sh) & 31);
        }
        __builtin_memcpy(dst, w, sizeof w);
    } else {
        uint64_t buf = 0;
        uint32_t have = 0;
#pragma unroll
        for (int e = 0; e < 32; ++e) {
            buf |= (uint64_t)vals[e] << have;
            have += wb;
            if (have >= 32) {
                *dst++ = (uint32_t)buf;
                buf >>= 32;
                have -= 32;
            }
        }
    }
}

// InitAT on every counter, clock and census reset.
__global__ void __launch_bounds__(256) k_init_x(Geo G, uint32_t *__restrict__ pool32, uint64_t ngroups,
                                                DevState *__restrict__ st, unsigned long long *__restrict__ copies)
{
    uint32_t vals[32];
#pragma unroll
    for (int e = 0; e < 32; ++e) vals[e] = inactive_value(G);
    for (uint64_t gi = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; gi < ngroups;
         gi += (uint64_t)gridDim.x * blockDim.x)
        write_group<0>(pool32 + gi * G.wb, G.wb, vals);
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

// Census of group gi and its activity bitmap word: distances below k are
// counted into hist (LDS) when given, else into the census.  A group inside
// one block (nearly all of them) has one ACT: its counters are tested without
// a branch, and only the active ones take the histogram's LDS atomic.
template <int WB>
__device__ __forceinline__ void census_group_x(const Geo &G, const uint32_t *__restrict__ pool32, uint64_t gi,
                                               uint32_t bact0, uint32_t *hist, unsigned long long *census,
                                               uint8_t *__restrict__ bitmap)
{
    const uint32_t inact = inactive_value(G);
    uint32_t vals[32];
    read_group<WB>(pool32 + gi * G.wb, G.wb, vals);
    const uint64_t p0 = gi * 32;
    uint32_t bid0 = 0, act0 = 0;
    uint64_t next = 0;
    bool one = G.dr != 0;
    if (G.fast_blocks && !G.dr) {
        bid0 = block_of(G, (uint32_t)p0);
        act0 = block_act(G, bact0, bid0);
        next = block_start(G, bid0 + 1);
        one = p0 + 32 <= next;
    }
    uint32_t bits = 0;
    if (WB > 0 && one && hist) {     // (the batched kernels keep their registers for the container widths)
        const uint32_t top = act0 + G.twok;
#pragma unroll
        for (int e = 0; e < 32; ++e) {
            const uint32_t u = top - vals[e];                       // ACT + 2k - value
            // (one bit holds no AT; the second of the minimum wraps when u < 2k)
            const uint32_t d = WB == 1 || G.dr ? vals[e] : min(u, u - G.twok);
            if (vals[e] != inact && d < G.k) {
                bits |= 1u << e;
                atomicAdd(&hist[d], 1u);
            }
        }
    } else {
#pragma unroll
        for (int e = 0; e < 32; ++e) {
            const uint32_t val = vals[e];
            if (val == inact) continue;
            uint32_t d;
            if (G.dr) {
                d = val;
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
    }
    reinterpret_cast<uint32_t *>(bitmap)[gi] = bits;
}

// Census and activity bitmap (one bitmap word per group).  Bound by its
// instructions: with a group's shifts and word indexes known at compile time
// 2^27 10-bit ATs of steady traffic (k = 300, 168 MB) take 44 us instead of
// 158, 2^28 9-bit DRs (302 MB) 81 instead of 196.
template <int WB>
__global__ void __launch_bounds__(256) k_census_x(Geo G, const uint32_t *__restrict__ pool32, uint64_t ngroups,
                                                  DevState *__restrict__ st, uint8_t *__restrict__ bitmap,
                                                  unsigned long long *__restrict__ copies, bool direct)
{
    __shared__ uint32_t hist[kCensusLdsBins];
    const bool lds = G.k <= kCensusLdsBins;
    if (lds)
        for (uint32_t d = threadIdx.x; d < G.k; d += blockDim.x) hist[d] = 0;
    __syncthreads();
    const uint32_t bact0 = st->bact0;
    for (uint64_t gi = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; gi < ngroups;
         gi += (uint64_t)gridDim.x * blockDim.x)
        census_group_x<WB>(G, pool32, gi, bact0, lds ? hist : nullptr, census_of(st), bitmap);
    __syncthreads();
    if (lds) census_flush(G, st, hist, copies, direct);
}

// Alg. 3 on the two blocks whose ACT is 0 or k; thread j < max_groups takes
// a group of the first block, the rest groups of the second (a group in both
// ranges is handled once, by the first).
template <int WB>
__device__ __forceinline__ void preserve_group_x(const Geo &G, uint32_t *__restrict__ pool32, uint32_t bact0,
                                                 uint64_t j, uint64_t max_groups)
{
    const uint32_t i0 = bact0 == 0 ? 0 : G.twok - bact0;                        // (BACT^0 + i0) mod 2k == 0
    const uint32_t i1 = bact0 <= G.k ? G.k - bact0 : G.twok + G.k - bact0;      // == k
    const uint64_t s0 = block_start(G, i0), e0 = block_start(G, i0 + 1);
    const uint64_t s1 = block_start(G, i1), e1 = block_start(G, i1 + 1);
    const uint64_t g0lo = s0 / 32, g0hi = s0 < e0 ? (e0 + 31) / 32 : g0lo;
    const uint64_t g1lo = s1 / 32, g1hi = s1 < e1 ? (e1 + 31) / 32 : g1lo;
    if (j >= 2 * max_groups) return;
    const bool second = j >= max_groups;
    const uint64_t gi = second ? g1lo + (j - max_groups) : g0lo + j;
    if (gi >= (second ? g1hi : g0hi)) return;
    if (second && gi >= g0lo && gi < g0hi) return;
    uint32_t *words = pool32 + gi * G.wb;
    uint32_t vals[32];
    read_group<WB>(words, G.wb, vals);
    bool changed = false;
#pragma unroll
    for (int e = 0; e < 32; ++e) {
        const uint64_t p = gi * 32 + e;
        const bool in0 = p >= s0 && p < e0, in1 = p >= s1 && p < e1;
        if (!in0 && !in1) continue;
        const uint32_t val = vals[e];
        bool mark;
        if (in0)   // ACT == 0: 0 <= Value <= k
            mark = val <= G.k;
        else       // ACT == k: k <= Value <= 2k-1, or Value == 0
            mark = (val >= G.k && val <= G.twok - 1) || val == 0;
        if (mark && val != G.twok) {
            vals[e] = G.twok;
            changed = true;
        }
    }
    if (changed) write_group<WB>(words, G.wb, vals);
}

template <int WB>
__global__ void __launch_bounds__(256) k_preserve_x(Geo G, uint32_t *__restrict__ pool32, DevState *st,
                                                    uint64_t max_groups, bool ends)
{
    const uint32_t bact0 = ends ? next_bact0(G, st->bact0) : st->bact0;
    for (uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; j < 2 * max_groups;
         j += (uint64_t)gridDim.x * blockDim.x)
        preserve_group_x<WB>(G, pool32, bact0, j, max_groups);
    if (ends && last_workgroup(&st->ticket)) advance_clock(G, st);
}

// DR maintenance: every counter of group gi grows by one, saturating at k
// (2^28 9-bit DRs, 302 MB read and what changed written: 87 us, with run-time
// shifts 187).
template <int WB>
__device__ __forceinline__ void dr_maintain_group_x(const Geo &G, uint32_t *__restrict__ pool32, uint64_t gi)
{
    uint32_t *words = pool32 + gi * G.wb;
    uint32_t vals[32];
    read_group<WB>(words, G.wb, vals);
    uint32_t changed = 0;
#pragma unroll
    for (int e = 0; e < 32; ++e) {
        const uint32_t up = vals[e] < G.k ? 1u : 0u;
        vals[e] += up;
        changed |= up;
    }
    if (changed) write_group<WB>(words, G.wb, vals);
}

template <int WB>
__global__ void __launch_bounds__(256) k_dr_maintain_x(Geo G, uint32_t *__restrict__ pool32, uint64_t ngroups,
                                                       DevState *__restrict__ st)
{
    if (blockIdx.x == 0) advance_clock(G, st);
    for (uint64_t gi = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; gi < ngroups;
         gi += (uint64_t)gridDim.x * blockDim.x)
        dr_maintain_group_x<WB>(G, pool32, gi);
}
