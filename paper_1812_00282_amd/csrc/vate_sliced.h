// Lookups against LDS copies of the activity bitmap, slice after slice: pools
// of up to 2^23 ATs.  Included into vate.hip inside namespace vate.
//
// A gather of one bit is a request to L2 each, and L2 serves about 2.7e11 of
// them a second, whatever their size.  Here a workgroup of 1024 threads, one
// per CU, hashes the VATs of a group of hosts into registers (P per thread),
// copies the pool's slices of 2^20 activity bits to LDS one after the other
// (128 KiB, the next slice's loads in flight while the current one is tested),
// and tests every VAT against every slice: VATs of other slices read one common
// zero word, which costs no bank conflict.  A test is seven vector instructions
// and an LDS read, so the cost grows with the slices; the lookups of a host are
// counted (or its live VATs' values gathered) when all have been tested.  A
// pool of one slice is copied once per workgroup.
//
// 512M lookups (g = 1024, closed form): 2^20 ATs 298 us, 2^21 553, 2^22 892,
// 2^23 1551; by gathers through L2 1545, 1755, 1900 and 1970 us.

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr uint32_t kSlicedThreads = 1024;
constexpr uint32_t kSlicedLog2 = 23;         // largest pool (log2)
constexpr uint32_t kSlicedLoads = kBmWords / 4u / kSlicedThreads;   // 16-byte loads per thread and slice

// 16-byte groups of a slice's bits (a pool below 2^20 is one short slice), and
// LDS words with the zero word after them.
__host__ __device__ __forceinline__ uint32_t sliced_groups(const Geo &G) { return G.c >= kSliceLog2 ? kBmWords / 4u : G.c > 7 ? 1u << (G.c - 7) : 1u; }
__host__ __device__ __forceinline__ uint32_t sliced_words(const Geo &G) { return 4u * sliced_groups(G) + 4u; }

__device__ __forceinline__ void sliced_load(const u32x4 *__restrict__ src, uint32_t nv, u32x4 (&v)[kSlicedLoads])
{
    uint32_t t = threadIdx.x;
    asm volatile("" : "+v"(t));       // (addresses are formed here, not kept)
#pragma unroll
    for (uint32_t u = 0; u < kSlicedLoads; ++u) v[u] = src[min(t + u * kSlicedThreads, nv - 1u)];
}

__device__ __forceinline__ void sliced_store(uint32_t *bits, uint32_t nv, const u32x4 (&v)[kSlicedLoads])
{
    u32x4 *dst = reinterpret_cast<u32x4 *>(bits);
#pragma unroll
    for (uint32_t u = 0; u < kSlicedLoads; ++u)
        if (threadIdx.x + u * kSlicedThreads < nv) dst[threadIdx.x + u * kSlicedThreads] = v[u];
    if (threadIdx.x == 0) dst[nv] = (u32x4)0u;
}

// The slices of a pool (a power of two).
__host__ __device__ __forceinline__ uint32_t sliced_slices(const Geo &G) { return G.c > kSliceLog2 ? 1u << (G.c - kSliceLog2) : 1u; }

// ONE: a pool of one slice, copied before the first sliced_masks (the whole
// workgroup calls).
__device__ __forceinline__ void sliced_begin(const Geo &G, const uint8_t *__restrict__ bitmap, uint32_t *bits)
{
    u32x4 v[kSlicedLoads];
    sliced_load(reinterpret_cast<const u32x4 *>(bitmap), sliced_groups(G), v);
    sliced_store(bits, sliced_groups(G), v);
    __syncthreads();
}

// Registers: with one slice the kernels keep to 64 (two workgroups per CU
// where the bits are small); with several, the next slice's 32 are in flight.
template <bool ONE>
constexpr uint32_t kSlicedWaves = ONE ? 8 : 4;

// Which of this thread's VATs are active (bit u of mask: VAT pid[u]; a pid of
// ~0 is none).  The whole workgroup calls; `bits`: sliced_words of LDS.
template <uint32_t P, bool ONE>
__device__ __forceinline__ void sliced_masks(const Geo &G, const uint8_t *__restrict__ bitmap, uint32_t *bits,
                                             u32x4 (&v)[kSlicedLoads], const uint32_t (&pid)[P], uint32_t &mask)
{
    static_assert(P <= 32, "one mask word");
    const uint32_t nv = sliced_groups(G), cap = 128u * nv, ns = ONE ? 1u : sliced_slices(G);
    const u32x4 *src = reinterpret_cast<const u32x4 *>(bitmap);
    mask = 0;
    for (uint32_t s = 0; s < ns; ++s) {
        if constexpr (!ONE) {
            __syncthreads();               // the last slice's tests are done
            sliced_store(bits, nv, v);
            if (s + 1 < ns) sliced_load(src + (size_t)(s + 1) * nv, nv, v);
            __syncthreads();
        }
        const uint32_t base = s << kSliceLog2;
        // eight LDS reads in flight; more of them at once would spill
#pragma unroll
        for (uint32_t u0 = 0; u0 < P; u0 += 8) {
            uint32_t a[8], w[8];
#pragma unroll
            for (uint32_t u = 0; u < 8; ++u) {
                a[u] = min(pid[u0 + u] - base, cap);         // another slice's AT: the zero word
                w[u] = bits[a[u] >> 5];
            }
#pragma unroll
            for (uint32_t u = 0; u < 8; ++u) mask |= __builtin_amdgcn_ubfe(w[u], a[u], 1u) << (u0 + u);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// VATs i0, i0 + lanes, ... of a host (independent VATs: no locality blocks).
template <uint32_t P>
__device__ __forceinline__ void sliced_pids(const Geo &G, uint32_t key, bool valid, uint32_t i0, uint32_t lanes,
                                            uint32_t (&pid)[P])
{
    const uint32_t end = valid ? G.g : 0u;
    // opaque per group of hosts: hoisted out of that loop, the VATs' products
    // and bounds would not fit the registers
    asm volatile("" : "+v"(i0));
#pragma unroll
    for (uint32_t u = 0; u < P; ++u) {
        const uint32_t i = i0 + u * lanes, x = mix(key ^ (i * kPhi)) >> G.shift;
        pid[u] = i < end ? x : ~0u;
        if (u % 8 == 7) __builtin_amdgcn_sched_barrier(0);
    }
}

// Live VATs of this thread for k', from the masks (and the values of the
// active ones where k' < k).
template <int W, uint32_t P>
__device__ __forceinline__ uint32_t sliced_live(const Geo &G, const uint8_t *__restrict__ pool, uint32_t kprime,
                                                uint32_t bact0, const uint32_t (&pid)[P],
                                                uint32_t mask)
{
    if (kprime >= G.k) return __popc(mask);
    uint32_t live = 0;
#pragma unroll
    for (uint32_t u0 = 0; u0 < P; u0 += 8) {
        uint32_t val[8];
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u)
            val[u] = (mask >> (u0 + u)) & 1u ? load_at<W>(pool, pid[u0 + u], G.wb) : 0u;
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u)
            if (((mask >> (u0 + u)) & 1u) && value_dist(G, bact0, pid[u0 + u], val[u]) < kprime)
                ++live;
        __builtin_amdgcn_sched_barrier(0);
    }
    return live;
}

__device__ __forceinline__ uint32_t sum_lanes_log2(uint32_t x, uint32_t lg)
{
    for (uint32_t off = 1; off < 1u << lg; off <<= 1) x += __shfl_xor(x, (int)off, 64);
    return x;
}

// The closed form: 2^lg lanes per host, P VATs each at a time.
template <int W, uint32_t P, bool ONE>
__global__ void __launch_bounds__(kSlicedThreads, kSlicedWaves<ONE>) k_sliced(Geo G, const uint8_t *__restrict__ pool,
                                                          const DevState *__restrict__ st,
                                                          const uint8_t *__restrict__ bitmap,
                                                          const uint32_t *__restrict__ hosts, uint32_t n, uint32_t lg,
                                                          uint32_t kprime, float *__restrict__ est,
                                                          uint32_t *__restrict__ live_out)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t bits[];
    const uint32_t per = kSlicedThreads >> lg, sub = threadIdx.x & ((1u << lg) - 1u);
    const uint32_t bact0 = st->bact0;
    const uint64_t active_pool = pool_active(st, kprime);
    if constexpr (ONE) sliced_begin(G, bitmap, bits);
    for (uint64_t h0 = (uint64_t)blockIdx.x * per; h0 < n; h0 += (uint64_t)gridDim.x * per) {
        const uint64_t h = h0 + (threadIdx.x >> lg);
        const bool valid = h < n;
        const uint32_t key = host_key(G, valid ? hosts[h] : 0u);
        uint32_t live = 0;
        for (uint32_t i0 = 0; i0 < G.g; i0 += P << lg) {
            u32x4 v[kSlicedLoads];
            if constexpr (!ONE) sliced_load(reinterpret_cast<const u32x4 *>(bitmap), sliced_groups(G), v);
            uint32_t pid[P], mask;
            sliced_pids<P>(G, key, valid, i0 + sub, 1u << lg, pid);
            sliced_masks<P, ONE>(G, bitmap, bits, v, pid, mask);
            live += sliced_live<W, P>(G, pool, kprime, bact0, pid, mask);
        }
        live = sum_lanes_log2(live, lg);
        if (valid && sub == 0) {
            est[h] = estimate_from_counts(G.g - live, G.N - active_pool, G.g, G.c);
            if (live_out) live_out[h] = live;
        }
    }
}

// With histograms, several windows or the learned estimate (finish_hosts):
// the live VATs' distances are counted into LDS rows behind the bits.
template <int W, int MODE, uint32_t P, bool ONE>
__global__ void __launch_bounds__(kSlicedThreads, MODE == kFinLearned ? 4 : kSlicedWaves<ONE>) k_sliced_hist(Geo G, const uint8_t *__restrict__ pool,
                                                               const DevState *__restrict__ st,
                                                               const uint8_t *__restrict__ bitmap,
                                                               const uint32_t *__restrict__ hosts, uint32_t n,
                                                               uint32_t lg, uint32_t rowp, uint32_t kprime,
                                                               float *__restrict__ est, uint32_t *__restrict__ live_out,
                                                               uint32_t *__restrict__ hist_out, Windows win,
                                                               const mlp::Packed *__restrict__ N,
                                                               float *__restrict__ cf_out)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t bits[];
    __shared__ unsigned long long act[MODE == kFinMulti ? kMaxWindows : 1u];
    uint32_t *hist = bits + sliced_words(G);
    const uint32_t t = threadIdx.x;
    if constexpr (MODE == kFinMulti)
        if (t < 64) window_counts(G, st, win, act);
    const uint32_t per = kSlicedThreads >> lg, sub = t & ((1u << lg) - 1u);
    const uint32_t bact0 = st->bact0;
    uint32_t *row = hist + (t >> lg) * rowp;
    if constexpr (ONE) sliced_begin(G, bitmap, bits);
    for (uint64_t h0 = (uint64_t)blockIdx.x * per; h0 < n; h0 += (uint64_t)gridDim.x * per) {
        const uint32_t nh = (uint32_t)min((uint64_t)per, n - h0);
        for (uint32_t q = t; q < nh * rowp; q += kSlicedThreads) hist[q] = 0;
        const uint64_t h = h0 + (t >> lg);
        const bool valid = h < n;
        const uint32_t key = host_key(G, valid ? hosts[h] : 0u);
        __syncthreads();
        for (uint32_t i0 = 0; i0 < G.g; i0 += P << lg) {
            u32x4 v[kSlicedLoads];
            if constexpr (!ONE) sliced_load(reinterpret_cast<const u32x4 *>(bitmap), sliced_groups(G), v);
            uint32_t pid[P], mask;
            sliced_pids<P>(G, key, valid, i0 + sub, 1u << lg, pid);
            sliced_masks<P, ONE>(G, bitmap, bits, v, pid, mask);
#pragma unroll
            for (uint32_t u0 = 0; u0 < P; u0 += 8) {
                uint32_t val[8];
#pragma unroll
                for (uint32_t u = 0; u < 8; ++u)
                    val[u] = (mask >> (u0 + u)) & 1u ? load_at<W>(pool, pid[u0 + u], G.wb) : 0u;
#pragma unroll
                for (uint32_t u = 0; u < 8; ++u)
                    if ((mask >> (u0 + u)) & 1u) {
                        const uint32_t d = value_dist(G, bact0, pid[u0 + u], val[u]);
                        if (d < G.k) atomicAdd(&row[d >> 1], 1u << ((d & 1u) << 4));
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();
        finish_hosts<MODE, kSlicedThreads>(G, st, hist, rowp, nh, (uint32_t)h0, kprime, est, live_out, hist_out, win,
                                           act, N, cf_out);
        __syncthreads();
    }
}
