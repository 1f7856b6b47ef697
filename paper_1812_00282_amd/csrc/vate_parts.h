// The closed form for window k by gathers of one part of the bitmap per XCD:
// hosts with several gathers each on pools of 2^26 ATs and more, where the lookups
// are not partitioned (no workspace, or too few hosts).  Included into vate.hip
// inside namespace vate.
//
// Each XCD has an L2 of 4 MiB.  The bitmap of 2^28 ATs is 32 MiB, and gathers
// from anywhere in it fill lines from beyond L2, 6.5e10 a second on the chip; a
// bitmap that L2 holds gives 2.65e11.  So the bitmap is cut into up to eight
// parts, and the workgroups of one XCD (blockIdx mod 8) look up one part's VATs
// only, of all hosts (with fewer parts, of a share of them): every VAT is hashed
// once per part, and each host's counts from the parts are added with atomics
// into its live count, from which a last kernel forms the estimate.  Bound by
// the hashing: 17 instructions per VAT and part.  2^28 byte ATs, g = 1024: 4,000
// hosts 68 -> 32 us, 16,000 264 -> 94, 250,000 3,861 -> 1,088; 1M hosts with
// blocks of 64 VATs (16 gathers each) 253 -> 164; 2^26 ATs 64,000 hosts 554 ->
// 276.

constexpr uint32_t kPartsThreads = 256;
constexpr uint32_t kPartsU = 16;           // gathers in flight per lane
constexpr uint32_t kPartsBlockU = 8;       // and blocks, two words each at a time
constexpr uint64_t kPartsMin = 3u << 19;   // gathers from which they go by parts (2M on 2^28: 37 us before, 22)

// log2 of the parts: 2^25 ATs (4 MiB) each, eight at most.
__host__ __device__ __forceinline__ uint32_t parts_log2(uint32_t c) { return c <= 25 ? 0u : c >= 28 ? 3u : c - 25u; }

__global__ void __launch_bounds__(256) k_parts_clear(uint32_t n, uint32_t *__restrict__ acc)
{
    for (uint64_t h = (uint64_t)blockIdx.x * 256 + threadIdx.x; h < n; h += (uint64_t)gridDim.x * 256) acc[h] = 0;
}

// 2^lg lanes per host; gridDim.x is a multiple of 8.  BLOCKED: locality blocks
// of at least 32 VATs, whole words of the bitmap, counted with popcount.
template <bool BLOCKED>
__global__ void __launch_bounds__(kPartsThreads) k_parts_count(Geo G, const uint32_t *__restrict__ bitmap,
                                                              const uint32_t *__restrict__ hosts, uint32_t n,
                                                              uint32_t lg, uint32_t *__restrict__ acc)
{
    const uint32_t pl = parts_log2(G.c), xcd = blockIdx.x & 7u;
    const uint32_t part = xcd & ((1u << pl) - 1u);
    // the workgroups of this part, numbered
    const uint32_t j = (blockIdx.x >> 3) * (8u >> pl) + (xcd >> pl), nj = (gridDim.x >> 3) * (8u >> pl);
    const uint32_t ps = G.c - pl;              // ATs per part = 2^ps
    const uint32_t per = kPartsThreads >> lg, lanes = 1u << lg, sub = threadIdx.x & (lanes - 1u);
    for (uint64_t h0 = (uint64_t)j * per; h0 < n; h0 += (uint64_t)nj * per) {
        const uint64_t h = h0 + (threadIdx.x >> lg);
        const bool valid = h < n;
        const uint32_t key = host_key(G, valid ? hosts[h] : 0u);
        uint32_t live = 0;
        if constexpr (BLOCKED) {
            const uint32_t beta = 1u << G.blog, words = beta >> 5, nb = valid ? (G.g + beta - 1u) >> G.blog : 0u;
            constexpr uint32_t U = kPartsBlockU;
            for (uint32_t q0 = sub; q0 < nb; q0 += U * lanes)
                for (uint32_t x = 0; x < words; x += 2) {
                    uint32_t a[U], b[U];
#pragma unroll
                    for (uint32_t u = 0; u < U; ++u) {
                        const uint32_t q = q0 + u * lanes, base = vat_pid(G, key, q << G.blog);
                        const bool in = q < nb && base >> ps == part;
                        const uint32_t *w = bitmap + (base >> 5) + x;
                        a[u] = in ? w[0] : 0u;
                        b[u] = in && x + 1 < words ? w[1] : 0u;
                    }
#pragma unroll
                    for (uint32_t u = 0; u < U; ++u) {      // VATs of the block past g do not count
                        const uint32_t q = q0 + u * lanes;
                        const uint32_t left = q < nb ? G.g - (q << G.blog) : 0u;
                        const uint32_t la = left > 32u * x ? left - 32u * x : 0u, lb = la > 32u ? la - 32u : 0u;
                        live += __popc(la >= 32u ? a[u] : a[u] & ((1u << la) - 1u));
                        live += __popc(lb >= 32u ? b[u] : b[u] & ((1u << lb) - 1u));
                    }
                }
        } else {
            const uint8_t *bytes = reinterpret_cast<const uint8_t *>(bitmap);
            const uint32_t end = valid ? G.g : 0u;
            for (uint32_t i0 = sub; i0 < end; i0 += kPartsU * lanes) {
                uint32_t pid[kPartsU], byte[kPartsU];
#pragma unroll
                for (uint32_t u = 0; u < kPartsU; ++u) pid[u] = vat_pid(G, key, i0 + u * lanes);
#pragma unroll
                for (uint32_t u = 0; u < kPartsU; ++u)
                    byte[u] = pid[u] >> ps == part && i0 + u * lanes < end ? (uint32_t)bytes[pid[u] >> 3] : 0u;
#pragma unroll
                for (uint32_t u = 0; u < kPartsU; ++u) live += (byte[u] >> (pid[u] & 7u)) & 1u;
            }
        }
        for (uint32_t off = 1; off < lanes; off <<= 1) live += __shfl_xor(live, (int)off, 64);
        if (valid && sub == 0 && live) atomicAdd(&acc[h], live);
    }
}

// acc may be est's own memory.
__global__ void __launch_bounds__(256) k_parts_finish(Geo G, const DevState *__restrict__ st, uint32_t n,
                                                      const uint32_t *acc, float *est)
{
    const uint64_t active_pool = pool_active(st, G.k);
    for (uint64_t h = (uint64_t)blockIdx.x * 256 + threadIdx.x; h < n; h += (uint64_t)gridDim.x * 256)
        est[h] = estimate_from_counts(G.g - acc[h], G.N - active_pool, G.g, G.c);
}
