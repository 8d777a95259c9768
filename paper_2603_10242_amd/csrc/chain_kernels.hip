// chain_kernels.hip -- segments of the SHA-256 hash chain the consensus
// section uses as its clock.  Included by ace_api.hip after ace_kernels.hip.

namespace ace {

// ------------------------------------------------------------------------------------------
// Hash-chain segments (the consensus section's clock: H_{i+1} = SHA-256(H_i)
// over the 32 digest bytes).  One segment per lane: steps[i] single-block
// hashes from start[i], compared with end[i].
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ State load_chain_state(const uint8_t *q)
{
    const uint32_t *p = reinterpret_cast<const uint32_t *>(q);
    const U4 a = load16(p), b = load16(p + 4);
    return State{{bswap32(a.x), bswap32(a.y), bswap32(a.z), bswap32(a.w), bswap32(b.x), bswap32(b.y),
                  bswap32(b.z), bswap32(b.w)}};
}

// Compares segment i's final state with end[i] and writes the wave's results
// (segments i0 .. i0 + 63).
__device__ __forceinline__ void poh_result(const State &h, bool live, uint64_t i, uint64_t i0, uint64_t n,
                                           const uint8_t *__restrict__ end, uint32_t *__restrict__ bitmask,
                                           unsigned long long *__restrict__ count, bool store)
{
    uint32_t d = 0;
    if (live) {
        const State e = load_chain_state(end + 32ull * i);
#pragma unroll
        for (int k = 0; k < 8; ++k) d = or_xor(d, h.h[k], e.h[k]);
    }
    const unsigned long long m = __ballot(live && d == 0);
    if (lane_id() == 0) {
        bitmask[i0 >> 5] = (uint32_t)m;
        if (i0 + 32 < n) bitmask[(i0 >> 5) + 1] = (uint32_t)(m >> 32);
        const unsigned long long c = __popcll(m);
        if (store) *count = c;
        else if (c) atomicAdd(count, c);
    }
}

__global__ void k_poh_zero(unsigned long long *count) { *count = 0; }

__global__ void __launch_bounds__(kWG) ACE_WAVES(8) k_poh_verify(const uint8_t *__restrict__ start,
                                                   const uint8_t *__restrict__ end,
                                                   const uint32_t *__restrict__ steps,
                                                   uint32_t uniform_steps, uint64_t n,
                                                   uint32_t *__restrict__ bitmask,
                                                   unsigned long long *__restrict__ count)
{
    const uint64_t i0 = 64ull * ((uint64_t)blockIdx.x * kWavesPerWG + (threadIdx.x >> 6));
    if (i0 >= n) return;  // whole wave past the end
    const uint64_t i = i0 + lane_id();
    const bool live = i < n;
    State h;
    uint32_t T = 0;
    if (live) {
        h = load_chain_state(start + 32ull * i);
        T = steps ? steps[i] : uniform_steps;
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) h.h[k] = 0;
    }
    for (uint32_t t = 0;; ++t) {
        const bool run = live && t < T;
        if (__ballot(run) == 0) break;
        if (run) {
            // the 32-byte value, 0x80, zeros, bit length 256: one block
            uint32_t W[16];
#pragma unroll
            for (int k = 0; k < 8; ++k) W[k] = h.h[k];
            W[8] = 0x80000000u;
#pragma unroll
            for (int k = 9; k < 15; ++k) W[k] = 0u;
            W[15] = 256u;
            State s = initial_state();
            compress_fold(s, W);  // words 8..15 are constants
            h = s;
        }
    }
    poh_result(h, live, i, i0, n, end, bitmask, count, false);
}

// Two waves per 64 segments (pair_kernels.hip), for up to one wave tile per CU.
// `solo`: the call is one workgroup, which stores the count itself.
__global__ void __launch_bounds__(128) k_poh_pair(const uint8_t *__restrict__ start,
                                                  const uint8_t *__restrict__ end,
                                                  const uint32_t *__restrict__ steps,
                                                  uint32_t uniform_steps, uint64_t n,
                                                  uint32_t *__restrict__ bitmask,
                                                  unsigned long long *__restrict__ count, uint32_t solo)
{
    __shared__ PairLds L;
    __shared__ uint32_t longest;
    const bool first = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == 0;
    const uint64_t i0 = 64ull * blockIdx.x;
    const uint64_t i = i0 + lane_id();
    const bool live = i < n;
    State h{};
    uint32_t T = 0;
    if (first) {
        if (live) {
            h = load_chain_state(start + 32ull * i);
            T = steps ? steps[i] : uniform_steps;
        }
        uint32_t m = 0;
        for (unsigned long long more; (more = __ballot(T > m)) != 0;)
            m = __builtin_amdgcn_readlane(T, __builtin_ctzll(more));
        if (lane_id() == 0) longest = m;
    }
    __syncthreads();
    const uint32_t most = uniform32(longest);
    if (!first) {
        for (uint32_t t = 0; t < most; ++t) pair_tail_schedule<256>(L);
        return;  // no barrier follows
    }
    for (uint32_t t = 0; t < most; ++t) {
        State s = initial_state();
        pair_tail_rounds<256>(L, s, h);
#pragma unroll
        for (int k = 0; k < 8; ++k) h.h[k] = t < T ? s.h[k] : h.h[k];
    }
    poh_result(h, live, i, i0, n, end, bitmask, count, solo != 0);
}

}  // namespace ace
