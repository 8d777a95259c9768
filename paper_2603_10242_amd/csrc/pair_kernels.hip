// pair_kernels.hip -- two waves for the work of one, where a call is too small to
// give every SIMD a wave.
//
// A lane's chain of compressions is serial, but of a block only the rounds
// depend on the chain: a second wave can expand the schedule of a block whose
// words are known (about 750 instructions with loading and padding) while the
// first runs the 64 rounds of the block before (about 900) on K[t] + W[t] read
// from LDS.  Where a block's words are the chain itself (HMAC's outer block,
// HKDF, the hash chain), the first wave starts its rounds 0..15 at once and the
// second expands the words of rounds 16..63 sixteen at a time ahead of it; the
// two midstates of a key go one to each wave.
//
// Bound by that chain: a lone wave takes 2.5 us for a whole compression and
// about 1.8 for the first wave's part.  It needs two waves' SIMDs per 64 lanes,
// so it serves up to half as many wave tiles as there are SIMDs (verify), or one
// per CU (derivations and hash chains, whose waves meet every sixteen rounds).
//
//   k_derive_pair    64 identities of one (salt, info) stream per workgroup.
//   k_poh_pair       64 hash-chain segments per workgroup.
// (k_verify_pair is with the other verify forms.)
//
// Included by ace_kernels.hip after hkdf_kernels.hip.

namespace ace {

struct alignas(16) Q4 {  // one 16-byte LDS access
    uint32_t x, y, z, w;
};
struct PairLds {
    Q4 tail[12][64];  // K[t] + W[t] of rounds 16..63 of a block made from the chain: [t / 4][lane]
    Q4 down[2][64];   // eight words per lane from the first wave to the second
    Q4 up[2][64];     // and back
};

__device__ __forceinline__ void put8(Q4 (&x)[2][64], const State &s)
{
    const uint32_t l = lane_id();
    x[0][l] = Q4{s.h[0], s.h[1], s.h[2], s.h[3]};
    x[1][l] = Q4{s.h[4], s.h[5], s.h[6], s.h[7]};
}
__device__ __forceinline__ State get8(const Q4 (&x)[2][64])
{
    const uint32_t l = lane_id();
    const Q4 a = x[0][l], b = x[1][l];
    return State{{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w}};
}

// 16 N rounds from K[t] + W[t] in LDS.  All the words are read first (the
// compiler, left to itself, reads them just before their rounds and waits).
template <int N>
__device__ __forceinline__ void rounds16(uint32_t (&v)[8], const Q4 (*kw)[64])
{
    const uint32_t l = lane_id();
    Q4 k[4 * N];
#pragma unroll
    for (int c = 0; c < 4 * N; ++c) k[c] = kw[c][l];
    asm volatile("" ::: "memory");
#pragma unroll
    for (int c = 0; c < 4 * N; ++c) {
        const uint32_t w[4] = {k[c].x, k[c].y, k[c].z, k[c].w};
#pragma unroll
        for (int j = 0; j < 4; ++j)
            round_step(v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], w[j], 0u);
    }
}
__device__ __forceinline__ void add_state(State &s, const uint32_t (&v)[8])
{
#pragma unroll
    for (int i = 0; i < 8; ++i) s.h[i] += v[i];
}

// Sixteen schedule words W[16 q ..] (q > 0: from the sixteen before) to LDS
// with their round constants added.
template <int Q>
__device__ __forceinline__ void expand16(uint32_t (&W)[16], Q4 (*kw)[64])
{
    const uint32_t l = lane_id();
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        uint32_t o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int j = 4 * c + i;
            if (Q > 0)
                W[j] = small_sigma1(W[(j - 2) & 15]) + W[(j - 7) & 15] + small_sigma0(W[(j - 15) & 15]) + W[j];
            o[i] = W[j] + kRound[16 * Q + j];
        }
        kw[c][l] = Q4{o[0], o[1], o[2], o[3]};
    }
}

// s <- F(s, m || 0x80 || 0 || BITS) for a 32-byte message m (768: after a 64-byte
// key block): the first wave's part, and the second's (four barriers each).
template <uint32_t BITS>
__device__ __forceinline__ void pair_tail_rounds(PairLds &L, State &s, const State &m)
{
    put8(L.down, m);
    __syncthreads();
    uint32_t v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = s.h[i];
#pragma unroll
    for (int t = 0; t < 16; ++t) {
        const uint32_t w = t < 8 ? m.h[t & 7] : (t == 8 ? 0x80000000u : (t == 15 ? BITS : 0u));
        round_step(v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], w, kRound[t]);
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        __syncthreads();
        rounds16<1>(v, &L.tail[4 * q]);
    }
    add_state(s, v);
}
template <uint32_t BITS>
__device__ __forceinline__ void pair_tail_schedule(PairLds &L)
{
    __syncthreads();
    const State m = get8(L.down);
    uint32_t W[16];
#pragma unroll
    for (int i = 0; i < 8; ++i) W[i] = m.h[i];
    W[8] = 0x80000000u;
#pragma unroll
    for (int i = 9; i < 15; ++i) W[i] = 0u;
    W[15] = BITS;
    expand16<1>(W, &L.tail[0]);
    __syncthreads();
    expand16<2>(W, &L.tail[4]);
    __syncthreads();
    expand16<3>(W, &L.tail[8]);
    __syncthreads();
}

// A block's whole schedule.
__device__ __forceinline__ void pair_schedule(uint32_t (&W)[16], Q4 (*kw)[64])
{
    expand16<0>(W, kw);
    expand16<1>(W, kw + 4);
    expand16<2>(W, kw + 8);
    expand16<3>(W, kw + 12);
}
__device__ __forceinline__ void pair_rounds(State &s, const Q4 (*kw)[64])
{
    uint32_t v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = s.h[i];
    rounds16<4>(v, kw);
    add_state(s, v);
}

// HKDF and both midstates of the derived key (as derive_lane), the steps shared
// out: the first wave ends with the key and its ipad midstate, the opad midstate
// is in L.up after the next barrier.  rv: root entropy words as loaded.
// `between` runs on the second wave while it would wait for the expand block.
__device__ __forceinline__ void pair_derive_first(PairLds &L, const HkdfPrep &prep, const uint32_t (&rv)[8],
                                                  State &key, State &ipad)
{
    State m, x, prk;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        m.h[k] = bswap32(rv[k]);
        x.h[k] = prep.salt_ipad[k];
        prk.h[k] = prep.salt_opad[k];
    }
    pair_tail_rounds<768>(L, x, m);
    pair_tail_rounds<768>(L, prk, x);
    put8(L.down, prk);
    __syncthreads();
    State pi = hmac_midstate<0x36363636u>(prk);
    const uint32_t nq = prep.info_blocks;
    for (uint32_t q = 0; q < nq; ++q) compress_kw(pi, prep.info_kw[q]);
    __syncthreads();
    key = get8(L.up);
    pair_tail_rounds<768>(L, key, pi);
    put8(L.down, key);
    __syncthreads();
    ipad = hmac_midstate<0x36363636u>(key);
}
template <class Between>
__device__ __forceinline__ void pair_derive_second(PairLds &L, const HkdfPrep &prep, Between between)
{
    (void)prep;
    pair_tail_schedule<768>(L);
    pair_tail_schedule<768>(L);
    __syncthreads();
    put8(L.up, hmac_midstate<0x5c5c5c5cu>(get8(L.down)));
    between();
    __syncthreads();
    pair_tail_schedule<768>(L);
    __syncthreads();
    put8(L.up, hmac_midstate<0x5c5c5c5cu>(get8(L.down)));
}

__device__ __forceinline__ const HkdfParams &param_set(const HkdfParams &p, uint32_t) { return p; }
__device__ __forceinline__ const StreamParams &param_set(const MultiHkdf &p, uint32_t y) { return p.s[y]; }
__device__ __forceinline__ uint32_t first_set(const HkdfParams &) { return 0; }
__device__ __forceinline__ uint32_t first_set(const MultiHkdf &p) { return p.first; }

// 64 identities under parameter set first_set + blockIdx.y, as k_derive (whose
// `zero` it has) and k_derive_multi.
template <class Params>
__global__ void __launch_bounds__(128) k_derive_pair(const uint8_t *__restrict__ rev, uint32_t n_id,
                                                     uint8_t *__restrict__ key_out,
                                                     uint32_t *__restrict__ mid_out, Params mp,
                                                     unsigned long long *zero)
{
    if (zero && blockIdx.x == 0 && threadIdx.x == 0) *zero = 0;
    __shared__ PairLds L;
    __shared__ HkdfPrep prep;
    const bool first = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == 0;
    const uint32_t j = 64 * blockIdx.x + lane_id();
    const bool live = j < n_id;
    RevRaw x{};
    if (first && live) x = load_rev(rev, j);
    hkdf_prepare(param_set(mp, blockIdx.y), prep);
    __syncthreads();
    const uint64_t row = (uint64_t)(first_set(mp) + blockIdx.y) * n_id + j;
    if (first) {
        const uint32_t rv[8] = {x.a.x, x.a.y, x.a.z, x.a.w, x.b.x, x.b.y, x.b.z, x.b.w};
        State key, ipad;
        pair_derive_first(L, prep, rv, key, ipad);
        if (live && key_out) {
            uint32_t *q = reinterpret_cast<uint32_t *>(key_out + 32ull * row);
#pragma unroll
            for (int i = 0; i < 8; ++i) q[i] = bswap32(key.h[i]);
        }
        if (live && mid_out) {
            uint32_t *q = mid_out + 16ull * row;
#pragma unroll
            for (int i = 0; i < 8; ++i) q[i] = ipad.h[i];
        }
    } else {
        pair_derive_second(L, prep, [] {});
        if (live && mid_out) {
            const State opad = get8(L.up);  // this lane's own
            uint32_t *q = mid_out + 16ull * row + 8;
#pragma unroll
            for (int i = 0; i < 8; ++i) q[i] = opad.h[i];
        }
    }
}

}  // namespace ace
