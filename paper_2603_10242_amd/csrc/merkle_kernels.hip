// merkle_kernels.hip -- Merkle roots of the block header's transaction and
// attestation lists (App. C, block header fields tx_merkle_root and
// attest_merkle_root; a validator recomputes the attestation root, Alg. 4).
//
// Reading (the paper fixes neither): leaf node = SHA-256(leaf bytes); parent
// = SHA-256(left || right); at a level with an odd number of nodes the last
// one moves up unchanged; a tree without leaves has the root SHA-256("").
//
// Layout: node j of level k of a tree whose leaves start at global leaf
// index leaf0 lives in slot leaf0 + j * 2^k of one node array (8 native
// words per slot).  A parent overwrites its left child's slot, so levels are
// reduced in place, and an unpaired last node is already where the next
// level expects it.
//
//   k_merkle_leaves  one leaf per lane: SHA-256 of its bytes into its slot.
//   k_merkle_plan    per reducing stage (one workgroup each), exclusive prefix
//                    of each tree's groups.
//   k_merkle_level   one parent per lane at level k -> k + 1 (two blocks:
//                    the 64 child bytes, then the constant padding block).
//   k_merkle_chunk   the narrow levels: a workgroup reduces up to kTopNodes
//                    nodes of a tree in LDS; the last such stage writes the roots.
//
// Bound by VALU issue where a level fills the chip and by one wave's chain of
// two compressions per level where it does not.  (Groups of eight leaves or
// nodes reduced in a lane's registers, three levels per launch, measured slower:
// 7.66M leaves of 256 trees 1,183 us against 1,163 with a launch per level, since
// the wide levels run at 95% of the issue rate as they are.)

namespace ace {

struct MerkleDesc {
    const uint8_t *data;
    const uint64_t *off;
    uint64_t n;      // leaves
    uint8_t *root;   // 32-byte output
    uint64_t leaf0;  // global index of the first leaf
};

// Trees passed by value to the kernel that writes the table (3,944 bytes of
// kernel arguments): two launches for 256 trees.
constexpr uint32_t kMerkleChunk = 140;
struct MerkleChunk {
    const uint8_t *data[kMerkleChunk];
    const uint64_t *off[kMerkleChunk];
    uint8_t *root[kMerkleChunk];
    uint32_t n[kMerkleChunk];
    uint32_t first;
    uint32_t count;
    uint64_t leaf0;  // global index of the chunk's first leaf
};

// The second block of every parent is the padding of a 64-byte message
// (0x80, zeros, bit length 512): its whole message schedule is known at
// compile time, so it is folded into the round constants, kw[t] = K[t] +
// W[t], and the block costs the 64 rounds and the feed-forward only.
constexpr uint32_t c_rotr(uint32_t x, int n) { return (x >> n) | (x << (32 - n)); }
struct ScheduleKW {
    uint32_t v[64];
};
constexpr ScheduleKW fold_pad64()
{
    ScheduleKW r{};
    uint32_t w[64] = {};
    w[0] = 0x80000000u;
    w[15] = 512u;
    for (int t = 16; t < 64; ++t) {
        const uint32_t s0 = c_rotr(w[t - 15], 7) ^ c_rotr(w[t - 15], 18) ^ (w[t - 15] >> 3);
        const uint32_t s1 = c_rotr(w[t - 2], 17) ^ c_rotr(w[t - 2], 19) ^ (w[t - 2] >> 10);
        w[t] = s1 + w[t - 7] + s0 + w[t - 16];
    }
    for (int t = 0; t < 64; ++t) r.v[t] = kRound[t] + w[t];
    return r;
}
__constant__ __attribute__((aligned(64))) ScheduleKW kPad64KW = fold_pad64();

__device__ __forceinline__ void compress_pad64(State &s)
{
    uint32_t a = s.h[0], b = s.h[1], c = s.h[2], d = s.h[3];
    uint32_t e = s.h[4], f = s.h[5], g = s.h[6], h = s.h[7];
#pragma nounroll
    for (int q = 0; q < 4; ++q) {
        const RoundConsts16 kq = *reinterpret_cast<const RoundConsts16 *>(&kPad64KW.v[16 * q]);
#pragma unroll
        for (int j = 0; j < 16; ++j) round_step(a, b, c, d, e, f, g, h, 0u, kq.k[j]);
    }
    s.h[0] += a; s.h[1] += b; s.h[2] += c; s.h[3] += d;
    s.h[4] += e; s.h[5] += f; s.h[6] += g; s.h[7] += h;
}

constexpr uint32_t kPutThreads = 256;
__global__ void __launch_bounds__(kPutThreads) k_merkle_put(MerkleDesc *table, MerkleChunk c)
{
    __shared__ uint64_t part[kPutThreads];
    const uint32_t t = threadIdx.x;
    const uint64_t n = t < c.count ? c.n[t] : 0;
    part[t] = n;
    __syncthreads();
    for (uint32_t s = 1; s < kPutThreads; s <<= 1) {  // inclusive scan (Hillis-Steele)
        const uint64_t add = t >= s ? part[t - s] : 0;
        __syncthreads();
        part[t] += add;
        __syncthreads();
    }
    if (t < c.count) table[c.first + t] = MerkleDesc{c.data[t], c.off[t], n, c.root[t], c.leaf0 + part[t] - n};
}

// Last i < n with key(i) <= x, for keys that do not decrease (equal keys:
// the last of them).  The lanes of a wave hold consecutive x, so the first
// active lane's x is searched once for the wave (a uniform loop on scalar
// loads); only lanes at or past the next key (a wave across two trees)
// search again, each on its own.
template <class Key>
__device__ __forceinline__ uint32_t last_at_or_below(uint32_t n, uint64_t x, Key key)
{
    const uint64_t x0 = uniform64(x);
    uint32_t lo = 0, hi = n;  // answer in [lo, hi)
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (key(mid) <= x0) lo = mid;
        else hi = mid;
    }
    if (lo + 1 < n && key(lo + 1) <= x) {
        uint32_t l = lo + 1, h = n;
        while (h - l > 1) {
            const uint32_t mid = (l + h) >> 1;
            if (key(mid) <= x) l = mid;
            else h = mid;
        }
        return l;
    }
    return lo;
}

// Tree of leaf g: the last tree whose first leaf is <= g (trees with no
// leaves are skipped by taking the last of equal starts).
__device__ __forceinline__ uint32_t merkle_tree_of(const MerkleDesc *__restrict__ table,
                                                   uint32_t n_trees, uint64_t g)
{
    return last_at_or_below(n_trees, g, [&](uint32_t i) { return table[i].leaf0; });
}

// SHA-256 of L bytes at p into S (from the initial value).  With
// overread_ok (the tree's data area extends at least 80 bytes past this
// leaf) whole 16-byte loads are used, whose bytes past the leaf's end feed
// only words the padding overwrites; otherwise every dword address is
// clamped to one that holds leaf bytes (for L == 0 none is read).
__device__ __forceinline__ void sha256_bytes(bool live, const uint8_t *p, uint64_t L, State &S,
                                             bool overread_ok = false)
{
    S = initial_state();
    const uint32_t nb = live ? (uint32_t)((L + 9 + 63) >> 6) : 0u;
    const uintptr_t addr = reinterpret_cast<uintptr_t>(p);
    const uint32_t sh = (uint32_t)addr & 3u;
    const uint32_t sel = 0x00010203u + sh * 0x01010101u;
    const uint64_t lim = (uint64_t)sh + L;
    const uint64_t last = lim ? ((lim - 1) >> 2) : 0;
    const uint32_t *A0 = reinterpret_cast<const uint32_t *>(addr - sh);
    const uint64_t bits = L << 3;
    for (uint32_t b = 0;; ++b) {
        const bool run = live && b < nb;
        if (__ballot(run) == 0) break;
        if (run) {
            uint32_t D[17], W[16];
            if (overread_ok) {
                const uint32_t *q = A0 + 16ull * b;
                const U4 v0 = load16(q), v1 = load16(q + 4), v2 = load16(q + 8), v3 = load16(q + 12);
                D[0] = v0.x; D[1] = v0.y; D[2] = v0.z; D[3] = v0.w;
                D[4] = v1.x; D[5] = v1.y; D[6] = v1.z; D[7] = v1.w;
                D[8] = v2.x; D[9] = v2.y; D[10] = v2.z; D[11] = v2.w;
                D[12] = v3.x; D[13] = v3.y; D[14] = v3.z; D[15] = v3.w;
                D[16] = load32(q + 16);
            } else {
#pragma unroll
                for (int k = 0; k < 17; ++k) {
                    const uint64_t idx = 16ull * b + k;
                    D[k] = lim ? load32(A0 + (idx < last ? idx : last)) : 0u;
                }
            }
#pragma unroll
            for (int j = 0; j < 16; ++j) W[j] = __builtin_amdgcn_perm(D[j + 1], D[j], sel);
            const int64_t rb = (int64_t)L - 64 * (int64_t)b;
            if (rb < 64) {
                const int32_t r0 = (int32_t)rb;
                const int32_t jf = r0 >> 2;
                const uint32_t c8 = ((uint32_t)r0 & 3u) << 3;
                const uint32_t keep = ~(0xFFFFFFFFu >> c8);
                const uint32_t pad = 0x80000000u >> c8;
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const uint32_t part = (W[j] & keep) | pad;
                    W[j] = j < jf ? W[j] : (j == jf ? part : 0u);
                }
                if (b + 1 == nb) {
                    W[14] = (uint32_t)(bits >> 32);
                    W[15] = (uint32_t)bits;
                }
            }
            compress_block(S, W);
        }
    }
}

// SHA-256 of a 72-byte leaf at p (4-byte alignment not required): the
// paper form's check record, obj_hash (32) || domain (8) || credential (32),
// the leaf of an attestation root.  Its second block holds 8 record bytes,
// then the 0x80 marker, zeros and the bit length 576: words 2..15 are
// constants there and fold into that block's schedule.  The 19 dwords from
// the aligned start hold the record at any alignment; the last one is read
// only when it holds record bytes.
constexpr uint64_t kRecordLeaf = 72;
__device__ __forceinline__ void sha256_record72(const uint8_t *p, State &S)
{
    const uintptr_t addr = reinterpret_cast<uintptr_t>(p);
    const uint32_t sh = (uint32_t)addr & 3u;
    const uint32_t sel = 0x00010203u + sh * 0x01010101u;
    const uint32_t *A0 = reinterpret_cast<const uint32_t *>(addr - sh);
    uint32_t D[19];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const U4 v = load16(A0 + 4 * c);
        D[4 * c] = v.x; D[4 * c + 1] = v.y; D[4 * c + 2] = v.z; D[4 * c + 3] = v.w;
    }
    D[16] = load32(A0 + 16);
    D[17] = load32(A0 + 17);
    D[18] = load32(A0 + (sh ? 18 : 17));
    uint32_t W[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) W[j] = __builtin_amdgcn_perm(D[j + 1], D[j], sel);
    S = initial_state();
    compress_block(S, W);
    W[0] = __builtin_amdgcn_perm(D[17], D[16], sel);
    W[1] = __builtin_amdgcn_perm(D[18], D[17], sel);
    W[2] = 0x80000000u;
#pragma unroll
    for (int j = 3; j < 15; ++j) W[j] = 0u;
    W[15] = (uint32_t)(kRecordLeaf * 8);
    compress_fold(S, W);
}

__global__ void __launch_bounds__(kWG) k_merkle_leaves(const MerkleDesc *__restrict__ table,
                                                       uint32_t n_trees, uint64_t n_leaves,
                                                       uint32_t *__restrict__ nodes)
{
    const uint64_t g = (uint64_t)blockIdx.x * kWG + threadIdx.x;
    const bool live = g < n_leaves;
    const uint8_t *p = nullptr;
    uint64_t L = 0;
    bool overread_ok = false;
    if (live) {
        const MerkleDesc d = table[merkle_tree_of(table, n_trees, g)];
        const uint64_t i = g - d.leaf0;
        const uint64_t a = d.off[i], e = d.off[i + 1];
        p = d.data + a;
        L = e >= a ? e - a : 0;  // decreasing offsets: the empty leaf
        // 17 dwords from the aligned start of the last block reach at most 76
        // bytes past the leaf's end; the tree's leaves end at off[n]
        overread_ok = e >= a && a + L + 80 <= d.off[d.n];
    }
    State S;
    if (__ballot(live && L != kRecordLeaf) == 0) {
        // every live leaf of the wave is a 72-byte record
        if (live) sha256_record72(p, S);
    } else {
        sha256_bytes(live, p, L, S, overread_ok);
    }
    if (live) {
        uint32_t *q = nodes + 8ull * g;
#pragma unroll
        for (int k = 0; k < 8; ++k) q[k] = S.h[k];
    }
}

// Parent of two nodes: SHA-256 of their 64 bytes, the second block of which is
// constant.
__device__ __forceinline__ State merkle_parent(const State &l, const State &r)
{
    uint32_t W[16];
#pragma unroll
    for (int j = 0; j < 8; ++j) { W[j] = l.h[j]; W[8 + j] = r.h[j]; }
    State S = initial_state();
    compress_block(S, W);
    compress_pad64(S);
    return S;
}

__device__ __forceinline__ State load_node(const uint32_t *q)
{
    const U4 a = load16(q), b = load16(q + 4);
    State S;
    S.h[0] = a.x; S.h[1] = a.y; S.h[2] = a.z; S.h[3] = a.w;
    S.h[4] = b.x; S.h[5] = b.y; S.h[6] = b.z; S.h[7] = b.w;
    return S;
}

__device__ __forceinline__ void store_node(uint32_t *q, const State &S)
{
#pragma unroll
    for (int j = 0; j < 8; ++j) q[j] = S.h[j];
}

// Row r of P: exclusive prefix over the trees of ceil(n / 2^shift[r]), the
// groups of the stage that reduces 2^shift[r] leaves to a node.  Workgroup r
// scans row r.
constexpr uint32_t kPlanThreads = 1024;
constexpr uint32_t kMaxStages = 32;  // levels of the largest tree
struct MerkleShifts {
    uint32_t shift[kMaxStages];
};
__device__ __forceinline__ uint64_t merkle_nodes(uint64_t n, uint32_t level)
{
    return (n + (1ull << level) - 1) >> level;
}

__global__ void __launch_bounds__(kPlanThreads) k_merkle_plan(const MerkleDesc *__restrict__ table,
                                                              uint32_t n_trees, MerkleShifts sh,
                                                              unsigned long long *__restrict__ P)
{
    __shared__ unsigned long long part[kPlanThreads];
    const uint32_t t = threadIdx.x;
    const uint32_t shift = sh.shift[blockIdx.x];
    unsigned long long *row = P + (uint64_t)blockIdx.x * (n_trees + 1);
    unsigned long long running = 0;
    for (uint32_t c = 0; c < n_trees; c += kPlanThreads) {
        const uint32_t b = c + t;
        const unsigned long long v = b < n_trees ? merkle_nodes(table[b].n, shift) : 0;
        part[t] = v;
        __syncthreads();
        // Hillis-Steele inclusive scan
        for (uint32_t s = 1; s < kPlanThreads; s <<= 1) {
            const unsigned long long add = t >= s ? part[t - s] : 0ull;
            __syncthreads();
            part[t] += add;
            __syncthreads();
        }
        if (b < n_trees) row[b] = running + part[t] - v;
        running += part[kPlanThreads - 1];
        __syncthreads();
    }
    if (t == 0) row[n_trees] = running;
}

// Group q of a stage: its tree, and its index among the tree's groups.
__device__ __forceinline__ uint32_t merkle_group(const unsigned long long *__restrict__ row,
                                                 uint32_t n_trees, uint64_t q, uint64_t &j)
{
    j = q;
    if (n_trees == 1) return 0;
    const uint32_t b = last_at_or_below(n_trees, q, [&](uint32_t i) { return row[i]; });
    j = q - row[b];
    return b;
}

__global__ void __launch_bounds__(kWG) k_merkle_level(const MerkleDesc *__restrict__ table,
                                                      uint32_t n_trees,
                                                      const unsigned long long *__restrict__ row,
                                                      uint64_t n_groups, uint32_t k,
                                                      uint32_t *__restrict__ nodes)
{
    const uint64_t q = (uint64_t)blockIdx.x * kWG + threadIdx.x;
    bool live = q < n_groups;
    State l = initial_state(), r = l;
    uint32_t *o = nodes;
    if (live) {
        uint64_t j;
        const MerkleDesc &d = table[merkle_group(row, n_trees, q, j)];
        live = 2 * j + 1 < merkle_nodes(d.n, k);  // an unpaired last node stays where it is
        o = nodes + 8ull * (d.leaf0 + ((2 * j) << k));
        if (live) {
            l = load_node(o);
            r = load_node(o + (8ull << k));
        }
    }
    if (__ballot(live) == 0) return;
    const State S = merkle_parent(l, r);
    if (live) store_node(o, S);
}

// The narrow levels: a workgroup takes a chunk of kTopNodes nodes of level k of
// a tree (row: prefix of the trees' chunks) and reduces it in LDS, one parent per
// lane and level, to the node of level k + kTopLog that it is.  `last`: every
// tree is one chunk, whose node is the root and goes to the caller.
constexpr uint32_t kTopWG = 512;
constexpr uint32_t kTopNodes = 2 * kTopWG;
constexpr uint32_t kTopLog = 10;
static_assert(kTopNodes == 1u << kTopLog, "a chunk is a full subtree");
__global__ void __launch_bounds__(kTopWG) k_merkle_chunk(const MerkleDesc *__restrict__ table,
                                                         uint32_t n_trees,
                                                         const unsigned long long *__restrict__ row,
                                                         uint32_t k, uint32_t last,
                                                         uint32_t *__restrict__ nodes)
{
    __shared__ uint32_t node[kTopNodes][8];
    uint64_t c = 0;
    const MerkleDesc d = table[last ? blockIdx.x : merkle_group(row, n_trees, blockIdx.x, c)];
    const uint32_t t = threadIdx.x;
    const uint64_t left = merkle_nodes(d.n, k) - (c << kTopLog);
    uint32_t m = left < kTopNodes ? (uint32_t)left : kTopNodes;
    if (m <= 1 && !last) return;  // the whole workgroup: the node is already in place
    uint32_t *const base = nodes + 8ull * (d.leaf0 + (c << (kTopLog + k)));
    for (uint32_t j = t; j < m; j += kTopWG) {
        const State S = load_node(base + (8ull * j << k));
        store_node(node[j], S);
    }
    __syncthreads();
    while (m > 1) {  // uniform
        const uint32_t pairs = m >> 1;
        const bool act = t < pairs;
        State S;
        if (act) {
            State l, r;
#pragma unroll
            for (int j = 0; j < 8; ++j) { l.h[j] = node[2 * t][j]; r.h[j] = node[2 * t + 1][j]; }
            S = merkle_parent(l, r);
        }
        // an unpaired last node moves up unchanged, to index `pairs`
        uint32_t carry[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) carry[j] = node[m - 1][j];
        __syncthreads();
        if (act) store_node(node[t], S);
        if ((m & 1) && t == 0) {
#pragma unroll
            for (int j = 0; j < 8; ++j) node[pairs][j] = carry[j];
        }
        __syncthreads();
        m = pairs + (m & 1);
    }
    if (last) {
        if (t >= 64) return;
        State S = initial_state();
        if (d.n == 0) {
            sha256_bytes(true, nullptr, 0, S);  // no leaves: SHA-256 of the empty string
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) S.h[j] = node[0][j];
        }
        uint32_t *o = reinterpret_cast<uint32_t *>(d.root);
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (t == 0) o[j] = bswap32(S.h[j]);
    } else if (t < 8) {
        base[t] = node[0][t];
    }
}

}  // namespace ace
