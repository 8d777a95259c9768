// ace_internal.h -- device-side data layout shared by the kernels and the
// host entry points of libace.so.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ace {

constexpr int kWG = 256;          // threads per workgroup (4 wave64)
constexpr int kWavesPerWG = kWG / 64;
constexpr int kTile = 2048;       // transactions per tile of the binning/finalize passes
constexpr int kBins = 64;         // bins by inner block count nb = ceil((L+9)/64); bin 63 = nb >= 64
constexpr uint32_t kMaxSalt = 1024;
constexpr uint32_t kMaxInfo = 255;
constexpr uint32_t kMaxInfoBlocks = 5;  // ceil((64 + 255 + 1 + 9) / 64) - 1

// One block of transactions as the kernels see it, plus its prefixes in the
// concatenated index spaces of a multi-block call.
struct DevBlock {
    const uint8_t *msg;
    const uint64_t *off;
    const uint32_t *id;
    const uint8_t *tag;
    uint32_t *bitmask;
    unsigned long long *count;
    uint64_t n;      // transactions
    uint64_t tx0;    // first global transaction index
    uint64_t tile0;  // first tile (kTile transactions per tile)
    uint64_t wave0;  // first wave tile of the in-order verify (64 per wave)
};

// How the local verify form shares a call's wave tiles among its workgroups.
// Workgroups first .. first + slots - 1 run at once and have one run of
// consecutive tiles among them, `base` tiles each and one more for the first
// `extra` of all.
struct LocalShare {
    uint32_t groups;
    uint32_t base;
    uint32_t extra;
    uint32_t slots;
};
constexpr uint32_t kLocalUnits = 64;  // most wave tiles per workgroup: 4,096 transactions

// `slots`: workgroups that run at once.  As many rounds of them as the wave
// tiles need, every workgroup with the same share, so that the last round is
// as full as the first.
__host__ __device__ inline LocalShare local_share(uint64_t waves, uint32_t slots)
{
    const uint32_t w = (uint32_t)waves;  // at most 2^26 of 64 transactions and 2^24 part-filled ones
    const uint32_t rounds = (w + slots * kLocalUnits - 1) / (slots * kLocalUnits);
    LocalShare s;
    s.groups = slots * (rounds ? rounds : 1u);
    s.base = w / s.groups;
    s.extra = w - s.base * s.groups;
    s.slots = slots;
    return s;
}

// The tiles of one workgroup.  A round deals out its run like cards, one to four
// consecutive tiles at a time, and each deal starts at another workgroup, so that
// input ordered by message length, with its long messages in one place or in
// alternating runs, gives every workgroup about the same work.  One consecutive
// share each, 1M transactions took 812 us sorted by length and 770 with the long
// ones in one place; dealt out 241 and 154 (shuffled 243 and 140).
//   tiles per deal   four where a workgroup has four to eight, one for each SIMD
//                    of its CU (a long message's chain takes the time there, and
//                    tiles apart cost it 4 us of 74), else two: the balance of
//                    single ones (four 169 us where two take 150, in one place)
//                    without their price where every block is an allocation of
//                    its own (256 blocks of 7.66M transactions 2,010 us, two
//                    1,715-1,755, consecutive 1,750).
//   starts           multiples of 27907/65536 of the round's workgroups, of 1,500
//                    tried the one that spreads long and short runs of equal
//                    length (1/128 of a deal to eight of them) most evenly; with
//                    the same start every time, 1M transactions in runs of 128
//                    tiles took 540 us against 360 (shuffled 341).
struct LocalTiles {
    uint32_t first_tile, slot, slots, shift, dealt, count;
};
__host__ __device__ inline LocalTiles local_tiles(const LocalShare &s, uint32_t group)
{
    LocalTiles t;
    const uint32_t first = group / s.slots * s.slots;  // of this round
    t.first_tile = first * s.base + (first < s.extra ? first : s.extra);
    t.slot = group - first;
    t.slots = s.slots;
    t.shift = s.base < 2 ? 0u : s.base < 4 ? 1u : s.base <= 8 ? 2u : 1u;
    t.dealt = s.base >> t.shift << t.shift;  // the others singly, from the first workgroup on
    t.count = s.base + (group < s.extra ? 1u : 0u);
    return t;
}
// Tile u of a workgroup, u < count; ascends with u.
__host__ __device__ inline uint32_t local_tile(const LocalTiles &t, uint32_t u)
{
    if (u >= t.dealt) return t.first_tile + u * t.slots + t.slot;
    const uint32_t deal = u >> t.shift;
    uint32_t at = t.slot + (((deal * 27907u & 0xFFFFu) * t.slots) >> 16);
    if (at >= t.slots) at -= t.slots;
    return t.first_tile + ((deal * t.slots + at) << t.shift) + (u & ((1u << t.shift) - 1u));
}

// Sizes of a call that a captured graph reads from device memory (they
// change from replay to replay while the kernel arguments stay fixed).
struct BatchHdr {
    uint32_t n_blocks;
    uint32_t pad_;
    uint64_t total_tx;
    uint64_t total_tiles;
    uint64_t total_waves;
    LocalShare share;
};

// Blocks of one call: a single block travels inline in the kernel arguments,
// several blocks in a device table.  When `hdr` is set, the block count and
// totals come from it and every block from the table.
struct Batch {
    DevBlock one;
    const DevBlock *table;
    const BatchHdr *hdr;
    uint32_t n_blocks;
    uint64_t total_tx;
    uint64_t total_tiles;
    uint64_t total_waves;
    LocalShare share;
};

// Control words of a bucketed pass (start of the workspace).  The per-tile
// bin counts live beside them in the workspace (see k_bin_count).
struct Ctrl {
    uint32_t bincount[kBins];  // transactions per bin (k_bin_scan)
    uint32_t ostart[kBins];    // bins in order o = 63 - bin (longest first): padded start
    uint32_t ocount[kBins];    // real transactions
    uint32_t opad[kBins];      // count rounded up to a multiple of 64
    uint32_t total_pos;        // sum of opad
    uint32_t work;             // wave-tile counter of the persistent verify
    uint32_t pad_[62];
};

// Persistent verify kernel: most wave tiles per atomic grab while a wave
// works on bin b (0: no cap), a kernel argument set from the launch tuning.
struct GrabCaps {
    uint8_t cap[kBins];
};

// HKDF parameters shared by all identities of a keyset (kernel argument), laid
// out by the host as big-endian message words so that the kernels assemble no
// bytes: the salt's key block K0 (RFC 2104) or, for a salt longer than the
// block, its padded message blocks (FIPS 180-4 sec. 5.1.1), and the expand
// input info || 0x01 padded as it follows the 64-byte key block.
constexpr uint32_t kMaxSaltBlocks = (kMaxSalt + 9 + 63) / 64;
struct HkdfParams {
    uint32_t salt_blocks;  // 0: salt_w[0..15] is K0; else padded blocks of a long salt
    uint32_t info_blocks;
    uint32_t salt_w[16 * kMaxSaltBlocks];
    uint32_t info_w[16 * kMaxInfoBlocks];
};

// Several HKDF parameter sets in one launch (one per grid row): short salts
// and infos only, so that the set fits the kernel's argument block.
constexpr uint32_t kMultiStreams = 16;
constexpr uint32_t kMultiSalt = 64;
constexpr uint32_t kMultiInfo = 64;
constexpr uint32_t kMultiInfoBlocks = (kMultiInfo + 1 + 9 + 63) / 64;
struct StreamParams {
    static constexpr uint32_t salt_blocks = 0;  // at most one block: K0 itself
    uint32_t info_blocks;
    uint32_t salt_w[16];
    uint32_t info_w[16 * kMultiInfoBlocks];
};
struct MultiHkdf {
    uint32_t first;  // index of s[0] among the call's streams
    uint32_t count;
    StreamParams s[kMultiStreams];
};

// Derived per-workgroup constants of an HKDF parameter set (built in LDS).
// The expand blocks (info || 0x01 and its padding) are the same for every
// identity, so they are held as their whole schedules with the round
// constants added: info_kw[q][t] = K[t] + W_q[t].
struct HkdfPrep {
    uint32_t salt_ipad[8];
    uint32_t salt_opad[8];
    alignas(16) uint32_t info_kw[kMaxInfoBlocks][64];
    uint32_t info_blocks;
};

// One transaction in bin order, written by the scatter pass so that the
// verify kernel reads contiguous records instead of gathering offsets and
// identities from scattered lines.
constexpr uint32_t kRecWide = 0xFFFFFFFFu;     // len: a wide message, re-read the offsets
constexpr uint64_t kRecMaxLen = 0x7FFFFFFFu;   // messages this long or longer are always wide
constexpr uint32_t kRecNearEnd = 0x80000000u;  // len flag: the block's message area ends within
                                               // kOverread bytes after this message
constexpr uint32_t kRecInvalid = 0xFFFFFFFFu;  // id: the transaction cannot be valid
struct TxRec {
    uint64_t addr;  // address of the first message byte
    uint32_t len;   // message length | kRecNearEnd, or kRecWide
    uint32_t id;    // identity index, or kRecInvalid
};

// Bytes past a message's end that the block loads of its last blocks may
// read: 17 dwords from the aligned start of the last block, whose message
// part is at least L - 64 * (nb - 1) > -9 bytes, give at most 76.
constexpr uint64_t kOverread = 80;

struct KeySource {
    const uint32_t *mid;   // [n_id][16] midstates, or NULL when keys come from rev
    const uint8_t *rev;    // [n_id][32] root entropy (per-transaction derivation)
    uint32_t n_id;
};

// A chunk of block descriptors passed by value to the kernel that writes
// them into the device table (no host staging buffer is needed).
constexpr int kDescChunk = 24;
struct DescChunk {
    DevBlock d[kDescChunk];
    uint32_t first;
    uint32_t count;
};

// Occupancy targets (waves per SIMD) that the hash kernels reach without
// spilling when the block computation is the looped form; the register
// allocator is asked for them explicitly because on its own it trades
// occupancy for scheduling freedom (about 120 VGPRs, 4 waves).
#ifndef ACE_WAVES_HINTS
#define ACE_WAVES_HINTS 1
#endif
#if ACE_WAVES_HINTS
#define ACE_WAVES(n) __attribute__((amdgpu_waves_per_eu(n, n)))
#else
#define ACE_WAVES(n)
#endif

__host__ __device__ inline uint32_t bin_of_length(uint64_t L)
{
    uint64_t nb = (L + 9 + 63) >> 6;
    return (uint32_t)(nb >= (uint64_t)kBins ? kBins : nb) - 1u;
}

}  // namespace ace
