// Parameter-server side of Algorithm 1: chunk-indexed Huffman decoding with an LDS lookup
// table (one lane per chunk), and the average of the reconstructed user gradients.
#include "co3_dev.h"
#include "kernels.h"

#include <type_traits>

#define DE_BLOCK 512           // most lanes of a workgroup of k_decode
#define DE_MIN_BLOCK 256       // load_tables wants this many threads

__device__ __forceinline__ const Co3Code *dcode_of(const void *codes, int u)
{
    return reinterpret_cast<const Co3Code *>(reinterpret_cast<const char *>(codes) + (size_t)u * CO3_CODE_BYTES);
}

// ------------------------------------------------------------------------------------------
// Per-lane stream window in LDS.  The stream is read in 16-byte blocks (4 pieces of 32 bits; piece q
// holds stream bits [32q, 32q+32), first bit on top; in memory the words are little-endian u64, so
// the two pieces of a word are swapped).  Each lane keeps the 4 most recent blocks of its chunk in
// a 16-dword ring, stored in descending piece order (piece q at ring index 16 - (q mod 16), and a
// copy of the piece with q mod 16 == 0 at index 0) so that pieces q+1 and q are ring entries j and
// j+1 of one two-address LDS read.  The rings of a wavefront are interleaved: entry j of lane l is
// dword j*64 + l of the wavefront's area, so the bank of an access depends on the lane only and
// lanes at different ring positions never conflict.  Blocks are requested one run (16 symbols, 32
// with the two-symbol table) ahead of their use, at a cadence that is the same for all lanes of the
// wavefront, so the global-load latency hides behind the decoding of the previous run.
// ------------------------------------------------------------------------------------------
#define RING_ROWS 17
#define RING_ROW_DW CO3_WAVE     // dwords between consecutive ring entries of one lane
#define DE_GROUP 16          // symbols per run: one ring refill point, one 16-byte store
#define DE_MISS_LEN 255u     // length field of a table entry that does not resolve a symbol
#define DE_PAIR_BITS 12      // prefix length of the two-symbol table used for alphabets of at most 16 symbols
// Table lookups between two reads of the ring: 4 x 14 bits lie in a window of 64.  That holds for hits alone: after a
// codeword that the table does not resolve (up to CO3_MAX_CODE_LEN bits) the window is read anew where it may fall short.
#define DE_REFILL 4
enum { DE_SHORT = 0, DE_LONG = 1, DE_PAIRS = 2, DE_RETRY = 3 };   // fast-path variants of decode_range

// AHEAD = 0: the blocks that the next run may need are requested, up to two, 16 bytes at any place.
// AHEAD = 4: 64 aligned bytes at a time, which wait in registers.  A full chip's lanes, each at a chunk of its own, have
// more 128-byte lines open than its L2 holds, and every visit of a line may fetch it again: 16 x 25 M E4M3 (a stream of
// 337 MB) read 1.18 GB in 306 us, now 1.01 GB in 281; a chip that is not full pays for the registers' shuffling (32 x
// 1 M E3M1 29 | 31 us) and keeps to 0, as the two-symbol table does (10 x 11.2 M E3M0 49 | 52).  With 128 bytes at a
// time the kernel took 305, with 32 291.
template <int AHEAD>
struct LaneStream {
    const uint4 *blocks;   // the user's stream from relative block 0 (the one that holds the chunk start) on, as 16-byte blocks
    uint64_t base_bit;     // stream position of relative block 0
    uint32_t nblocks;      // relative blocks inside the buffer; beyond read as zeros
    uint32_t phase;        // AHEAD: position of relative block 0 in its aligned group of AHEAD blocks
    uint32_t *slot;        // this lane's ring in LDS
    uint32_t rel;          // current bit position relative to block 0
    uint32_t loaded;       // relative blocks [loaded-4, loaded) are in the ring
    uint32_t have;         // blocks [loaded, loaded + have) are in ahead[] or on their way there
    uint4 ahead[AHEAD ? AHEAD : 2];

    __device__ __forceinline__ uint4 fetch(uint32_t relblk) const
    {
        return relblk < nblocks ? blocks[relblk] : make_uint4(0u, 0u, 0u, 0u);
    }
    __device__ __forceinline__ void put(uint32_t relblk, uint4 v)
    {
        uint32_t top = 16u - (relblk & 3u) * 4u;   // ring index of the block's first piece
        slot[(top - 3) * RING_ROW_DW] = v.z;
        slot[(top - 2) * RING_ROW_DW] = v.w;
        slot[(top - 1) * RING_ROW_DW] = v.x;
        slot[top * RING_ROW_DW] = v.y;
        if (top == 16u) slot[0] = v.y;
    }
    // the next block into the ring (have > 0)
    __device__ __forceinline__ void pop()
    {
        put(loaded, ahead[0]);
#pragma unroll
        for (int k = 0; k + 1 < (AHEAD ? AHEAD : 2); ++k) ahead[k] = ahead[k + 1];
        ++loaded;
        --have;
    }
    // AHEAD = 0: all that was requested into the ring
    __device__ __forceinline__ void land()
    {
        if (have >= 1u) put(loaded, ahead[0]);
        if (have == 2u) put(loaded + 1u, ahead[1]);
        loaded += have;
        have = 0;
    }
    // make pieces [.., need_dw) resident (synchronous; only used off the fast path).  Callers ask for
    // at most block cur+3, so the block overwritten (loaded-4) always lies behind the position.
    __device__ __forceinline__ void ensure(uint32_t need_dw)
    {
        if (AHEAD == 0) land();
        while (loaded * 4u < need_dw) {
            if (AHEAD && have) pop();
            else {
                put(loaded, fetch(loaded));
                ++loaded;
            }
        }
    }
    // words: the user's stream of cap_words 64-bit words, an even number
    __device__ __forceinline__ void open(const uint64_t *words, int64_t cap_words, uint64_t p0)
    {
        const uint64_t b0 = p0 >> 7, all = (uint64_t)cap_words / 2;
        blocks = reinterpret_cast<const uint4 *>(words) + b0;
        nblocks = b0 < all ? (uint32_t)(all - b0 < 0xffffffffull ? all - b0 : 0xffffffffull) : 0u;
        phase = AHEAD ? (uint32_t)(reinterpret_cast<uintptr_t>(blocks) >> 4) & (AHEAD - 1u) : 0u;
        base_bit = b0 << 7;
        rel = (uint32_t)(p0 & 127u);
        have = 0;
        uint4 a = fetch(0), b = fetch(1), c = fetch(2), d = fetch(3);
        put(0, a);
        put(1, b);
        put(2, c);
        put(3, d);
        loaded = 4;
    }
    // Start of a run of DE_GROUP symbols: what was requested at an earlier boundary enters the ring, so that it holds
    // four blocks from the current one on (the blocks they replace lie behind the position), and more is requested.
    __device__ __forceinline__ void group_boundary()
    {
        const uint32_t want = (rel >> 7) + 4u;
        if (AHEAD == 0) {
            land();
            if (loaded < want) {
                ahead[0] = fetch(loaded);
                have = 1;
                if (loaded + 1u < want) {
                    ahead[1] = fetch(loaded + 1u);
                    have = 2;
                }
            }
            return;
        }
        if (loaded < want && have) {
            pop();
            if (loaded < want && have) pop();
        }
        if (have == 0u) {
            const uint32_t cnt = AHEAD - ((phase + loaded) & (AHEAD - 1u));
            if (cnt == AHEAD && loaded + AHEAD <= nblocks) {
#pragma unroll
                for (int k = 0; k < AHEAD; ++k) ahead[k] = blocks[loaded + k];
            } else {                               // the first group, the end of the buffer
#pragma unroll
                for (int k = 0; k < AHEAD; ++k)
                    if ((uint32_t)k < cnt) ahead[k] = fetch(loaded + k);
            }
            have = cnt;
        }
    }
    // what a stretch of long codewords needs and has been requested is waited for
    __device__ __forceinline__ void hurry()
    {
        if (AHEAD == 0) land();
        else ensure((((rel + 240u) >> 7) + 1u) * 4u);
    }
    __device__ __forceinline__ uint64_t pos() const { return base_bit + rel; }
    // the 32 stream bits at the current position
    __device__ __forceinline__ uint32_t peek32() const
    {
        const uint32_t *pc = slot + (~(rel >> 5) & 15u) * RING_ROW_DW;
        uint64_t two = ((uint64_t)pc[RING_ROW_DW] << 32) | (uint64_t)pc[0];
        return (uint32_t)((two << (rel & 31u)) >> 32);
    }
    // The 64 stream bits at the negated position m = -rel.  With d = (rel - 1) / 32, whose ring index is bits
    // 5..8 of m, they lie in pieces d, d+1, d+2: three LDS reads and two funnel shifts by m mod 32.
    __device__ __forceinline__ uint64_t window64(uint32_t m) const
    {
        const uint32_t row = (m >> 5) & 15u;
        const uint32_t *pc = slot + row * RING_ROW_DW;
        const uint32_t d0 = pc[RING_ROW_DW], d1 = pc[0], d2 = slot[((row - 1u) & 15u) * RING_ROW_DW];
        return ((uint64_t)__builtin_amdgcn_alignbit(d0, d1, m) << 32) | __builtin_amdgcn_alignbit(d1, d2, m);
    }
    __device__ __forceinline__ uint32_t piece(uint32_t d) const { return slot[(16u - (d & 15u)) * RING_ROW_DW]; }
    __device__ __forceinline__ uint64_t peek64()
    {
        uint32_t d = rel >> 5, o = rel & 31u;
        ensure(d + 3u);
        uint64_t hi = ((uint64_t)piece(d) << 32) | (uint64_t)piece(d + 1u);
        uint64_t lo = (uint64_t)piece(d + 2u);
        return o ? ((hi << o) | (lo >> (32u - o))) : hi;
    }
};

// LDS-resident decoder tables of one code.  BITS: longest prefix the lookup table resolves.  The code
// blob stores a table of at most CO3_LUT_BITS_MAX bits; a workgroup that has LDS to spare widens it
// (DE_WIDE_BITS) while loading, so that fewer codewords take the canonical search.
#define DE_WIDE_BITS 14
// What the table leaves out lies above all it resolves (canonical codewords grow with their length): a second one,
// indexed by the distance from there, resolves codewords of up to as many bits as ENTRIES2 entries reach, and no more
// than are left of a window after the lookups since it was read.  It takes the place of a search over the lengths'
// limits, five LDS reads one after the other: one user's ResNet-18 in E4M3 (some wavefronts miss at most symbols) 60 ->
// 44 us, ten users' 119 -> 100, four users' under shared codes 105 -> 92.  Making it costs a workgroup a third of a
// microsecond: chunks of less than 256 symbols do without (10 x 11.2 M in chunks of 64 95 | 101 us).
template <int BITS, int ENTRIES2>
struct DecTablesT {
    static constexpr int kBits = BITS, kEntries2 = ENTRIES2;
    static constexpr bool kSecond = ENTRIES2 > 1;
    static constexpr int kBits2 = 64 - (DE_REFILL - 1) * BITS < 32 ? 64 - (DE_REFILL - 1) * BITS : 32;
    alignas(16) uint16_t lut[1 << BITS];
    uint16_t lut2[ENTRIES2];      // (1: none)
    uint32_t from2, shift2, n2;   // entry (prefix of 32 bits - from2) >> shift2, below n2 (0: none)
    uint64_t first_code[65];
    uint16_t count[66];
    uint16_t base[66];
    uint8_t sorted[256];
    uint64_t lim_incl[65];   // largest 64-bit window (codeword left-aligned, ones below) of a codeword of length <= l
    uint32_t maxlen, lut_bits;
};
typedef DecTablesT<CO3_LUT_BITS_MAX, 1> DecTablesPairs;     // beside the two-symbol table
typedef DecTablesT<CO3_LUT_BITS_MAX, 256> DecTables;      // shared per-layer codes: four of them a workgroup

template <class Tables>
__device__ __forceinline__ void load_tables(Tables &t, const Co3Code *cd)
{
    constexpr uint32_t BITS = Tables::kBits;
    const uint32_t lb = cd->lut_bits > CO3_LUT_BITS_MAX ? CO3_LUT_BITS_MAX : (cd->lut_bits < 1 ? 1 : cd->lut_bits);
    const uint32_t ml = cd->maxlen > 64 ? 64 : cd->maxlen;
    // table prefix here: the stored one, widened up to BITS when the code has longer codewords
    const uint32_t nb = (BITS > CO3_LUT_BITS_MAX && ml > lb) ? (ml < BITS ? ml : BITS) : lb;
    // Everything is requested before anything is stored: one trip to memory in all (at least 256 threads).  The
    // widened entries come from the stored ones and from the codewords that they leave out; reading a stored entry
    // and searching the lengths for each of the 2^14 took 8 to 10 us of a workgroup (32 x 1 M E3M1 44 -> 36 us,
    // 16 x 25 M E4M3 356 -> 324).
    constexpr uint32_t PIECES = sizeof(Co3Code::lut) / 8;                  // 4 stored entries each (blobs are 8-byte aligned)
    constexpr int ROUNDS = (PIECES + DE_MIN_BLOCK - 1) / DE_MIN_BLOCK;
    const uint2 *lut_g = reinterpret_cast<const uint2 *>(cd->lut);
    const int x = (int)threadIdx.x;
    const uint32_t step = blockDim.x;
    uint2 v[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const uint32_t q = (uint32_t)x + r * step;
        v[r] = q < PIECES && q * 4u < (1u << lb) ? lut_g[q] : make_uint2(0u, 0u);
    }
    const uint64_t fc = x < 65 ? cd->first_code[x] : 0;
    const uint16_t cn = x < 66 ? cd->count[x] : (uint16_t)0, ba = x < 66 ? cd->base[x] : (uint16_t)0;
    const uint8_t so = x < 256 ? cd->sorted[x] : (uint8_t)0;
    if (x < 65) t.first_code[x] = fc;
    if (x < 66) {
        t.count[x] = cn;
        t.base[x] = ba;
    }
    if (x < 256) t.sorted[x] = so;
    if (x == 0) {
        t.maxlen = ml;
        t.lut_bits = nb;
    }
    const uint32_t wide = nb - lb;                                         // each stored entry fills 2^wide
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const uint32_t q = (uint32_t)x + r * step;
        if (q >= PIECES || q * 4u >= (1u << lb)) continue;
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k) {
            uint32_t e = ((k < 2u ? v[r].x : v[r].y) >> (16 * (k & 1))) & 0xffffu;
            if ((e >> 8) == 0u) e = DE_MISS_LEN << 8;                      // longer than the prefix, or invalid
            const uint32_t at = q * 4u + k;
            if (at >= (1u << lb)) continue;                                // (a stored table of two entries)
            if (wide == 0u) {
                t.lut[at] = (uint16_t)e;
            } else if (wide == 1u) {
                reinterpret_cast<uint32_t *>(t.lut)[at] = e | (e << 16);
            } else {
                const uint32_t e2 = e | (e << 16);
                for (uint32_t h = 0; h < (1u << wide) / 4u; ++h)
                    reinterpret_cast<uint2 *>(t.lut)[(at << (wide - 2)) + h] = make_uint2(e2, e2);
            }
        }
    }
    const bool make2 = Tables::kSecond && ml > nb;
    __syncthreads();
    if (wide != 0u) {
        // the codewords of lengths lb+1 .. nb, a thread each, enter where their prefixes lie
        for (uint32_t l = lb + 1; l <= nb; ++l)
            for (uint32_t k = (uint32_t)x; k < t.count[l]; k += step) {
                const uint64_t code = t.first_code[l] + k;
                const uint16_t e = (uint16_t)((l << 8) | t.sorted[(t.base[l] + k) & 255u]);
                if (code < (1ull << l))
                    for (uint32_t h = 0; h < (1u << (nb - l)); ++h) t.lut[((uint32_t)code << (nb - l)) + h] = e;
            }
    }
    // (beside that, by the other end of the workgroup; the caller's barrier is the next)
    const int xr = BITS > CO3_LUT_BITS_MAX ? (int)step - 1 - x : x;
    if (ml > nb) {                    // only codes with codewords beyond the table prefix use the limits
        for (int l = xr; l < 65; l += (int)step) {
            int j = l < (int)ml ? l : (int)ml;
            while (j >= 1 && t.count[j] == 0) --j;     // canonical order: shorter codewords are numerically below
            uint64_t lim = 0;
            if (j >= 1) {
                const uint64_t last = t.first_code[j] + t.count[j] - 1;
                lim = j == 64 ? last : (last << (64 - j)) | ((~0ull) >> j);
            }
            t.lim_incl[l] = lim;
        }
    }
    if (Tables::kSecond && x == 0 && !make2) t.n2 = t.from2 = t.shift2 = 0u;
    if (make2) {
        const int lane = x & (CO3_WAVE - 1);
        const uint64_t end_nb = t.first_code[nb] + t.count[nb];          // uniform
        const uint64_t left = (1ull << nb) - end_nb;                     // prefixes of nb bits that are left out
        uint32_t top = nb;
        while (top < ml && top < (uint32_t)Tables::kBits2 && (left << (top + 1u - nb)) <= (uint64_t)Tables::kEntries2) ++top;
        const bool some = end_nb < (1ull << nb) && top > nb;             // (also of a damaged blob: within the array)
        const uint32_t n2 = some ? (uint32_t)left << (top - nb) : 0u;
        if (x == 0) {
            t.from2 = some ? (uint32_t)end_nb << (32u - nb) : 0u;
            t.shift2 = 32u - top;
            t.n2 = n2;
        }
        if (some) {
            // of every length the end of its range, as prefixes of `top` bits: lane l holds that of length l
            const bool mid = lane > (int)nb && lane <= (int)top;
            const uint64_t end = mid ? (t.first_code[lane] + t.count[lane]) << (top - lane) : 0ull;
            const uint64_t from = end_nb << (top - nb);
            const uint32_t mine = end < from ? 0u : end - from > 0xffffull ? 0xffffu : (uint32_t)(end - from);
            for (uint32_t i = (uint32_t)xr; i < n2; i += step) {
                uint32_t l = nb + 1u;
                for (uint32_t k = nb + 1u; k <= top; ++k)
                    l += i >= (uint32_t)__builtin_amdgcn_readlane((int)mine, (int)k) ? 1u : 0u;
                uint32_t e = DE_MISS_LEN << 8;
                if (l <= top) {
                    const uint64_t off = ((from + i) >> (top - l)) - t.first_code[l];
                    if (off < (uint64_t)t.count[l]) e = (l << 8) | t.sorted[(t.base[l] + (uint32_t)off) & 255u];
                }
                t.lut2[i] = (uint16_t)e;
            }
        }
    }
}

// Two-symbol table for small alphabets (most pairs of codewords fit DE_PAIR_BITS bits there): entry i
// describes the stream that starts with the DE_PAIR_BITS-bit prefix i.
//   bits 0..7 first symbol, 8..15 second symbol, 16..23 length of the first codeword (DE_MISS_LEN when
//   the prefix does not resolve it), 24..31 length of both codewords together, 0 when the prefix does
//   not hold the whole second codeword.
// NIB (symbols of at most four bits): both symbols share the low byte instead, the second one in its
// upper half, the form in which the averaging workspace stores them.
// The second codeword is looked up with the bits after the first one, zero-filled: a codeword that
// ends inside the prefix is determined by its own bits alone (prefix-free code).
template <bool NIB>
__device__ __forceinline__ void build_pairs(const DecTablesPairs &t, uint32_t *pairs)
{
    const uint32_t down = DE_PAIR_BITS - t.lut_bits;
    for (uint32_t i = threadIdx.x; i < (1u << DE_PAIR_BITS); i += blockDim.x) {
        const uint32_t e1 = t.lut[i >> down];
        const uint32_t l1 = e1 >> 8;
        uint32_t entry = DE_MISS_LEN << 16;
        if (l1 != DE_MISS_LEN) {
            entry = (e1 & 0xffu) | (l1 << 16);
            const uint32_t i2 = (i << l1) & ((1u << DE_PAIR_BITS) - 1u);
            const uint32_t e2 = t.lut[i2 >> down];
            const uint32_t l2 = e2 >> 8;
            if (l2 != DE_MISS_LEN && l1 + l2 <= DE_PAIR_BITS)
                entry |= ((e2 & 0xffu) << (NIB ? 4 : 8)) | ((l1 + l2) << 24);
        }
        pairs[i] = entry;
    }
}

// Canonical decoding of a codeword longer than the table prefix: the first length l whose l-bit
// prefix lies within that length's codeword range.  Returns the length, 0 if there is none.
template <class Tables>
__device__ __forceinline__ int decode_long(const Tables &t, uint64_t window, uint32_t *sym)
{
    for (uint32_t l = t.lut_bits + 1; l <= t.maxlen; ++l) {
        uint64_t off = (window >> (64 - l)) - t.first_code[l];
        if (off < (uint64_t)t.count[l]) {
            *sym = t.sorted[(t.base[l] + (uint32_t)off) & 255u];
            return (int)l;
        }
    }
    return 0;
}

// Careful decoding of `count` <= 16 symbols (any codeword length, any stream content): used for runs
// that the fast path could not vouch for and for the ragged end of a chunk.  Leaves blocks
// cur .. cur+2 resident.  Symbols are returned 4 per word, first in the lowest byte.
template <class Tables, class Stream>
__device__ __forceinline__ void decode_run_careful(const Tables &t, Stream &ls, int shift, int count, bool &ok,
                                                   uint32_t w[4])
{
    w[0] = w[1] = w[2] = w[3] = 0;
    for (int k = 0; k < count; ++k) {
        ls.ensure((ls.rel >> 5) + 2u);
        uint32_t e = t.lut[ls.peek32() >> shift];
        uint32_t l = e >> 8, s = e & 0xffu;
        if (l == DE_MISS_LEN) {
            l = (uint32_t)decode_long(t, ls.peek64(), &s);
            if (l == 0) {
                ok = false;
                l = 1;
                s = 0;
            }
        }
        ls.rel += l;
        uint32_t sh = s << (8 * (k & 3));
        if ((k >> 2) == 0) w[0] |= sh;
        else if ((k >> 2) == 1) w[1] |= sh;
        else if ((k >> 2) == 2) w[2] |= sh;
        else w[3] |= sh;
    }
    ls.ensure(((ls.rel >> 7) + 3u) * 4u);
}

// One lookup in the two-symbol table.  win: the stream from the negated position m on; read anew from the ring
// every DE_REFILL lookups (of at most DE_PAIR_BITS bits each).  An entry that holds only its first codeword is
// completed from a lookup of its own, in a branch that the wavefront skips when no lane needs it and that leaves
// a whole window behind.  mw: the last position at which the ring was read.
template <bool NIB, class Stream>
__device__ __forceinline__ uint32_t pair_step(const Stream &ls, const uint32_t *pairs, uint64_t &win, uint32_t &m,
                                              uint32_t &mw, bool &bad)
{
    uint32_t e = pairs[win >> (64 - DE_PAIR_BITS)];
    uint32_t l = e >> 24, drop = l;
    if (l == 0u) {
        const uint32_t l1 = (e >> 16) & 0xffu;
        if (l1 == DE_MISS_LEN) {     // not even the first codeword: the careful path takes the run
            bad = true;
            l = 2u;
        } else {
            const uint32_t e2 = pairs[(win << l1) >> (64 - DE_PAIR_BITS)];
            uint32_t l2 = (e2 >> 16) & 0xffu;
            if (l2 == DE_MISS_LEN) {
                bad = true;
                l2 = 1u;
            }
            e = (e & 0xffu) | ((e2 & 0xffu) << (NIB ? 4 : 8));
            l = l1 + l2;
        }
        drop = 0u;
        mw = m - l;
        win = ls.window64(mw);
    }
    m -= l;
    win <<= drop & 63u;
    return e;
}

// One lane decodes symbols [i0, i1) of its chunk; the stream is open at symbol i0.  Symbols leave in
// runs of 16: run r is stored at out + r * run_step (run_step = 16 gives the plain contiguous layout;
// the tiled layout used between decoding and averaging interleaves the runs of the 64 chunks of a
// wavefront so that each store instruction of the wavefront covers one contiguous KiB).  A range
// that does not start or end on a run boundary (tensor boundaries with one code per tensor, the end
// of the vector) takes the careful path for the partial runs and stores them byte by byte.
//
// The fast path decodes a run without a residency check per symbol and validates it afterwards:
// every window it read must lie inside the blocks that were resident when the run started, and
// every window must have started a codeword.  Otherwise the run is decoded again by the careful
// path from the saved position.  Codewords longer than the table prefix are resolved by a
// second table or a canonical search (the lengths' upper limits are ordered), in a branch the wavefront skips when
// no lane needs it: in place, symbol by symbol (DE_LONG), or after every four symbols (DE_RETRY).
//
// DE_SHORT is the instance for codes whose longest codeword fits the table prefix: there a miss can
// only come from an invalid stream; it advances by DE_MISS_LEN, more than 16 hits can, which the
// validation catches.  DE_PAIRS reads the two-symbol table `pairs`: one lookup per two symbols and one
// refill point per 32 symbols (with at most four bits per symbol on average the blocks requested at one
// boundary cover the symbols up to the next one); a lookup whose prefix does not hold both codewords
// takes the second one from a lookup of its own (in a branch the wavefront skips when no lane needs
// it), and a codeword longer than the prefix sends the run to the careful path.
template <int MODE, class Tables, class Stream>
__device__ __forceinline__ void decode_range(const Tables &t, Stream &ls, int i0, int i1, uint8_t *out,
                                             int64_t run_step, bool &ok, const uint32_t *pairs = nullptr)
{
    static_assert(DE_REFILL * Tables::kBits <= 64 && DE_REFILL == 4, "a window holds the lookups between two refills");
    static_assert(DE_GROUP * Tables::kBits < DE_MISS_LEN, "a miss must advance more than a run of hits can");
    constexpr bool AGAIN = MODE == DE_RETRY, SECOND = Tables::kSecond;
    const int shift = 32 - (int)t.lut_bits;
    int i = i0;
    // cnt < 16 symbols from symbol i on, inside one run
    auto partial = [&](int cnt) {
        ls.group_boundary();
        uint32_t w[4];
        decode_run_careful(t, ls, shift, cnt, ok, w);
        uint8_t *dst = out + (int64_t)(i >> 4) * run_step + (i & 15);
        for (int k = 0; k < cnt; ++k) {
            uint32_t word = (k >> 2) == 0 ? w[0] : (k >> 2) == 1 ? w[1] : (k >> 2) == 2 ? w[2] : w[3];
            dst[k] = (uint8_t)(word >> (8 * (k & 3)));
        }
        i += cnt;
    };
    if ((i & 15) != 0 && i < i1) partial(16 - (i & 15) < i1 - i ? 16 - (i & 15) : i1 - i);
    if (MODE == DE_PAIRS) {
#pragma unroll 1
        for (; i + 2 * DE_GROUP <= i1; i += 2 * DE_GROUP) {
            ls.group_boundary();
            const uint32_t rel0 = ls.rel;
            uint32_t w[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
            uint32_t m = 0u - rel0, mw = m;
            uint64_t win = 0;
            bool bad = false;
#pragma unroll
            for (int b = 0; b < DE_GROUP; ++b) {
                if (b % DE_REFILL == 0) win = ls.window64(mw = m);
                const uint32_t e = pair_step<false>(ls, pairs, win, m, mw, bad);
                w[b >> 1] = __builtin_amdgcn_alignbit(e, w[b >> 1], 16);
            }
            ls.rel = 0u - m;
            if (bad || 96u - mw > ls.loaded * 128u) {   // rare
                ls.rel = rel0;
                decode_run_careful(t, ls, shift, DE_GROUP, ok, w);
                decode_run_careful(t, ls, shift, DE_GROUP, ok, w + 4);
            }
            uint8_t *dst = out + (int64_t)(i >> 4) * run_step;
            *reinterpret_cast<uint4 *>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
            *reinterpret_cast<uint4 *>(dst + run_step) = make_uint4(w[4], w[5], w[6], w[7]);
        }
    }
#pragma unroll 1
    for (; i + DE_GROUP <= i1; i += DE_GROUP) {
        ls.group_boundary();
        // a stretch of long codewords (the last run took more than nine bits a symbol): what has just been
        // requested is waited for, which costs less than a run by the careful path
        if (MODE != DE_PAIRS && ls.rel + 240u > ls.loaded * 128u) ls.hurry();
        const uint32_t rel0 = ls.rel;
        uint32_t w[4] = {0u, 0u, 0u, 0u};
        // Work with the negated position m = -rel.  The next 64 stream bits wait in registers and are read anew
        // every DE_REFILL lookups, so that the chain from symbol to symbol holds one LDS access, the table's, in
        // place of two (one user of 65,536 elements 26.6 -> 19 us, 16 x 25 M E4M3 391 -> 381, 10 x 11.2 M E3M0 54 -> 49).
        uint32_t m = 0u - rel0, mw = m;
        uint64_t win = 0;
        bool bad = false;
        if (MODE == DE_PAIRS) {
#pragma unroll
            for (int b = 0; b < DE_GROUP / 2; ++b) {
                if (b % DE_REFILL == 0) win = ls.window64(mw = m);
                const uint32_t e = pair_step<false>(ls, pairs, win, m, mw, bad);
                w[b >> 1] = __builtin_amdgcn_alignbit(e, w[b >> 1], 16);
            }
        } else {
        // Codeword longer than the table prefix, at the start of the window w64: mostly from the second table.  Else the
        // first length whose largest left-aligned codeword is not below the window.  (The limits do not decrease with
        // the length and stay put beyond the longest codeword, so counting the limits below the window gives the
        // length; without the second table nearly all end within four bits of the prefix, compared without a loop.)
        // `again`: the window is not known to hold all of it and is read anew for that.
        auto search = [&](uint64_t &w64, bool again) -> uint32_t {
            if constexpr (SECOND) {
                const uint32_t i2 = ((uint32_t)(w64 >> 32) - t.from2) >> t.shift2;
                if (i2 < t.n2) {
                    const uint32_t e2 = t.lut2[i2];
                    if ((e2 >> 8) != DE_MISS_LEN) return e2;
                }
            }
            if (again) w64 = ls.window64(mw = m);
            const uint32_t l0 = t.lut_bits + 1u;
            uint32_t l = l0;
#pragma unroll
            for (uint32_t k = 0; k < 4u; ++k) l += w64 > t.lim_incl[l0 + k] ? 1u : 0u;
            if (l == l0 + 4u)
                for (uint32_t j = l0 + 4u; j < t.maxlen; ++j) l += w64 > t.lim_incl[j] ? 1u : 0u;
            const uint64_t off = (w64 >> (64u - l)) - t.first_code[l];
            if (off < (uint64_t)t.count[l]) return (l << 8) | t.sorted[(t.base[l] + (uint32_t)off) & 255u];
            bad = true;                   // no codeword starts here
            return 1u << 8;
        };
        // DE_RETRY tests for misses once per DE_REFILL symbols, after which the lane goes on one by one from the
        // first; DE_LONG tests at every symbol, and each lookup has to wait for the test of the last.  With the wide
        // table a miss is rare in data that the code was made for (about one in 2,000 symbols of an 8-bit format):
        // DE_LONG | DE_RETRY 16 x 25 M E4M3 306 | 284 us, 32 x 1 M E3M1 38 | 32; but one user's 62 tensors in E4M3, some
        // with stretches of long codewords, 44 | 54.  With the narrow table (one miss in 200 symbols) it is DE_LONG.
#pragma unroll
        for (int q = 0; q < DE_GROUP / DE_REFILL; ++q) {
            win = ls.window64(mw = m);
            uint32_t any = 0u, es[DE_REFILL];
#pragma unroll
            for (int b = 0; b < DE_REFILL; ++b) {
                uint32_t e = t.lut[(uint32_t)(win >> 32) >> shift];
                uint32_t drop = e >> 8;
                if (MODE == DE_LONG && drop == DE_MISS_LEN) {   // skipped by the wavefront when no lane is here
                    if constexpr (SECOND) {
                        if (mw - m > 64u - Tables::kBits2) win = ls.window64(mw = m);
                        e = search(win, true);
                        drop = e >> 8;
                        // the window is read anew where what is left of it may not hold the lookups to come
                        if (b + 1 < DE_REFILL && mw - (m - drop) + (DE_REFILL - 1 - b) * Tables::kBits > 64u) {
                            mw = m - drop;
                            win = ls.window64(mw);
                            drop = 0u;
                        }
                    } else {
                        win = ls.window64(m);
                        e = search(win, false);
                        drop = 0u;
                        mw = m - (e >> 8);
                        win = ls.window64(mw);
                    }
                }
                es[b] = e;
                any |= e;
                m -= e >> 8;
                win <<= drop & 63u;
                w[q] = __builtin_amdgcn_alignbit(e, w[q], 8);
            }
            if (AGAIN && (any & 0x8000u) != 0u) {      // of all lengths only that of a miss has its top bit set
                m = mw;
                int b = 0;                             // the first miss: what stands before it is right
#pragma unroll
                for (int k = 0; k < DE_REFILL - 1; ++k)
                    if (b == k && (es[k] & 0x8000u) == 0u) {
                        m -= es[k] >> 8;
                        b = k + 1;
                    }
                uint32_t e = DE_MISS_LEN << 8;
#pragma unroll 1
                for (;;) {
                    if ((e >> 8) == DE_MISS_LEN) {     // (hits since the last read have left win short of bits)
                        win = ls.window64(mw = m);
                        e = search(win, false);
                        if (!SECOND || (e >> 8) > (uint32_t)Tables::kBits2) win = ls.window64(mw = m - (e >> 8));
                        else win <<= e >> 8;
                    } else {
                        win <<= (e >> 8) & 63u;
                    }
                    m -= e >> 8;
                    w[q] = (w[q] & ~(0xffu << (8 * b))) | ((e & 0xffu) << (8 * b));
                    if (++b == DE_REFILL) break;
                    e = t.lut[(uint32_t)(win >> 32) >> shift];
                }
            }
        }
        }
        ls.rel = 0u - m;
        // every window read above (96 bits from the last one's position on) must have been resident
        if (bad || 96u - mw > ls.loaded * 128u ||
            (MODE == DE_SHORT && ls.rel - rel0 > DE_GROUP * Tables::kBits)) {   // rare
            ls.rel = rel0;
            decode_run_careful(t, ls, shift, DE_GROUP, ok, w);
        }
        *reinterpret_cast<uint4 *>(out + (int64_t)(i >> 4) * run_step) = make_uint4(w[0], w[1], w[2], w[3]);
    }
    if (i < i1) partial(i1 - i);
}

// A whole chunk of an alphabet of at most 16 symbols, written in the packed form of the averaging
// workspace: two symbols per byte (the earlier one in the low half), 32 symbols per 16-byte store, run r
// of 32 symbols at out + r * run_step.  One refill point per 32 symbols: with at most four bits per
// symbol on average the blocks requested at one boundary cover the symbols up to the next one.
__device__ __forceinline__ void decode_chunk_packed(const DecTablesPairs &t, LaneStream<0> &ls, int nsym, uint8_t *out,
                                                    int64_t run_step, bool &ok, const uint32_t *pairs)
{
    const int shift = 32 - (int)t.lut_bits;
    // cnt <= 32 symbols by the careful path, packed; the rest of the 16 bytes is zero
    auto careful = [&](int cnt, uint32_t w[4]) {
        uint32_t b[8];
        decode_run_careful(t, ls, shift, cnt < DE_GROUP ? cnt : DE_GROUP, ok, b);
        if (cnt > DE_GROUP) decode_run_careful(t, ls, shift, cnt - DE_GROUP, ok, b + 4);
        else b[4] = b[5] = b[6] = b[7] = 0u;
#pragma unroll
        for (int k = 0; k < 4; ++k) {      // bytes 0x0d0c0b0a, 0x0h0g0f0e -> nibbles 0xhgfedcba
            const uint32_t lo = b[2 * k], hi = b[2 * k + 1];
            const uint32_t l2 = (lo | (lo >> 4)) & 0x00ff00ffu, h2 = (hi | (hi >> 4)) & 0x00ff00ffu;
            w[k] = ((l2 | (l2 >> 8)) & 0xffffu) | (((h2 | (h2 >> 8)) & 0xffffu) << 16);
        }
    };
    int i = 0;
#pragma unroll 1
    for (; i + 2 * DE_GROUP <= nsym; i += 2 * DE_GROUP) {
        ls.group_boundary();
        const uint32_t rel0 = ls.rel;
        uint32_t w[4] = {0u, 0u, 0u, 0u};
        uint32_t m = 0u - rel0, mw = m;
        uint64_t win = 0;
        bool bad = false;
#pragma unroll
        for (int b = 0; b < DE_GROUP; ++b) {
            if (b % DE_REFILL == 0) win = ls.window64(mw = m);
            const uint32_t e = pair_step<true>(ls, pairs, win, m, mw, bad);
            w[b >> 2] = __builtin_amdgcn_alignbit(e, w[b >> 2], 8);
        }
        ls.rel = 0u - m;
        if (bad || 96u - mw > ls.loaded * 128u) {   // rare: see decode_range
            ls.rel = rel0;
            careful(2 * DE_GROUP, w);
        }
        *reinterpret_cast<uint4 *>(out + (int64_t)(i >> 5) * run_step) = make_uint4(w[0], w[1], w[2], w[3]);
    }
    if (i < nsym) {                        // ragged end of the vector
        ls.group_boundary();
        uint32_t w[4];
        careful(nsym - i, w);
        *reinterpret_cast<uint4 *>(out + (int64_t)(i >> 5) * run_step) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// TILED = false: sym_out is [U][stride] symbols in order.  TILED = true: sym_out is the averaging
// workspace, [U][tiles][chunk_syms/16][64 lanes][16 symbols] with tile = 64 consecutive chunks.
// PAIRS: the workgroup also builds the two-symbol table (launched for alphabets of at most 16
// symbols and chunks of at least 32); with TILED the workspace then holds two symbols per byte,
// [U][tiles][chunk_syms/32][64 lanes][32 symbols in 16 bytes].  SECOND: it makes the second table (larger alphabets, chunks
// of 256 symbols or more).  Without it a miss is searched as before there was one: with its tests left in (an empty table)
// 4 x 11.2 M in chunks of 64 took 104.8 us for 103.6, of codewords that all miss 274 for 269 (before: 104, 267).
template <bool TILED, bool PAIRS, bool SECOND, int AHEAD>
__global__ __launch_bounds__(DE_BLOCK) void k_decode(const uint64_t *__restrict__ words, int64_t cap_words,
                                                      const uint64_t *__restrict__ chunk_bitoff, int chunk_syms,
                                                      int64_t nchunks, int chunks_per_block, const void *__restrict__ codes,
                                                      int code_per_user, int64_t n, uint8_t *__restrict__ sym_out,
                                                      int64_t stride, int32_t *status)
{
    const int u = blockIdx.y;
    // tables first: their LDS offsets then fit the immediate field of the read instructions
    __shared__ struct {
        uint32_t pairs[PAIRS ? (1 << DE_PAIR_BITS) : 1];
        // one symbol per lookup: the widened table
        typename std::conditional<PAIRS, DecTablesPairs, DecTablesT<DE_WIDE_BITS, SECOND ? 256 : 1>>::type t;
    } lds;
    extern __shared__ __align__(256) uint32_t ring[];   // chunks_per_block * RING_ROWS
    auto &t = lds.t;
    uint32_t *const pairs = lds.pairs;

    // The chunk's stream position and its first blocks are requested before the tables are loaded, so
    // that the three memory latencies at the start of a workgroup overlap.
    const int64_t c = (int64_t)blockIdx.x * chunks_per_block + threadIdx.x;
    const bool active = (int)threadIdx.x < chunks_per_block && c < nchunks;   // further wavefronts load tables only
    const uint64_t *off = chunk_bitoff + (int64_t)u * (nchunks + 1);
    const uint64_t p0 = active ? off[c] : 0, p1 = active ? off[c + 1] : 0, all_bits = off[nchunks];
    LaneStream<AHEAD> ls;
    ls.slot = ring + (threadIdx.x / CO3_WAVE) * (RING_ROWS * RING_ROW_DW) + (threadIdx.x & (CO3_WAVE - 1));
    if (active) ls.open(words + (int64_t)u * cap_words, cap_words, p0);
    const int64_t first = c * chunk_syms;
    const int nsym = active ? (int)(n - first < chunk_syms ? n - first : chunk_syms) : 0;
    load_tables(t, dcode_of(codes, code_per_user ? u : 0));        // else one code shared by all users
    __syncthreads();
    if constexpr (PAIRS) {
        build_pairs<TILED>(t, pairs);
        __syncthreads();
    }
    if (!active) return;

    uint8_t *out;
    int64_t run_step;
    if (TILED) {
        const int64_t tile_bytes = (int64_t)CO3_WAVE * (PAIRS ? chunk_syms >> 1 : chunk_syms);
        out = sym_out + (int64_t)u * stride + (c >> 6) * tile_bytes + (c & 63) * 16;
        run_step = CO3_WAVE * 16;
    } else {
        out = sym_out + (int64_t)u * stride + first;
        run_step = 16;
    }
    // Whether the wavefront looks for codewords beyond the table at every symbol: where one of its chunks takes more than
    // eight bits a symbol, or half a bit a symbol more than the stream on average (chunks of 512: a third).  Chunks of
    // data that the code was made for scatter by a tenth to an eighth of a bit (256 symbols); those of tensors that it
    // was not made for lie beyond: one user's ResNet-18 in E4M3 44 us; with a line of 0.63 bits 53, of eight bits a
    // symbol alone 54; 10 x 11.2 M E5M2 of one law 98 | 99 | 96.  Five other layouts of 7 to 62 tensors whose scales lie
    // three decades apart, with this line | eight bits alone: E4M3 41 | 49, 69 | 69, 42 | 42, 59 | 59, 44 | 48 us, E5M2 44 |
    // 50, 80 | 85, 36 | 38, 50 | 50, 41 | 45; in E4M1, where a chunk is dense with fewer codewords beyond the table, 32.4 |
    // 30.3, 79 | 80, 31 | 29, 34 | 32, 36 | 38.  Smaller chunks scatter more and keep to eight bits.
    auto dense = [&]() -> bool {
        float line = 8.0f;
        if (SECOND) line = fminf(line, (float)all_bits / (float)n + 8.0f * rsqrtf((float)chunk_syms));
        return __any((float)(p1 - p0) > (float)nsym * line) != 0;
    };
    bool ok = true;
    if constexpr (PAIRS && TILED) decode_chunk_packed(t, ls, nsym, out, run_step, ok, pairs);
    else if constexpr (PAIRS) decode_range<DE_PAIRS>(t, ls, 0, nsym, out, run_step, ok, pairs);
    else if (t.maxlen <= t.lut_bits) decode_range<DE_SHORT>(t, ls, 0, nsym, out, run_step, ok);
    else if (dense()) decode_range<DE_LONG>(t, ls, 0, nsym, out, run_step, ok);
    else decode_range<DE_RETRY>(t, ls, 0, nsym, out, run_step, ok);
    if (!(ok && ls.pos() == p1)) co3_raise(status, CO3_EBADSTREAM);
}

// Decompression with one code per tensor shared by all users (Sec. III (ii) as stated).  The workgroup
// walks the tensors of its range of elements with the tables of four neighbouring tensors resident
// (tensor s in slot s mod 4): a lane decodes the part of its chunk that lies in the tensor at its
// position as soon as that tensor's tables are there, so the chunks on both sides of a tensor
// boundary are decoded at the same time, each lane reading the table of its own tensor; a chunk that
// straddles tensors goes on into the next tensor while that tensor's tables are in the window.  Lanes
// whose tensor is more than three tensors away from the first one of the range wait for the window:
// tensors much smaller than a workgroup's range (512 chunks) are better given a code together with a
// neighbour.
//
// The second tables are made for chunks of any size: the 12 bits of the first resolve so much less than the 14 of the
// per-user decoder that they pay even where a workgroup walks 65 tensors (one user of 300,000 elements in tensors of 2,000,
// E4M3, chunks of 64, 256: without 107, 1,240 us, with 97, 1,170).
#define DL_BLOCK 512
#define DL_SLOTS 4

// Compiled for the two workgroups that a unit's LDS holds.
template <bool TILED, int AHEAD>
__global__ __launch_bounds__(DL_BLOCK) __attribute__((amdgpu_waves_per_eu(4)))
void k_decode_layers(const uint64_t *__restrict__ words, int64_t cap_words, const uint64_t *__restrict__ chunk_bitoff,
                     int chunk_syms, int64_t nchunks, const void *__restrict__ codes, const int64_t *__restrict__ seg_off,
                     int nseg, int64_t n, uint8_t *__restrict__ sym_out, int64_t stride, int32_t *status)
{
    const int u = blockIdx.y;
    __shared__ DecTables t[DL_SLOTS];
    __shared__ uint32_t ring[DL_BLOCK * RING_ROWS];
    if (threadIdx.x < DL_SLOTS) {
        t[threadIdx.x].maxlen = 0;
        t[threadIdx.x].lut_bits = 1;
    }

    const int64_t c = (int64_t)blockIdx.x * DL_BLOCK + threadIdx.x;
    const bool active = c < nchunks;
    const uint64_t *off = chunk_bitoff + (int64_t)u * (nchunks + 1);
    LaneStream<AHEAD> ls;
    ls.slot = ring + (threadIdx.x / CO3_WAVE) * (RING_ROWS * RING_ROW_DW) + (threadIdx.x & (CO3_WAVE - 1));
    const int64_t first = c * chunk_syms;
    const int nsym = active ? (int)(n - first < chunk_syms ? n - first : chunk_syms) : 0;
    uint8_t *out;
    int64_t run_step;
    if (TILED) {
        out = sym_out + (int64_t)u * stride + (c >> 6) * ((int64_t)CO3_WAVE * chunk_syms) + (c & 63) * 16;
        run_step = CO3_WAVE * 16;
    } else {
        out = sym_out + (int64_t)u * stride + first;
        run_step = 16;
    }
    // tensors touched by the workgroup's range of elements (uniform)
    const int64_t b_first = (int64_t)blockIdx.x * DL_BLOCK * chunk_syms;
    int64_t b_last = b_first + (int64_t)DL_BLOCK * chunk_syms;
    b_last = (b_last < n ? b_last : n) - 1;
    const int b_lo = co3_find_seg(seg_off, nseg, b_first), b_hi = co3_find_seg(seg_off, nseg, b_last);

    bool ok = true;
    int cur = 0;                                                        // next symbol of the chunk to decode
    int cur_seg = nsym > 0 ? co3_find_seg(seg_off, nseg, first) : -1;   // the tensor that holds it
    if (nsym > 0) ls.open(words + (int64_t)u * cap_words, cap_words, off[c]);
    for (int sg = b_lo; sg <= b_hi; ++sg) {
        __syncthreads();                 // nobody reads the slot that is replaced any more
        if (sg == b_lo) {
            for (int k = 0; k < DL_SLOTS - 1 && sg + k <= b_hi; ++k)
                load_tables(t[(sg + k) & (DL_SLOTS - 1)], dcode_of(codes, sg + k));
        }
        if (sg + DL_SLOTS - 1 <= b_hi)
            load_tables(t[(sg + DL_SLOTS - 1) & (DL_SLOTS - 1)], dcode_of(codes, sg + DL_SLOTS - 1));
        __syncthreads();
        bool any_long = false;           // uniform
        for (int k = 0; k < DL_SLOTS; ++k) any_long |= t[k].maxlen > t[k].lut_bits;
        // a chunk that straddles tensors goes on at once while the next tensor's tables are in the window
        // (if it waited for the next step it would start its second part when all other lanes have finished
        // their whole chunks)
        while (cur < nsym && cur_seg >= sg && cur_seg < sg + DL_SLOTS) {
            const DecTables &tl = t[cur_seg & (DL_SLOTS - 1)];
            const int64_t seg_end = seg_off[cur_seg + 1] - first;
            const int i1 = seg_end < nsym ? (int)seg_end : nsym;
            if (i1 <= cur) break;        // boundaries that do not increase: the chunk stays unfinished and is reported
            if (any_long) decode_range<DE_LONG>(tl, ls, cur, i1, out, run_step, ok);
            else decode_range<DE_SHORT>(tl, ls, cur, i1, out, run_step, ok);
            cur = i1;
            if (cur < nsym) cur_seg = co3_find_seg(seg_off, nseg, first + cur);
        }
    }
    if (nsym > 0) {
        ok = ok && cur == nsym && ls.pos() == off[c + 1];
    }
    if (!ok) co3_raise(status, CO3_EBADSTREAM);
}

// ---- average of the reconstructed gradients: users added in index order, one division -----
// Average from the tiled workspace: one thread owns the 16 bytes of one run, 16 consecutive elements
// (NIB, two symbols per byte: 32).  A workgroup of PT_WAVES wavefronts takes that many consecutive runs
// of one tile of 64 chunks.
#define PT_WAVES(NIB) ((NIB) ? 2 : 4)

// TABLE != 0 (one tensor, i.e. one anchor per user): the values of every user's symbols are computed
// once per block into LDS, and an element costs one LDS read and one add.  TABLE = 1 keeps all K
// values; TABLE = 2 (larger alphabets) keeps the K/2 magnitudes and applies the sign bit after the
// read, halving the LDS footprint.  TABLE = 3 (several tensors): a step whose elements lie in one tensor takes
// its K/2 magnitudes of every user from LDS as TABLE = 2 does (U * K/2 values computed for 4096 * U symbols;
// 16 users of 11.2 M elements in 62 tensors, E4M3: 113 -> 76 us); the other steps look up a tensor per run or element.
//
// Bound by latency and, with many users, by issue: how many wavefronts a SIMD holds counts, and how many users' symbols
// are on their way at once (PT_AHEAD).  Registers are set by the runs that straddle tensors, though few do: an address
// per element kept from user to user, and 64-bit comparisons to find its tensor, had brought them to 227.  One user's
// symbols at a time | as now: one tensor, 32 users of 1 M E3M1 23 | 15.4 us, 16 of 25 M E4M3 121 | 101, 10 of 11.2 M E3M0
// 28.4 | 27.4; 62 tensors of 11.2 M elements in E4M3, one user 21 | 16.7, two 26.7 | 19.2, four 29 | 24, ten 55 | 45.6; six
// in E3M0 38 | 30.  Runs that straddle tensors read their symbols by themselves, a user at a time: taking what was requested
// cost the others more (4 M elements in tensors of 200, ten users E4M3 56 -> 62 us), requesting only where none straddles
// likewise (two users 16.0 -> 18.5).  In 33,333 tensors of three: E3M0 ten users 54 us.
//
// Wavefronts per SIMD that the compiler has to leave room for.  With NIB and a table four (128 registers): with three the
// long sums slow down (16 x 25 M E3M0 66 -> 75 us), with five registers are stored away (4 x 11.2 M 17.6 -> 20.2).  One
// user's bytes at a time seven, the most without that (eight: 25 M of one user 25 -> 29 us); four users' five (six 16 x 25 M
// E4M3 102 -> 106).  Several tensors three and four: what the straddling runs' registers allow.
template <int TABLE, bool NIB, int PT_AHEAD>
__global__ __launch_bounds__(PT_WAVES(NIB) * CO3_WAVE)
__attribute__((amdgpu_waves_per_eu(TABLE == 1 || TABLE == 2 ? (NIB ? 4 : PT_AHEAD == 1 ? 7 : 5) : (NIB ? 3 : 4))))
void k_ps_sum_tiled(const uint8_t *__restrict__ symt, int64_t n, int U, int64_t ws_stride, int chunk_syms, int64_t nruns,
                    const int32_t *__restrict__ anchor, const float *__restrict__ scale,
                    const int64_t *__restrict__ seg_off_g, int nseg, co3_fmt fmt, const float *acc_in, float divisor,
                    float *avg_out)
{
    constexpr int EPT = NIB ? 32 : 16;     // elements per thread
    constexpr int WAVES = PT_WAVES(NIB), PT_BLOCK = WAVES * CO3_WAVE;
    const FmtC fc(fmt);
    const int EM = fc.E + fc.M, M = fc.M, F = fc.F;
    const uint32_t cmask = (uint32_t)fc.codemax;
    const int runs_per_chunk = chunk_syms / EPT;
    const float recip = divisor > 0.f ? 1.0f / divisor : 0.f;
    const bool pow2 = (__float_as_uint(divisor) & 0x7fffffu) == 0u;      // (a whole number below 2^31)
    // value of symbol s of user u in tensor sg; with multipliers (scale != NULL) the level is divided by
    // the user's multiplier, one fp32 rounding
    auto value = [&](uint32_t s, int u, int sg) -> float {
        const int e_min = anchor[(int64_t)u * nseg + sg] - F + 1;
        float v = __uint_as_float(__float_as_uint(co3_code_value(s & cmask, e_min, M)) | ((s >> EM) << 31));
        if (scale) v = v / scale[(int64_t)u * nseg + sg];
        return v;
    };
    // symbol k of the 16 bytes w
    auto symbol = [&](const uint32_t (&w)[4], int k) -> uint32_t {
        return NIB ? (w[k >> 3] >> (4 * (k & 7))) & 0xfu : (w[k >> 2] >> (8 * (k & 3))) & 0xffu;
    };
    constexpr bool ONE = TABLE == 1 || TABLE == 2;               // one tensor, nothing to look up
    constexpr bool HALF = TABLE == 2 || TABLE == 3;              // the magnitudes alone
    __shared__ int64_t seg_cache[ONE ? 1 : CO3_SEG_CACHE];
    const int64_t *seg_off = ONE ? seg_off_g : co3_cache_segs(seg_off_g, nseg, seg_cache);
    extern __shared__ float value_of[];    // [U][K] or [U][K/2], TABLE only
    int table_seg = -1;                    // TABLE 3: the tensor whose values are there
    if (ONE) {
        const int sh = EM + (HALF ? 0 : 1);                    // (K is a power of two)
        for (int j = threadIdx.x; j < U << sh; j += PT_BLOCK) value_of[j] = value((uint32_t)j & ((1u << sh) - 1u), j >> sh, 0);
        __syncthreads();
    }
    // One block step covers one tile (64 chunks) x WAVES consecutive runs: each wavefront one run, each
    // lane one chunk (a chunk has a multiple of WAVES runs).  The WAVES * EPT results per chunk are
    // contiguous in the output; they pass through LDS so that every store instruction of a wavefront
    // writes 256 contiguous bytes.
    constexpr int ROW = WAVES * EPT;       // 64 elements in both layouts
    __shared__ float out_s[CO3_WAVE][ROW + 1];
    for (int64_t rb = (int64_t)blockIdx.x * PT_BLOCK; rb < nruns; rb += (int64_t)gridDim.x * PT_BLOCK) {
        // r enumerates (tile, run within chunk, lane) with the lane fastest: the workspace order
        const int64_t r = rb + threadIdx.x;
        const int lane = (int)(r & 63);
        const int wr = threadIdx.x >> 6;
        const int64_t q = r >> 6;
        const int run = (int)(q & (runs_per_chunk - 1));             // runs per chunk: a power of two
        const int64_t tile = q >> __builtin_ctz((unsigned)runs_per_chunk);
        const int64_t i0 = (tile * CO3_WAVE + lane) * chunk_syms + (int64_t)run * EPT;
        const uint8_t *src = symt + r * 16;
        // Users are taken PT_AHEAD at a time, their symbols requested together, the first ones before anything is looked
        // up: a step that waited for one user's after the other took 0.7 us a user where few steps fill the chip.  (A
        // single user: the registers for more cost 20 % where its steps fill the chip.)
        uint4 ahead[PT_AHEAD];
        auto request = [&](int u0) {
#pragma unroll
            for (int q = 0; q < PT_AHEAD; ++q)
                if (u0 + q < U) ahead[q] = ld_stream_u4(src + (int64_t)(u0 + q) * ws_stride);
        };
        if (i0 < n) request(0);
        // add(u, w): a user's 16 bytes
        auto each_user = [&](auto add) {
            for (int u0 = 0; u0 < U; u0 += PT_AHEAD) {
                if (u0) request(u0);
#pragma unroll
                for (int q = 0; q < PT_AHEAD; ++q) {
                    if (u0 + q >= U) break;
                    const uint32_t w[4] = {ahead[q].x, ahead[q].y, ahead[q].z, ahead[q].w};
                    add(u0 + q, w);
                }
            }
        };
        // the sum starts at zero, or continues a sum over users before these (acc_in may be avg_out: every
        // element is read and written by the same workgroup, the reads first)
        float acc[EPT];
#pragma unroll
        for (int k = 0; k < EPT; ++k) acc[k] = 0.f;
        if (acc_in && i0 < n) {
            if (i0 + EPT <= n) {
#pragma unroll
                for (int k = 0; k < EPT; k += 4) {
                    const float4 a = *reinterpret_cast<const float4 *>(acc_in + i0 + k);
                    acc[k] = a.x, acc[k + 1] = a.y, acc[k + 2] = a.z, acc[k + 3] = a.w;
                }
            } else {
#pragma unroll
                for (int k = 0; k < EPT; ++k)
                    if (i0 + k < n) acc[k] = acc_in[i0 + k];
            }
        }
        bool from_table = ONE;
        if (TABLE == 3) {
            // the elements of the whole step lie between those of its first and last lane
            const int64_t b0 = tile * CO3_WAVE * chunk_syms + (int64_t)(run - wr) * EPT;
            const int64_t b1 = b0 + (int64_t)(CO3_WAVE - 1) * chunk_syms + ROW - 1;
            const int bs = co3_find_seg(seg_off, nseg, b0 < n ? b0 : n - 1);
            from_table = bs == co3_find_seg(seg_off, nseg, b1 < n ? b1 : n - 1);     // the same for all threads
            if (from_table && bs != table_seg) {       // (every read of the last values lies before a barrier below)
                const int sh = EM + (HALF ? 0 : 1);            // (K is a power of two)
                for (int j = threadIdx.x; j < U << sh; j += PT_BLOCK)
                    value_of[j] = value((uint32_t)j & ((1u << sh) - 1u), j >> sh, bs);
                table_seg = bs;
                __syncthreads();
            }
        }
        int s_lo = 0, s_hi = 0;                // first and last tensor of the run
        if (!from_table) {
            s_lo = co3_find_seg(seg_off, nseg, i0 < n ? i0 : n - 1);       // (lanes past the end store nothing)
            s_hi = co3_find_seg(seg_off, nseg, i0 + EPT - 1 < n ? i0 + EPT - 1 : n - 1);
        }
        if (i0 >= n) {
        } else if (from_table) {
            each_user([&](int u, const uint32_t (&w)[4]) {
                const float *vu = value_of + u * (HALF ? fc.K >> 1 : fc.K);
#pragma unroll
                for (int k = 0; k < EPT; ++k) {
                    const uint32_t sy = symbol(w, k);
                    if (!HALF) acc[k] += vu[sy & ((uint32_t)fc.K - 1u)];
                    else acc[k] += __uint_as_float(__float_as_uint(vu[sy & cmask]) ^ (((sy >> EM) & 1u) << 31));
                }
            });
        } else if (s_lo == s_hi) {
            each_user([&](int u, const uint32_t (&w)[4]) {
                const int e_min = anchor[(int64_t)u * nseg + s_lo] - F + 1;
                const float c = scale ? scale[(int64_t)u * nseg + s_lo] : 1.0f;
                if (!scale && __all((uint32_t)(e_min + 125) <= (uint32_t)(253 - F))) {
                    // Anchors as the conversion makes them: the code in the exponent and mantissa of a float that is
                    // subnormal where the field is 0, times a power of two -- exact.  (21 -> 16 us for one user's 62
                    // tensors of 11.2 M elements.)
#pragma unroll
                    for (int k = 0; k < EPT; ++k) {
                        const uint32_t s = symbol(w, k);
                        acc[k] += ldexpf(__uint_as_float(((s & cmask) << (23 - M)) | ((s >> EM) << 31)), e_min + 126);
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < EPT; ++k) {
                        uint32_t s = symbol(w, k);
                        float val = co3_code_value(s & cmask, e_min, M);
                        val = __uint_as_float(__float_as_uint(val) | ((s >> EM) << 31));
                        acc[k] += scale ? val / c : val;
                    }
                }
            });
        } else {                           // the run straddles tensors: anchor per element
            uint32_t seg_of[EPT];          // looked up once, not for every user
            uint32_t sg = (uint32_t)s_lo;
            int next = s_lo < s_hi ? (int)(seg_off[sg + 1] - i0) : EPT;        // where the tensor after sg begins
#pragma unroll
            for (int k = 0; k < EPT; ++k) {
                while (k >= next) {
                    ++sg;
                    next = sg < (uint32_t)s_hi ? (int)(seg_off[sg + 1] - i0) : EPT;
                }
                seg_of[k] = sg;
            }
            for (int u = 0; u < U; ++u) {      // (few runs: their registers are not worth more requests at a time)
                const int32_t *anchor_u = anchor + (int64_t)u * nseg;
                const float *scale_u = scale ? scale + (int64_t)u * nseg : nullptr;
                uint4 v = *reinterpret_cast<const uint4 *>(src + (int64_t)u * ws_stride);
                uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int k = 0; k < EPT; ++k) {
                    asm volatile("" : "+v"(seg_of[k]));    // addresses made from it stay inside the loop (see above)
                    const uint32_t s = symbol(w, k);
                    float val = co3_code_value(s & cmask, anchor_u[seg_of[k]] - F + 1, M);
                    val = __uint_as_float(__float_as_uint(val) | ((s >> EM) << 31));
                    acc[k] += scale_u ? val / scale_u[seg_of[k]] : val;
                }
            }
        }
        if (divisor > 0.f) {
            // one division, rounded once: by a power of two (a single user among them) it is a multiplication
            if (pow2) {
#pragma unroll
                for (int k = 0; k < EPT; ++k) acc[k] *= recip;
            } else {
#pragma unroll
                for (int k = 0; k < EPT; ++k) acc[k] = acc[k] / divisor;
            }
        }
#pragma unroll
        for (int k = 0; k < EPT; ++k) out_s[lane][wr * EPT + k] = acc[k];
        __syncthreads();
        const int64_t run0 = (int64_t)(run - wr) * EPT;      // first element (within a chunk) of the block's runs
#pragma unroll 4
        for (int j = 0; j < CO3_WAVE; j += WAVES) {
            const int idx = (j + wr) * CO3_WAVE + (threadIdx.x & 63);   // element of the [64][ROW] tile, row-major
            const int cc = idx / ROW, e = idx % ROW;
            const int64_t i = (tile * CO3_WAVE + cc) * chunk_syms + run0 + e;
            if (i < n) __builtin_nontemporal_store(out_s[cc][e], avg_out + i);   // not read again here
        }
        __syncthreads();
    }
}

// Chunks (lanes) per workgroup of k_decode.  A chip that the chunks do not fill: as few wavefronts a workgroup as
// spread them over all compute units (the lookups of the wavefronts of one unit share its LDS).  A full chip:
// eight, so that two workgroups share a unit and one loads its tables while the other decodes; us with 8 | 16
// wavefronts: 16 x 25 M E4M3 324 | 349, 10 x 11.2 M E4M3 118 | 126, 1 x 100 M E5M2 91 | 99, 10 x 11.2 M E3M0 48.4 | 49.3
// (ten wavefronts 325, 125, 108, 52; twelve 350, 131, 92, 54).
static int decode_chunks_per_block(int64_t nchunks, int U)
{
    const int known = co3_device_cus(), cus = known > 0 ? known : 256;
    const int64_t waves = (nchunks + CO3_WAVE - 1) / CO3_WAVE * U;
    const int64_t w = (waves + cus - 1) / cus;
    return (int)(w < 1 ? 1 : w > DE_BLOCK / CO3_WAVE ? DE_BLOCK / CO3_WAVE : w) * CO3_WAVE;
}

// Lanes of a workgroup of k_decode: those that have no chunk help with the tables.  The two-symbol table has 4,096
// entries to be made from the code's (chunks of 64, 256 | 512 lanes: 3,000 elements 10.9 | 9.8 us, 32 users of 30,000
// 9.2 | 8.0).
static int decode_lanes(int per_block, bool pairs)
{
    const int least = pairs ? DE_BLOCK : DE_MIN_BLOCK;
    return per_block < least ? least : per_block;
}

// seg_off != NULL selects one code per tensor (codes[tensor], shared by the users) instead of codes[user]
hipError_t co3_launch_decode(const uint64_t *words, int64_t cap_words, const uint64_t *chunk_bitoff, int chunk_syms,
                             const void *codes, const int64_t *seg_off, int nseg, int K, int64_t n, int U,
                             uint8_t *sym_out, int64_t stride, int tiled, int32_t *status, hipStream_t st)
{
    const int64_t nchunks = (n + chunk_syms - 1) / chunk_syms;
    if (nchunks <= 0) return hipSuccess;
    const int per_block = decode_chunks_per_block(nchunks, U);
    const unsigned blocks = (unsigned)((nchunks + per_block - 1) / per_block);
    // 64 bytes at a time (LaneStream): where the chunks fill the chip more than once and a lane's lie a line or more apart
    const int known = co3_device_cus(), cus = known > 0 ? known : 256;
    const bool wide_requests = chunk_syms >= 256 && (nchunks + CO3_WAVE - 1) / CO3_WAVE * U >= 20 * (int64_t)cus;
    const unsigned lblocks = (unsigned)((nchunks + DL_BLOCK - 1) / DL_BLOCK);
    // Shared codes, whose tables take the LDS of all but two workgroups a unit: the same from half as many wavefronts on,
    // and where a workgroup decodes more than it walks from tensor to tensor (E4M3, us with 16 | 64 bytes at a time: 4 x
    // 11 M in tensors of 500,000 elements, chunks of 64 59 | 63, of 128 82 | 77, of 256 98 | 80, of 512 (1,344 wavefronts)
    // 124 | 127; 10 x 11 M, tensors of 100,000, chunks of 256 200 | 188; 4 x 11 M, tensors of 20,000 and 5,000, chunks of
    // 256 217 | 227 and 550 | 616; one user of 11 M 66 | 68).
    const bool wide_layers = chunk_syms >= 128 && (nchunks + CO3_WAVE - 1) / CO3_WAVE * U >= 8 * (int64_t)cus &&
                             n / (nseg > 0 ? nseg : 1) >= (int64_t)DL_BLOCK * chunk_syms / 4;
#define CO3_DECODE_LAUNCH(T, P, S, A)                                                                              \
    hipLaunchKernelGGL((k_decode<T, P, S, A>), dim3(blocks, U), dim3(decode_lanes(per_block, P)),                     \
                       (size_t)per_block * RING_ROWS * sizeof(uint32_t), st, words, cap_words, chunk_bitoff, chunk_syms, \
                       nchunks, per_block, codes, code_per_user, n, sym_out, stride, status)
#define CO3_LAYERS_LAUNCH(T, A)                                                                                    \
    hipLaunchKernelGGL((k_decode_layers<T, A>), dim3(lblocks, U), dim3(DL_BLOCK), 0, st, words, cap_words, chunk_bitoff, \
                       chunk_syms, nchunks, codes, seg_off, nseg, n, sym_out, stride, status)
    Co3LaunchTimer tm(CO3_K_DECODE, st);
    // one code for everything, shared by the users: the per-user kernels with every user reading codes[0]
    const int code_per_user = seg_off == nullptr;
    if (seg_off && nseg == 1) seg_off = nullptr;
    if (seg_off && wide_layers) {
        if (tiled) CO3_LAYERS_LAUNCH(true, 4);
        else CO3_LAYERS_LAUNCH(false, 4);
    } else if (seg_off) {
        if (tiled) CO3_LAYERS_LAUNCH(true, 0);
        else CO3_LAYERS_LAUNCH(false, 0);
    }
    else if (co3_ws_packed(K, chunk_syms, 0)) {
        if (tiled) CO3_DECODE_LAUNCH(true, true, false, 0);
        else CO3_DECODE_LAUNCH(false, true, false, 0);
    } else if (chunk_syms < 256) {
        if (tiled) CO3_DECODE_LAUNCH(true, false, false, 0);
        else CO3_DECODE_LAUNCH(false, false, false, 0);
    } else if (wide_requests) {
        if (tiled) CO3_DECODE_LAUNCH(true, false, true, 4);
        else CO3_DECODE_LAUNCH(false, false, true, 4);
    } else {
        if (tiled) CO3_DECODE_LAUNCH(true, false, true, 0);
        else CO3_DECODE_LAUNCH(false, false, true, 0);
    }
#undef CO3_DECODE_LAUNCH
#undef CO3_LAYERS_LAUNCH
    return hipGetLastError();
}

hipError_t co3_launch_ps_sum_tiled(const uint8_t *symt, int64_t n, int U, int64_t ws_stride, int chunk_syms,
                                   const int32_t *anchor, const float *scale, const int64_t *seg_off, int nseg,
                                   co3_fmt fmt, int packed, const float *acc_in, float divisor, float *avg_out,
                                   hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const int64_t nchunks = (n + chunk_syms - 1) / chunk_syms;
    const int64_t ntiles = (nchunks + CO3_WAVE - 1) / CO3_WAVE;
    const int64_t nruns = ntiles * (chunk_syms >> (packed ? 5 : 4)) * CO3_WAVE;   // 16-byte pieces of one user
    const int threads = PT_WAVES(packed) * CO3_WAVE;
    int64_t b = (nruns + threads - 1) / threads;
    unsigned blocks = (unsigned)(b < 16384 ? b : 16384);
    Co3LaunchTimer tm(CO3_K_PS_SUM, st);
    const size_t full_bytes = (size_t)U * (size_t)(1 << (1 + fmt.exp_bits + fmt.mant_bits)) * sizeof(float);
    // Several tensors: the values of one in LDS pay where a workgroup's steps stay in it and there are users to share what
    // they cost, which is half the alphabet's values a user (us with | without; 11 M elements in tensors of 400,000: three
    // users E3M1 24.9 | 25.7, ten 39 | 45, six in E4M3 32.1 | 33.6; of 100,000: three users E3M0 25.5 | 25.8, E4M3 27.4 | 26.7,
    // eight 37.6 | 38.2; of 40,000: ten in E3M0 46.0 | 46.5, sixteen 60.5 | 61.8, E4M3 62.5 | 61.4; of 15,000: three 34.4 |
    // 31.5, ten 78 | 75; ResNet-18's 62: three in E3M0 25.1 | 25.4, ten 42.1 | 45.5, E4M3 three 27.2 | 26.4, ten 44.6 | 45.0).
    const int64_t each = n / (nseg > 0 ? nseg : 1);
    const bool few_values = fmt.exp_bits + fmt.mant_bits <= 5;
    const bool tables_pay = nseg > 1 && (few_values ? each >= 32768 && U >= (each >= 65536 ? 3 : 10) : each >= 65536 && U >= 6);
#define CO3_SUM_LAUNCH(T, P, A, BYTES)                                                                             \
    hipLaunchKernelGGL((k_ps_sum_tiled<T, P, A>), dim3(blocks), dim3(threads), BYTES, st, symt, n, U, ws_stride,  \
                       chunk_syms, nruns, anchor, scale, seg_off, nseg, fmt, acc_in, divisor, avg_out)
    const size_t half_bytes = full_bytes / 2;
    const int known = co3_device_cus(), cus = known > 0 ? known : 256;
    // A table of few values: four users at a time; one where there are many that long (E3M1, one | four at a time, four users
    // of 25 M 36.9 | 34.2 us, sixteen of 18 M 62 | 59.5, of 40 M 130.6 | 128.8, thirty-two of 18 M 111 | 107, but twenty-four
    // of 25 M 116 | 120, thirty-two 147 | 158).  Two at a time where the registers of more would cost wavefronts.
    const bool long_sums = U > 16 && blocks >= 20u * (unsigned)cus;
    if (packed) {       // alphabets of at most 16 symbols: the full table is 64 bytes per user
        if (nseg == 1 && U == 1) CO3_SUM_LAUNCH(1, true, 1, full_bytes);
        else if (nseg == 1 && full_bytes <= 4096) CO3_SUM_LAUNCH(1, true, 2, full_bytes);
        else if (tables_pay && half_bytes <= 32768) CO3_SUM_LAUNCH(3, true, 2, half_bytes);
        else if (U == 1) CO3_SUM_LAUNCH(0, true, 1, 0);
        else CO3_SUM_LAUNCH(0, true, 2, 0);
    } else if (nseg == 1 && U == 1) CO3_SUM_LAUNCH(1, false, 1, full_bytes);
    else if (nseg == 1 && full_bytes <= 4096 && long_sums) CO3_SUM_LAUNCH(1, false, 1, full_bytes);
    else if (nseg == 1 && full_bytes <= 4096) CO3_SUM_LAUNCH(1, false, 4, full_bytes);
    else if (nseg == 1 && half_bytes <= 32768) CO3_SUM_LAUNCH(2, false, 4, half_bytes);
    else if (tables_pay && half_bytes <= 32768) CO3_SUM_LAUNCH(3, false, 2, half_bytes);
    else if (U == 1) CO3_SUM_LAUNCH(0, false, 1, 0);
    else CO3_SUM_LAUNCH(0, false, 2, 0);
#undef CO3_SUM_LAUNCH
    return hipGetLastError();
}
