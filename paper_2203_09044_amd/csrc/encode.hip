// Compression h_Hf (Algorithm 1, user side): coded size of every tile of 1024 symbols, exclusive scan
// of the tile sizes per user, then bit packing.  In the packing pass one wavefront takes one tile (16
// symbols per lane): it looks the codewords up, scans the lengths and packs its bits in an LDS staging
// window -- its own, or one of four consecutive tiles -- from which every 64-bit word whose first bit
// lies in the window's tiles leaves, the last one completed with the leading codewords of the following
// symbols, so that each word of the stream is written exactly once, with plain coalesced stores.
#include "co3_dev.h"
#include "kernels.h"

#include <atomic>

#define EN_BLOCK 256
#define EN_WAVES (EN_BLOCK / CO3_WAVE)
#define EN_LSYM 16                             // symbols per lane
#define EN_STAGE_WORDS 128                     // staging window of a tile: 8192 bits = 8 bits/symbol on average
#define EN_LONG_STAGE_WORDS 448                // where the LDS is there anyway: 28 bits/symbol
static_assert(CO3_WAVE * EN_LSYM == CO3_PACK_SYMS, "tile geometry");
#define EN_WG_SYMS (EN_WAVES * CO3_PACK_SYMS)  // symbols of a workgroup's tiles
#define EN_WG_WORDS 640                        // staging window of a workgroup: 10 bits/symbol on average
#define EN_MOST_BLOCKS (CO3_PACK_GROUP / EN_WAVES) // blocks of a group
#define EN_ALL_WORDS 2016                      // its two windows, and the room of a block of up to 31 bits/symbol

__device__ __forceinline__ const Co3Code *code_of(const void *codes, int u)
{
    return reinterpret_cast<const Co3Code *>(reinterpret_cast<const char *>(codes) + (size_t)u * CO3_CODE_BYTES);
}

// Eight symbols stored two per byte (the earlier one in the low half) -> two words of four symbol bytes.
__device__ __forceinline__ void unpack_nib8(uint32_t w, uint32_t &b0, uint32_t &b1)
{
    const uint32_t lo = w & 0x0f0f0f0fu, hi = (w >> 4) & 0x0f0f0f0fu;      // symbols 0 2 4 6 / 1 3 5 7, one per byte
    b0 = (lo & 0xffu) | ((hi & 0xffu) << 8) | ((lo & 0xff00u) << 8) | ((hi & 0xff00u) << 16);
    b1 = ((lo >> 16) & 0xffu) | (((hi >> 16) & 0xffu) << 8) | ((lo >> 24) << 16) | ((hi >> 24) << 24);
}

// The 16 symbols from element i (a multiple of 16) on, all below n; NIB: the array holds two symbols per byte.
__device__ __forceinline__ void load_syms16_full(const uint8_t *su, int64_t i, bool nib, uint32_t s[4])
{
    if (nib) {
        const uint2 a = *reinterpret_cast<const uint2 *>(su + (i >> 1));
        unpack_nib8(a.x, s[0], s[1]);
        unpack_nib8(a.y, s[2], s[3]);
    } else {
        const uint4 a = *reinterpret_cast<const uint4 *>(su + i);
        s[0] = a.x; s[1] = a.y; s[2] = a.z; s[3] = a.w;
    }
}

__device__ __forceinline__ uint32_t load_sym1(const uint8_t *su, int64_t j, bool nib)
{
    return nib ? ((uint32_t)su[j >> 1] >> (4 * (int)(j & 1))) & 0xfu : (uint32_t)su[j];
}

// Loads the 16 symbols of this lane into s[0..4) (4 per word, first symbol in the low byte);
// returns how many lie below n.
__device__ __forceinline__ int load_syms16(const uint8_t *su, int64_t i, int64_t n, uint32_t s[4], bool nib = false)
{
    if (i + EN_LSYM <= n) {
        load_syms16_full(su, i, nib, s);
        return EN_LSYM;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) s[k] = 0;
    int c = 0;
    for (int64_t j = i; j < n; ++j, ++c) s[c >> 2] |= load_sym1(su, j, nib) << (8 * (c & 3));
    return c;
}

__device__ __forceinline__ void wave_lds_sync() { co3_wave_lds_sync(); }

__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += (uint64_t)__shfl_xor((long long)v, o, CO3_WAVE);
    return v;
}

// ---- pass 1: coded size of every tile; a wavefront takes 4 consecutive tiles with all loads in
// flight before the first table lookup.  The 16 tiles of a workgroup form a group: the kernel
// leaves each tile's offset within its group in tilesum[] and the group's size in groupsum[], so
// the serial scan of pass 2 runs over 16 times fewer entries. ------------------------------------
#define SZ_TILES 4
#define SZ_GROUP (EN_WAVES * SZ_TILES)        // tiles per workgroup = CO3_PACK_GROUP

__global__ __launch_bounds__(EN_BLOCK) void k_enc_sizes(const uint8_t *__restrict__ sym, int64_t n, int64_t stride,
                                                         const void *__restrict__ codes, int K,
                                                         uint64_t *__restrict__ tilesum, int64_t nblk,
                                                         uint64_t *__restrict__ groupsum, int64_t ngrp,
                                                         int32_t *status, int sym_nib, int newest_last)
{
    // (the order of the users: see co3_launch_encode)
    const int u = newest_last ? (int)(gridDim.y - 1 - blockIdx.y) : (int)blockIdx.y;
    const Co3Code *cd = code_of(codes, u);
    __shared__ uint8_t len_s[256];
    __shared__ uint8_t pairlen_s[256];     // symbols two per byte: both lengths together, bit 7 set when one of them is 0
    __shared__ uint32_t tile_bits[SZ_GROUP];
    len_s[threadIdx.x] = (int)threadIdx.x < K ? cd->len[threadIdx.x] : (uint8_t)0;
    if (threadIdx.x < SZ_GROUP) tile_bits[threadIdx.x] = 0;
    if (sym_nib) {
        const int lo = threadIdx.x & 15, hi = threadIdx.x >> 4;
        const uint32_t l0 = lo < K ? cd->len[lo] : 0u, l1 = hi < K ? cd->len[hi] : 0u;
        pairlen_s[threadIdx.x] = (uint8_t)((l0 + l1) | (l0 == 0u || l1 == 0u ? 0x80u : 0u));
    }
    __syncthreads();

    const int lane = threadIdx.x & (CO3_WAVE - 1);
    const int wave = threadIdx.x / CO3_WAVE;
    const int64_t tb0 = ((int64_t)blockIdx.x * EN_WAVES + wave) * SZ_TILES;
    const bool nib = sym_nib != 0;
    const uint8_t *su = sym + (int64_t)u * (nib ? stride / 2 : stride);
    uint32_t s[SZ_TILES][4];
    bool nocode = false;
    if (tb0 >= nblk) {                                // uniform: nothing for this wavefront
    } else if (nib && (tb0 + SZ_TILES) * CO3_PACK_SYMS <= n) {     // uniform: four complete tiles, two symbols per byte
        uint2 raw[SZ_TILES];
#pragma unroll
        for (int t = 0; t < SZ_TILES; ++t)
            raw[t] = *reinterpret_cast<const uint2 *>(su + (((tb0 + t) * CO3_PACK_SYMS + (int64_t)lane * EN_LSYM) >> 1));
#pragma unroll
        for (int t = 0; t < SZ_TILES; ++t) {
            uint32_t bits = 0, flags = 0;    // one lookup per byte
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const uint32_t e = pairlen_s[((c < 4 ? raw[t].x : raw[t].y) >> (8 * (c & 3))) & 0xffu];
                bits += e & 0x7fu;
                flags |= e;
            }
            nocode |= (flags & 0x80u) != 0u;
            bits = wave_sum_u32(bits);
            if (lane == 0) tile_bits[wave * SZ_TILES + t] = bits;
        }
    } else if ((tb0 + SZ_TILES) * CO3_PACK_SYMS <= n) {     // uniform: all four tiles are complete
#pragma unroll
        for (int t = 0; t < SZ_TILES; ++t) {
            // ordinary (cached) loads: the packing pass reads the same symbols next
            load_syms16_full(su, (tb0 + t) * CO3_PACK_SYMS + (int64_t)lane * EN_LSYM, nib, s[t]);
        }
#pragma unroll
        for (int t = 0; t < SZ_TILES; ++t) {
            uint32_t bits = 0, minlen = 255u;
#pragma unroll
            for (int c = 0; c < EN_LSYM; ++c) {
                uint32_t l = len_s[(s[t][c >> 2] >> (8 * (c & 3))) & 0xffu];
                bits += l;
                minlen = min(minlen, l);
            }
            nocode |= minlen == 0u;
            bits = wave_sum_u32(bits);
            if (lane == 0) tile_bits[wave * SZ_TILES + t] = bits;
        }
    } else {                                          // the end of the vector
        for (int t = 0; t < SZ_TILES && tb0 + t < nblk; ++t) {
            const int64_t i = (tb0 + t) * CO3_PACK_SYMS + (int64_t)lane * EN_LSYM;
            const int nvalid = i < n ? load_syms16(su, i, n, s[0], nib) : 0;
            uint32_t bits = 0;
#pragma unroll
            for (int c = 0; c < EN_LSYM; ++c) {
                uint32_t l = len_s[(s[0][c >> 2] >> (8 * (c & 3))) & 0xffu];
                bits += c < nvalid ? l : 0u;
                nocode |= c < nvalid && l == 0u;
            }
            bits = wave_sum_u32(bits);
            if (lane == 0) tile_bits[wave * SZ_TILES + t] = bits;
        }
    }
    if (nocode) co3_raise(status, CO3_ENOCODE);
    __syncthreads();
    if (threadIdx.x < SZ_GROUP) {
        const int64_t tb = (int64_t)blockIdx.x * SZ_GROUP + threadIdx.x;
        uint32_t before = 0, all = 0;
#pragma unroll
        for (int k = 0; k < SZ_GROUP; ++k) {
            const uint32_t b = tile_bits[k];
            before += k < (int)threadIdx.x ? b : 0u;
            all += b;
        }
        if (tb < nblk) tilesum[(int64_t)u * nblk + tb] = before;
        if (threadIdx.x == 0) groupsum[(int64_t)u * ngrp + blockIdx.x] = all;
    }
}

// The same pass for one code per tensor shared by all users (Sec. III (ii) as stated): a wavefront keeps
// the length table of the tensor it is in, reloading it when a tile lies in another tensor; symbols of
// a tile that straddles tensors read their lengths from the code blobs directly.
__global__ __launch_bounds__(EN_BLOCK) void k_enc_sizes_layers(const uint8_t *__restrict__ sym, int64_t n,
                                                                int64_t stride, const void *__restrict__ codes, int K,
                                                                const int64_t *__restrict__ seg_off_g, int nseg,
                                                                uint64_t *__restrict__ tilesum, int64_t nblk,
                                                                uint64_t *__restrict__ groupsum, int64_t ngrp,
                                                                int32_t *status)
{
    const int u = blockIdx.y;
    __shared__ uint32_t len_w[EN_WAVES][256 / 4];
    __shared__ uint32_t tile_bits[SZ_GROUP];
    __shared__ int64_t seg_cache[CO3_SEG_CACHE];
    if (threadIdx.x < SZ_GROUP) tile_bits[threadIdx.x] = 0;
    const int64_t *seg_off = co3_cache_segs(seg_off_g, nseg, seg_cache);
    __syncthreads();

    const int lane = threadIdx.x & (CO3_WAVE - 1);
    const int wave = threadIdx.x / CO3_WAVE;
    const int64_t tb0 = ((int64_t)blockIdx.x * EN_WAVES + wave) * SZ_TILES;
    const uint8_t *su = sym + (int64_t)u * stride;
    const uint8_t *len_b = reinterpret_cast<const uint8_t *>(len_w[wave]);
    bool nocode = false;
    int cached = -1;
    for (int t = 0; t < SZ_TILES && tb0 + t < nblk; ++t) {
        const int64_t t_lo = (tb0 + t) * CO3_PACK_SYMS;
        const int64_t t_hi = (t_lo + CO3_PACK_SYMS < n ? t_lo + CO3_PACK_SYMS : n) - 1;
        const int s_lo = co3_find_seg(seg_off, nseg, t_lo), s_hi = co3_find_seg(seg_off, nseg, t_hi);
        const int64_t i = t_lo + (int64_t)lane * EN_LSYM;
        uint32_t s[4];
        const int nvalid = i < n ? load_syms16(su, i, n, s) : 0;
        uint32_t bits = 0;
        if (s_lo == s_hi) {              // uniform
            if (cached != s_lo) {
                wave_lds_sync();
                len_w[wave][lane] = reinterpret_cast<const uint32_t *>(code_of(codes, s_lo)->len)[lane];
                wave_lds_sync();
                cached = s_lo;
            }
#pragma unroll
            for (int c = 0; c < EN_LSYM; ++c) {
                const uint32_t sy = (s[c >> 2] >> (8 * (c & 3))) & 0xffu;
                const uint32_t l = (int)sy < K ? len_b[sy] : 0u;
                bits += c < nvalid ? l : 0u;
                nocode |= c < nvalid && l == 0u;
            }
        } else if (nvalid > 0) {
            // a tile that straddles tensors: lengths from the code blobs.  The lane's 16 symbols mostly lie in
            // one tensor: then one lookup of the tensor and 16 independent loads (a lookup and a load per
            // symbol in turn put 16 memory latencies into this wavefront, and the kernel ends with its
            // slowest one)
            const int c_first = co3_find_seg(seg_off, nseg, i), c_last = co3_find_seg(seg_off, nseg, i + nvalid - 1);
            const uint8_t *len_first = code_of(codes, c_first)->len;
#pragma unroll
            for (int c = 0; c < EN_LSYM; ++c) {
                const uint32_t sy = (s[c >> 2] >> (8 * (c & 3))) & 0xffu;
                const uint8_t *lp = c_first == c_last ? len_first
                                                      : code_of(codes, co3_find_seg(seg_off, nseg, c < nvalid ? i + c : i))->len;
                const uint32_t l = c < nvalid && (int)sy < K ? lp[sy] : 0u;
                bits += l;
                nocode |= c < nvalid && l == 0u;
            }
        }
        bits = wave_sum_u32(bits);
        if (lane == 0) tile_bits[wave * SZ_TILES + t] = bits;
    }
    if (nocode) co3_raise(status, CO3_ENOCODE);
    __syncthreads();
    if (threadIdx.x < SZ_GROUP) {
        const int64_t tb = (int64_t)blockIdx.x * SZ_GROUP + threadIdx.x;
        uint32_t before = 0, all = 0;
#pragma unroll
        for (int k = 0; k < SZ_GROUP; ++k) {
            const uint32_t b = tile_bits[k];
            before += k < (int)threadIdx.x ? b : 0u;
            all += b;
        }
        if (tb < nblk) tilesum[(int64_t)u * nblk + tb] = before;
        if (threadIdx.x == 0) groupsum[(int64_t)u * ngrp + blockIdx.x] = all;
    }
}

// ---- pass 2: per user, exclusive scan of the group sizes (in place), stream length and capacity
// check --------------------------------------------------------------------------------------
#define SC_BLOCK 1024
#define SC_PER 8

__global__ __launch_bounds__(SC_BLOCK) void k_enc_scan(uint64_t *__restrict__ tilesum, int64_t nblk, int64_t cap_words,
                                                        uint64_t *__restrict__ chunk_bitoff, int64_t nchunks,
                                                        uint64_t *__restrict__ total_bits, int32_t *status)
{
    const int u = blockIdx.x;
    uint64_t *bs = tilesum + (int64_t)u * nblk;
    const int lane = threadIdx.x & (CO3_WAVE - 1);
    const int wave = threadIdx.x / CO3_WAVE;
    __shared__ uint64_t wave_tot[SC_BLOCK / CO3_WAVE];
    __shared__ uint64_t carry_s;
    if (threadIdx.x == 0) carry_s = 0;
    __syncthreads();

    // the sizes of the next step are requested before the current step is scanned
    uint64_t nxt[SC_PER];
#pragma unroll
    for (int k = 0; k < SC_PER; ++k) {
        const int64_t i = (int64_t)threadIdx.x * SC_PER + k;
        nxt[k] = i < nblk ? bs[i] : 0;
    }
    for (int64_t base = 0; base < nblk; base += SC_BLOCK * SC_PER) {
        int64_t i0 = base + (int64_t)threadIdx.x * SC_PER;
        uint64_t v[SC_PER];
        uint64_t mine = 0;
#pragma unroll
        for (int k = 0; k < SC_PER; ++k) {
            v[k] = nxt[k];
            mine += v[k];
        }
#pragma unroll
        for (int k = 0; k < SC_PER; ++k) {
            const int64_t i = i0 + (int64_t)SC_BLOCK * SC_PER + k;
            nxt[k] = i < nblk ? bs[i] : 0;
        }
        uint64_t incl = mine;   // wave inclusive scan of 64-bit values
#pragma unroll
        for (int o = 1; o < CO3_WAVE; o <<= 1) {
            uint64_t t = (uint64_t)__shfl_up((long long)incl, o, CO3_WAVE);
            if (lane >= o) incl += t;
        }
        if (lane == CO3_WAVE - 1) wave_tot[wave] = incl;
        __syncthreads();
        uint64_t off = carry_s, tile_tot = 0;
        for (int w = 0; w < SC_BLOCK / CO3_WAVE; ++w) {
            uint64_t t = wave_tot[w];
            if (w < wave) off += t;
            tile_tot += t;
        }
        uint64_t running = off + incl - mine;
#pragma unroll
        for (int k = 0; k < SC_PER; ++k) {
            if (i0 + k < nblk) bs[i0 + k] = running;
            running += v[k];
        }
        __syncthreads();
        if (threadIdx.x == 0) carry_s += tile_tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const uint64_t total = carry_s;
        total_bits[u] = total;
        chunk_bitoff[(int64_t)u * (nchunks + 1) + nchunks] = total;
        if ((total + 63) / 64 > (uint64_t)cap_words) co3_raise(status, CO3_ECAP);
    }
}

// ---- pass 3: bit packing ------------------------------------------------------------------
// Codewords of the lane's 16 symbols, concatenated four at a time.
// `entry(symbol, k)` returns the packed (codeword << 6 | length) of the lane's k-th symbol.
template <bool FULL, class Entry>
__device__ __forceinline__ void lookup_runs(Entry entry, const uint32_t s[4], int nvalid,
                                            uint64_t run[EN_LSYM / 4], uint32_t runbits[EN_LSYM / 4], uint32_t &mybits,
                                            bool &wide)
{
#pragma unroll
    for (int g = 0; g < EN_LSYM / 4; ++g) {
        uint64_t acc = 0;
        uint32_t nb = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            uint64_t e = (FULL || 4 * g + k < nvalid) ? entry((s[g] >> (8 * k)) & 0xffu, 4 * g + k) : 0ull;
            uint32_t l = (uint32_t)(e & 63u);
            acc = (acc << l) | (e >> 6);
            nb += l;
        }
        wide |= nb > 64u;
        run[g] = acc;
        runbits[g] = nb;
        mybits += nb;
    }
}

// The same for codes of at most 16 bits (then (codeword << 6 | length) sits in the low dword of a
// table entry and two codewords fit 32 bits): pairs are joined with 32-bit operations.
__device__ __forceinline__ void lookup_runs_short(const uint64_t *enc_s, const uint32_t s[4],
                                                  uint64_t run[EN_LSYM / 4], uint32_t runbits[EN_LSYM / 4],
                                                  uint32_t &mybits)
{
    const uint32_t *enc32 = reinterpret_cast<const uint32_t *>(enc_s);
#pragma unroll
    for (int g = 0; g < EN_LSYM / 4; ++g) {
        uint32_t e0 = enc32[2 * (s[g] & 0xffu)], e1 = enc32[2 * ((s[g] >> 8) & 0xffu)];
        uint32_t e2 = enc32[2 * ((s[g] >> 16) & 0xffu)], e3 = enc32[2 * (s[g] >> 24)];
        uint32_t l1 = e1 & 63u, l3 = e3 & 63u;
        uint32_t p01 = ((e0 >> 6) << l1) | (e1 >> 6);
        uint32_t p23 = ((e2 >> 6) << l3) | (e3 >> 6);
        uint32_t n23 = (e2 & 63u) + l3;
        uint32_t nb = (e0 & 63u) + l1 + n23;
        run[g] = ((uint64_t)p01 << n23) | (uint64_t)p23;
        runbits[g] = nb;
        mybits += nb;
    }
}

// Symbols stored two per byte (alphabets of at most 16 symbols: no codeword exceeds 15 bits): one lookup per
// byte in a table of codeword pairs, (both codewords joined << 6 | both lengths), the earlier symbol's
// codeword on top; the two pairs of four consecutive symbols make a run of at most 60 bits.
__device__ __forceinline__ void lookup_runs_pairs(const uint64_t *penc_s, uint2 raw, uint64_t run[EN_LSYM / 4],
                                                  uint32_t runbits[EN_LSYM / 4], uint32_t &mybits)
{
#pragma unroll
    for (int g = 0; g < EN_LSYM / 4; ++g) {
        const uint32_t w = (g < 2 ? raw.x : raw.y) >> (16 * (g & 1));
        const uint64_t p0 = penc_s[w & 0xffu], p1 = penc_s[(w >> 8) & 0xffu];
        const uint32_t l1 = (uint32_t)(p1 & 63u);
        const uint32_t nb = (uint32_t)(p0 & 63u) + l1;
        run[g] = ((p0 >> 6) << l1) | (p1 >> 6);
        runbits[g] = nb;
        mybits += nb;
    }
}

// ORs `nb` bits (right-aligned in `acc`, 1 <= nb <= 64) into the staging window at stream position
// `pos` (bits, relative to the first word of the tile); only words inside the window are touched.
template <int STAGE>
__device__ __forceinline__ void stage_bits(unsigned long long *stage, int64_t win_w0, uint64_t acc, int nb,
                                           uint64_t pos)
{
    uint64_t v = acc << (64 - nb);
    int64_t w = (int64_t)(pos >> 6) - win_w0;
    int o = (int)(pos & 63);
    if (w >= 0 && w < STAGE) atomicOr(&stage[w], (unsigned long long)(v >> o));
    if (o + nb > 64 && w + 1 >= 0 && w + 1 < STAGE) atomicOr(&stage[w + 1], (unsigned long long)(v << (64 - o)));
}

// ---- whole blocks of four tiles packed by a workgroup together ---------------------------------
// A window per wavefront made the packer short-lived wavefronts of 7,500 cycles, half of them spent before the first
// codeword: a workgroup takes up to four blocks in a row, its tables built once, the next block's symbols requested
// while one is packed, one barrier a block, and only the last block looks ahead: the unfinished last word of a block
// is handed to the window of the next.  What is the same for a wavefront is kept in scalar registers, and codewords are
// joined in table entries of 32 bits (16 symbols of a lane: 267 -> 175 vector instructions in an 8-bit format, 237 -> 117
// with two symbols per byte).  Fewer instructions alone gave nothing: a workgroup per block with the same packing took
// 198 and 49 us below.  10 x 11.2 M E3M0 52 -> 34 us, E4M3 57 -> 46; 16 x 25 M E4M3 199 -> 158 (737 MB at 4.7 TB/s, the
// rate of a copy); 4 x 11.2 M E4M3 under shared codes 50 -> 31.
//
// A block of more than 10 bits a symbol takes the windows' LDS alone (encoding 10 x 11.2 M in E4M3, a fifth | all of the
// blocks at 23 bits a symbol 136 -> 88 | 328 -> 155 us; with such blocks tile by tile one after the other 163 | 377).
//
// An entry is codeword << 8 | length; a codeword of 24 bits or more has only its length there and the top bit set.  A
// lane with such a codeword, or with two neighbours of 32 bits together, packs its symbols one by one.
#define EN_FAR_PAIR 0x60u                      // bits of the sum of two lengths
#define EN_FAR_ENTRY 0x80000000u
struct PackLds {
    uint64_t enc[256];                         // as in the code
    uint32_t tab[256];                         // per symbol; symbols two per byte: per pair of symbols
    unsigned long long win[EN_ALL_WORDS];      // word r of a window that begins at word b at b + EN_WG_WORDS - 1 - r
};

__device__ __forceinline__ uint32_t pack_entry(uint64_t code, uint32_t l)
{
    return l >= 24u ? EN_FAR_ENTRY | l : ((uint32_t)code << 8) | l;
}

// Two windows, of blocks in turn; one that takes the whole array, for a block that does not fit these.
#define EN_WIN_BITS ((EN_WG_WORDS + 2) * 64u)                       // distance of the two windows
#define EN_WIDE_BITS ((EN_ALL_WORDS - 2 - EN_WG_WORDS) * 64u)       // where the one window begins

// ORs the `nb` <= 64 bits of v (right-aligned) into the windows.  d: distance of their start from the end of the first
// window (for the others their beginning more), on return that of their end; what of v lies before the word that holds
// their end goes to the word before, which is the next one in the array.
__device__ __forceinline__ void pack_put(PackLds &L, uint64_t v, uint32_t nb, uint32_t &d)
{
    d -= nb;
    unsigned long long *w = L.win + (d >> 6);
    atomicOr(w, (unsigned long long)(v << (d & 63u)));
    if ((d & 63u) + nb > 64u) atomicOr(w + 1, (unsigned long long)(v >> ((0u - d) & 63u)));
}

// Up to `blocks` blocks from element i0 on, all of one code.  where(request(lane), tid, group_base, group_end): stream
// positions of their group of tiles and of its end (made behind the first barrier, when what is requested beside the
// symbols and the table has arrived); toff: positions of their tiles in the group, up to tile `tiles_end` (from the
// first block's on), where the group ends.  Takes the blocks up to the first one that does not fit a window or ends
// behind the stream's capacity; a first one that fits the whole array alone.  Returns their number (to all threads).
template <bool NIB, class Request, class Where>
__device__ __forceinline__ int pack_blocks(PackLds &L, const uint8_t *su, const Co3Code *cd, int K, int64_t n, int64_t i0,
                                            int blocks, int wave, int tid, Request request, Where where,
                                            const uint64_t *__restrict__ toff, int tiles_end, uint64_t *__restrict__ wu,
                                            int64_t cap_words, int chunk_syms, uint64_t *__restrict__ chunk_off)
{
    constexpr int G = EN_LSYM / 4;
    const int lane = tid & (CO3_WAVE - 1);
    const int64_t iw = i0 + (int64_t)wave * CO3_PACK_SYMS;
    const uint8_t *src = su + (NIB ? iw >> 1 : iw);                      // uniform
    const uint32_t lane_at = (uint32_t)lane * (NIB ? EN_LSYM / 2 : EN_LSYM);
    auto load = [&]() -> uint4 {
        if (NIB) {
            const uint2 a = *reinterpret_cast<const uint2 *>(src + lane_at);
            return make_uint4(a.x, a.y, 0u, 0u);
        }
        return *reinterpret_cast<const uint4 *>(src + lane_at);
    };
    uint4 nxt = load();
    const uint64_t requested = request(lane);
    // offsets of the tiles in the group, one a lane (they fit 32 bits)
    const uint32_t tile_offs = lane < tiles_end ? (uint32_t)toff[lane] : 0u;
    // the symbols that follow the last block: their codewords complete its last word
    int64_t i_end = i0 + (int64_t)blocks * EN_WG_SYMS;
    bool ahead = wave == EN_WAVES - 1 && lane < CO3_WAVE - 1 && i_end + lane < n;
    uint32_t next_sym = ahead ? load_sym1(su, i_end + lane, NIB) : 0u;
    {
        const int j = tid;
        static_assert(EN_BLOCK == 256, "a table entry per thread");
        const uint64_t e = j < K ? cd->enc[j] : 0ull;
        L.enc[j] = e;
        if (NIB) {
            const int lo = j & 15, hi = j >> 4;
            const uint64_t e0 = lo < K ? cd->enc[lo] : 0ull, e1 = hi < K ? cd->enc[hi] : 0ull;
            const uint32_t l1 = (uint32_t)(e1 & 63u);
            L.tab[j] = pack_entry(((e0 >> 6) << l1) | (e1 >> 6), (uint32_t)(e0 & 63u) + l1);
        } else {
            L.tab[j] = pack_entry(e >> 6, (uint32_t)(e & 63u));
        }
        for (int q = j; q < EN_WG_WORDS + 2; q += EN_BLOCK)
            reinterpret_cast<ulonglong2 *>(L.win)[q] = make_ulonglong2(0ull, 0ull);
    }
    __syncthreads();
    uint64_t group_base, group_end;
    where(requested, tid, group_base, group_end);
    const uint32_t last_off = (uint32_t)(group_end - group_base);
    const uint32_t offs = lane < tiles_end ? tile_offs : last_off;
    auto tile_off = [&](int t) -> uint32_t { return (uint32_t)__builtin_amdgcn_readlane((int)offs, t); };
    const uint32_t off0 = tile_off(0);
    bool wide = false;                         // one block, alone in the whole array
    {
        const uint64_t cap_bits = (uint64_t)cap_words * 64u;
        const uint64_t left = cap_bits > group_base ? cap_bits - group_base : 0ull;
        const uint32_t most = left < 0xffffffffull ? (uint32_t)left : 0xffffffffu;
        // lane 4 k: the end of block k, from the lane four on (row_shl:4; a group has 16 tiles, a row of lanes: its last
        // block ends with it)
        static_assert(CO3_PACK_GROUP == 16 && EN_WAVES == 4, "a block's end lies four lanes on in a row of 16");
        const uint32_t to = (uint32_t)__builtin_amdgcn_update_dpp((int)last_off, (int)offs, 0x104, 0xf, 0xf, false);
        const uint32_t size = to - offs;
        const uint32_t fits = (uint32_t)__ballot(to <= most && size <= EN_WG_WORDS * 64u - 63u);
        const int fit = __builtin_ctz((~fits & 0x1111u) | 0x10000u) / EN_WAVES;
        if (fit < blocks) {
            if (fit == 0) {
                if ((__ballot(to <= most && size <= (EN_ALL_WORDS - 2) * 64u - 63u) & 1u) == 0u) return 0;
                wide = true;
            }
            blocks = wide ? 1 : fit;
            i_end = i0 + (int64_t)blocks * EN_WG_SYMS;
            ahead = wave == EN_WAVES - 1 && lane < CO3_WAVE - 1 && i_end + lane < n;
            next_sym = ahead ? load_sym1(su, i_end + lane, NIB) : 0u;
        }
        if (wide) {
            for (int q = tid + 2 * (EN_WG_WORDS + 2); q < EN_ALL_WORDS; q += EN_BLOCK) L.win[q] = 0ull;
            __syncthreads();
        }
    }

    uint64_t base = group_base + off0;
    bool foreign = (base & 63u) != 0u;         // the window's first word begins before element i0
    const bool chunk_lane = ((lane * EN_LSYM) & (chunk_syms - 1)) == 0;  // (chunk sizes are powers of two)
    const uint32_t chunk_sh = (uint32_t)__builtin_ctz((unsigned)chunk_syms);
    const uint32_t chunk_at = (uint32_t)(lane * EN_LSYM) >> chunk_sh;
    int64_t tile_i = iw;
#pragma unroll 1
    for (int k = 0; k < blocks; ++k) {
        const bool last = k + 1 == blocks;
        const uint32_t s[4] = {nxt.x, nxt.y, nxt.z, nxt.w};
        src += NIB ? EN_WG_SYMS / 2 : EN_WG_SYMS;
        if (!last) nxt = load();
        const uint32_t tile_rel = tile_off(k * EN_WAVES + wave) - tile_off(k * EN_WAVES);
        const uint64_t base_next = group_base + tile_off((k + 1) * EN_WAVES);
        const uint32_t base_bit = (uint32_t)base & 63u;
        const uint32_t win = wide ? EN_WIDE_BITS : k & 1 ? EN_WIN_BITS : 0u;

        // codewords of four symbols joined, right-aligned
        uint64_t run[G];
        uint32_t nb[G], far_pair = 0u, far_entry = 0u;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (NIB) {                         // two pairs of codewords from the table
                const uint32_t w = s[g >> 1] >> (16 * (g & 1));
                const uint32_t e0 = L.tab[w & 0xffu], e1 = L.tab[(w >> 8) & 0xffu];
                run[g] = ((uint64_t)(e0 >> 8) << (e1 & 63u)) | (e1 >> 8);
                nb[g] = (e0 + e1) & 0xffu;
                far_entry |= e0 | e1;
            } else {                           // two pairs of codewords
                const uint32_t e0 = L.tab[s[g] & 0xffu], e1 = L.tab[(s[g] >> 8) & 0xffu];
                const uint32_t e2 = L.tab[(s[g] >> 16) & 0xffu], e3 = L.tab[s[g] >> 24];
                const uint32_t t01 = e0 + e1, t23 = e2 + e3;
                const uint32_t p01 = ((e0 >> 8) << (e1 & 31u)) | (e1 >> 8), p23 = ((e2 >> 8) << (e3 & 31u)) | (e3 >> 8);
                run[g] = ((uint64_t)p01 << (t23 & 63u)) | p23;
                nb[g] = (t01 + t23) & 0xffu;
                far_pair |= t01 | t23;
                far_entry |= e0 | e1 | e2 | e3;
            }
        }
        const uint32_t n01 = nb[0] + nb[1], n23 = nb[2] + nb[3];
        const uint32_t mybits = n01 + n23;
        const uint32_t pos = base_bit + tile_rel + wave_scan_incl_u32(mybits, lane) - mybits;
        if ((tile_i & (int64_t)(chunk_syms - 1) & ~(int64_t)(CO3_PACK_SYMS - 1)) == 0) {       // uniform
            // chunk index: stream position of every chunk that starts at this lane's first symbol
            if (chunk_lane) (chunk_off + (tile_i >> chunk_sh))[chunk_at] = (base - base_bit) + pos;
        }
        tile_i += EN_WG_SYMS;
        uint32_t d = win + EN_WG_WORDS * 64u - pos;
        const uint32_t far = NIB ? ((n01 | n23) & 0x40u) | (far_entry & EN_FAR_ENTRY)
                                 : (far_pair & EN_FAR_PAIR) | (far_entry & EN_FAR_ENTRY);
        if (far == 0u) {
            if (NIB) {
                pack_put(L, (run[0] << (nb[1] & 63u)) | run[1], n01, d);
                pack_put(L, (run[2] << (nb[3] & 63u)) | run[3], n23, d);
            } else {
#pragma unroll
                for (int g = 0; g < G; ++g) pack_put(L, run[g], nb[g], d);
            }
        } else {
#pragma unroll 1
            for (int c = 0; c < EN_LSYM; ++c) {
                const int per = NIB ? 8 : 4, q = c / per;
                const uint32_t w = q == 0 ? s[0] : q == 1 ? s[1] : q == 2 ? s[2] : s[3];
                const uint64_t e = L.enc[(w >> (c % per * (32 / per))) & (NIB ? 0xfu : 0xffu)];
                pack_put(L, e >> 6, (uint32_t)(e & 63u), d);
            }
        }
        const uint32_t end = base_bit + (uint32_t)(base_next - base);    // of the block in the window
        if (last && wave == EN_WAVES - 1 && (end & 63u)) {               // complete the last word
            const uint64_t e = ahead ? L.enc[next_sym] : 0ull;
            const uint32_t l = (uint32_t)(e & 63u);
            const uint32_t o = wave_scan_incl_u32(l, lane) - l + (end & 63u);
            uint32_t at = (win >> 6) + EN_WG_WORDS - 1 - (end >> 6);
            asm volatile("" : "+v"(at));       // one word for all lanes: the compiler would gather them one by one
            if (l && o < 64u) atomicOr(L.win + at, (unsigned long long)(((e >> 6) << (64u - l)) >> o));
        }
        __syncthreads();
        // Words leave in order; what has been read is cleared for the block after the next.
        const uint32_t whole = end >> 6, nw = (end + 63u) >> 6;
        uint64_t *dst = wu + (base >> 6);
        for (uint32_t r = (uint32_t)tid; r < nw; r += EN_BLOCK) {
            unsigned long long *w = L.win + ((win >> 6) + EN_WG_WORDS - 1 - r);
            const unsigned long long v = *w;
            *w = 0ull;
            if (r >= whole && !last) {         // (one thread) the unfinished word: the next window's first
                uint32_t at = ((EN_WIN_BITS - win) >> 6) + EN_WG_WORDS - 1;
                asm volatile("" : "+v"(at));
                atomicOr(L.win + at, v);
            } else if (r != 0u || !foreign) dst[r] = v;
        }
        foreign = foreign && whole == 0u;
        base = base_next;
    }
    return blocks;
}

// The general path: a wavefront packs its own tile tb, of any size and with any codes, through a window of its own.
// s: the lane's 16 symbols, four a word; raw: a complete tile of symbols stored two per byte stays in that form, one
// lookup per byte; next_sym: the symbols that follow the tile (their codewords complete its last word).
__device__ __forceinline__ void load_tile(const uint8_t *su, bool nib, int64_t n, int64_t tb, int lane, uint32_t (&s)[4],
                                          uint2 &raw, int &nvalid, uint32_t &next_sym, bool &has_next)
{
    const int64_t t0 = tb * CO3_PACK_SYMS;               // the wavefront's tile: elements [t0, t1)
    const int64_t t1 = t0 + CO3_PACK_SYMS < n ? t0 + CO3_PACK_SYMS : n;
    const int64_t i = t0 + (int64_t)lane * EN_LSYM;
    s[0] = s[1] = s[2] = s[3] = 0u;
    raw = make_uint2(0u, 0u);
    nvalid = EN_LSYM;
    if (t1 - t0 != CO3_PACK_SYMS) nvalid = i < t1 ? load_syms16(su, i, t1, s, nib) : 0;
    else if (nib) raw = *reinterpret_cast<const uint2 *>(su + (i >> 1));
    else load_syms16_full(su, i, nib, s);
    has_next = t1 > t0 && lane < CO3_WAVE - 1 && t1 + lane < n;
    next_sym = has_next ? load_sym1(su, t1 + lane, nib) : 0u;
}

// LAYERS: a tile that straddles tensors (look-ahead included) reads its entries from the code blobs, tensor by element.
// STAGE: words of the window; a tile of short codewords uses EN_STAGE_WORDS of them.
template <bool LAYERS, int STAGE>
__device__ __forceinline__ void pack_tile(const uint32_t (&s)[4], uint2 raw, int nvalid, uint32_t next_sym, bool has_next,
                                          bool nib, int64_t n, const void *codes, int K, const int64_t *seg_off, int nseg,
                                          int64_t tb, int lane, uint64_t *enc_s, const uint64_t *penc_s,
                                          unsigned long long *stage, uint32_t maxlen, uint64_t B0, uint64_t *wu,
                                          int64_t cap_words, int chunk_syms, uint64_t *chunk_off)
{
    const int64_t t0 = tb * CO3_PACK_SYMS;
    const int64_t t1 = t0 + CO3_PACK_SYMS < n ? t0 + CO3_PACK_SYMS : n;
    const bool whole_tile = t1 - t0 == CO3_PACK_SYMS;
    const int64_t i = t0 + (int64_t)lane * EN_LSYM, i2 = t1 + lane;
    const bool raw_tile = nib && whole_tile;

    bool one_tensor = true;
    if (LAYERS) {
        // tensors of the tile and of the at most 63 following symbols whose codewords complete its last word
        int64_t t_hi = t0 + CO3_PACK_SYMS + CO3_WAVE - 1;
        t_hi = (t_hi < n ? t_hi : n) - 1;
        const int s_lo = co3_find_seg(seg_off, nseg, t0), s_hi = co3_find_seg(seg_off, nseg, t_hi);
        one_tensor = s_lo == s_hi;
        maxlen = 64u;                    // a mixed tile takes the general path
        if (one_tensor) {
            const Co3Code *cd = code_of(codes, s_lo);
            wave_lds_sync();
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int q = lane + k * CO3_WAVE;
                enc_s[q] = q < K ? cd->enc[q] : 0ull;
            }
            maxlen = cd->maxlen;
            wave_lds_sync();
        }
    }

    // packed (codeword << 6 | length) of symbol sy at element idx.  (The table is read as what it is, LDS: the compiler
    // joined its reads with those of the code blobs to accesses of either kind, each waited for by itself: 4 x 11 M E4M3
    // under shared codes 79 -> 86 us.)
    const __attribute__((address_space(3))) uint64_t *enc_l = (const __attribute__((address_space(3))) uint64_t *)enc_s;
    auto entry_at = [&](uint32_t sy, int64_t idx) -> uint64_t {
        if (!LAYERS || one_tensor) return enc_l[sy];
        return (int)sy < K ? code_of(codes, co3_find_seg(seg_off, nseg, idx))->enc[sy] : 0ull;
    };
    // the lane's own symbols in a tile that straddles tensors: mostly one tensor, looked up once, so that the
    // 16 reads from its code blob are independent
    int c_first = 0, c_last = 0;
    if (LAYERS && !one_tensor && nvalid > 0) {
        c_first = co3_find_seg(seg_off, nseg, i);
        c_last = co3_find_seg(seg_off, nseg, i + nvalid - 1);
    }
    const uint64_t *enc_first = LAYERS ? code_of(codes, c_first)->enc : nullptr;
    auto entry = [&](uint32_t sy, int k) -> uint64_t {
        if (!LAYERS || one_tensor) return enc_l[sy];
        if (c_first == c_last) return (int)sy < K ? enc_first[sy] : 0ull;
        return entry_at(sy, i + k);
    };

    // One table lookup per symbol: the codewords of every 4 symbols are concatenated into one run
    // (kept in registers) as long as the run fits 64 bits, which it always does for codes of at most
    // 16 bits; a lane that meets a longer run falls back to symbol-by-symbol packing below.
    uint64_t run[EN_LSYM / 4];
    uint32_t runbits[EN_LSYM / 4];
    uint32_t mybits = 0;
    bool wide = false;
    if (raw_tile) {
        lookup_runs_pairs(penc_s, raw, run, runbits, mybits);
    } else if (whole_tile) {    // uniform: every symbol of the tile exists
        if (maxlen <= 16u)
            lookup_runs_short(enc_s, s, run, runbits, mybits);
        else
            lookup_runs<true>(entry, s, nvalid, run, runbits, mybits, wide);
    } else
        lookup_runs<false>(entry, s, nvalid, run, runbits, mybits, wide);
    const uint32_t incl = wave_scan_incl_u32(mybits, lane);
    const uint32_t excl = incl - mybits;
    const uint32_t tilebits = (uint32_t)__builtin_amdgcn_readlane((int)incl, CO3_WAVE - 1);

    const uint64_t B1 = B0 + tilebits;

    // chunk index: stream position of every chunk that starts at this lane's first symbol
    // (chunk sizes are powers of two: a shift, not a 64-bit division that every lane of the wavefront would sit through)
    if (nvalid > 0 && (i & (int64_t)(chunk_syms - 1)) == 0)
        chunk_off[i >> __builtin_ctz((unsigned)chunk_syms)] = B0 + excl;
    // beyond the capacity nothing is written (the scan pass has reported it); uniform over the wavefront
    if ((B1 + 63) / 64 > (uint64_t)cap_words || tilebits == 0) return;

    const int64_t gw0 = (int64_t)(B0 >> 6);          // first and last stream word the tile touches
    const int64_t gwl = (int64_t)((B1 - 1) >> 6);
    const int64_t first_owned = (B0 & 63) ? gw0 + 1 : gw0;   // words whose first bit lies in the tile
    const uint64_t rel0 = (B0 & 63) + excl;          // position of this lane's bits, relative to word gw0

    if ((B0 & 63) + tilebits <= EN_STAGE_WORDS * 64u && !__any(wide)) {
        // usual case: the tile fits one staging window and every run fits 64 bits
#pragma unroll
        for (int j = 0; j < EN_STAGE_WORDS / CO3_WAVE; ++j) stage[lane + j * CO3_WAVE] = 0ull;
        wave_lds_sync();
        uint32_t pos = (uint32_t)rel0;
#pragma unroll
        for (int g = 0; g < EN_LSYM / 4; ++g) {
            const uint32_t nb = runbits[g];
            if (nb) {
                const uint64_t v = run[g] << (64u - nb);
                const uint32_t w = pos >> 6, o = pos & 63u;
                atomicOr(&stage[w], (unsigned long long)(v >> o));
                if (o + nb > 64u) atomicOr(&stage[w + 1], (unsigned long long)(v << (64u - o)));
            }
            pos += nb;
        }
        const uint32_t last_rel = (uint32_t)(gwl - gw0);
        if (B1 & 63) {          // complete the last word with the codewords that follow the tile
            uint64_t e = has_next ? entry_at(next_sym, i2) : 0ull;
            uint32_t l = (uint32_t)(e & 63u);
            uint32_t o = wave_scan_incl_u32(l, lane) - l;
            const uint32_t used = (uint32_t)(B1 & 63);
            if (l && used + o < 64u)
                atomicOr(&stage[last_rel], (unsigned long long)(((e >> 6) << (64 - l)) >> (used + o)));
        }
        wave_lds_sync();
        const uint32_t first_rel = (uint32_t)(first_owned - gw0);
#pragma unroll
        for (int j = 0; j < EN_STAGE_WORDS / CO3_WAVE; ++j) {
            const uint32_t r = lane + j * CO3_WAVE;
            if (r >= first_rel && r <= last_rel) wu[gw0 + r] = stage[r];
        }
        return;
    }

    for (int64_t win_w0 = 0; gw0 + win_w0 <= gwl; win_w0 += STAGE) {
#pragma unroll
        for (int j = 0; j < STAGE / CO3_WAVE; ++j) stage[lane + j * CO3_WAVE] = 0ull;
        wave_lds_sync();
        if (!wide) {
            uint64_t pos = rel0;
#pragma unroll
            for (int g = 0; g < EN_LSYM / 4; ++g) {
                if (runbits[g]) stage_bits<STAGE>(stage, win_w0, run[g], (int)runbits[g], pos);
                pos += runbits[g];
            }
        } else {
            // runs of at most 64 bits, symbol by symbol
            uint64_t acc = 0, pos = rel0;
            int accbits = 0;
            for (int c = 0; c < nvalid; ++c) {
                uint64_t e = entry((s[c >> 2] >> (8 * (c & 3))) & 0xffu, c);
                int l = (int)(e & 63u);
                if (l) {
                    if (accbits + l > 64) {
                        stage_bits<STAGE>(stage, win_w0, acc, accbits, pos);
                        pos += accbits;
                        acc = 0;
                        accbits = 0;
                    }
                    acc = (acc << l) | (e >> 6);
                    accbits += l;
                }
            }
            if (accbits) stage_bits<STAGE>(stage, win_w0, acc, accbits, pos);
        }
        // The last word of the tile is completed with the first codewords of the symbols that follow
        // (at most 63 bits, hence at most 63 symbols), clipped at the word end.
        const int64_t last_rel = gwl - gw0 - win_w0;
        if ((B1 & 63) && last_rel >= 0 && last_rel < STAGE) {
            uint64_t e = has_next ? entry_at(next_sym, i2) : 0ull;
            uint32_t l = (uint32_t)(e & 63u);
            uint32_t o = wave_scan_incl_u32(l, lane) - l;
            const uint32_t used = (uint32_t)(B1 & 63);
            if (l && used + o < 64u)
                atomicOr(&stage[last_rel], (unsigned long long)(((e >> 6) << (64 - l)) >> (used + o)));
        }
        wave_lds_sync();
#pragma unroll
        for (int j = 0; j < STAGE / CO3_WAVE; ++j) {
            int64_t gw = gw0 + win_w0 + lane + j * CO3_WAVE;
            if (gw >= first_owned && gw <= gwl) wu[gw] = stage[lane + j * CO3_WAVE];
        }
        wave_lds_sync();
    }
}

// The user's codewords for the general path; called by all threads of the workgroup.  Returns the longest length.
__device__ __forceinline__ uint32_t load_tile_tables(uint64_t *enc_s, uint64_t *penc_s, const Co3Code *cd, int K, bool nib,
                                                     int tid)
{
    for (int j = tid; j < 256; j += EN_BLOCK) {
        enc_s[j] = j < K ? cd->enc[j] : 0ull;
        if (nib) {
            const int lo = j & 15, hi = j >> 4;
            const uint64_t e0 = lo < K ? cd->enc[lo] : 0ull, e1 = hi < K ? cd->enc[hi] : 0ull;
            const uint32_t l1 = (uint32_t)(e1 & 63u);
            penc_s[j] = ((((e0 >> 6) << l1) | (e1 >> 6)) << 6) | (uint64_t)((uint32_t)(e0 & 63u) + l1);
        }
    }
    return cd->maxlen;
}

// SCAN: groupoff holds the sizes of at most 64 groups as the sizes pass left them.  Every wavefront takes them with
// one load (lane g: group g), beside those it makes anyway, and scans them in registers; `report`: the first one of a
// user writes what the scan kernel would.  That saves the kernel (3.3 us and its place in a chain of small ones: one
// user of 65,536 elements 53.9 -> 50.0 us a pass).  With up to 682 groups a form of this took 59 us against 51 and the
// kernel's 5.  Returns the stream positions at which the groups up to each lane's end.
__device__ __forceinline__ uint32_t scan_groups(uint32_t bits, int lane, bool report, uint64_t *total_bits_u, uint64_t *chunk_last,
                                                int64_t cap_words, int32_t *status)
{
    const uint32_t upto = wave_scan_incl_u32(bits, lane);
    if (report && lane == CO3_WAVE - 1) {      // the last lane holds the stream's length
        *total_bits_u = upto;
        *chunk_last = upto;
        if (((uint64_t)upto + 63) / 64 > (uint64_t)cap_words) co3_raise(status, CO3_ECAP);
    }
    return upto;
}

template <bool LAYERS, int STAGE>
struct TileLds {
    uint64_t enc_all[LAYERS ? EN_WAVES * 256 : 256];
    uint64_t penc_s[LAYERS ? 1 : 256];           // codeword pairs, symbols two per byte
    unsigned long long stage_all[EN_WAVES][STAGE];
};

// A tile per wavefront.  LAYERS = false: one code per user (codes[u]), its table shared by the workgroup.  LAYERS = true:
// one code per tensor shared by all users (codes[tensor]); each wavefront keeps the table of its tile's tensor.
// The per-user form is compiled for eight wavefronts per SIMD (64 registers; a few spills on the rarely taken
// paths): it is bound by the latency of its per-tile chain, and residency is what hides it.
template <bool LAYERS, bool SCAN>
__global__ __launch_bounds__(EN_BLOCK) __attribute__((amdgpu_waves_per_eu(LAYERS ? 5 : 8, LAYERS ? 5 : 8)))
void k_enc_pack(const uint8_t *__restrict__ sym, int64_t n, int64_t stride, const void *__restrict__ codes, int K,
                const int64_t *__restrict__ seg_off_g, int nseg, const uint64_t *__restrict__ tileoff, int64_t nblk,
                const uint64_t *__restrict__ groupoff, int64_t ngrp, uint64_t *__restrict__ words, int64_t cap_words,
                int chunk_syms, uint64_t *__restrict__ chunk_bitoff, int64_t nchunks, int sym_nib,
                uint64_t *__restrict__ total_bits, int32_t *status)
{
    const int u = blockIdx.y;
    const bool nib = !LAYERS && sym_nib != 0;
    __shared__ TileLds<LAYERS, EN_STAGE_WORDS> lds;
    __shared__ int64_t seg_cache[LAYERS ? CO3_SEG_CACHE : 1];
    const int lane = threadIdx.x & (CO3_WAVE - 1);
    const int wave = threadIdx.x / CO3_WAVE;
    const int64_t tb = (int64_t)blockIdx.x * EN_WAVES + wave;
    // Everything the wavefront reads from memory apart from the tables is requested first, so that its latency
    // and that of the table load below (with its barrier) overlap.
    const bool live = tb < nblk;                     // uniform: the wavefront has a tile
    uint32_t s[4], next_sym;
    uint2 raw;
    int nvalid;
    bool has_next;
    load_tile(sym + (int64_t)u * (nib ? stride / 2 : stride), nib, n, tb, lane, s, raw, nvalid, next_sym, has_next);
    uint64_t group_base = 0;
    uint32_t group_bits = 0;
    if (SCAN) group_bits = lane < (int)ngrp ? (uint32_t)groupoff[(int64_t)u * ngrp + lane] : 0u;   // (64 groups fit 32 bits)
    else if (live) group_base = groupoff[(int64_t)u * ngrp + tb / CO3_PACK_GROUP];
    const uint64_t tile_base = live ? tileoff[(int64_t)u * nblk + tb] : 0ull;
    uint64_t *chunk_off = chunk_bitoff + (int64_t)u * (nchunks + 1);

    uint32_t maxlen = 0u;
    const int64_t *seg_off = seg_off_g;
    if (LAYERS) seg_off = co3_cache_segs(seg_off_g, nseg, seg_cache);
    else maxlen = load_tile_tables(lds.enc_all, lds.penc_s, code_of(codes, u), K, nib, (int)threadIdx.x);
    __syncthreads();
    if (tb >= nblk) return;
    if (SCAN) {
        const uint32_t upto = scan_groups(group_bits, lane, tb == 0, total_bits + u, chunk_off + nchunks, cap_words, status);
        const int grp = __builtin_amdgcn_readfirstlane((int)(tb / CO3_PACK_GROUP));
        group_base = grp ? (uint32_t)__builtin_amdgcn_readlane((int)upto, grp - 1) : 0u;
    }
    pack_tile<LAYERS, EN_STAGE_WORDS>(s, raw, nvalid, next_sym, has_next, nib, n, codes, K, seg_off, nseg, tb, lane,
                                      lds.enc_all + (LAYERS ? wave * 256 : 0), lds.penc_s, lds.stage_all[wave], maxlen,
                                      group_base + tile_base, words + (int64_t)u * cap_words, cap_words, chunk_syms, chunk_off);
}

// A workgroup takes a group of tiles: blocks that are whole and of one code together, up to four in a row, the others
// (the end of a user's vector, blocks that hold a tensor boundary, that end behind the capacity or that take more than 31
// bits a symbol) tile by tile.
template <bool LAYERS, bool SCAN, bool NIB>
__global__ __launch_bounds__(EN_BLOCK) __attribute__((amdgpu_waves_per_eu(LAYERS ? 5 : 8, LAYERS ? 5 : 8)))
void k_enc_pack_blocks(const uint8_t *__restrict__ sym, int64_t n, int64_t stride, const void *__restrict__ codes, int K,
                       const int64_t *__restrict__ seg_off_g, int nseg, const uint64_t *__restrict__ tileoff, int64_t nblk,
                       const uint64_t *__restrict__ groupoff, int64_t ngrp, uint64_t *__restrict__ words, int64_t cap_words,
                       int chunk_syms, uint64_t *__restrict__ chunk_bitoff, int64_t nchunks, int /*sym_nib*/,
                       uint64_t *__restrict__ total_bits, int32_t *status)
{
    const int u = blockIdx.y;
    __shared__ union {
        PackLds wg;
        TileLds<LAYERS, EN_LONG_STAGE_WORDS> tile;
    } lds;
    __shared__ int64_t seg_cache[LAYERS ? CO3_SEG_CACHE : 1];
    const int64_t grp = blockIdx.x, tb0 = grp * CO3_PACK_GROUP, i0 = tb0 * CO3_PACK_SYMS;
    const uint8_t *su = sym + (int64_t)u * (NIB ? stride / 2 : stride);
    uint64_t *wu = words + (int64_t)u * cap_words;
    uint64_t *chunk_off = chunk_bitoff + (int64_t)u * (nchunks + 1);
    const uint64_t *toff = tileoff + (int64_t)u * nblk + tb0;
    // Stream positions of the workgroup's group of tiles and of its end: requested beside the symbols, made when needed.
    // SCAN: lane g the bits of group g (64 groups fit 32 bits); else an even lane the first position, an odd one the last.
    auto request = [&](int lane) -> uint64_t {
        int64_t of_user = (int64_t)u * ngrp;
        asm volatile("" : "+s"(of_user));          // (not before the loop: it would be waited for before all other requests)
        const uint64_t *g = groupoff + of_user;
        if (SCAN) return lane < (int)ngrp ? g[lane] : 0ull;
        const uint64_t *next = grp + 1 < ngrp ? g + grp + 1 : total_bits + u;
        return *(lane & 1 ? next : g + grp);
    };
    auto where = [&](uint64_t requested, int tid, uint64_t &group_base, uint64_t &group_end) {
        const uint32_t lo = (uint32_t)requested, hi = (uint32_t)(requested >> 32);
        if (SCAN) {
            const uint32_t upto = scan_groups(lo, tid & (CO3_WAVE - 1), blockIdx.x == 0 && tid < CO3_WAVE, total_bits + u,
                                              chunk_off + nchunks, cap_words, status);
            group_base = grp ? (uint32_t)__builtin_amdgcn_readlane((int)upto, (int)grp - 1) : 0u;
            group_end = (uint32_t)__builtin_amdgcn_readlane((int)upto, (int)grp);
        } else {
            auto of_lane = [&](int l) -> uint64_t {
                const uint32_t h = (uint32_t)__builtin_amdgcn_readlane((int)hi, l);
                return (uint64_t)h << 32 | (uint32_t)__builtin_amdgcn_readlane((int)lo, l);
            };
            group_base = of_lane(0);
            group_end = of_lane(1);
        }
    };
    const int64_t *seg_off = LAYERS ? co3_cache_segs(seg_off_g, nseg, seg_cache) : seg_off_g;
    const int tiles_end = nblk - tb0 < CO3_PACK_GROUP ? (int)(nblk - tb0) : CO3_PACK_GROUP;

    // (looking for blocks of one code costs more than it finds: see pack_by_groups)
    const bool short_codes = LAYERS && n < nseg * (int64_t)EN_MOST_BLOCKS * EN_WG_SYMS;
    bool together = false, apart = false;                // how the LDS is used since the last barrier
#pragma unroll 1
    for (int k = 0; k * EN_WAVES < tiles_end;) {
        // What is made from it stays inside the loop: the registers are all in use, and what the compiler stored away before
        // the loop, 27 MB for a full chip, took room in the last-level cache from the kernels behind (an average 82 -> 87 us).
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int lane = tid & (CO3_WAVE - 1), wave = __builtin_amdgcn_readfirstlane(tid / CO3_WAVE);
        const int64_t ik = i0 + (int64_t)k * EN_WG_SYMS;
        // blocks to pack together: whole ones, of one code with the at most 63 symbols behind each (its last word)
        int64_t room = n - ik;
        int code = u;
        if (LAYERS && short_codes) room = 0;
        else if (LAYERS) {
            code = __builtin_amdgcn_readfirstlane(co3_find_seg(seg_off, nseg, ik));
            const int64_t end = code + 1 < nseg ? seg_off[code + 1] : n;
            if (end < n) room = end - (CO3_WAVE - 1) - ik;
        }
        const int most = (EN_MOST_BLOCKS - k) * EN_WG_SYMS;
        int m = __builtin_amdgcn_readfirstlane((room < 0 ? 0 : room < most ? (int)room : most) / EN_WG_SYMS);
        if (m > 0) {
            if (together || apart) __syncthreads();
            together = true;
            apart = false;
            m = pack_blocks<NIB>(lds.wg, su, code_of(codes, code), K, n, ik, m, wave, tid, request, where, toff + k * EN_WAVES,
                                 tiles_end - k * EN_WAVES, wu, cap_words, chunk_syms, chunk_off);
        }
        if (m == 0) {                                    // one block tile by tile
            m = 1;
            if (together || (!LAYERS && apart)) __syncthreads();
            together = false;
            apart = true;
            uint32_t maxlen = 0u;
            if (!LAYERS) maxlen = load_tile_tables(lds.tile.enc_all, lds.tile.penc_s, code_of(codes, u), K, NIB, tid);
            if (!LAYERS) __syncthreads();
            const uint64_t requested = request(lane);
            const int64_t tb = tb0 + k * EN_WAVES + wave;
            const uint64_t tile_base = tb < nblk ? toff[k * EN_WAVES + wave] : 0ull;
            uint32_t s[4], next_sym;
            uint2 raw;
            int nvalid;
            bool has_next;
            load_tile(su, NIB, n, tb, lane, s, raw, nvalid, next_sym, has_next);
            uint64_t group_base, group_end;
            where(requested, tid, group_base, group_end);
            if (tb < nblk)
                pack_tile<LAYERS, EN_LONG_STAGE_WORDS>(
                    s, raw, nvalid, next_sym, has_next, NIB, n, codes, K, seg_off, nseg, tb, lane,
                    lds.tile.enc_all + (LAYERS ? wave * 256 : 0), lds.tile.penc_s, lds.tile.stage_all[wave], maxlen,
                    group_base + tile_base, wu, cap_words, chunk_syms, chunk_off);
        }
        k += m;
    }
}

hipError_t co3_launch_enc_scan(uint64_t *sizes, int64_t nsizes, int U, int64_t cap_words, uint64_t *chunk_bitoff,
                               int64_t nchunks, uint64_t *total_bits, int32_t *status, hipStream_t st)
{
    Co3LaunchTimer tm(CO3_K_ENC_SCAN, st);
    hipLaunchKernelGGL(k_enc_scan, dim3(U), dim3(SC_BLOCK), 0, st, sizes, nsizes, cap_words, chunk_bitoff, nchunks,
                       total_bits, status);
    return hipGetLastError();
}

// Whether a workgroup of the packer takes a group of four blocks (else a tile per wavefront).  Few workgroups end sooner
// with little each (packer of one user, us with a tile per wavefront | four blocks: 8 M E3M0 8.8 | 9.4, E4M3 9.4 | 11.1;
// 16 M 12.6 | 11.6 and 13.7 | 14.0; 20 M 14.7 | 12.7 and 15.6 | 15.2): from 4,096 blocks on.  And the groups have to hold
// blocks that can be packed together.  Codes per user: a last group that holds one block, or one or two and a ragged end,
// takes as long as a whole one or longer, which shows where users have few groups (encoding 100 M symbols in E4M3 by users
// of one block 83 | 92 us, of two 72 | 64.5, three 70 | 59, four 70 | 58, five 72 | 80, six 70 | 70, nine 69 | 60.5; 200 M
// by users of 10,000 symbols 173 | 180).
// Shared codes of groups of tensors that are no longer than the packer's mostly hold a boundary and go tile by tile,
// which pays for a full chip alone (encoding in E4M3 under codes of 3,000 symbols, 4 x 11 M 363 | 351, 30 M of one user 293
// | 321, 10 x 11 M 800 | 740; of 5,000 277 | 261, 235 | 240, 610 | 555; of 9,000 226 | 226, 180 | 194, 484 | 473; of 17,000
// 184 | 165, 154 | 138, 385 | 338; of 40,000 91 | 73, 96 | 77, 197 | 148).
static bool pack_by_groups(int64_t n, int U, int ncodes)
{
    const int64_t block = EN_WG_SYMS, group = EN_MOST_BLOCKS * block, last = n % group;
    if ((n + block - 1) / block * U < 4096) return false;
    if (ncodes) return n / ncodes >= group || (n + block - 1) / block * U >= 16384;
    return n >= 2 * group || last >= 3 * block || (last % block == 0 && last != block);
}

// seg_off != NULL selects one code per tensor (codes[tensor], shared by the users) instead of codes[user].
// newest_last: the symbols were written user by user, the last user's last.  The sizes pass then takes the users from
// the last to the first, and the packer from the first on: each begins with what the pass before it has left in the
// last-level cache (16 x 25 M E4M3, 400 MB of symbols against 256 MB of cache: sizes 120 -> 84 us, packer 162 -> 165).
hipError_t co3_launch_encode(const uint8_t *sym, int64_t n, int U, int64_t stride, const void *codes, int K,
                             const int64_t *seg_off, int nseg, uint64_t *words, int64_t cap_words, int chunk_syms,
                             uint64_t *chunk_bitoff, uint64_t *total_bits, uint64_t *tilesum, int32_t *status,
                             hipStream_t st, int sym_nib, int newest_last)
{
    if (sym_nib && (seg_off || K > 16)) return hipErrorInvalidValue;
    static_assert(SZ_GROUP == CO3_PACK_GROUP, "group size of the sizes pass");
    const int64_t nblk = (n + CO3_PACK_SYMS - 1) / CO3_PACK_SYMS;
    const int64_t ngrp = (nblk + CO3_PACK_GROUP - 1) / CO3_PACK_GROUP;
    const int64_t nchunks = (n + chunk_syms - 1) / chunk_syms;
    uint64_t *groupsum = tilesum + (int64_t)U * (nblk > 0 ? nblk : 1);     // workspace: [U][nblk] then [U][ngrp]
    if (nblk > 0) {
        Co3LaunchTimer tm(CO3_K_ENC_SIZES, st);
        if (seg_off)
            hipLaunchKernelGGL(k_enc_sizes_layers, dim3((unsigned)ngrp, U), dim3(EN_BLOCK), 0, st, sym, n, stride, codes,
                               K, seg_off, nseg, tilesum, nblk, groupsum, ngrp, status);
        else
            hipLaunchKernelGGL(k_enc_sizes, dim3((unsigned)ngrp, U), dim3(EN_BLOCK), 0, st, sym, n, stride, codes, K,
                               tilesum, nblk, groupsum, ngrp, status, sym_nib, newest_last);
    }
    static_assert((int64_t)CO3_WAVE * CO3_PACK_GROUP * CO3_PACK_SYMS * 64 < (1ll << 32), "64 groups fit 32 bits");
    const bool scan_in_pack = !seg_off && nblk > 0 && ngrp <= CO3_WAVE;
    if (!scan_in_pack &&
        co3_launch_enc_scan(groupsum, ngrp, U, cap_words, chunk_bitoff, nchunks, total_bits, status, st) != hipSuccess)
        return hipGetLastError();
    if (nblk > 0) {
        const bool groups = pack_by_groups(n, U, seg_off ? nseg : 0);
        const unsigned gx = (unsigned)(groups ? ngrp : (nblk + EN_WAVES - 1) / EN_WAVES);
        Co3LaunchTimer tm(CO3_K_ENC_PACK, st);
#define CO3_PACK_LAUNCH(...)                                                                                           \
    hipLaunchKernelGGL((__VA_ARGS__), dim3(gx, U), dim3(EN_BLOCK), 0, st, sym, n, stride, codes, K, seg_off, nseg,      \
                       (const uint64_t *)tilesum, nblk, (const uint64_t *)groupsum, ngrp, words, cap_words, chunk_syms, \
                       chunk_bitoff, nchunks, sym_nib, total_bits, status)
        if (groups) {
            if (seg_off) CO3_PACK_LAUNCH(k_enc_pack_blocks<true, false, false>);
            else if (scan_in_pack && sym_nib) CO3_PACK_LAUNCH(k_enc_pack_blocks<false, true, true>);
            else if (scan_in_pack) CO3_PACK_LAUNCH(k_enc_pack_blocks<false, true, false>);
            else if (sym_nib) CO3_PACK_LAUNCH(k_enc_pack_blocks<false, false, true>);
            else CO3_PACK_LAUNCH(k_enc_pack_blocks<false, false, false>);
        } else if (seg_off) CO3_PACK_LAUNCH(k_enc_pack<true, false>);
        else if (scan_in_pack) CO3_PACK_LAUNCH(k_enc_pack<false, true>);
        else CO3_PACK_LAUNCH(k_enc_pack<false, false>);
#undef CO3_PACK_LAUNCH
    }
    return hipGetLastError();
}

// ---- the encoder's workspace for callers that cannot allocate --------------------------------------
// A fixed array in the library's device image (every GPU that loads the library holds its own copy until
// the process ends).  On the host the array's name is only a handle: its device address is looked up once
// per device and kept; kernels and copies only ever see that address.
static __device__ __align__(256) unsigned char scratch[CO3_ENCODE_STATIC_WS_BYTES];

#define CO3_MAX_DEVICES 64
hipError_t co3_static_encode_workspace(void **ptr_out)
{
    static std::atomic<void *> ptr_of[CO3_MAX_DEVICES];      // zero-initialised: nothing looked up yet
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= CO3_MAX_DEVICES) return hipErrorInvalidDevice;
    void *p = ptr_of[dev].load(std::memory_order_acquire);
    if (!p) {
        // two threads may both look it up: they get the same address
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        ptr_of[dev].store(p, std::memory_order_release);
    }
    *ptr_out = p;
    return hipSuccess;
}
