// Huffman code construction (Sec. III (ii)) by one workgroup of 1024 or 256 lanes: code lengths by the
// two-queue merge, canonical codewords, and the decoder tables of the code blob, from K <= 256 integer weights.
//
// A few codes on a chip that is otherwise idle: what counts is the length of the dependent chain.  With one merged
// node a step in one lane, and loops over LDS entries one at a time around it, K = 256 took 255 steps of about 250
// cycles; it now takes one round per level of the tree (20 - 24 rounds of 650 - 1,250 cycles on the 8-bit formats).
// At most 16 leaves still take a step per node.  Launch to launch in a graph, before | now: K = 256 52 | 19 us, 64
// 22 | 16, 32 15.6 | 13.5, 16 11.6 | 8.8, 8 6.3 | 6.4; with the ragged end of 11.2 M elements in E4M3 58 | 23 us.
#pragma once
#include "co3_dev.h"

#define CO3_HB_BLOCK 1024       // lanes for a few codes; many take 256 (co3_launch_build_code)
#define CO3_HB_STEPS 16         // most leaves that are merged a node a step
#define CO3_LEN_CAP 62          // lengths are clipped here; above CO3_MAX_CODE_LEN the status word says so

template <int V> struct Co3Const { static constexpr int value = V; };

struct Co3BuildLds {
    // weights and keys are whole numbers below 2^53 (a key is weight << 8 | symbol, a sum at most 2^40): exact as
    // doubles, whose comparison and addition are single instructions; where all weights together stay below 2^30 the
    // merge keeps them in 32 bits
    __attribute__((aligned(16))) double key[256];
    double leaf_w[256 + CO3_WAVE];            // leaves in (weight, symbol) order, then "no item" (see Co3MergeF64, Co3MergeU32)
    double node_w[256 + CO3_WAVE];            // merged nodes in creation order, then "no item"
    double ord[256 + 2];                      // a round's items in merged order
    unsigned long long total;                 // of the weights
    uint32_t rank[256];
    uint32_t up[256];                         // of a node: an ancestor | steps to it << 16
    int32_t at[CO3_LUT_BITS_MAX + 2];
    uint32_t maxlen, nact;
    uint16_t parent[512 + 1];                 // of leaf j: [j]; of node i: [256 + i]; the parent's node number
    uint8_t leaf_sym[256];
    uint8_t len[256];
    uint8_t sorted[256];
    uint16_t wave_cnt[4][CO3_WAVE];           // symbols of each length among the 64 symbols of wavefront w
};

// LDS operations of one wavefront are carried out in order: a hand-over between its lanes needs no wait, only
// that the compiler keeps the order.
__device__ __forceinline__ void co3_lds_order()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

// The weights of the merge in 32 bits (their sum is below 2^30) or as doubles.  `none` stands behind the last item:
// above every weight, and it stays that when something is added.
struct Co3MergeU32 {
    typedef uint32_t W;
    static __device__ __forceinline__ W none() { return 0x7fffffffu; }
    static __device__ __forceinline__ W least(W a, W b) { return a < b ? a : b; }
    static __device__ __forceinline__ W lane(W v, int l) { return (W)__builtin_amdgcn_readlane((int)v, l); }
    static __device__ __forceinline__ W next(W v)      // the value of the lane above (used in lane 0)
    {
        return (W)__builtin_amdgcn_update_dpp(0, (int)v, 0x101, 0xf, 0xf, true);      // row_shl:1
    }
    static __device__ __forceinline__ int not_below(W a, W b) { return (int)((b - a - 1u) >> 31); }     // a >= b, neither above none
};
struct Co3MergeF64 {
    typedef double W;
    static __device__ __forceinline__ W none() { return __builtin_huge_val(); }
    static __device__ __forceinline__ W least(W a, W b) { return fmin(a, b); }
    static __device__ __forceinline__ W join(uint32_t lo, uint32_t hi)
    {
        return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
    }
    static __device__ __forceinline__ W lane(W v, int l)
    {
        const uint64_t b = (uint64_t)__double_as_longlong(v);
        return join((uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l),
                    (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l));
    }
    static __device__ __forceinline__ W next(W v)
    {
        const uint64_t b = (uint64_t)__double_as_longlong(v);
        return join((uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, 0x101, 0xf, 0xf, true),
                    (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), 0x101, 0xf, 0xf, true));
    }
    static __device__ __forceinline__ int not_below(W a, W b) { return __builtin_amdgcn_readfirstlane(a >= b ? 1 : 0); }
};

// Number of entries of the ascending list a[0, count) that are below w (OR_EQUAL: not above it); top: the largest
// power of two not above count, 0 for no search.
template <bool OR_EQUAL, class W>
__device__ __forceinline__ int co3_count_below(const W *a, int count, int top, W w)
{
    int c = 0;
    for (int b = top; b >= 1; b >>= 1) {
        const int t = c + b;
        const W v = a[(t <= count ? t : 1) - 1];
        if (t <= count && (OR_EQUAL ? v <= w : v < w)) c = t;
    }
    return c;
}

// The two-queue merge by one wavefront, in rounds.  With s the sum of the two smallest items, every leaf of weight
// at most s and every node present (their weights do not exceed s: merged weights never decrease) comes before the
// node that s creates; so the sequential procedure pairs these items two by two in their merged order before it
// meets a new node, and one round does all of it.  An odd item out, the last one, stays in front of its queue.  A
// leaf precedes a node of equal weight, as in the sequential rule, so the tree is the same, ties included.
//
// The fronts of both queues stay in registers, lane j holding the j-th leaf and the j-th node that is left; a
// round of at most 63 of each finds the merged order by a four-way search (three chained LDS reads; going through
// the other list item by item with lane reads took 44 cycles an item, up to 3,400 a round) and passes the items
// through LDS once.  Larger rounds (many equal weights) take more steps.  One wavefront alone pays for every way
// between vector and scalar unit and for every branch: all lanes go the same way, those without an item writing to
// a slot that nothing reads.
template <class T>
__device__ __forceinline__ void co3_merge_rounds(Co3BuildLds &L, const int lane, const int nact)
{
    typedef typename T::W W;
    W *leaf_w = reinterpret_cast<W *>(L.leaf_w), *node_w = reinterpret_cast<W *>(L.node_w), *ord = reinterpret_cast<W *>(L.ord);
    int q1 = 0, nb = 0, ne = 0;               // leaves from q1 on and nodes [nb, ne) are not merged yet
    W lw = leaf_w[lane], nw = T::none();
    while (nact - q1 + ne - nb > 1) {
        const W s = T::lane(T::least(T::least(lw + T::next(lw), nw + T::next(nw)), lw + nw), 0);
        const int mn = ne - nb;
        int nl = __popcll(__ballot(lw <= s));
        if (mn < CO3_WAVE && nl < CO3_WAVE) {
            int lrank = lane, nrank = lane;
            if (nl && mn) {
                // lane j's leaf: how many nodes lie below it; lane i's node: how many leaves do not lie above it.  Each
                // step narrows four ways with three independent reads per list.  What stands behind the last item of
                // the round lies above every item of the other list, so no step needs a bound.
                const int big = mn > nl ? mn : nl;
                const W *leaf = leaf_w + q1, *node = node_w + nb;
                int cl = 0, cn = 0;
                auto narrow = [&](auto step) {
                    constexpr int B = decltype(step)::value;
                    const W n1 = node[cl + B - 1], n2 = node[cl + 2 * B - 1], n3 = node[cl + 3 * B - 1];
                    const W l1 = leaf[cn + B - 1], l2 = leaf[cn + 2 * B - 1], l3 = leaf[cn + 3 * B - 1];
                    cl += B * ((n1 < lw ? 1 : 0) + (n2 < lw ? 1 : 0) + (n3 < lw ? 1 : 0));
                    cn += B * ((l1 <= nw ? 1 : 0) + (l2 <= nw ? 1 : 0) + (l3 <= nw ? 1 : 0));
                };
                if (big > 15) narrow(Co3Const<16>());
                if (big > 3) narrow(Co3Const<4>());
                narrow(Co3Const<1>());
                lrank += cl;
                nrank += cn;
            }
            const int m = mn + nl, pairs = m >> 1;
            // whether the odd item out is a node: there is one, and no leaf of the round lies above the last one
            const int last_is_node = T::not_below(T::lane(nw, (mn - 1) & (CO3_WAVE - 1)), T::lane(lw, (nl - 1) & (CO3_WAVE - 1)));
            const int node_last = m & ((-mn) >> 31) & (last_is_node | ~((-nl) >> 31)) & 1;
            ord[lane < nl ? lrank : 256] = lw;
            ord[lane < mn ? nrank : 256] = nw;
            // (of the odd one out a parent is written that its own round replaces)
            L.parent[lane < nl ? q1 + lane : 512] = (uint16_t)(ne + (lrank >> 1));
            L.parent[lane < mn ? 256 + nb + lane : 512] = (uint16_t)(ne + (nrank >> 1));
            q1 += nl - (m & (node_last ^ 1));
            nb = ne - node_last;
            co3_lds_order();
            const int p = lane - node_last;
            const int t = p < 0 ? m - 1 : p < pairs ? 2 * p : 0;
            const W a = ord[t], b = ord[t + 1];
            lw = leaf_w[q1 + lane];
            nw = p < pairs ? (p < 0 ? a : a + b) : T::none();
            node_w[p >= 0 && p < pairs ? ne + p : 256 + CO3_WAVE - 1] = nw;      // (what the last slot holds nothing reads)
            ne += pairs;
            co3_lds_order();
            continue;
        }
        const W *leaf = leaf_w + q1, *node = node_w + nb;
        while (q1 + nl < 256) {               // (behind the last leaf stands "no item")
            const int c = __popcll(__ballot(leaf[nl + lane] <= s));
            nl += c;
            if (c < CO3_WAVE) break;
        }
        const int m = mn + nl;
        const int big = mn > nl ? mn : nl;
        const int top_n = nl && mn ? 1 << (31 - __builtin_clz(mn)) : 0;
        const int top_l = nl && mn ? 1 << (31 - __builtin_clz(nl)) : 0;
        for (int j = lane; j < big; j += CO3_WAVE) {
            if (j < nl) {
                const W w = leaf[j];
                const int r = j + co3_count_below<false, W>(node, mn, top_n, w);
                ord[r] = w;
                L.parent[q1 + j] = (uint16_t)(ne + (r >> 1));
            }
            if (j < mn) {
                const W w = node[j];
                const int r = j + co3_count_below<true, W>(leaf, nl, top_l, w);
                ord[r] = w;
                L.parent[256 + nb + j] = (uint16_t)(ne + (r >> 1));
            }
        }
        const bool odd = m & 1;
        // (the same in all lanes: said to the compiler, so that the queue positions stay scalar)
        const bool node_last =
            __builtin_amdgcn_readfirstlane(odd && mn > 0 && (nl == 0 || node[mn - 1] >= leaf[nl - 1]) ? 1 : 0) != 0;
        co3_lds_order();
        for (int p = lane; p < m >> 1; p += CO3_WAVE) node_w[ne + p] = ord[2 * p] + ord[2 * p + 1];
        q1 += nl - (odd && !node_last ? 1 : 0);
        nb = ne - (node_last ? 1 : 0);
        ne += m >> 1;
        co3_lds_order();
        lw = leaf_w[q1 + lane];
        nw = nb + lane < ne ? node_w[nb + lane] : T::none();
    }
}

// The two-queue merge of few leaves, one node a step in one lane.  A step reads the two fronts of each queue and
// takes one of three outcomes: two leaves, two nodes, or the first leaf with the first node.  A skewed code of few
// symbols has nearly as many levels as nodes, and a round costs three steps or more: steps | rounds, skewed weights,
// K = 8 6.4 | 7.9 us, 16 8.8 | 10.9, 32 12.1 | 13.5; but the model's law at K = 32 10.3 | 8.6, K = 64 16.4 | 12.3.
template <class T>
__device__ __forceinline__ void co3_merge_steps(Co3BuildLds &L, const int lane, const int nact)
{
    typedef typename T::W W;
    const W *leaf_w = reinterpret_cast<const W *>(L.leaf_w);
    W *node_w = reinterpret_cast<W *>(L.node_w);
    if (lane == 0) {
        int q1 = 0, q2 = 0;
        for (int ne = 0; ne < nact - 1; ++ne) {
            const W l0 = leaf_w[q1], l1 = leaf_w[q1 + 1], n0 = node_w[q2], n1 = node_w[q2 + 1];
            const bool leaves = l1 <= n0, nodes = !leaves && n1 < l0;
            L.parent[nodes ? 256 + q2 + 1 : q1] = (uint16_t)ne;
            L.parent[leaves ? q1 + 1 : 256 + q2] = (uint16_t)ne;
            node_w[ne] = leaves ? l0 + l1 : nodes ? n0 + n1 : l0 + n0;
            q1 += leaves ? 2 : nodes ? 0 : 1;
            q2 += leaves ? 0 : nodes ? 2 : 1;
        }
    }
    co3_lds_order();
}

// Code lengths = depths of the leaves, by the same wavefront: every node's way up is doubled until it ends at the
// root (log2 of the depth steps instead of one step per level).
__device__ __forceinline__ void co3_leaf_depths(Co3BuildLds &L, const int lane, const int nact)
{
    const int root = nact - 2;                // the last node
    uint32_t e[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int v = lane + k * CO3_WAVE;
        e[k] = v < root ? (uint32_t)L.parent[256 + v] | (1u << 16) : (uint32_t)(root < 0 ? 0 : root);
        L.up[v] = e[k];
    }
    co3_lds_order();
    for (int step = 0; step < 8; ++step) {    // (255 nodes: eight doublings reach any root)
        bool done = true;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t p = L.up[e[k] & 0xffu];
            e[k] = (p & 0xffffu) | ((e[k] & 0xffff0000u) + (p & 0xffff0000u));
            done &= (int)(e[k] & 0xffffu) == root || root < 0;
        }
        co3_lds_order();
#pragma unroll
        for (int k = 0; k < 4; ++k) L.up[lane + k * CO3_WAVE] = e[k];
        co3_lds_order();
        if (__all(done)) break;
    }
    uint32_t longest = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int leaf = lane + k * CO3_WAVE;
        if (leaf < nact) {
            const uint32_t depth = nact == 1 ? 1u : 1u + (L.up[L.parent[leaf] & 0xffu] >> 16);
            L.len[L.leaf_sym[leaf]] = (uint8_t)(depth > CO3_LEN_CAP ? CO3_LEN_CAP : depth);
            longest = longest > depth ? longest : depth;
        }
    }
    longest = wave_max_u32(longest);
    if (lane == 0) L.maxlen = longest;
}

// weight: of symbol tid, for tid < 256 (0 from K on).  out: the user's code blob.  All BLOCK lanes of the workgroup
// call it.
template <int BLOCK>
__device__ __forceinline__ void co3_build_code_group(Co3BuildLds &L, const int tid, const uint32_t weight, const int K,
                                                     Co3Code *out, int32_t *status)
{
    const int lane = tid & (CO3_WAVE - 1), wave = __builtin_amdgcn_readfirstlane(tid / CO3_WAVE);
    if (tid < 256) {
        L.key[tid] = weight ? (double)(((uint64_t)weight << 8) | (uint64_t)tid) : __builtin_huge_val();
        L.rank[tid] = 0;
        L.len[tid] = 0;
        L.sorted[tid] = 0;
    }
    if (tid == 0) {
        L.nact = 0;
        L.total = 0;
    }
    __syncthreads();

    // leaves in (weight, symbol) order: a symbol's place is the number of keys below its own; PARTS lanes per
    // symbol, each comparing with its share of the keys (all lanes of a wavefront read the same two entries at a
    // time, a broadcast)
    constexpr int PARTS = BLOCK / 256;
    static_assert(PARTS * 256 == BLOCK, "whole alphabets of lanes");
    if ((tid & 255) < (K + CO3_WAVE - 1) / CO3_WAVE * CO3_WAVE) {
        const int sy = tid & 255, part = tid >> 8, per = (K + 2 * PARTS - 1) / (2 * PARTS) * 2;      // keys per part, an even number
        const double mine = L.key[sy];
        const int k0 = part * per, k1 = k0 + per < 256 ? k0 + per : 256;
        uint32_t below = 0;
#pragma unroll 8
        for (int i = k0; i < k1; i += 2) {
            const double2 kk = *reinterpret_cast<const double2 *>(&L.key[i]);
            below += (kk.x < mine ? 1u : 0u) + (kk.y < mine ? 1u : 0u);
        }
        if (below) atomicAdd(&L.rank[sy], below);
        if (part == 0) {
            const int c = __popcll(__ballot(weight != 0));
            unsigned long long t = weight;
#pragma unroll
            for (int o = 1; o < CO3_WAVE; o <<= 1) t += (unsigned long long)__shfl_xor((long long)t, o, CO3_WAVE);
            if (lane == 0 && c) {
                atomicAdd(&L.nact, (uint32_t)c);
                atomicAdd(&L.total, t);
            }
        }
    }
    __syncthreads();
    const int nact = (int)L.nact;
    const bool small = L.total < (1ull << 30);        // uniform
    if (tid < 256 && weight) {
        const uint32_t r = L.rank[tid];
        if (small) reinterpret_cast<uint32_t *>(L.leaf_w)[r] = weight;
        else L.leaf_w[r] = (double)weight;
        L.leaf_sym[r] = (uint8_t)tid;
    }
    for (int j = tid; j < 256 + CO3_WAVE; j += BLOCK) {
        if (small) {
            if (j >= nact) reinterpret_cast<uint32_t *>(L.leaf_w)[j] = Co3MergeU32::none();
            reinterpret_cast<uint32_t *>(L.node_w)[j] = Co3MergeU32::none();
        } else {
            if (j >= nact) L.leaf_w[j] = Co3MergeF64::none();
            L.node_w[j] = Co3MergeF64::none();
        }
    }
    __syncthreads();
    if (wave == 0) {
        if (nact <= CO3_HB_STEPS && small) co3_merge_steps<Co3MergeU32>(L, lane, nact);
        else if (nact <= CO3_HB_STEPS) co3_merge_steps<Co3MergeF64>(L, lane, nact);
        else if (small) co3_merge_rounds<Co3MergeU32>(L, lane, nact);
        else co3_merge_rounds<Co3MergeF64>(L, lane, nact);
        co3_leaf_depths(L, lane, nact);
    }
    __syncthreads();
    const uint32_t maxlen = L.maxlen;
    if (tid == 0 && maxlen > CO3_MAX_CODE_LEN) co3_raise(status, CO3_EINVAL);

    // A symbol's rank among the symbols of its length: within its wavefront by ballots, one per length; lane l then
    // holds the wavefront's number of symbols of length l.
    const uint32_t top_len = maxlen < CO3_LEN_CAP ? maxlen : CO3_LEN_CAP;
    const uint32_t l = tid < 256 ? L.len[tid] : 0u;
    uint32_t rank = 0;
    if (wave < 4) {
        uint32_t mine = 0;
#pragma unroll 4
        for (uint32_t k = 1; k <= top_len; ++k) {
            const uint64_t b = __ballot(l == k);
            if (l == k) rank = (uint32_t)__popcll(b & ((1ull << lane) - 1ull));
            if ((uint32_t)lane == k) mine = (uint32_t)__popcll(b);
        }
        L.wave_cnt[wave][lane] = (uint16_t)mine;
    }
    __syncthreads();
    // canonical numbering, in every wavefront for itself, lane l for length l: base = symbols of shorter lengths,
    // first code = sum over the shorter lengths j of count[j] << (l - j)
    uint32_t cnt = 0, lower = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const uint32_t c = L.wave_cnt[w][lane];
        cnt += c;
        lower += w < wave ? c : 0u;
    }
    const uint32_t base = wave_scan_incl_u32(cnt, lane) - cnt;
    uint64_t first;
    {
        // as a sum of shares of the code space: count[j] << (63 - j) over the shorter lengths, shifted back
        uint64_t incl = (uint64_t)cnt << (63 - lane), mine = incl;
        auto step = [&](auto dpp, auto rows) {
            const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)incl, dpp.value, rows.value, 0xf, false);
            const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(incl >> 32), dpp.value, rows.value, 0xf, false);
            incl += ((uint64_t)hi << 32) | lo;
        };
        step(Co3Const<0x111>(), Co3Const<0xf>());
        step(Co3Const<0x112>(), Co3Const<0xf>());
        step(Co3Const<0x114>(), Co3Const<0xf>());
        step(Co3Const<0x118>(), Co3Const<0xf>());
        step(Co3Const<0x142>(), Co3Const<0xa>());
        step(Co3Const<0x143>(), Co3Const<0xc>());
        first = (incl - mine) >> (63 - lane);
    }

    if (wave < 4) {
        const uint64_t first_l = (uint64_t)__shfl((long long)first, (int)l, CO3_WAVE);
        rank += (uint32_t)__shfl((int)lower, (int)l, CO3_WAVE);
        const uint32_t base_l = (uint32_t)__shfl((int)base, (int)l, CO3_WAVE);
        if (l) L.sorted[base_l + rank] = (uint8_t)tid;
        out->len[tid] = (uint8_t)l;
        out->enc[tid] = l ? ((first_l + rank) << 6) | (uint64_t)l : 0ull;
    }
    if (wave == BLOCK / CO3_WAVE - 1) {       // (with 1024 lanes one that has no symbols)
        out->first_code[lane] = first;
        out->count[lane] = (uint16_t)cnt;
        out->base[lane] = (uint16_t)base;
        if (lane < CO3_LUT_BITS_MAX + 2) L.at[lane] = (int32_t)base - (int32_t)(uint32_t)first;    // prefix -> place in sorted[]
        if (lane < 2) {                       // beyond every length
            out->count[CO3_WAVE + lane] = 0;
            out->base[CO3_WAVE + lane] = (uint16_t)nact;
        }
        if (lane == 0) out->first_code[CO3_WAVE] = 0;
    }
    const uint32_t lut_bits = maxlen < 1 ? 1 : (maxlen > CO3_LUT_BITS_MAX ? CO3_LUT_BITS_MAX : maxlen);
    if (tid == 0) {
        out->nact = (uint32_t)nact;
        out->maxlen = maxlen;
        out->lut_bits = lut_bits;
        out->reserved = 0;
    }
    __syncthreads();
    if (tid < 256 / 4) reinterpret_cast<uint32_t *>(out->sorted)[tid] = reinterpret_cast<const uint32_t *>(L.sorted)[tid];

    // decoder table: entry i decodes the lut_bits-bit prefix i by the canonical rule.  Canonical codewords grow with
    // their length, so the prefixes resolved by length <= k form the range [0, limit[k]) with
    // limit[k] = (first_code[k] + count[k]) << (lut_bits - k): the entry's length is the first k whose limit exceeds
    // i (the limits do not decrease: their number at or below i, plus one).  They are uniform over the wavefront
    // (lane k of every wavefront holds that of length k).  A lane makes four entries in a row and counts for the
    // first and the last: between them the length is mostly the same.
    uint32_t lim[CO3_LUT_BITS_MAX + 1];
    {
        const uint64_t end = first + cnt;
        const uint32_t mylim = lane >= 1 && lane <= (int)lut_bits ? (uint32_t)(end << (lut_bits - lane)) : 0xffffffffu;
#pragma unroll
        for (int k = 1; k <= CO3_LUT_BITS_MAX; ++k) lim[k] = (uint32_t)__builtin_amdgcn_readlane((int)mylim, k);
    }
    auto length_of = [&](uint32_t i) -> uint32_t {
        uint32_t k = 1;
#pragma unroll
        for (int j = 1; j <= CO3_LUT_BITS_MAX; ++j) k += i >= lim[j] ? 1u : 0u;
        return k;
    };
    auto entry = [&](uint32_t i, uint32_t k) -> uint32_t {
        return k > lut_bits ? 0u : (k << 8) | L.sorted[(uint32_t)((int)(i >> (lut_bits - k)) + L.at[k]) & 255u];
    };
    for (uint32_t i = 4 * tid; i < (1u << lut_bits); i += 4 * BLOCK) {
        const uint32_t ka = length_of(i), kd = length_of(i + 3);
        uint32_t kb = ka, kc = ka;
        if (ka != kd) {
            kb = length_of(i + 1);
            kc = length_of(i + 2);
        }
        const uint32_t e01 = entry(i, ka) | (entry(i + 1, kb) << 16), e23 = entry(i + 2, kc) | (entry(i + 3, kd) << 16);
        *reinterpret_cast<uint2 *>(out->lut + i) = make_uint2(e01, e23);
    }
}
