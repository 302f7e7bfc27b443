// Huffman code construction (Sec. III (ii)): one workgroup per user builds code lengths,
// canonical codewords and the decoder tables from K <= 256 integer weights.
#include "co3_dev.h"
#include "co3_huffman.h"
#include "kernels.h"

// The weights of a user -> its code.
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_build_code(const uint32_t *__restrict__ weights, int K, char *codes,
                                                              int32_t *status)
{
    const int u = blockIdx.x;
    const int tid = threadIdx.x;
    __shared__ Co3BuildLds lds;
    const uint32_t wt = tid < K ? weights[(size_t)u * K + tid] : 0u;
    co3_build_code_group<BLOCK>(lds, tid, wt, K, reinterpret_cast<Co3Code *>(codes + (size_t)u * CO3_CODE_BYTES), status);
}

// What is left of a user's steps before compression when a resident grid has converted everything but the
// ragged end of the vector (Algorithm 1, the user's conversion, memory update and code design; Sec. III
// (i)-(iii)): one workgroup per user converts elements [n_full, n) with the user's anchor, counts their
// symbols, adds the grid's partial count tables to them and builds the user's code.  A latency chain like the
// code build itself: the partial tables are requested first, the ragged end (at most 12,287 elements) takes 16
// bytes per lane and step.
__global__ __launch_bounds__(CO3_HB_BLOCK) void k_user_finish(const float *__restrict__ g, float *__restrict__ err,
                                                               uint8_t *__restrict__ sym, int64_t n, int64_t n_full,
                                                               int64_t stride, const int64_t *__restrict__ seg_off, int nseg,
                                                               const int32_t *__restrict__ anchor, float gamma,
                                                               co3_fmt fmt, int sym_nib, const uint32_t *__restrict__ counts_rep,
                                                               uint32_t *__restrict__ counts, char *codes,
                                                               int32_t *status, int first_user, int U)
{
    const FmtC fc(fmt);
    const int K = fc.K;
    const int tid = threadIdx.x;
    const int u = first_user + blockIdx.x;       // users first_user .. first_user + gridDim.x - 1 of the batch of U
    __shared__ Co3BuildLds lds;
    __shared__ uint32_t hist[256];
    constexpr int PARTS = CO3_HB_BLOCK / 256, PER = CO3_COOP_COUNT_REPS / PARTS;
    static_assert(CO3_COOP_COUNT_REPS % PARTS == 0, "partial tables per lane");
    uint32_t part[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k)                // (independent loads, all in flight before the ragged end is converted)
        part[k] = (tid & 255) < K ? counts_rep[((size_t)((tid >> 8) + k * PARTS) * U + u) * K + (tid & 255)] : 0u;
    if (tid < 256) hist[tid] = 0u;
    __syncthreads();
    // one anchor per (user, tensor): anchor is [U][nseg]
    const float *gu = g + (int64_t)u * stride;
    float *eu = err + (int64_t)u * stride;
    uint8_t *su = sym + (int64_t)u * (sym_nib ? stride / 2 : stride);
    const int32_t *anchor_u = anchor + (int64_t)u * nseg;
    // four consecutive elements per thread and step (n_full is a multiple of 256: loads are aligned, and with two
    // symbols per byte the bytes a thread writes are its own)
    for (int64_t i = n_full + 4 * (int64_t)tid; i < n; i += 4 * CO3_HB_BLOCK) {
        uint32_t q[4] = {0u, 0u, 0u, 0u};
        const int cnt = n - i < 4 ? (int)(n - i) : 4;
        float gv[4] = {0.f, 0.f, 0.f, 0.f}, ev[4] = {0.f, 0.f, 0.f, 0.f};
        if (cnt == 4) {
            const float4 a = *reinterpret_cast<const float4 *>(gu + i), b = *reinterpret_cast<const float4 *>(eu + i);
            gv[0] = a.x, gv[1] = a.y, gv[2] = a.z, gv[3] = a.w;
            ev[0] = b.x, ev[1] = b.y, ev[2] = b.z, ev[3] = b.w;
        } else {
            for (int c = 0; c < 3; ++c)
                if (c < cnt) gv[c] = gu[i + c], ev[c] = eu[i + c];
        }
        const int s_first = co3_find_seg(seg_off, nseg, i), s_last = co3_find_seg(seg_off, nseg, i + cnt - 1);
        const int A_first = anchor_u[s_first];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (c >= cnt) break;
            const float x = gv[c] + gamma * ev[c];          // no contraction (build flag): one rounding per operation
            const int A = s_first == s_last ? A_first : anchor_u[co3_find_seg(seg_off, nseg, i + c)];
            float v;
            co3_quantize(x, A - fc.F + 1, A, fc.E, fc.M, fc.codemax, q[c], v);
            ev[c] = x - v;
            atomicAdd(&hist[q[c]], 1u);
        }
        if (cnt == 4) *reinterpret_cast<float4 *>(eu + i) = make_float4(ev[0], ev[1], ev[2], ev[3]);
        else
            for (int c = 0; c < 3; ++c)
                if (c < cnt) eu[i + c] = ev[c];
        if (sym_nib) {
            su[i >> 1] = (uint8_t)(q[0] | (q[1] << 4));
            if (cnt > 2) su[(i >> 1) + 1] = (uint8_t)(q[2] | (q[3] << 4));
        } else {
            for (int c = 0; c < 4; ++c)
                if (c < cnt) su[i + c] = (uint8_t)q[c];
        }
    }
    {
        uint32_t sum = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) sum += part[k];
        if (sum) atomicAdd(&hist[tid & 255], sum);
    }
    __syncthreads();
    uint32_t wt = 0u;
    if (tid < K) {
        wt = hist[tid];
        counts[(size_t)u * K + tid] = wt;
    }
    co3_build_code_group<CO3_HB_BLOCK>(lds, tid, wt, K, reinterpret_cast<Co3Code *>(codes + (size_t)u * CO3_CODE_BYTES), status);
}

hipError_t co3_launch_user_finish(const float *g, float *err, uint8_t *sym, int64_t n, int64_t n_full, int64_t stride, int U,
                                  const int64_t *seg_off, int nseg, const int32_t *anchor, float gamma, co3_fmt fmt,
                                  int sym_nib, const uint32_t *counts_rep, uint32_t *counts, void *codes,
                                  int32_t *status, hipStream_t st, int first_user, int users)
{
    if (U <= 0 || users <= 0) return hipSuccess;
    Co3LaunchTimer tm(CO3_K_BUILD, st);
    hipLaunchKernelGGL(k_user_finish, dim3(users), dim3(CO3_HB_BLOCK), 0, st, g, err, sym, n, n_full, stride, seg_off, nseg, anchor, gamma, fmt,
                       sym_nib, counts_rep, counts, reinterpret_cast<char *>(codes), status, first_user, U);
    return hipGetLastError();
}

hipError_t co3_launch_build_code(const uint32_t *weights, int U, int K, void *codes, int32_t *status, hipStream_t st)
{
    if (U <= 0) return hipSuccess;
    Co3LaunchTimer tm(CO3_K_BUILD, st);
    // More codes than two large workgroups per compute unit hold at a time: what counts is how many are under way, and
    // one wavefront does the merge (256 | 1024 lanes, 400, 700 and 4,000 codes: K = 256 25 | 23 us, 27 | 40, 70 | 164;
    // K = 32 17.8 | 17.5, 19 | 30, 46 | 120).  The tables of up to 8 symbols gain nothing from more lanes (300 codes of
    // K = 8 7.2 | 7.9).
    const int known = co3_device_cus(), cus = known > 0 ? known : 256;
    if (U > 2 * cus || K <= 8)
        hipLaunchKernelGGL(k_build_code<256>, dim3(U), dim3(256), 0, st, weights, K, reinterpret_cast<char *>(codes), status);
    else
        hipLaunchKernelGGL(k_build_code<CO3_HB_BLOCK>, dim3(U), dim3(CO3_HB_BLOCK), 0, st, weights, K,
                           reinterpret_cast<char *>(codes), status);
    return hipGetLastError();
}
