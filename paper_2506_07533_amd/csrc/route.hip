// moqae_route_chunks: router MLP (Eq. (1), Sec. 3.2), token top-1 and chunk majority vote
// (Eq. (2)), routing freezing (Sec. 3.4).
//
// route_kernel (chunks of 64 tokens or more): one wavefront per (sequence, KV head, chunk).  A lane owns one token: it
// requests its whole 256-byte key row at once (no LDS, no barrier in the loop) and runs
// the 2*M length-D dot products as sequential binary32 sums (the products of two fp16 values
// are exact in binary32, so a fused multiply-add rounds exactly like multiply-then-add), which
// is what makes the integer result reproducible bit for bit.  The router weights are
// wave-uniform: they are read through uniform 32-bit loads of the caller's fp16 arrays.
//
// route_short_kernel (chunks of 8, 16 and 32 tokens): 64/N consecutive chunks of a row share a window of 64 lanes, which
// route_kernel would leave half to seven eighths idle; a chunk's votes are its lanes' bits of the ballots.  Persistent
// wavefronts that go by half rows (64 dims): the next half rows are requested, in whole 128-byte lines, before the current
// ones are multiplied, and reach their lanes through LDS.  32-token chunks, 2.1 M rows: 104 us against 156 (5.2 TB/s; the
// multiply-adds in their order alone take about 70).  For one window per chunk and more it is not the better one: 231 us
// against 224 for 128-token chunks, 5.2 M rows.  The windows begin after a row's frozen chunks, whose keys are not read:
// 256 rows of 64 chunks of 32 tokens, 1 frozen 28.3 us a call against 28.8 with windows over all of them, 3 frozen 26.9
// against 28.9, 60 or all frozen 11.6 (a call's launch) against 28.9.
#include "moqae_dev.hpp"
#include "moqae_kernels.hpp"
#include "pack_dev.hpp"
#include "route_dev.hpp"
#include <algorithm>

namespace moqae {

constexpr int kRouteThreads = 64;         // one wavefront per workgroup, one lane per token

template <int M>
__global__ __launch_bounds__(kRouteThreads) void route_kernel(RouteArgs a) {
    __shared__ float w3f[72];                        // W3 as binary32, then the optional bias

    const int c = a.chunk_begin + (int)blockIdx.x;
    const int u = (int)blockIdx.y;
    const int tid = (int)threadIdx.x;
    const int64_t eidx = (int64_t)u * a.expert_stride + c;

    if (c < a.freeze_chunks) {                       // routing freezing: never routed, FP16 expert
        if (tid == 0) a.expert[eidx] = (uint8_t)a.e16;
        if (a.votes && tid < M) a.votes[eidx * M + tid] = 0;
        return;
    }
    if (tid < M * M) w3f[tid] = half_bits_to_float(a.W3[tid]);
    if (a.bias && tid < M) w3f[64 + tid] = a.bias[tid];
    __syncthreads();

    const int b = u / a.Hkv, h = u % a.Hkv;
    const uint16_t *Kc = a.K + (int64_t)b * a.stride_b + (int64_t)h * a.stride_h + (int64_t)c * a.N * a.stride_s;
    const uint32_t *W1w = reinterpret_cast<const uint32_t *>(a.W1);
    const uint32_t *W2w = reinterpret_cast<const uint32_t *>(a.W2);

    int cnt[M];                                      // votes, identical in every lane
    route_tokens<M>(Kc, a.N, a.stride_s, W1w, W2w, w3f, a.bias != nullptr, tid, cnt);
    if (tid == 0) {
        int best = 0, cbest = cnt[0];
#pragma unroll
        for (int k = 1; k < M; k++) if (cnt[k] > cbest) { best = k; cbest = cnt[k]; }
        a.expert[eidx] = (uint8_t)best;
    }
    if (a.votes) {
#pragma unroll
        for (int k = 0; k < M; k++) if (tid == k) a.votes[eidx * M + k] = cnt[k];
    }
}

// Few chunks of more than 64 tokens (a decode step that flushes a chunk per head): one wavefront per 64 tokens of a chunk,
// the votes added up in LDS.  A wavefront that takes a chunk's passes one after the other has nobody to hide its latency.
// One chunk of 128 tokens for each of 32 heads: 6.9 us against 10.2; calls on 64 chunks of 256 tokens: 11.5 us against 18.4.
// From half a wavefront per SIMD on, the other chunks' wavefronts hide it.
template <int M>
__global__ __launch_bounds__(256) void route_split_kernel(RouteArgs a) {
    __shared__ float w3f[72];                        // W3 as binary32, then the optional bias
    __shared__ int votes_s[8];
    const int c = a.chunk_begin + (int)blockIdx.x;
    const int u = (int)blockIdx.y;
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t eidx = (int64_t)u * a.expert_stride + c;
    if (c < a.freeze_chunks) {                       // routing freezing: never routed, FP16 expert
        if (tid == 0) a.expert[eidx] = (uint8_t)a.e16;
        if (a.votes && tid < M) a.votes[eidx * M + tid] = 0;
        return;
    }
    if (tid < M * M) w3f[tid] = half_bits_to_float(a.W3[tid]);
    if (a.bias && tid < M) w3f[64 + tid] = a.bias[tid];
    if (tid < 8) votes_s[tid] = 0;
    __syncthreads();
    const uint16_t *Kc = a.K + (int64_t)(u / a.Hkv) * a.stride_b + (int64_t)(u % a.Hkv) * a.stride_h + ((int64_t)c * a.N + wave * 64) * a.stride_s;
    int cnt[M];
    route_tokens<M>(Kc, min(64, a.N - wave * 64), a.stride_s, reinterpret_cast<const uint32_t *>(a.W1),
                    reinterpret_cast<const uint32_t *>(a.W2), w3f, a.bias != nullptr, lane, cnt);
#pragma unroll
    for (int k = 0; k < M; k++) if (lane == k) atomicAdd(&votes_s[k], cnt[k]);
    __syncthreads();
    if (tid == 0) {
        int best = 0;
        for (int k = 1; k < M; k++) if (votes_s[k] > votes_s[best]) best = k;   // strict: the first maximum wins
        a.expert[eidx] = (uint8_t)best;
    }
    if (a.votes && tid < M) a.votes[eidx * M + tid] = votes_s[tid];
}

constexpr int kShortWaves = 4;            // independent wavefronts of a workgroup: they share the copy of W3
constexpr int kShortWgPerCu = 4;

template <int M>
__global__ __launch_bounds__(kShortWaves * 64) void route_short_kernel(RouteArgs a) {
    __shared__ float w3f[72];                        // W3 as binary32, then the optional bias
    __shared__ __attribute__((aligned(16))) uint8_t tbuf[kShortWaves * 64 * kTRow];
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);           // wave-uniform, kept scalar
    if (tid < M * M) w3f[tid] = half_bits_to_float(a.W3[tid]);
    if (a.bias && tid < M) w3f[64 + tid] = a.bias[tid];
    __syncthreads();

    // routing freezing: the first chunks of every row are never routed
    const int n_frozen = min(max(a.freeze_chunks - a.chunk_begin, 0), a.n_chunks);
    const uint32_t win0 = (uint32_t)wave * gridDim.x + blockIdx.x, stride = gridDim.x * kShortWaves;
    const int c_begin = a.chunk_begin + n_frozen, n_chunks = a.n_chunks - n_frozen;
    const int N = a.N, cpw = 64 / N;                 // chunks of a window
    const int per_row = max((n_chunks + cpw - 1) / cpw, 1);
    const const_words W1w = reinterpret_cast<const_words>(reinterpret_cast<uintptr_t>(a.W1));
    const const_words W2w = reinterpret_cast<const_words>(reinterpret_cast<uintptr_t>(a.W2));

    // window t of row u, from win0 on in steps of all wavefronts of the grid, on the scalar unit
    const int step_u = (int)(stride / (uint32_t)per_row), step_t = (int)(stride % (uint32_t)per_row);
    int u = n_chunks > 0 ? (int)(win0 / (uint32_t)per_row) : a.BH, t = (int)(win0 % (uint32_t)per_row), h = 0;
    auto advance = [&]() {
        t += step_t; u += step_u;
        if (t >= per_row) { t -= per_row; u++; }
    };
    auto tokens_of = [&](int st) { return min(cpw, n_chunks - st * cpw) * N; };
    auto store = [&](int su, int st, const int (&cnt)[M]) {   // lane j: chunk j of the window
        const int c = c_begin + st * cpw + lane;
        if (lane >= cpw || c >= c_begin + n_chunks) return;
        int best = 0, cbest = cnt[0];
#pragma unroll
        for (int k = 1; k < M; k++) if (cnt[k] > cbest) { best = k; cbest = cnt[k]; }
        const int64_t eidx = (int64_t)su * a.expert_stride + c;
        a.expert[eidx] = (uint8_t)best;
        if (a.votes) {
#pragma unroll
            for (int k = 0; k < M; k++) a.votes[eidx * M + k] = cnt[k];
        }
    };
    uint4 v[8];                                      // half rows as loaded: register j, piece lane%8 of row 8j + lane/8
    const int r8 = lane >> 3, p8 = lane & 7;
    auto request = [&]() {                           // rows past the window's tokens read its last row
        const uint16_t *Kc = a.K + (int64_t)(u / a.Hkv) * a.stride_b + (int64_t)(u % a.Hkv) * a.stride_h
                           + (int64_t)(c_begin + t * cpw) * N * a.stride_s + h * 64;
        const int last = tokens_of(t) - 1;
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = nt_load(reinterpret_cast<const uint4 *>(Kc + (int64_t)min(8 * j + r8, last) * a.stride_s) + p8);
    };
    float accA[M], accB[M];
#pragma unroll
    for (int k = 0; k < M; k++) { accA[k] = 0.0f; accB[k] = 0.0f; }
    uint8_t *mine = tbuf + wave * (64 * kTRow);
    if (u < a.BH) request();
#pragma unroll 1
    while (u < a.BH) {
        const int cu = u, ct = t, ch = h;
        uint4 x[8];
#pragma unroll
        for (int j = 0; j < 8; j++) *reinterpret_cast<uint4 *>(mine + (8 * j + r8) * kTRow + p8 * 16) = v[j];
        h ^= 1;                                      // the next half rows
        if (h == 0) advance();
        if (u < a.BH) request();
        wave_lds_sync();
#pragma unroll
        for (int k = 0; k < 8; k++) x[k] = *reinterpret_cast<const uint4 *>(mine + lane * kTRow + k * 16);
        wave_lds_sync();
        route_half_row<M>(x, ch * 64, W1w, W2w, accA, accB);
        if (ch == 0) continue;
        const bool active = lane < tokens_of(ct);
        const int top = route_top<M>(accA, accB, w3f, a.bias != nullptr);
        int cnt[M];
#pragma unroll
        for (int k = 0; k < M; k++) {
            accA[k] = 0.0f; accB[k] = 0.0f;
            const unsigned long long mask = __ballot(active && top == k);
            cnt[k] = lane < cpw ? __popcll((mask >> (lane * N)) & ((1ull << N) - 1ull)) : 0;
        }
        store(cu, ct, cnt);
    }
    // frozen chunks take the FP16 expert
    for (uint32_t ru = win0; n_frozen > 0 && ru < (uint32_t)a.BH; ru += stride) {
        const int64_t e0 = (int64_t)ru * a.expert_stride + a.chunk_begin;
        for (int c = lane; c < n_frozen; c += 64) {
            a.expert[e0 + c] = (uint8_t)a.e16;
            if (a.votes) {
#pragma unroll
                for (int k = 0; k < M; k++) a.votes[(e0 + c) * M + k] = 0;
            }
        }
    }
}

template <int M>
static hipError_t launch_m(const RouteArgs &a, int n_cu, hipStream_t s) {
    if (a.N > 64 && (long long)a.n_chunks * a.BH <= 2LL * n_cu) {   // fewer wavefronts than half of the SIMDs
        hipLaunchKernelGGL(route_split_kernel<M>, dim3((unsigned)a.n_chunks, (unsigned)a.BH), dim3((unsigned)((a.N + 63) / 64 * 64)), 0, s, a);
    } else if (a.N >= 64) {
        hipLaunchKernelGGL(route_kernel<M>, dim3((unsigned)a.n_chunks, (unsigned)a.BH), dim3(kRouteThreads), 0, s, a);
    } else {
        const int cpw = 64 / a.N, n_frozen = std::min(std::max(a.freeze_chunks - a.chunk_begin, 0), a.n_chunks);
        const long long windows = (long long)a.BH * ((a.n_chunks - n_frozen + cpw - 1) / cpw);
        // a window per workgroup as long as there are compute units, then all four wavefronts of a workgroup
        long long n_wg = (windows + kShortWaves - 1) / kShortWaves;
        if (n_wg < n_cu) n_wg = windows < n_cu ? windows : n_cu;
        if (n_wg < 1) n_wg = std::min(a.BH, n_cu);   // frozen chunks only: a row per wavefront
        if (n_wg > (long long)kShortWgPerCu * n_cu) n_wg = (long long)kShortWgPerCu * n_cu;
        hipLaunchKernelGGL(route_short_kernel<M>, dim3((unsigned)n_wg), dim3(kShortWaves * 64), 0, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_route(const RouteArgs &a, int M, int n_cu, hipStream_t s) {
    if (a.n_chunks <= 0 || a.BH <= 0) return hipSuccess;
    switch (M) {
        case 1: return launch_m<1>(a, n_cu, s);
        case 2: return launch_m<2>(a, n_cu, s);
        case 3: return launch_m<3>(a, n_cu, s);
        case 4: return launch_m<4>(a, n_cu, s);
        case 5: return launch_m<5>(a, n_cu, s);
        case 6: return launch_m<6>(a, n_cu, s);
        case 7: return launch_m<7>(a, n_cu, s);
        case 8: return launch_m<8>(a, n_cu, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace moqae
