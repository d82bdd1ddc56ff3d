// moqae_route_chunks: router MLP (Eq. (1), Sec. 3.2), token top-1 and chunk majority vote
// (Eq. (2)), routing freezing (Sec. 3.4).
//
// route_kernel: persistent wavefronts over windows of 64 tokens: a part of a chunk, or (chunks of 8, 16 and 32 tokens) 64/N
// consecutive chunks of a row, whose votes are their lanes' bits of the ballots.  The decision is defined by sequential
// binary32 sums over the dims; it is taken from the same sums on the matrix cores where these tell it with certainty
// (certain_top), and from the sums in order, for the tokens they leave open, where they do not.  The rows come in whole lines, half a window
// ahead, and reach the lanes of the matrix products through LDS.
// What bounds it: HBM, and for small calls latency.  5.2 M rows in 128-token chunks 211 us a call (6.35 TB/s) against 241 with a
// lane per token and the sums in order (whose 1024 multiply-adds alone took 170); 524 288 rows 24.3 us against 29.6, 131 072 rows 9.3 to
// 10.3 against 10.2 to 12.5, 32 768 rows in 32-token chunks 6.6 against 7.2 (9.4 while open tokens sent their whole window through
// the sums in order).  Two workgroups of four wavefronts per compute unit: three and four (128 registers) 213 and 220 us; a whole
// window ahead 211, and 25.3 and 10.8 us for 524 288 and 131 072 rows; rows requested in the operands' own shape, four 16-byte
// pieces of a row per load, 228.
// The windows begin after a row's frozen chunks, whose keys are not read.
//
// route_split_kernel: few chunks.
#include "moqae_dev.hpp"
#include "moqae_kernels.hpp"
#include "pack_dev.hpp"
#include "route_dev.hpp"
#include <algorithm>

namespace moqae {

constexpr int kRouteWaves = 4;            // independent wavefronts of a workgroup: they share the copy of W3
constexpr int kRouteWgPerCu = 2;

// Half a window of 64 tokens: the blocks of 16 tokens `pair` and `pair` + 2 (see gather_sums), row r of them = token
// 16 pair + r + (r < 16 ? 0 : 16).  Requested in whole rows (streaming loads: nothing is read twice), handed to the lanes of the
// matrix products through LDS: piece p of row r at 16 r + (p ^ r % 16), so that both ways every bank is touched once.
constexpr int kHalfPieces = 32 * 16;
struct HalfRows { uint4 v[8]; };
__device__ __forceinline__ void request_half(const uint16_t *Kc, int64_t stride_s, int n_tok, int pair, int lane, HalfRows &h) {
    const int piece = lane & 15, r4 = lane >> 4;
    if (n_tok == 64 && stride_s < (1 << 24)) {   // scalar row addresses, one 32-bit offset per lane
        const uint32_t off = (uint32_t)r4 * (uint32_t)stride_s * 2u + (uint32_t)piece * 16u;
#pragma unroll
        for (int j = 0; j < 8; j++)
            h.v[j] = nt_load(reinterpret_cast<const uint4 *>(reinterpret_cast<const uint8_t *>(Kc + (16 * pair + 4 * j + (j < 4 ? 0 : 16)) * stride_s) + off));
        return;
    }
#pragma unroll
    for (int j = 0; j < 8; j++)           // rows past the window's tokens read its last row
        h.v[j] = nt_load(reinterpret_cast<const uint4 *>(Kc + (int64_t)min(16 * pair + 4 * j + (j < 4 ? 0 : 16) + r4, n_tok - 1) * stride_s) + piece);
}
__device__ __forceinline__ void stage_half(const HalfRows &h, int lane, uint4 *buf) {
    const int piece = lane & 15, r4 = lane >> 4;
#pragma unroll
    for (int j = 0; j < 8; j++) buf[(4 * j + r4) * 16 + (piece ^ ((4 * j + r4) & 15))] = h.v[j];
}
template <int M>
__device__ __forceinline__ void half_sums(const RouterWeights &w, const uint4 *buf, int pair, int lane, v4f_r (&val)[M <= 4 ? 2 : 4], v4f_r (&bnd)[M <= 4 ? 2 : 4]) {
    const int x = lane & 15, q = lane >> 4;
    v4f_r c[2], d[2];
#pragma unroll
    for (int h = 0; h < 2; h++) {
        c[h] = v4f_r{0.0f, 0.0f, 0.0f, 0.0f}; d[h] = c[h];
#pragma unroll
        for (int s = 0; s < 4; s++) router_step(w, s, buf[(16 * h + x) * 16 + ((4 * s + q) ^ x)], c[h], d[h]);
    }
    if constexpr (M <= 4) { val[pair] = pick_pair(c[0], c[1], lane); bnd[pair] = pick_pair(d[0], d[1], lane); }
    else { val[pair] = c[0]; val[pair + 2] = c[1]; bnd[pair] = d[0]; bnd[pair + 2] = d[1]; }
}
template <int M>
__device__ __forceinline__ int window_top(v4f_r (&val)[M <= 4 ? 2 : 4], v4f_r (&bnd)[M <= 4 ? 2 : 4], const RouterSums<M> &floor, const uint16_t *Kc, int64_t stride_s, int n_tok,
                                          int lane, const RouteArgs &a, const uint32_t *raw, const float *w3f) {
    RouterSums<M> v, s;
    gather_sums<M>(val, v); gather_sums<M>(bnd, s);
    RouterValues<M> o;
    int top;
    const bool sure = certain_top<M>(v, s, floor, w3f, a.bias != nullptr, o, top);
    settle_in_order<M, 16>(__ballot(!sure && lane < n_tok), [&](int t, int p) { return reinterpret_cast<const uint4 *>(Kc + (int64_t)t * stride_s)[p]; },
                       n_tok, raw, a.W1, a.W2, w3f, a.bias != nullptr, lane, top);
    return top;
}

// Persistent wavefronts over windows of up to 64 tokens: 64/N consecutive chunks of a row (SHORT), or a part of a chunk, whose
// wavefront takes all its parts one after the other.
// DIRECT: one expert (whose sums decide nothing), or two and a window per wavefront: sums in order, a lane per token, from the rows as they lie.  Their 512
// multiply-adds are done before the operands of the matrix products would be (131 072 rows in 32-token chunks 7.5 us against
// 8.6); with four experts it is the other way round (10.0 against 9.4).
template <int M, bool SHORT, bool DIRECT>
__global__ __launch_bounds__(kRouteWaves * 64, kRouteWgPerCu) void route_kernel(RouteArgs a) {
    __shared__ float w3f[kW3Words];
    __shared__ uint32_t raw[kD * M];
    __shared__ uint4 rows[kRouteWaves][kHalfPieces];
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);           // wave-uniform, kept scalar
    uint4 *buf = &rows[wave][0];

    // routing freezing: the first chunks of every row are never routed
    const int n_frozen = min(max(a.freeze_chunks - a.chunk_begin, 0), a.n_chunks);
    const uint32_t item0 = (uint32_t)wave * gridDim.x + blockIdx.x, stride = gridDim.x * kRouteWaves;
    const int c_begin = a.chunk_begin + n_frozen, n_chunks = a.n_chunks - n_frozen;
    const int N = a.N, cpw = SHORT ? 64 / N : 1;     // chunks of an item
    const int per_row = max((n_chunks + cpw - 1) / cpw, 1), parts = SHORT ? 1 : (N + 63) / 64;

    // item t of row u, part h, from item0 on in steps of all wavefronts of the grid, on the scalar unit
    const int step_u = (int)(stride / (uint32_t)per_row), step_t = (int)(stride % (uint32_t)per_row);
    int u = n_chunks > 0 ? (int)(item0 / (uint32_t)per_row) : a.BH, t = (int)(item0 % (uint32_t)per_row), h = 0;
    auto tokens_of = [&](int st, int sh) { return SHORT ? min(cpw, n_chunks - st * cpw) * N : min(64, N - 64 * sh); };
    auto window = [&](int su, int st, int sh) {
        return a.K + (int64_t)(su / a.Hkv) * a.stride_b + (int64_t)(su % a.Hkv) * a.stride_h
             + ((int64_t)(c_begin + st * cpw) * N + 64 * sh) * a.stride_s;
    };
    HalfRows hr;
    if (!DIRECT && u < a.BH) request_half(window(u, t, 0), a.stride_s, tokens_of(t, 0), 0, lane, hr);
    RouterWeights w;
    RouterSums<M> floor;
    if (n_chunks > 0) {                              // all frozen: 2.3 us a call, 3.1 with the weights
        if constexpr (!DIRECT) stage_router_weights<M>(a.W1, a.W2, raw, tid, kRouteWaves * 64);
        stage_w3<M, !DIRECT>(a.W3, a.bias, w3f, tid);
        __syncthreads();
        if constexpr (!DIRECT) { load_router_weights<M>(raw, lane, w); floor = bound_floor<M>(w.e); }
    }
    int cnt[M];
#pragma unroll 1
    while (u < a.BH) {
        const int cu = u, ct = t, ch = h, n_tok = tokens_of(ct, ch);
        if (++h == parts) {                          // the next window
            h = 0; t += step_t; u += step_u;
            if (t >= per_row) { t -= per_row; u++; }
        }
        int top;
        if constexpr (DIRECT) {
            const uint4 *row = reinterpret_cast<const uint4 *>(window(cu, ct, ch) + (int64_t)min(lane, n_tok - 1) * a.stride_s);
            top = ordered_top<M>([&](int p) { return row[p]; }, a.W1, a.W2, w3f, a.bias != nullptr);
        } else {
            v4f_r val[M <= 4 ? 2 : 4], bnd[M <= 4 ? 2 : 4];
            stage_half(hr, lane, buf);
            request_half(window(cu, ct, ch), a.stride_s, n_tok, 1, lane, hr);
            wave_lds_sync();
            half_sums<M>(w, buf, 0, lane, val, bnd);
            wave_lds_sync();
            stage_half(hr, lane, buf);
            if (u < a.BH) request_half(window(u, t, h), a.stride_s, tokens_of(t, h), 0, lane, hr);
            wave_lds_sync();
            half_sums<M>(w, buf, 1, lane, val, bnd);
            wave_lds_sync();
            top = window_top<M>(val, bnd, floor, window(cu, ct, ch), a.stride_s, n_tok, lane, a, raw, w3f);
        }
        if (ch == 0) {
#pragma unroll
            for (int k = 0; k < M; k++) cnt[k] = 0;
        }
#pragma unroll
        for (int k = 0; k < M; k++) {
            const unsigned long long mask = __ballot(lane < n_tok && top == k);
            if constexpr (SHORT) cnt[k] = lane < cpw ? __popcll((mask >> (lane * N)) & ((1ull << N) - 1ull)) : 0;
            else                 cnt[k] += __popcll(mask);
        }
        if (ch != parts - 1) continue;
        const int c = c_begin + ct * cpw + (SHORT ? lane : 0);           // SHORT: lane j stores chunk j of the window
        if (SHORT ? (lane < cpw && c < c_begin + n_chunks) : lane == 0) {
            int best = 0, cbest = cnt[0];
#pragma unroll
            for (int k = 1; k < M; k++) if (cnt[k] > cbest) { best = k; cbest = cnt[k]; }
            const int64_t eidx = (int64_t)cu * a.expert_stride + c;
            a.expert[eidx] = (uint8_t)best;
            if (a.votes) {
#pragma unroll
                for (int k = 0; k < M; k++) a.votes[eidx * M + k] = cnt[k];
            }
        }
    }
    // frozen chunks take the FP16 expert
    for (uint32_t ru = item0; n_frozen > 0 && ru < (uint32_t)a.BH; ru += stride) {
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

// Few chunks of more than 64 tokens (a decode step that flushes a chunk per head): one wavefront per 64 tokens of a chunk, its
// whole window requested at once, the votes added up in LDS.  A wavefront that takes a chunk's windows one after the other has
// nobody to hide its latency.  From three to four workgroups per compute unit on, the other chunks' wavefronts hide it.  Up to two
// experts: sums in order, see DIRECT.
// 64 to 256 chunks of 128 tokens 4.7 to 4.9 us (a token per lane, sums in order: 7.1 to 7.2), 32 to 128 chunks of 256 tokens 5.4 to
// 7.0 (7.5 to 7.7), 512 of them 10.4 (10.8).
template <int M>
__global__ __launch_bounds__(kRouteWaves * 64) void route_split_kernel(RouteArgs a) {
    constexpr bool kMatrix = M > 2;
    __shared__ float w3f[kW3Words];
    __shared__ uint32_t raw[kMatrix ? kD * M : 1];
    __shared__ uint4 rows[kMatrix ? kRouteWaves : 1][kHalfPieces];
    __shared__ int votes_s[8];
    const int c = a.chunk_begin + (int)blockIdx.x;
    const int u = (int)blockIdx.y;
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);           // wave-uniform, kept scalar
    const int64_t eidx = (int64_t)u * a.expert_stride + c;
    if (c < a.freeze_chunks) {                       // routing freezing: never routed, FP16 expert
        if (tid == 0) a.expert[eidx] = (uint8_t)a.e16;
        if (a.votes && tid < M) a.votes[eidx * M + tid] = 0;
        return;
    }
    const int n_tok = min(64, a.N - wave * 64);
    const uint16_t *Kc = a.K + (int64_t)(u / a.Hkv) * a.stride_b + (int64_t)(u % a.Hkv) * a.stride_h + ((int64_t)c * a.N + wave * 64) * a.stride_s;
    HalfRows hr[2];
    if constexpr (kMatrix) {
#pragma unroll
        for (int k = 0; k < 2; k++) request_half(Kc, a.stride_s, n_tok, k, lane, hr[k]);
        stage_router_weights<M>(a.W1, a.W2, raw, tid, (int)blockDim.x);
    }
    stage_w3<M, kMatrix>(a.W3, a.bias, w3f, tid);
    if (tid < 8) votes_s[tid] = 0;
    __syncthreads();
    int top;
    if constexpr (kMatrix) {
        RouterWeights w;
        load_router_weights<M>(raw, lane, w);
        const RouterSums<M> floor = bound_floor<M>(w.e);
        v4f_r val[M <= 4 ? 2 : 4], bnd[M <= 4 ? 2 : 4];
        uint4 *buf = &rows[wave][0];
#pragma unroll
        for (int k = 0; k < 2; k++) {
            stage_half(hr[k], lane, buf);
            wave_lds_sync();
            half_sums<M>(w, buf, k, lane, val, bnd);
            wave_lds_sync();
        }
        top = window_top<M>(val, bnd, floor, Kc, a.stride_s, n_tok, lane, a, raw, w3f);
    } else {
        const uint4 *row = reinterpret_cast<const uint4 *>(Kc + (int64_t)min(lane, n_tok - 1) * a.stride_s);
        top = ordered_top<M>([&](int p) { return row[p]; }, a.W1, a.W2, w3f, a.bias != nullptr);
    }
#pragma unroll
    for (int k = 0; k < M; k++) {
        const int cnt = __popcll(__ballot(lane < n_tok && top == k));
        if (lane == k) atomicAdd(&votes_s[k], cnt);
    }
    __syncthreads();
    if (tid == 0) {
        int best = 0;
        for (int k = 1; k < M; k++) if (votes_s[k] > votes_s[best]) best = k;   // strict: the first maximum wins
        a.expert[eidx] = (uint8_t)best;
    }
    if (a.votes && tid < M) a.votes[eidx * M + tid] = votes_s[tid];
}

template <int M>
static hipError_t launch_m(const RouteArgs &a, int n_cu, hipStream_t s) {
    // as long as the chunks' workgroups are at most one round and mostly wait for their rows: 528 / 768 / 1024 chunks of 128 tokens
    // 7.3 / 8.8 / 10.5 us against 8.0 / 9.7 / 12.0 with route_kernel, of 256 tokens 11.1 / 12.4 / 16.6 against 13.2 / 12.9 / 15.3
    // (two experts, 1024 chunks: 12.7 against 14.3)
    if (a.N > 64 && (long long)a.n_chunks * a.BH <= (a.N <= 128 || M <= 2 ? 4LL : 3LL) * n_cu) {
        hipLaunchKernelGGL(route_split_kernel<M>, dim3((unsigned)a.n_chunks, (unsigned)a.BH), dim3((unsigned)((a.N + 63) / 64 * 64)), 0, s, a);
    } else {
        const int cpw = a.N < 64 ? 64 / a.N : 1, n_frozen = std::min(std::max(a.freeze_chunks - a.chunk_begin, 0), a.n_chunks);
        const long long items = (long long)a.BH * ((a.n_chunks - n_frozen + cpw - 1) / cpw);
        // an item per workgroup as long as there are compute units, then all four wavefronts of a workgroup
        long long n_wg = (items + kRouteWaves - 1) / kRouteWaves;
        if (n_wg < n_cu) n_wg = items < n_cu ? items : n_cu;
        if (n_wg < 1) n_wg = std::min(a.BH, n_cu);   // frozen chunks only: a row per wavefront
        if (n_wg > (long long)kRouteWgPerCu * n_cu) n_wg = (long long)kRouteWgPerCu * n_cu;
        const dim3 grid((unsigned)n_wg), block(kRouteWaves * 64);
        if constexpr (M <= 2) {                      // one expert: every token's, no key is read (5.2 M rows in 128-token chunks 194 -> 8.6 us)
            if (M == 1 || items * ((a.N + 63) / 64) <= (long long)kRouteWgPerCu * kRouteWaves * n_cu) {
                if (a.N < 64) hipLaunchKernelGGL((route_kernel<M, true, true>), grid, block, 0, s, a);
                else          hipLaunchKernelGGL((route_kernel<M, false, true>), grid, block, 0, s, a);
                return hipGetLastError();
            }
        }
        if constexpr (M > 1) {
            if (a.N < 64) hipLaunchKernelGGL((route_kernel<M, true, false>), grid, block, 0, s, a);
            else          hipLaunchKernelGGL((route_kernel<M, false, false>), grid, block, 0, s, a);
        }
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
