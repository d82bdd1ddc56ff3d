// Device code of the router shared by the routing, the fused route + pack and the training kernels (Eq. (1)-(2), Sec. 3.2).
#pragma once
#include "moqae_dev.hpp"

namespace moqae {

// exp(x) with a fixed evaluation order: 2^n * P(r), t = x*log2(e), n = rint(t), r = t - n,
// P = degree-6 Taylor polynomial of 2^r in Horner form, every operation rounded separately.
__device__ __forceinline__ float exp_pinned(float x) {
    const float LOG2E = 0x1.715476p+0f;
    const float C1 = 0x1.62e430p-1f, C2 = 0x1.ebfbe0p-3f, C3 = 0x1.c6b08ep-5f;
    const float C4 = 0x1.3b2ab6p-7f, C5 = 0x1.5d87fep-10f, C6 = 0x1.430912p-13f;
    x = fminf(fmaxf(x, -80.0f), 80.0f);
    float t = __fmul_rn(x, LOG2E);
    float n = rintf(t);
    float r = __fsub_rn(t, n);
    float p = C6;
    p = __fadd_rn(__fmul_rn(p, r), C5);
    p = __fadd_rn(__fmul_rn(p, r), C4);
    p = __fadd_rn(__fmul_rn(p, r), C3);
    p = __fadd_rn(__fmul_rn(p, r), C2);
    p = __fadd_rn(__fmul_rn(p, r), C1);
    p = __fadd_rn(__fmul_rn(p, r), 1.0f);
    float s = __builtin_bit_cast(float, (uint32_t)((int)n + 127) << 23);
    return __fmul_rn(p, s);
}

// 64 dims of a key row (eight 16-byte pieces xr[0..7], dims dbase..dbase+63) into the two running sums per expert,
// in ascending order of the dims.  W1w, W2w: the fp16 weight matrices as 32-bit words (wave-uniform loads; WP: a plain
// pointer, or const_words where the compiler would not see by itself that nothing in the kernel writes them; dbase should
// then vary in a loop around the call, or the weights of the whole row are loaded ahead of it).
typedef const uint32_t __attribute__((address_space(4))) *const_words;
template <int M, typename WP>
__device__ __forceinline__ void route_half_row(const uint4 *xr, int dbase, WP W1w, WP W2w,
                                               float (&accA)[M], float (&accB)[M]) {
    // two key dims (two rows of the weight matrices) per step so that the fp16 pairs fall on 32-bit words
#pragma unroll
    for (int p = 0; p < 8; p++) {
        const uint32_t xw[4] = {xr[p].x, xr[p].y, xr[p].z, xr[p].w};
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            const int d = dbase + p * 8 + e;      // even; rows d, d+1 of W = 2*M halves = M words
            const float x0 = half_bits_to_float(xw[e >> 1] & 0xffffu);
            const float x1 = half_bits_to_float(xw[e >> 1] >> 16);
            uint32_t w1[M], w2[M];
#pragma unroll
            for (int m = 0; m < M; m++) { w1[m] = W1w[d / 2 * M + m]; w2[m] = W2w[d / 2 * M + m]; }
#pragma unroll
            for (int m = 0; m < M; m++) {
                const int i0 = m, i1 = M + m;     // half index inside the two-row block
                const float wa0 = half_bits_to_float((w1[i0 >> 1] >> (16 * (i0 & 1))) & 0xffffu);
                const float wb0 = half_bits_to_float((w2[i0 >> 1] >> (16 * (i0 & 1))) & 0xffffu);
                accA[m] = fmaf(x0, wa0, accA[m]);
                accB[m] = fmaf(x0, wb0, accB[m]);
                const float wa1 = half_bits_to_float((w1[i1 >> 1] >> (16 * (i1 & 1))) & 0xffffu);
                const float wb1 = half_bits_to_float((w2[i1 >> 1] >> (16 * (i1 & 1))) & 0xffffu);
                accA[m] = fmaf(x1, wa1, accA[m]);
                accB[m] = fmaf(x1, wb1, accB[m]);
            }
        }
        __builtin_amdgcn_sched_barrier(0);        // keeps the uniform weight loads of later steps from piling up
    }
}

// The token's expert from the two sums per expert: SiLU of their product, times W3 (plus the bias), first maximum.
// w3f: W3 as binary32 (M*M values) and the optional bias at [64..64+M), in LDS.
template <int M>
__device__ __forceinline__ int route_top(const float (&accA)[M], const float (&accB)[M], const float *w3f, bool has_bias) {
    float hid[M];
#pragma unroll
    for (int m = 0; m < M; m++) {
        const float z = __fmul_rn(accA[m], accB[m]);
        const float e = exp_pinned(-z);
        hid[m] = __fdiv_rn(z, __fadd_rn(1.0f, e));              // SiLU(z) = z / (1 + exp(-z))
    }
    int top = 0; float ptop = 0.0f;
#pragma unroll
    for (int k = 0; k < M; k++) {
        float acc = 0.0f;
#pragma unroll
        for (int j = 0; j < M; j++) acc = __fadd_rn(acc, __fmul_rn(hid[j], w3f[j * M + k]));
        if (has_bias) acc = __fadd_rn(acc, w3f[64 + k]);
        if (k == 0) ptop = acc;
        else if (acc > ptop) { top = k; ptop = acc; }           // strict: the first maximum wins
    }
    return top;
}

// One token's expert from its whole key row in registers (sixteen 16-byte pieces): the same operations in the same
// order as route_tokens.
template <int M>
__device__ __forceinline__ int route_row(const uint4 (&x)[16], const uint32_t *W1w, const uint32_t *W2w, const float *w3f,
                                         bool has_bias) {
    float accA[M], accB[M];
#pragma unroll
    for (int m = 0; m < M; m++) { accA[m] = 0.0f; accB[m] = 0.0f; }
    route_half_row<M>(&x[0], 0, W1w, W2w, accA, accB);
    route_half_row<M>(&x[8], 64, W1w, W2w, accA, accB);
    return route_top<M>(accA, accB, w3f, has_bias);
}

// One wavefront routes the n_tok tokens whose key rows start at Kc (row stride stride_s elements), one lane per
// token and pass of 64 tokens; W1w, W2w: the fp16 weight matrices as 32-bit words (wave-uniform loads), w3f: W3 as
// binary32 (M*M values) and the optional bias at [64..64+M), in LDS.  Returns the votes per expert, the same in
// every lane.  STAGE: every lane also leaves its rows in `stage` (LDS, kStageRow 16-byte pieces per row, row = token
// counted from Kc), so that a quantiser that follows reads the keys from there and not from memory again.
constexpr int kStageRow = 17;                     // 16 pieces of data + 1 of padding: the lanes' writes fall on different banks
template <int M, bool STAGE = false>
__device__ __forceinline__ void route_tokens(const uint16_t *Kc, int n_tok, int64_t stride_s, const uint32_t *W1w,
                                             const uint32_t *W2w, const float *w3f, bool has_bias, int lane, int (&cnt)[M],
                                             uint4 *stage = nullptr) {
#pragma unroll
    for (int k = 0; k < M; k++) cnt[k] = 0;

    float accA[M], accB[M];
    // The loop runs over half rows (64 dims = one 128-byte line per lane); the next half row is
    // requested before the current one is consumed, across the 64-token passes too.
    const int n_half = 2 * ((n_tok + 64 - 1) / 64);
    auto half_ptr = [&](int hr) {
        const int row = (hr >> 1) * 64 + lane;
        return reinterpret_cast<const uint4 *>(Kc + (int64_t)(row < n_tok ? row : 0) * stride_s) + (hr & 1) * 8;
    };
    uint4 xn[8];
    {
        const uint4 *hp = half_ptr(0);
#pragma unroll
        for (int p = 0; p < 8; p++) xn[p] = hp[p];
    }
#pragma unroll 1
    for (int hr = 0; hr < n_half; hr++) {
        const int row0 = (hr >> 1) * 64;
        const bool active = row0 + lane < n_tok;        // the last pass may be partly empty
        uint4 xr[8];
#pragma unroll
        for (int p = 0; p < 8; p++) xr[p] = xn[p];
        if constexpr (STAGE) {
            if (active) {
#pragma unroll
                for (int p = 0; p < 8; p++) stage[(row0 + lane) * kStageRow + (hr & 1) * 8 + p] = xr[p];
            }
        }
        if (hr + 1 < n_half) {
            const uint4 *hp = half_ptr(hr + 1);
#pragma unroll
            for (int p = 0; p < 8; p++) xn[p] = hp[p];
        }
        if (!(hr & 1)) {
#pragma unroll
            for (int m = 0; m < M; m++) { accA[m] = 0.0f; accB[m] = 0.0f; }
        }
        route_half_row<M>(xr, (hr & 1) * 64, W1w, W2w, accA, accB);
        if (!(hr & 1)) continue;
        const int top = route_top<M>(accA, accB, w3f, has_bias);
#pragma unroll
        for (int k = 0; k < M; k++) cnt[k] += __popcll(__ballot(active && top == k));
    }
}

// ---- decisions on the matrix cores -----------------------------------------------------------
// The decision is defined by binary32 sums in the order of the dims: 1024 dependent-order multiply-adds per token at four
// experts, which bound the kernels that route.  The same sums on v_mfma_f32_16x16x32_f16 (products exact, binary32 sums in an
// order of their own) differ from them by rounding only, so that nearly every token's arg-max can be told from them with
// certainty.  Every addition errs by at most its rounding times the absolute sum so far: in order, dim d is in 128 - d additions of
// relative error 2^-24; in the matrix core, in at most 32 per step of 32 dims, from its own step on.  There a subnormal number
// counts with the smallest normal exponent (a zero not at all): the 32 products of a step are cut off at 2^-24 of the largest
// power of two among them, that of a key of 2^-24 times 8 being 2^-14 * 8 (measured: at most 23 of the 32 allowed, normal numbers
// 4 times 2^-24 of the absolute sum).  So the two differ by at most
//   sum_d ((128 - d) + 32 (4 - d / 32)) 2^-24 max(|x_d|, 2^-14) max(|w_d|, 2^-14),
// and a maximum is at most the sum: it comes from a second product, |x| times the weights scaled so, plus 2^-14 and rounded up, and
// from 2^-14 times the sum of those weights (bound_floor), and is carried through SiLU and W3.  A token whose two best logits are closer
// than that (ties, else about one in a thousand) is settled by the sums in order.  The result is the same, bit for bit, always.
typedef float v4f_r __attribute__((ext_vector_type(4)));
typedef uint32_t v4u_r __attribute__((ext_vector_type(4)));
typedef _Float16 v8h_r __attribute__((ext_vector_type(8)));
constexpr float kSumErr = 256.0f / 16777216.0f;           // the factor of |x_0 w_0|; the others relative to it
constexpr int kW3Max = 72, kBiasMax = 80, kW3Words = 84;  // w3f: also the largest |W3| of every row, the largest |bias|

// The workgroup's copy of W3 as binary32 and (BOUND) what the bound needs of it.
template <int M, bool BOUND = true>
__device__ __forceinline__ void stage_w3(const uint16_t *W3, const float *bias, float *w3f, int tid) {
    if (tid < M * M) w3f[tid] = half_bits_to_float(W3[tid]);
    if (tid < M) {
        w3f[64 + tid] = bias ? bias[tid] : 0.0f;
    }
    if constexpr (!BOUND) return;
    if (tid < M) {
        float m = 0.0f;
#pragma unroll
        for (int k = 0; k < M; k++) m = fmaxf(m, fabsf(half_bits_to_float(W3[tid * M + k])));
        w3f[kW3Max + tid] = m;
    }
    if (tid == M) {
        float m = 0.0f;
        if (bias) for (int k = 0; k < M; k++) m = fmaxf(m, fabsf(bias[k]));
        w3f[kBiasMax] = m;
    }
}

// Operand A, held by every wavefront: row i = an output, lane 16q + i holds its weights of dims 32s + 8q .. + 7 in w[s].
// Up to four experts: rows 0..3 = the columns of W1, 4..7 = of W2, 8..15 = 0..7 again; else rows 0..7 and 8..15.
struct RouterWeights { v4u_r w[4], e[4]; };              // e: the weights of the bound
// The two weight matrices as they are, in LDS (2 * kD * M halves), by all threads of the workgroup; then, behind a barrier, the operand.
template <int M>
__device__ __forceinline__ void stage_router_weights(const uint16_t *W1, const uint16_t *W2, uint32_t *raw, int tid, int n_threads) {
    constexpr int n = kD * M / 2;                         // words of a matrix
    for (int i = tid; i < n; i += n_threads) {
        raw[i] = reinterpret_cast<const uint32_t *>(W1)[i];
        raw[n + i] = reinterpret_cast<const uint32_t *>(W2)[i];
    }
}
template <int M>
__device__ __forceinline__ void load_router_weights(const uint32_t *raw, int lane, RouterWeights &r) {
    constexpr int H = M <= 4 ? 4 : 8;
    const int i = lane & (2 * H - 1), q = lane >> 4, m = i & (H - 1);
    const uint16_t *W = reinterpret_cast<const uint16_t *>(raw) + (i < H ? 0 : kD * M) + min(m, M - 1) + 8 * q * M;
#pragma unroll
    for (int s = 0; s < 4; s++) {
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const uint32_t w0 = m < M ? (uint32_t)W[(32 * s + 2 * k) * M] : 0u, w1 = m < M ? (uint32_t)W[(32 * s + 2 * k + 1) * M] : 0u;
            r.w[s][k] = w0 | (w1 << 16);
            // at least 2^-14 each; cutting off loses up to 2^-10 of a value
            const float f0 = (float)(256 - 64 * s - 2 * k - 8 * q) * ((1.0f + 0x1p-8f) / 256.0f), f1 = f0 - (1.0f + 0x1p-8f) / 256.0f;
            const auto e = __builtin_amdgcn_cvt_pkrtz(fmaf(fabsf(half_bits_to_float(w0)), f0, 0x1.01p-14f), fmaf(fabsf(half_bits_to_float(w1)), f1, 0x1.01p-14f));
            r.e[s][k] = __builtin_bit_cast(uint32_t, e);
        }
    }
}

__device__ __forceinline__ v4f_r mfma_router(v4u_r a, v4u_r b, v4f_r c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h_r, a), __builtin_bit_cast(v8h_r, b), c, 0, 0, 0);
}
// k-step s of a block of 16 tokens: lane 16q + x holds the 16-byte piece 4s + q of token x's row.  sum and bound: row 4q + n
// of the outputs for token x.
__device__ __forceinline__ void router_step(const RouterWeights &r, int s, const uint4 &x, v4f_r &sum, v4f_r &bound) {
    const v4u_r b = {x.x, x.y, x.z, x.w};
    sum = mfma_router(r.w[s], b, sum);
    bound = mfma_router(r.e[s], b & 0x7fff7fffu, bound);
}

// Outputs of 64 tokens -> every lane's own token: blocks 0..3 of 16 tokens as two pairs (0, 2) and (1, 3).  Up to four experts a
// pair is one register set already (lanes 0..31 keep the first block, the others the second), see pick_pair.
template <int M> struct RouterSums { static constexpr int H = M <= 4 ? 4 : 8; float A[H], B[H]; };
__device__ __forceinline__ v4f_r pick_pair(const v4f_r &lo, const v4f_r &hi, int lane) {
    v4f_r r;
#pragma unroll
    for (int n = 0; n < 4; n++) r[n] = lane < 32 ? lo[n] : hi[n];
    return r;
}
__device__ __forceinline__ void swap16(float &a, float &b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), false, false);
    a = __builtin_bit_cast(float, (uint32_t)r[0]); b = __builtin_bit_cast(float, (uint32_t)r[1]);
}
__device__ __forceinline__ void swap32(float &a, float &b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), false, false);
    a = __builtin_bit_cast(float, (uint32_t)r[0]); b = __builtin_bit_cast(float, (uint32_t)r[1]);
}
// c[b]: block b (up to four experts: c[0] = pair (0, 2), c[1] = pair (1, 3))
template <int M>
__device__ __forceinline__ void gather_sums(v4f_r (&c)[M <= 4 ? 2 : 4], RouterSums<M> &o) {
#pragma unroll
    for (int n = 0; n < 4; n++) {
        if constexpr (M <= 4) {
            float a = c[0][n], b = c[1][n];
            swap16(a, b);
            o.A[n] = a; o.B[n] = b;
        } else {
            float t0 = c[0][n], t1 = c[1][n], t2 = c[2][n], t3 = c[3][n];
            swap32(t0, t2); swap32(t1, t3);               // t0, t1: outputs 0..7, t2, t3: 8..15
            swap16(t0, t1); swap16(t2, t3);
            o.A[n] = t0; o.A[4 + n] = t1; o.B[n] = t2; o.B[4 + n] = t3;
        }
    }
}

// The part of the bound that does not depend on the keys, the same in every lane: 2^-14 times the sums of an output's bound weights.
template <int M>
__device__ __forceinline__ RouterSums<M> bound_floor(const v4u_r (&e)[4]) {
    const v4f_r zero = {0.0f, 0.0f, 0.0f, 0.0f};
    const v4u_r least = {0x04000400u, 0x04000400u, 0x04000400u, 0x04000400u};
    const v4f_r c = mfma_router(e[1], least, mfma_router(e[0], least, zero)) + mfma_router(e[3], least, mfma_router(e[2], least, zero));
    v4f_r all[M <= 4 ? 2 : 4];
#pragma unroll
    for (int k = 0; k < (M <= 4 ? 2 : 4); k++) all[k] = c;
    RouterSums<M> o;
    gather_sums<M>(all, o);
    return o;
}

// What the sums of a token lead to: SiLU of their products and its sigmoid, the logits.
template <int M> struct RouterValues { float z[M], sg[M], hid[M], logit[M]; };
template <int M>
__device__ __forceinline__ void router_values(const RouterSums<M> &v, const float *w3f, bool has_bias, RouterValues<M> &o) {
#pragma unroll
    for (int m = 0; m < M; m++) {
        o.z[m] = v.A[m] * v.B[m];
        o.sg[m] = __builtin_amdgcn_rcpf(1.0f + fast_exp2(fminf(-o.z[m], 80.0f) * 1.44269504f));
        o.hid[m] = o.z[m] * o.sg[m];
    }
#pragma unroll
    for (int k = 0; k < M; k++) {
        o.logit[k] = has_bias ? w3f[64 + k] : 0.0f;
#pragma unroll
        for (int j = 0; j < M; j++) o.logit[k] = fmaf(o.hid[j], w3f[j * M + k], o.logit[k]);
    }
}

// The token's expert from the sums and their bounds (s + floor); false if they do not tell it from the expert by the sums in order.
template <int M>
__device__ __forceinline__ bool certain_top(const RouterSums<M> &v, const RouterSums<M> &s, const RouterSums<M> &floor, const float *w3f, bool has_bias,
                                            RouterValues<M> &o, int &top) {
    float err = 0.0f;
    router_values<M>(v, w3f, has_bias, o);
#pragma unroll
    for (int m = 0; m < M; m++) {
        const float ea = kSumErr * (s.A[m] + floor.A[m]), eb = kSumErr * (s.B[m] + floor.B[m]);
        // |z - z'| of the two products, times the slope of SiLU: the slope at z and what the second derivative, at most
        // s (1 - s) (2 + |z|), adds within 1/4; 1.1 anywhere
        const float ez = fmaf(fabsf(v.A[m]), eb, fmaf(fabsf(v.B[m]), ea, ea * eb));
        const float sg = o.sg[m];
        const float near = fmaf(ez * 1.45f * fmaf(-sg, sg, sg), 2.0f + fabsf(o.z[m]), fabsf(fmaf(o.hid[m], 1.0f - sg, sg)));
        const float slope = ez <= 0.25f ? near : 1.1f;
        // exponential, division and W3's sums on either side: (|z| + 8) 2^-21 and 2^-19 of the hidden value
        err = fmaf(fmaf(fmaf(fabsf(o.z[m]), 0x1p-21f, 0x1p-18f + 0x1p-19f), fabsf(o.hid[m]), ez * slope), w3f[kW3Max + m], err);
    }
    float best = o.logit[0], second = -INFINITY;
    top = 0;
#pragma unroll
    for (int k = 1; k < M; k++) {
        const bool more = o.logit[k] > best;
        second = fmaxf(second, more ? best : o.logit[k]);
        top = more ? k : top; best = more ? o.logit[k] : best;
    }
    if (has_bias) err = fmaf(w3f[kBiasMax], 0x1p-19f, err);
    // rows of zeros (the largest product of any other row stays in s): the same logits on both sides.  NaN: not certain
    return M == 1 || best - second > 2.1f * err || s.A[0] == 0.0f;
}

// A token per lane by the sums in order; piece(p): the 16-byte piece p of the lane's row.
template <int M, typename F>
__device__ __forceinline__ int ordered_top(F piece, const uint16_t *W1, const uint16_t *W2, const float *w3f, bool has_bias) {
    float accA[M], accB[M];
#pragma unroll
    for (int m = 0; m < M; m++) { accA[m] = 0.0f; accB[m] = 0.0f; }
#pragma unroll 1
    for (int h = 0; h < 2; h++) {
        uint4 x[8];
#pragma unroll
        for (int p = 0; p < 8; p++) x[p] = piece(8 * h + p);
        route_half_row<M>(x, 64 * h, reinterpret_cast<const_words>(reinterpret_cast<uintptr_t>(W1)),
                          reinterpret_cast<const_words>(reinterpret_cast<uintptr_t>(W2)), accA, accB);
    }
    return route_top<M>(accA, accB, w3f, has_bias);
}

// The tokens of `open` (one bit per token of a window of 64, those certain_top could not settle) by the sums in order; `top`:
// the lane's own token's expert.  A lane adds up ONE of a token's 2 M sums, so that eight tokens (more than four experts: four)
// are settled at once in 128 dependent multiply-adds: with a token per lane all 64 wait for 1024, 5 us on an idle chip.
// piece(t, p): the 16-byte piece p of token t's row, AHEAD of them requested at once; raw: the weights in LDS (stage_router_weights).
// Windows with many of them (a router whose experts tie) take a token per lane all the same.
template <int M, int AHEAD, typename F>
__device__ __forceinline__ void settle_in_order(unsigned long long open, F piece, int n_tok, const uint32_t *raw, const uint16_t *W1,
                                                const uint16_t *W2, const float *w3f, bool has_bias, int lane, int &top) {
    if (open == 0ull) return;
    if (__popcll(open) > 24) {
        top = ordered_top<M>([&](int p) { return piece(min(lane, n_tok - 1), p); }, W1, W2, w3f, has_bias);
        return;
    }
    constexpr int H = M <= 4 ? 4 : 8, TPL = 2 * H, NT = 64 / TPL;
    const int k = lane % TPL, slot = lane / TPL;
    const uint16_t *w = reinterpret_cast<const uint16_t *>(raw) + (k < H ? 0 : kD * M) + min(k & (H - 1), M - 1);
    while (open != 0ull) {                               // the same for all lanes
        int tok = 0, src = -1;                            // the token this lane works on; the lane that will hold its own token's expert
#pragma unroll
        for (int s = 0; s < NT; s++) {
            if (open != 0ull) {
                const int t = __ffsll((long long)open) - 1;
                open &= open - 1ull;
                tok = slot >= s ? t : tok;                // slots without a token repeat the last one
                src = lane == t ? s * TPL : src;
            }
        }
        float acc = 0.0f;
#pragma unroll 1
        for (int p0 = 0; p0 < 16; p0 += AHEAD) {
            uint4 x[AHEAD];
#pragma unroll
            for (int p = 0; p < AHEAD; p++) x[p] = piece(tok, p0 + p);
#pragma unroll
            for (int p = 0; p < AHEAD; p++) {
                const uint32_t xw[4] = {x[p].x, x[p].y, x[p].z, x[p].w};
#pragma unroll
                for (int e = 0; e < 8; e++)
                    acc = fmaf(half_bits_to_float((xw[e >> 1] >> (16 * (e & 1))) & 0xffffu), half_bits_to_float(w[(8 * (p0 + p) + e) * M]), acc);
                if (p & 1) __builtin_amdgcn_sched_barrier(0);    // keeps the weights of later pieces out of the registers
            }
        }
        float A[M], B[M];
#pragma unroll
        for (int m = 0; m < M; m++) { A[m] = __shfl(acc, slot * TPL + m); B[m] = __shfl(acc, slot * TPL + H + m); }
        const int found = __shfl(route_top<M>(A, B, w3f, has_bias), max(src, 0));
        top = src >= 0 ? found : top;
    }
}

}  // namespace moqae
