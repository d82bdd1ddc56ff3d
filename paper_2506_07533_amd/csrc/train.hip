// moqae_router_loss_grad: the router fine-tuning loss of Sec. 3.3 (Eq. (3)-(5)) and its gradient with respect to
// the router weights, over cached key rows, in one pass.
//
//   L = (1/T) sum_i p^i_j * (lambda * L_nll * pen_model_j + (1 - lambda) * pen_mem_j),  j = the token's top-1 expert,
//   p^i = softmax of the token's logits.  The top-1 index is the routing decision (route_kernel) bit for bit; everything
//   after it is plain binary32.
//
// One wavefront per tile of 64 tokens, eight wavefronts per workgroup, one workgroup per compute unit; a wavefront keeps
// its gradient accumulators over all its tiles.
//   rows      requested in whole rows, a tile ahead, and staged in LDS (pieces XOR-swizzled: reads by row and by piece both
//             touch every bank), from where the forward pass takes a row per lane and the weight gradient a piece per lane.
//   forward   up to five experts (one and two: in large calls): xW1, xW2 and the bound on their distance from the sums in order on the matrix cores (see
//             certain_top), a lane per token afterwards; the tokens whose top-1 index they leave open take it from the sums in
//             order.  Else one lane per token, route_half_row (more than five experts: the operands and the eight tiles of results would not
//             fit the registers beside the rest: 7 experts 189 us against 134).  Then the token's loss and its gradient down to
//             d(loss)/d(xW1), d(loss)/d(xW2) (2M values per token, handed over through LDS).
//   dW1, dW2  = x^T [128 x 64 tokens] times those values [64 tokens x 2M] on v_mfma_f32_16x16x32_f16: x is fp16 as it is; a
//             value is scaled by a power of two of its own column (expert and matrix) and tile and split into two fp16 numbers,
//             the second holding what the first leaves: 22 bits and more of every value that is not 2^28 times smaller than
//             its column's largest in the tile.  One scale for all columns would lose the experts whose gradients are small
//             beside another's (a saturated router has such): relative error of a column 2^-34 (2^-44) of the largest 4e-6
//             (2.5e-3), with its own scale 1e-7 as with the binary32 multiply-adds this took before (+2 % of time at 4
//             experts, +5 % at 7).  Elsewhere the error against binary64 is that of those multiply-adds or below: their
//             accumulators rounded once per token, these once per 32.  A row i of tile rt = dim 8i + rt, and the tokens
//             are taken in the order 4j + r, so that the operands of a lane are the fp16 halves of row pieces it can read
//             with one load each.  Binary32 matrix products (16x16x4) took 27 us of the matrix pipe at 1.05 M rows and
//             128 conversions per tile: 111 us in all.
//   fold      dW3, the bias gradient and the loss are per-lane sums; everything meets in LDS, then ONE atomic add per
//             address and workgroup.  Device-wide atomic steps on one address run at about nine per microsecond here: one
//             wavefront at a time, each with its own atomic adds (4096 per address), took 0.8 ms of the 0.89 ms that the
//             gradient over 1.05 M rows needed.
// 1.05 M rows: 2 / 4 / 5 / 8 experts 53 / 60 / 75 / 180 us (54 / 77 / 95 / 182 with the forward pass in order for all), 0.26 M rows,
// 4 experts: 29.0 (34.3), 64 rows: 12.6 (14.7); 8k to 32k rows, three experts: 15.7 to 17.1 (15.1 to 16.9), five: 18.7 to 21.1 (19.8
// to 21.0), where the few open tokens of one tile hold up the call.  The rows alone are 38 us at the read ceiling of the chip; what is
// left are the 110 KiB of LDS traffic of a tile and the arithmetic per token, at two wavefronts per SIMD.  Error against binary64 5e-8
// to 7e-7 of an array either way (it changes from run to run with the order of the atomic adds).  With 7 and 8 experts the 256
// registers that eight wavefronts leave are not enough: 116 and 164 bytes of scratch a lane; with 5 experts 36.
#include "moqae_dev.hpp"
#include "moqae_kernels.hpp"
#include "pack_dev.hpp"
#include "route_dev.hpp"

namespace moqae {

constexpr int kTrainWaves = 8;
// The fp16 halves of the 2M values per token, in the order of the B operand: [32-token step h][token % 4][column][j], token
// = 32h + 4j + token % 4; the steps of token % 4 and h are padded so that they start on different banks.
constexpr int kTrainCol = 8, kTrainR4 = 16 * kTrainCol + 8, kTrainH = 4 * kTrainR4 + 32;

typedef float v4f_t __attribute__((ext_vector_type(4)));
typedef uint32_t v4u_t __attribute__((ext_vector_type(4)));
typedef _Float16 v8h_t __attribute__((ext_vector_type(8)));

__device__ __forceinline__ uint32_t word4(const uint4 &v, int i) { return i == 0 ? v.x : (i == 1 ? v.y : (i == 2 ? v.z : v.w)); }

__device__ __forceinline__ v4f_t mfma_train(v4u_t a, v4u_t b, v4f_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h_t, a), __builtin_bit_cast(v8h_t, b), c, 0, 0, 0);
}

// Largest of every one of P columns (a power of two; v[i]: the lane's entry of column i, compared as an unsigned number) over
// the wavefront: lane l returns that of column l / (64 / P).  Every step halves the columns a lane carries, then the lanes of
// a column meet: 26 instructions for 8 columns, where a reduction of each would take 48.
template <int P>
__device__ __forceinline__ uint32_t column_max(uint32_t (&v)[P], int lane) {
#pragma unroll
    for (int i = 0; i < P / 2; i++) {                 // lanes 32.. take the upper half of the columns
        const auto r = __builtin_amdgcn_permlane32_swap(v[i], v[i + P / 2], false, false);
        v[i] = max(r[0], r[1]);
    }
#pragma unroll
    for (int i = 0; i < (P >= 4 ? P / 4 : 1); i++) {  // odd rows of 16 lanes the upper half of those
        const auto r = __builtin_amdgcn_permlane16_swap(v[i], v[P >= 4 ? i + P / 4 : i], false, false);
        v[i] = max(r[0], r[1]);
    }
#pragma unroll
    for (int i = 0; i < (P >= 8 ? P / 8 : 1); i++) {
        const uint32_t other = v[P >= 8 ? i + P / 8 : i];
        v[i] = max((lane & 8) ? other : v[i], dpp_u<0x128>((lane & 8) ? v[i] : other));   // row_ror:8
    }
    {
        const uint32_t other = v[P >= 16 ? 1 : 0];
        v[0] = max((lane & 4) ? other : v[0], dpp_u<DPP_HALF_MIRROR>((lane & 4) ? v[0] : other));
    }
    v[0] = max(v[0], dpp_u<DPP_XOR2>(v[0]));
    return max(v[0], dpp_u<DPP_XOR1>(v[0]));
}

// kMatrix: the forward pass on the matrix cores
template <int M, bool kMatrix>
__global__ __launch_bounds__(kTrainWaves * 64) void router_train_kernel(TrainArgs a) {
    constexpr int NS = M * M + M + 2;                 // sums that every lane keeps: dW3, bias, the two losses
    __shared__ float w3f[kW3Words];
    __shared__ float sums[kTrainWaves][NS];
    __shared__ uint4 stage[kTrainWaves][64 * 16];     // key rows: piece p of row r at 16r + (p ^ (r % 16)); the fold's dW at the end
    constexpr int NB = M <= 4 ? 1 : 2;                // B operands: columns 0..7 first halves, 8..15 second ones, or one each
    __shared__ v4u_r wop[kMatrix ? 2 : 1][4][64];     // its operand A and that of its bound (registers are short)
    __shared__ RouterSums<M> floor;
    __shared__ uint32_t raw[kMatrix ? kD * M : 1];    // the weights for the tokens that it leaves open
    __shared__ __attribute__((aligned(16))) uint16_t dabs[kTrainWaves][2 * kTrainH];
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);           // wave-uniform, kept scalar
    if constexpr (!kMatrix) {                         // first of all: behind the accumulators' set-up eight experts take 236 bytes of scratch instead of 164
        stage_w3<M, false>(a.W3, a.bias, w3f, tid);
        __syncthreads();
    }
    const const_words W1w = reinterpret_cast<const_words>(reinterpret_cast<uintptr_t>(a.W1));
    const const_words W2w = reinterpret_cast<const_words>(reinterpret_cast<uintptr_t>(a.W2));
    uint4 *mine = &stage[wave][0];
    uint16_t *dab = &dabs[wave][0];
    for (int i = lane; i < 2 * kTrainH; i += 64) dab[i] = 0;   // the columns nobody writes stay zero

    v4f_t gw[8];                                      // C tiles: row 4*(l/16) + n of tile rt = dim 8*row + rt, column l%16
    float g3[M][M], gb[M], lsum[2] = {0.0f, 0.0f};
#pragma unroll
    for (int rt = 0; rt < 8; rt++) gw[rt] = v4f_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int m = 0; m < M; m++) {
        gb[m] = 0.0f;
#pragma unroll
        for (int k = 0; k < M; k++) g3[m][k] = 0.0f;
    }
    // tile (row u, tile tr of the row); the wavefront's first is wave * gridDim + block, then steps of gridDim * kTrainWaves,
    // all on the scalar unit
    const int tiles_per_row = (a.n_tok + 63) / 64;
    const uint32_t tile0 = (uint32_t)wave * gridDim.x + blockIdx.x, tw = gridDim.x * kTrainWaves;
    const int step_u = (int)(tw / (uint32_t)tiles_per_row), step_t = (int)(tw % (uint32_t)tiles_per_row);
    int u = (int)(tile0 / (uint32_t)tiles_per_row), tr = (int)(tile0 % (uint32_t)tiles_per_row);
    const int piece = lane & 15, r4 = lane >> 4;
    uint4 v[16];
    auto request = [&](int un, int tn) {              // rows past the tile's end read its last row
        const uint16_t *Kt = a.K + (int64_t)(un / a.Hkv) * a.stride_b + (int64_t)(un % a.Hkv) * a.stride_h + (int64_t)(a.token_begin + tn * 64) * a.stride_s;
        const int last = min(64, a.n_tok - tn * 64) - 1;
        if (last == 63 && a.stride_s < (1 << 28)) {   // scalar row addresses, one 32-bit offset per lane
            const uint32_t off = (uint32_t)r4 * (uint32_t)a.stride_s * 2u + (uint32_t)piece * 16u;
#pragma unroll
            for (int j = 0; j < 16; j++) v[j] = nt_load(reinterpret_cast<const uint4 *>(reinterpret_cast<const uint8_t *>(Kt + 4 * j * a.stride_s) + off));
            return;
        }
#pragma unroll
        for (int j = 0; j < 16; j++) v[j] = nt_load(reinterpret_cast<const uint4 *>(Kt + (int64_t)min(4 * j + r4, last) * a.stride_s) + piece);
    };
    if (u < a.BH) request(u, tr);                     // on their way while the weights are laid out
    if constexpr (kMatrix) {
        stage_router_weights<M>(a.W1, a.W2, raw, tid, kTrainWaves * 64);
        stage_w3<M>(a.W3, a.bias, w3f, tid);
        __syncthreads();
        if (wave == 0) {
            RouterWeights w;
            load_router_weights<M>(raw, lane, w);
#pragma unroll
            for (int s = 0; s < 4; s++) { wop[0][s][lane] = w.w[s]; wop[1][s][lane] = w.e[s]; }
            const RouterSums<M> f = bound_floor<M>(w.e);
            if (lane == 0) floor = f;
        }
        __syncthreads();
    }
    while (u < a.BH) {
        const int b = u / a.Hkv;
        const bool active = lane < a.n_tok - tr * 64;
        tr += step_t; u += step_u;                    // the next tile
        if (tr >= tiles_per_row) { tr -= tiles_per_row; u++; }
#pragma unroll
        for (int j = 0; j < 16; j++) mine[(4 * j + r4) * 16 + (piece ^ ((4 * j + r4) & 15))] = v[j];
        if (u < a.BH) request(u, tr);
        wave_lds_sync();
        RouterSums<M> v1;                             // xW1, xW2
        RouterValues<M> f;
        int top;
        if constexpr (kMatrix) {
            // ---- forward: block b of 16 tokens takes the pieces 4s + l/16 of its rows in k-step s
            constexpr int NP = M <= 4 ? 2 : 4;
            v4f_r c[4], d[4], val[NP], bnd[NP];
#pragma unroll
            for (int k = 0; k < 4; k++) { c[k] = v4f_r{0.0f, 0.0f, 0.0f, 0.0f}; d[k] = c[k]; }
#pragma unroll
            for (int s = 0; s < 4; s++) {
                const v4u_r ww = wop[0][s][lane], we = wop[kMatrix ? 1 : 0][s][lane];
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const uint4 x = mine[(16 * k + piece) * 16 + ((4 * s + r4) ^ piece)];
                    const v4u_r xb = {x.x, x.y, x.z, x.w};
                    c[k] = mfma_router(ww, xb, c[k]);
                    d[k] = mfma_router(we, xb & 0x7fff7fffu, d[k]);
                }
            }
#pragma unroll
            for (int k = 0; k < NP; k++) {
                val[k] = M <= 4 ? pick_pair(c[k], c[(k + 2) & 3], lane) : c[k];
                bnd[k] = M <= 4 ? pick_pair(d[k], d[(k + 2) & 3], lane) : d[k];
            }
            RouterSums<M> e;
            gather_sums<M>(val, v1); gather_sums<M>(bnd, e);
            const bool sure = certain_top<M>(v1, e, floor, w3f, a.bias != nullptr, f, top);       // by every lane: f and top are used below
            settle_in_order<M, 2>(__ballot(active && !sure), [&](int t, int p) { return mine[t * 16 + (p ^ (t & 15))]; }, 64, raw, a.W1, a.W2,
                               w3f, a.bias != nullptr, lane, top);
        } else {
            // ---- forward, the routing arithmetic: sequential binary32 sums over d (products of two fp16 values are exact)
            float accA[M], accB[M];
#pragma unroll
            for (int m = 0; m < M; m++) { accA[m] = 0.0f; accB[m] = 0.0f; }
#pragma unroll 1
            for (int hr = 0; hr < 2; hr++) {
                uint4 xr[8];
#pragma unroll
                for (int p = 0; p < 8; p++) xr[p] = mine[lane * 16 + ((hr * 8 + p) ^ piece)];
                route_half_row<M>(xr, hr * 64, W1w, W2w, accA, accB);
            }
#pragma unroll
            for (int m = 0; m < M; m++) {
                v1.A[m] = accA[m]; v1.B[m] = accB[m];
                f.z[m] = __fmul_rn(accA[m], accB[m]);
                const float den = __fadd_rn(1.0f, exp_pinned(-f.z[m]));
                f.hid[m] = __fdiv_rn(f.z[m], den);
                f.sg[m] = 1.0f / den;
            }
            top = 0;
            float ltop = 0.0f;
#pragma unroll
            for (int k = 0; k < M; k++) {
                float acc = 0.0f;
#pragma unroll
                for (int j = 0; j < M; j++) acc = __fadd_rn(acc, __fmul_rn(f.hid[j], w3f[j * M + k]));
                if (a.bias) acc = __fadd_rn(acc, w3f[64 + k]);
                f.logit[k] = acc;
                if (k == 0) ltop = acc;
                else if (acc > ltop) { top = k; ltop = acc; }   // strict: the first maximum wins
            }
        }
        // ---- loss of the token and its gradient down to xW1, xW2
        float mx = f.logit[0];
#pragma unroll
        for (int k = 1; k < M; k++) mx = fmaxf(mx, f.logit[k]);
        float p[M], den = 0.0f;
#pragma unroll
        for (int k = 0; k < M; k++) { p[k] = __expf(f.logit[k] - mx); den += p[k]; }
        const float rden = 1.0f / den;
        float ptop = 0.0f, pm = 0.0f, pe = 0.0f;
#pragma unroll
        for (int k = 0; k < M; k++) { p[k] *= rden; if (k == top) { ptop = p[k]; pm = a.pen_model[k]; pe = a.pen_mem[k]; } }
        const float nll = a.nll[b];
        const float act = active ? 1.0f : 0.0f;
        lsum[0] += act * ptop * nll * pm; lsum[1] += act * ptop * pe;
        const float w = act * (a.lambda * nll * pm + (1.0f - a.lambda) * pe) * ptop * a.inv_T;
        float dl[M];
#pragma unroll
        for (int k = 0; k < M; k++) { dl[k] = w * ((k == top ? 1.0f : 0.0f) - p[k]); gb[k] += dl[k]; }
        float dx[2 * M];
#pragma unroll
        for (int m = 0; m < M; m++) {
            float dh = 0.0f;
#pragma unroll
            for (int k = 0; k < M; k++) { dh = fmaf(dl[k], w3f[m * M + k], dh); g3[m][k] = fmaf(f.hid[m], dl[k], g3[m][k]); }
            const float dz = dh * (f.sg[m] * (1.0f + f.z[m] * (1.0f - f.sg[m])));
            dx[m] = dz * v1.B[m]; dx[M + m] = dz * v1.A[m];
        }
        // ---- dW1, dW2.  A scale for every column: 2^ef <= its largest < 2^(ef+1): value * 2^(14 - ef) is below 2^15
        constexpr int P = M <= 1 ? 2 : (M <= 2 ? 4 : 8);                        // columns of a reduction, padded
        constexpr int R = M <= 4 ? 1 : 2, CR = 2 * M / R;                       // all at once, or W1's and W2's (fewer registers: 8 experts 204 us at once, 184 so)
        uint32_t upbits[R];
        float down = 0.0f;
#pragma unroll
        for (int r = 0; r < R; r++) {
            uint32_t mag[P] = {};
#pragma unroll
            for (int i = 0; i < CR; i++) mag[i] = __builtin_bit_cast(uint32_t, fabsf(dx[r * CR + i]));
            const int ef = min(max((int)(column_max(mag, lane) >> 23) - 127, -110), 127);   // of column r * CR + lane / (64 / P)
            upbits[r] = (uint32_t)(127 + 14 - ef) << 23;
            const float dn = __shfl(__builtin_bit_cast(float, (uint32_t)max(127 - 14 + ef, 1) << 23), ((NB == 1 ? piece & 7 : piece) - r * CR) * (64 / P));
            if (r == 0 || piece >= CR) down = dn;
        }
        uint16_t *mydab = dab + (lane >> 5) * kTrainH + (lane & 3) * kTrainR4 + ((lane >> 2) & 7);
        uint32_t lo[2 * M];
#pragma unroll
        for (int m = 0; m < 2 * M; m++) {
            const float s = dx[m] * __builtin_bit_cast(float, (uint32_t)__builtin_amdgcn_readlane((int)upbits[m / CR], (m % CR) * (64 / P)));
            const uint32_t hi = float_to_half_bits(s);
            lo[m] = float_to_half_bits((s - half_bits_to_float(hi)) * 2048.0f);
            mydab[m * kTrainCol] = (uint16_t)hi;
            if constexpr (NB == 1) mydab[(8 + m) * kTrainCol] = (uint16_t)lo[m];
        }
        wave_lds_sync();
        v4u_t B[NB][2];
#pragma unroll
        for (int h = 0; h < 2; h++) B[0][h] = *reinterpret_cast<const v4u_t *>(dab + h * kTrainH + r4 * kTrainR4 + piece * kTrainCol);
        if constexpr (NB == 2) {
            wave_lds_sync();
#pragma unroll
            for (int m = 0; m < 2 * M; m++) mydab[m * kTrainCol] = (uint16_t)lo[m];
            wave_lds_sync();
#pragma unroll
            for (int h = 0; h < 2; h++) B[1][h] = *reinterpret_cast<const v4u_t *>(dab + h * kTrainH + r4 * kTrainR4 + piece * kTrainCol);
        }
        const float down_lo = down * (1.0f / 2048.0f), down_c = NB == 1 && piece >= 8 ? down_lo : down;
        v4f_t c[8];
#pragma unroll
        for (int h = 0; h < 2; h++) {
            uint4 xv[8];
#pragma unroll
            for (int j = 0; j < 8; j++) { const int row = 32 * h + 4 * j + r4; xv[j] = mine[row * 16 + (piece ^ (row & 15))]; }
#pragma unroll
            for (int rt = 0; rt < 8; rt++) {
                v4u_t A;
#pragma unroll
                for (int i = 0; i < 4; i++) {         // dim rt of the tokens j = 2i (low half) and 2i + 1
                    const uint32_t w0 = word4(xv[2 * i], rt >> 1), w1 = word4(xv[2 * i + 1], rt >> 1);
                    A[i] = __builtin_amdgcn_perm(w1, w0, (rt & 1) ? 0x07060302u : 0x05040100u);
                }
                const v4f_t zero = {0.0f, 0.0f, 0.0f, 0.0f};
                if constexpr (NB == 1) {
                    c[rt] = mfma_train(A, B[0][h], h ? c[rt] : zero);
                } else {                              // the registers do not allow a second set of tiles: added up at once
                    const v4f_t c0 = mfma_train(A, B[0][h], zero), c1 = mfma_train(A, B[NB - 1][h], zero);
#pragma unroll
                    for (int n = 0; n < 4; n++) gw[rt][n] = fmaf(c0[n], down, fmaf(c1[n], down_lo, gw[rt][n]));
                }
            }
        }
        if constexpr (NB == 1) {
#pragma unroll
            for (int rt = 0; rt < 8; rt++) {
#pragma unroll
                for (int n = 0; n < 4; n++) gw[rt][n] = fmaf(c[rt][n], down_c, gw[rt][n]);
            }
        }
        wave_lds_sync();                              // rows and values are consumed
    }
    // ---- fold: lanes, then wavefronts through LDS, then the workgroups by atomic adds
#pragma unroll
    for (int m = 0; m < M; m++) {
#pragma unroll
        for (int k = 0; k < M; k++) { const float v = wave_sum(g3[m][k]); if (lane == 0) sums[wave][m * M + k] = v; }
        const float v = wave_sum(gb[m]);
        if (lane == 0) sums[wave][M * M + m] = v;
    }
    {
        const float lm = wave_sum(lsum[0]) * a.inv_T, le = wave_sum(lsum[1]) * a.inv_T;
        if (lane == 0) { sums[wave][M * M + M] = lm; sums[wave][M * M + M + 1] = le; }
    }
    float *fold = reinterpret_cast<float *>(mine);    // [dim][2M] per wavefront
#pragma unroll
    for (int rt = 0; rt < 8; rt++) {
#pragma unroll
        for (int n = 0; n < 4; n++) {
            float v = gw[rt][n];
            if constexpr (NB == 1) v += __shfl_xor(v, 8);   // first and second halves
            if (piece < 2 * M) fold[(8 * (4 * r4 + n) + rt) * (2 * M) + piece] = v;
        }
    }
    __syncthreads();
    for (int k = tid; k < kD * 2 * M; k += kTrainWaves * 64) {
        const int i = (int)((uint32_t)(k + (int)blockIdx.x * 64) % (uint32_t)(kD * 2 * M));   // workgroups end together: each starts elsewhere
        float v = 0.0f;
#pragma unroll
        for (int wv = 0; wv < kTrainWaves; wv++) v += reinterpret_cast<const float *>(&stage[wv][0])[i];
        const int d = i / (2 * M), c = i % (2 * M);
        atomicAdd(c < M ? &a.dW1[d * M + c] : &a.dW2[d * M + c - M], v);
    }
    if (tid < NS) {
        float v = 0.0f;
#pragma unroll
        for (int wv = 0; wv < kTrainWaves; wv++) v += sums[wv][tid];
        if (tid < M * M) atomicAdd(&a.dW3[tid], v);
        else if (tid < M * M + M) { if (a.dbias) atomicAdd(&a.dbias[tid - M * M], v); }
        else atomicAdd(&a.loss3[1 + tid - M * M - M], v);
    }
    if (tid == NS) {
        float lm = 0.0f, le = 0.0f;
#pragma unroll
        for (int wv = 0; wv < kTrainWaves; wv++) { lm += sums[wv][M * M + M]; le += sums[wv][M * M + M + 1]; }
        atomicAdd(&a.loss3[0], a.lambda * lm + (1.0f - a.lambda) * le);
    }
}

__global__ void train_zero_kernel(TrainArgs a) {
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < kD * a.M) { a.dW1[i] = 0.0f; a.dW2[i] = 0.0f; }
    if (i < a.M * a.M) a.dW3[i] = 0.0f;
    if (i < a.M && a.dbias) a.dbias[i] = 0.0f;
    if (i < 3) a.loss3[i] = 0.0f;
}

template <int M>
static hipError_t launch_t(const TrainArgs &a, unsigned n_wg, bool many, hipStream_t s) {
    // one and two experts: 128 or 256 multiply-adds a row are done before the weights are laid out and the open tokens settled,
    // which two tiles per wavefront pay for (two experts, 16384 / 131072 / 262144 / 1.05 M rows: 13.0 / 20.3 / 26.5 / 53.8 us in
    // order, 14.2 / 21.7 / 26.6 / 53.0)
    const dim3 grid(n_wg), block(kTrainWaves * 64);
    if constexpr (M <= 2) {
        if (many) hipLaunchKernelGGL((router_train_kernel<M, true>), grid, block, 0, s, a);
        else      hipLaunchKernelGGL((router_train_kernel<M, false>), grid, block, 0, s, a);
    } else hipLaunchKernelGGL((router_train_kernel<M, (M <= 5)>), grid, block, 0, s, a);
    return hipGetLastError();
}

hipError_t launch_router_train(const TrainArgs &a, int n_cu, hipStream_t s) {
    hipLaunchKernelGGL(train_zero_kernel, dim3((kD * 8 + 255) / 256), dim3(256), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const long long n_tiles = (long long)a.BH * ((a.n_tok + 63) / 64);
    long long n_wg = (n_tiles + kTrainWaves - 1) / kTrainWaves;
    if (n_wg > n_cu) n_wg = n_cu;                      // every wavefront keeps its accumulators over many tiles
    const bool many = n_tiles >= 2LL * kTrainWaves * n_cu;
    switch (a.M) {
        case 1: return launch_t<1>(a, (unsigned)n_wg, many, s);
        case 2: return launch_t<2>(a, (unsigned)n_wg, many, s);
        case 3: return launch_t<3>(a, (unsigned)n_wg, many, s);
        case 4: return launch_t<4>(a, (unsigned)n_wg, many, s);
        case 5: return launch_t<5>(a, (unsigned)n_wg, many, s);
        case 6: return launch_t<6>(a, (unsigned)n_wg, many, s);
        case 7: return launch_t<7>(a, (unsigned)n_wg, many, s);
        case 8: return launch_t<8>(a, (unsigned)n_wg, many, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace moqae
