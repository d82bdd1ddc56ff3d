// moqae_decode_attn: single-token decode attention over the mixed-precision packed cache with
// de-quantisation in registers and a binary32 online softmax ("Limitations" section of the
// paper: the quantised keys are de-quantised before they meet the query; softmax needs high
// precision).
//
// attn_prep_kernel    zeroes the ticket counters and counts the units of every (sequence, KV head) row (not for short calls).
// attn_split_kernel   one persistent workgroup per CU (8 wavefronts).  A workgroup owns an interval
//                     of the rows, balanced by units; inside a row its wavefronts draw tickets
//                     (one "unit" each) from counters shared by the workgroups of the row.  A unit is
//                     up to 4 KiB of K codes plus the matching 4 KiB of V codes (128 / 64 / 32 / 16
//                     tokens at 2 / 4 / 8 / 16 bits), loaded with one 16-byte load per lane per KiB.
//                     Codes are never converted one by one.  The zero-points are factored out,
//                       q.k^   = sum_g scale_g * (sum_d code_d q_d) + zero_g * (sum_{d in g} q_d)
//                       sum p v^ = sum_t (p_t scale_tg) code_td  +  sum_t p_t zero_tg,
//                     and the code sums run on the matrix cores:
//                     - one query head per KV head: byte-wise masks leave one code per byte and
//                       v_mfma_i32_16x16x64_i8 multiplies them with the base-128 digits of a
//                       fixed-point copy of q (scores) or of the softmax weights (values);
//                     - grouped queries: masking a word leaves two codes in the mantissa fields of an
//                       fp16 pair (subnormal values code * 4^k * 2^-24, which the matrix core keeps)
//                       and v_mfma_f32_16x16x32_f16 multiplies them with pre-scaled copies of q / of
//                       the weights, all heads of the group in one product;
//                     - raw fp16 rows (16-bit chunks, FP16 residual): v_dot2_f32_f16 / mixed FMAs.
//                     Every workgroup writes one partial (m, l, o[D]) per row it touched.
// attn_merge_kernel   log-sum-exp merge of the partials of one query head, normalisation (not where a row has one workgroup).
#include <type_traits>
#include "moqae_dev.hpp"
#include "moqae_kernels.hpp"

namespace moqae {

constexpr float kTwo24 = 16777216.0f;
constexpr float kTwoM24 = 1.0f / 16777216.0f;

template <int BITS> struct BW {
    static constexpr int E = 128 / BITS;                 // codes in a 16-byte slot
    static constexpr int SPR = BITS;                     // slots (= lanes) per token row of 128 dims
    static constexpr int TT = 64 / BITS;                 // tokens per KiB of codes
    static constexpr int PS = E / 2;                     // fp16 pairs per slot
    static constexpr int PPW = BITS == 16 ? 1 : 16 / BITS;   // pairs per 32-bit word
    static constexpr int KD = BITS == 2 ? 5 : (BITS == 4 ? 2 : 1);  // pairs whose bits stay below the fp16 exponent
    static constexpr int SH = BITS == 2 ? 10 : 8;        // shift that brings the remaining pairs down
    static constexpr uint32_t MASK = BITS == 16 ? 0xffffffffu : ((1u << BITS) - 1u) * 0x00010001u;
    static constexpr int BI = BITS == 2 ? 0 : (BITS == 4 ? 1 : (BITS == 8 ? 2 : 3));
};

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int kDescCap = 1024;                            // chunks of a row segment (descriptors held in LDS)
constexpr int kUnitCap = 8192;                            // units of a row segment
constexpr int kCounterStride = 64;                        // uint32 slots between two ticket counters (256 bytes)
constexpr int kMaxWeightedRowsLds = 1024;                // == kMaxWeightedRows
constexpr int kMaxBatches = 64;                           // ticket batches a workgroup can be granted per row segment
constexpr uint32_t kRowSetupCost = 40u * 16u;             // a row's set-up in the cost unit of attn_prep_kernel (512 bytes of codes)

template <int G, int REP, int NWV> struct alignas(16) AttnLds {
    static constexpr int NG = kD / G;
    uint32_t qtab[REP][64];                              // q as fp16 pairs in the order of the raw fp16 rows
    // one query head per KV head: operands and constants of the integer matrix-core path (see iq_build_q)
    v4i qa[REP == 1 ? 8 : 1][64];
    v4i wa[REP == 1 ? NWV : 1][2][64];                   // per wavefront: weight digits of up to two token blocks
    uint32_t wpos[REP == 1 ? 3 : 1][8][64];
    uint4 kx[REP == 1 ? NWV : 1][4 * 72];                // per wavefront: the K codes of a unit on their way to the lanes that use them
    alignas(16) uint32_t pcq[REP == 1 ? NWV : 1][4][kD]; // keys quantised per channel: q * scale of up to four token groups of a unit, two fp16 numbers each
    int iq[kD];
    int iqs16[8];
    float iqpart[3][8][2];
    float iqscale[4];
    alignas(16) float sc[NWV][REP][128];                             // scores (log2 domain) / fp16-path weights of a unit
    static constexpr int WLS = 136;                      // weight row stride in halfs: rows fall on different banks
    alignas(16) uint16_t wl[NWV][REP][NG][WLS];                     // fp16 softmax weight * V scale, pre-scaled per pair
    uint16_t zrow[WLS];                                  // zeros: the weight row of the unused tile rows
    float qsumg[REP][NG];                                // sum of q over a group, times 2^-24
    v4u qmc[REP > 1 ? 3 : 1][4][REP > 1 ? 64 : 1];       // grouped queries: score operands A per (bit-width, pass, lane)
    alignas(8) float comb[NWV][REP][kD + 2];                        // per-wavefront (o, m, l) at the end of a row segment
    uint32_t qraw[REP * 64];                             // the row's queries as loaded (fp16 pairs)
    unsigned long long desc[kDescCap];                   // chunk descriptors of the current pass: offset | log2 bits (Gather: offsets, ordered by bit-width)
    // ticket queue of the workgroup: local tickets [0, limit) are granted; batch i maps local
    // tickets from bl[i] on to the row's tickets from bg[i] on
    uint16_t ustart[REP > 1 ? kDescCap : 0];             // grouped queries: first unit of every chunk of the segment
    uint16_t inv[kUnitCap];                              // unit -> chunk of the segment, with one head per KV head | unit of the
                                                         // chunk << 10 (not with Gather, whose units follow from the counts)
    uint32_t wscan[NWV], wscan2[NWV];
    uint32_t U[kMaxWeightedRowsLds + 1], r0, uneven;            // prefix sums of the rows' units
    uint32_t next, limit, done, fetching, g_seen, nb;
    uint32_t bl[kMaxBatches], bg[kMaxBatches];
};

// Orders this wavefront's LDS traffic between phases that exchange data across lanes.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <int REP> struct WaveState {
    float m[REP], lsum[REP], z[REP];
    float acc[REP][2];                                   // raw fp16 rows: dims 8 (l % 16) + 2 (l / 16), + 1, in units of 2^-24
    float accq[REP][8];                                  // quantised V, one head per KV head: dims 16*ct + l%16, this lane's token slices only
    v4f accA[8];                                         // quantised V, grouped queries: matrix-core tile ct, rows 4*(l/16)..+3
};

// scale of the k-th pair of a word after masking: 2^(BITS*k') with k' counted from the shift
template <int BITS> __device__ __forceinline__ int pair_exp(int k) {
    return BITS * (k < BW<BITS>::KD ? k : k - BW<BITS>::KD);
}

// New running maximum of head r: every accumulator of the head is scaled by 2^(old - new).
template <int G, int REP>
__device__ __forceinline__ void rescale(WaveState<REP> &st, int r, float unit_max, int lane) {
    const float m_new = fmaxf(st.m[r], unit_max);
    const float alpha = (m_new == -INFINITY) ? 1.0f : fast_exp2(st.m[r] - m_new);   // first unit: exp2(-inf) = 0; nothing seen yet: unchanged
    st.m[r] = m_new;
    st.lsum[r] *= alpha; st.z[r] *= alpha; st.acc[r][0] *= alpha; st.acc[r][1] *= alpha;
    if constexpr (REP == 1) {
#pragma unroll
        for (int ct = 0; ct < 8; ct++) st.accq[r][ct] *= alpha;
    } else {
        if (alpha != 1.0f) {                              // wave-uniform; rare once the maximum has settled
            constexpr int NG = kD / G;
            const int qd = lane >> 4;
#pragma unroll
            for (int n = 0; n < 4; n++) {
                const float f = ((4 * qd + n) / NG == r) ? alpha : 1.0f;         // tile rows >= REP*NG hold zeros
#pragma unroll
                for (int ct = 0; ct < 8; ct++) st.accA[ct][n] *= f;
            }
        }
    }
}

// A unit: up to 4 KiB of K codes (nsub KiB) with the matching V codes.  All fields are
// wave-uniform and live in scalar registers; lgb = log2(bit-width) (1, 2, 3; 4 = raw fp16).
struct Unit {
    int lgb, nsub, nvalid;                               // nvalid: valid rows of an fp16 unit
    int tail_rows;                                       // residual units: valid residual rows from the unit's first row on (else huge)
    const uint8_t *kb, *vb;                              // bases: the chunk block (both), or the residual K and V rows of the row
    uint32_t kc, km, vc, vm;                             // byte offsets of the unit's K codes / K meta (from kb), V codes / V meta (from vb)
    // units of several short chunks (see Gather): kb = the arena, the blocks' offsets in it desc[first .. last]
    bool gath, half;                                     // half: 8 tokens at 2 bits, every second run of 8 tokens of the unit does not exist
    int first, last;
};

// a ? x : y field by field: a choice between the two objects would keep them in memory, whose loads the waits would count.
__device__ __forceinline__ Unit either(bool a, Unit x, Unit y) {
    Unit r;
    r.lgb = a ? x.lgb : y.lgb; r.nsub = a ? x.nsub : y.nsub; r.nvalid = a ? x.nvalid : y.nvalid; r.tail_rows = a ? x.tail_rows : y.tail_rows;
    r.kb = a ? x.kb : y.kb; r.vb = a ? x.vb : y.vb;
    r.kc = a ? x.kc : y.kc; r.km = a ? x.km : y.km; r.vc = a ? x.vc : y.vc; r.vm = a ? x.vm : y.vm;
    r.gath = a ? x.gath : y.gath; r.half = a ? x.half : y.half; r.first = a ? x.first : y.first; r.last = a ? x.last : y.last;
    return r;
}

// Units of short chunks (8, 16, 32 tokens; one query head per KV head).  A unit of one such chunk would hold a few hundred
// bytes to 2 KiB of codes instead of 8 KiB and cost nearly as much as a full one, so a unit takes as many chunks of the same
// bit-width as fill it: the row's block offsets are ordered by bit-width at the set-up (the order of the tokens does not
// matter to a softmax) and every lane's 16
// bytes are addressed through the entry of the lane's chunk, so that the registers hold what a unit of one long chunk would.  A chunk counts
// as NV tokens: N, but 16 for 8 tokens at 2 bits, whose V slice is half empty (the second half of the K tokens is masked).
// The chunk and the place inside it are a part that depends on the lane, computed once, plus a scalar part per register;
// entries past the unit's last chunk read the last one again.
// Units that are one chunk or a part of one anyway (8 bits at 32 tokens, raw rows) and the residual keep a scalar base: the
// look-ups gain them nothing.  Both branches of a loader issue the same number of loads in the same order, so that the
// waits on them can be counted exactly.
// 8 sequences x 32 heads x 8k tokens, 60/30/5/5 % at 2/4/8/16 bits, 32-token chunks: 71 us a call against 122 with a unit per
// chunk, 16 tokens 70 against 207, 8 tokens 90 against 385.  One bit-width alone (4 sequences x 32 heads x 4k tokens, groups of
// 64): 32 tokens 22.5 / 28.1 / 38.4 / 53.1 us at 2 / 4 / 8 / 16 bits against 43.7 / 41.0 / 39.3 / 54.1 (with look-ups for all
// units, and the unit's fields in memory, 23.9 / 30.9 / 40.7 / 55.5), 8 tokens at 16 bits 82 against 84 (90).
// Grouped queries keep a unit per chunk: their kernel is bound by instruction issue and at its register limit (tried: 0.26 to
// 1.17 of the speed), as do 64-token chunks, where only 2-bit units gain (the mix 0.95).
struct Gather {
    int lgb, lgnv, N;                                    // lgb 1, 2, 3: raw rows are not gathered
    __device__ __forceinline__ Gather(const Unit &u, int N_) : lgb(u.lgb), N(N_), arena(u.kb) {
        lgnv = max(31 - __builtin_clz((unsigned)N_), u.lgb == 1 ? 4 : 3);
    }
    const uint8_t *arena;
    template <typename LDS> __device__ __forceinline__ const uint8_t *block(const LDS &L, int entry) const { return arena + L.desc[entry]; }
    __device__ __forceinline__ uint32_t code_bytes() const { return (uint32_t)N << (4 + lgb); }
    __device__ __forceinline__ uint32_t vcode_bytes() const { return (uint32_t)max(N, lgb == 1 ? 16 : 8) << (4 + lgb); }
};
// The entry of bit-width lgb; by value, for the reason given at either()
__device__ __forceinline__ int of_width(int lgb, int a, int b, int c, int d) { return lgb == 1 ? a : (lgb == 2 ? b : (lgb == 3 ? c : d)); }
// log2 of the units a chunk of 2^lgnv tokens takes (positive), or of the chunks a unit takes (negative)
__host__ __device__ __forceinline__ int gather_shift(int N, int lgb) {
    const int lgn = 31 - __builtin_clz((unsigned)N), least = lgb == 4 || lgb == 1 ? 4 : 3;
    return (lgn > least ? lgn : least) - (8 - lgb);
}

template <int G> struct KRegs {
    static constexpr int GSMAX = 2;                      // a 2-bit slot of 64 codes spans two groups of 32; per-channel keys: two dims
    uint4 c[4];
    uint32_t m[4][GSMAX];
};
template <int G> struct VRegs {
    static constexpr int MV = 2 * (kD / G);              // V meta words per lane of the largest unit (2 bits)
    uint4 c[4];
    uint32_t m[MV];
};

// Loads through a scalar base plus a 32-bit per-lane byte offset (no 64-bit vector address
// arithmetic: the base of every KiB is computed on the scalar unit).  The cache is read exactly once
// per call, so every load of it is a streaming (nontemporal) load: a plain read-only kernel moves
// 6.9 TB/s with them on this chip and 6.0 TB/s with ordinary loads.
__device__ __forceinline__ uint4 ld16(const uint8_t *sbase, uint32_t voff) {
    const v4u v = __builtin_nontemporal_load(reinterpret_cast<const v4u *>(sbase + voff));
    return uint4{v[0], v[1], v[2], v[3]};
}
__device__ __forceinline__ uint32_t ld4(const uint8_t *sbase, uint32_t voff) {
    return __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(sbase + voff));
}

// The V side: the 16-byte slots 64*j + l of the unit's V KiBs and its (token, group) meta
// words 64*jj + l, same conventions.
// GATH: units of several short chunks, see Gather.
// SMALL (chunks of 8, 16 or 32 tokens, one unit per quantised chunk; grouped queries): the chunk is one token block of QD = 1, 2 or
// 4 slices, its V codes are 2 (8 bits: 4) tiles of 16*QD slots.  With QD < 4 lanes 0..16*QD-1 take tile i into c[i]
// as the lanes of the first slices of a full block would; the lanes of the absent slices and the registers of the
// absent tiles / second block hold zeros.  The meta words of a short chunk are fewer than 64: the lanes past
// them read the last one (their tokens have weight 0).
template <int G, bool SMALL, bool GATH, typename LDS>
__device__ __forceinline__ void load_v(const Unit &u, int lane, VRegs<G> &v, int N, const LDS &L) {
    constexpr int NG = kD / G;
    if (GATH && u.gath) {
        // register i: tile cg of token block bu of a full unit, lane slice qd = lane / 16; the slice's tokens lie in one chunk
        const Gather g(u, N);
        const int qd = lane >> 4;
        const int lgqd = min(2, g.lgnv - (u.lgb == 1 ? 4 : 3));           // log2 of the slices of a chunk's token block
        const uint32_t vbase = g.code_bytes() + (uint32_t)N * (NG * 4);
        {
            const int lchunk = u.first + (qd >> lgqd);
            const uint32_t loff = vbase + (uint32_t)((qd & ((1 << lgqd) - 1)) * 16 + (lane & 15)) * 16u;
            const uint8_t *b0 = g.block(L, min(lchunk, u.last)) + loff;
            const uint8_t *b1 = g.block(L, min(lchunk + (u.lgb < 3 ? 1 << (2 - lgqd) : 0), u.last)) + loff;   // 8 bits: one block of four tiles
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const uint32_t tile = u.lgb == 3 ? (uint32_t)i : (uint32_t)(i & 1);
                v.c[i] = ld16(i < 2 ? b0 : b1, tile << (8 + lgqd));
            }
        }
        {
            const int s2 = g.lgnv + (NG == 2 ? 1 : 2);                    // log2 of the meta words of a chunk (as NV tokens)
            const int words = N * NG;
            const int lchunk = u.first + (lane >> s2);
            const uint32_t loff = vbase + g.vcode_bytes() + (uint32_t)(lane & (words - 1)) * 4u;
#pragma unroll
            for (int jj = 0; jj < VRegs<G>::MV; jj++)
                v.m[jj] = ld4(g.block(L, min(lchunk + ((64 * jj) >> s2), u.last)) + loff, (uint32_t)((64 * jj) & (words - 1)) * 4u);
        }
        return;
    }
    constexpr bool PART = SMALL && !GATH;                 // a gathering kernel's other units are whole
    const int nw = u.nvalid * NG;                                         // SMALL: meta words of the unit (u.nsub counts whole KiB of codes)
    const uint32_t vv = u.vc + (uint32_t)lane * 16u, vmo = u.vm + (uint32_t)(PART ? min(lane, nw - 1) : lane) * 4u;
    const int nvm = u.lgb == 4 ? 1 : (PART ? max(nw >> 6, 1) : (u.nsub * NG) >> u.lgb);   // rows of 64 meta words, >= 1
    // slots per tile (64 for whole 1-KiB tiles) and tiles of the chunk's one block; one code path for both shapes, so
    // that the waits on the loads around these can be counted exactly
    const int ts = PART && u.lgb < 4 ? min(64, (max(N, u.lgb == 1 ? 16 : 8) << 4) >> (u.lgb == 1 ? 4 : 3)) : 64;
    const bool part = PART && ts < 64;
    const int ntile = u.lgb == 3 ? 4 : 2;
    const uint32_t vh = u.vc + (uint32_t)(lane & (ts - 1)) * 16u;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const uint4 t = ld16(u.vb, vh + (part ? (uint32_t)(min(i, ntile - 1) * ts) * 16u : (uint32_t)min(i, u.nsub - 1) * 1024u));
        const bool ok = !part || (lane < ts && i < ntile);
        v.c[i] = PART ? uint4{ok ? t.x : 0u, ok ? t.y : 0u, ok ? t.z : 0u, ok ? t.w : 0u} : t;
    }
#pragma unroll
    for (int jj = 0; jj < VRegs<G>::MV; jj++) v.m[jj] = ld4(u.vb, vmo + (uint32_t)min(jj, nvm - 1) * 256u);
}

// Softmax weights of a quantised unit: fp16(p * V scale / pair scale) per (head, group, token) into LDS.
template <int BITS, int G, int REP, int NWV>
__device__ __forceinline__ void value_weights(const VRegs<G> &v, int lane, int wave,
                                              AttnLds<G, REP, NWV> &L, WaveState<REP> &st) {
    using B = BW<BITS>;
    constexpr int NG = kD / G;
    constexpr int MAXVM = (4 * B::TT * NG / 64) > 0 ? (4 * B::TT * NG / 64) : 1;
    // ---- softmax weights, one lane per V (token, group) meta word
    constexpr int n = 32 / BITS;
#pragma unroll
    for (int jj = 0; jj < MAXVM; jj++) {
        const int idx = 64 * jj + lane, tv = idx / NG, g = idx % NG;
        const float sV = half_bits_to_float(v.m[jj] & 0xffffu);
        const float zV = half_bits_to_float(v.m[jj] >> 16);
        const int kk = (tv % n) >> 1;
        const int kp = BITS * (kk < B::KD ? kk : kk - B::KD);
        const float pre = sV * __builtin_bit_cast(float, (uint32_t)(127 - kp) << 23);
#pragma unroll
        for (int r = 0; r < REP; r++) {
            const float p = fast_exp2(L.sc[wave][r][tv] - st.m[r]);   // tokens past a short unit: score -inf, p = 0
            if (g == 0) st.lsum[r] += p;
            st.z[r] = fmaf(p, zV, st.z[r]);
            L.wl[wave][r][g][tv] = (uint16_t)float_to_half_bits(p * pre);
        }
    }

    wave_sync();
}

// v[i] summed over the 16 lanes of a row, P values at once: a step in which a lane and its partner each hand over half of their
// values takes half of the instructions of the step before, 45 for 16 values where a reduction of each takes 128.  Lane x of a
// row is left with value x P / 16 (P < 16: several lanes hold the same one; P = 32: and the next).
template <int BIT, int CTRL, int P, int PT>
__device__ __forceinline__ void row_fold_step(float (&v)[PT], int lane) {
    if constexpr (P > 1) {
#pragma unroll
        for (int i = 0; i < P / 2; i++) {
            const float keep = (lane & BIT) ? v[i + P / 2] : v[i], give = (lane & BIT) ? v[i] : v[i + P / 2];
            v[i] = keep + dpp_f<CTRL>(give);
        }
    } else {
        v[0] += dpp_f<CTRL>(v[0]);
    }
}
template <int P>
__device__ __forceinline__ void row_fold(float (&v)[P], int lane) {
    row_fold_step<8, 0x128, P>(v, lane);                             // row_ror:8
    row_fold_step<4, DPP_HALF_MIRROR, (P + 1) / 2>(v, lane);
    row_fold_step<2, DPP_XOR2, (P + 3) / 4>(v, lane);
    row_fold_step<1, DPP_XOR1, (P + 7) / 8>(v, lane);
}

// ---- one unit of raw fp16 rows (16-bit chunks and the FP16 residual) -----------------------
// 16 rows: lane l holds dims 8*(l%16)..+7 of row 4*j + l/16, for K and for V alike.  One head: every lane of
// a row ends up with the row's score, so the weights p1 need no trip through LDS and wait in registers for the value phase.
// Several heads: one score per lane (see row_fold), the weights wait in LDS.  Registers decide here (four heads: 85 spilled before,
// 39 with it; with the same scores but all weights read back at once 90, reloads in the unit loop and 131 us): four sequences of 128k
// tokens, 8 KV heads x 4 queries 121.5 -> 113.5 us a call, four new tokens on 32 heads x 32k 52.1 -> 48.0.
// Several queries per sequence (nq > 1; head r belongs to query r / rep_in): query t does not see the residual rows of
// the queries after it, the last nq - 1 - t valid rows.
template <int G, int REP, int NWV, typename KR>
__device__ __forceinline__ void fp16_scores(const Unit &u, const KR &k, int lane, int wave, float scale_log2, int nq, int rep_in,
                                            AttnLds<G, REP, NWV> &L, WaveState<REP> &st, float (&p4)[REP][4]) {
    const int part = lane & 15, tok_l = lane >> 4;
    if constexpr (REP > 1) {
        // one score per lane (8 heads: two): value 4r + j is head r, row 4j + l / 16
        constexpr int P = 4 * REP, PK = P / 16 > 0 ? P / 16 : 1, DUP = P < 16 ? 16 / P : 1;
        float v[P];
#pragma unroll
        for (int r = 0; r < REP; r++) {
            const uint4 qv = *reinterpret_cast<const uint4 *>(&L.qtab[r][part * 4]);
#pragma unroll
            for (int j = 0; j < 4; j++) {
                float ps = dot2(k.c[j].x, qv.x, 0.0f);
                ps = dot2(k.c[j].y, qv.y, ps);
                ps = dot2(k.c[j].z, qv.z, ps);
                v[4 * r + j] = dot2(k.c[j].w, qv.w, ps);
            }
        }
        row_fold<P>(v, lane);
        const int idx = part * P / 16, head = idx >> 2;              // PK consecutive values lie in one head
        int nvalid = u.nvalid;
        if (nq > 1) {
#pragma unroll
            for (int r = 0; r < REP; r++) nvalid = head == r ? min(u.nvalid, u.tail_rows - (nq - 1 - r / rep_in)) : nvalid;
        }
        float lmax = -INFINITY;
#pragma unroll
        for (int i = 0; i < PK; i++) {
            v[i] = 4 * ((idx & 3) + i) + tok_l < nvalid ? v[i] * scale_log2 : -INFINITY;
            lmax = fmaxf(lmax, v[i]);
        }
        lmax = group_max<16 / REP>(lmax);                            // over the lanes of a head in a row, then the rows
        {
            const auto x = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, lmax), __builtin_bit_cast(uint32_t, lmax), false, false);
            lmax = fmaxf(__builtin_bit_cast(float, (uint32_t)x[0]), __builtin_bit_cast(float, (uint32_t)x[1]));
            const auto y = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, lmax), __builtin_bit_cast(uint32_t, lmax), false, false);
            lmax = fmaxf(__builtin_bit_cast(float, (uint32_t)y[0]), __builtin_bit_cast(float, (uint32_t)y[1]));
        }
        float m = 0.0f;
#pragma unroll
        for (int r = 0; r < REP; r++) {
            rescale<G, REP>(st, r, __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, lmax), r * (16 / REP))), lane);
            m = head == r ? st.m[r] : m;
        }
        float *dst = &L.sc[wave][0][tok_l * P + idx], sum = 0.0f;
#pragma unroll
        for (int i = 0; i < PK; i++) {
            const float p = v[i] == -INFINITY ? 0.0f : fast_exp2(v[i] - m);         // masked rows
            dst[i] = p;
            sum += p;
        }
        if (DUP > 1 && (part & (DUP - 1)) != 0) sum = 0.0f;
#pragma unroll
        for (int r = 0; r < REP; r++) st.lsum[r] += head == r ? sum : 0.0f;
        wave_sync();
        return;
    }
#pragma unroll
    for (int r = 0; r < REP; r++) {
        const uint4 qv = *reinterpret_cast<const uint4 *>(&L.qtab[r][part * 4]);
        float s4[4], lmax = -INFINITY;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            float ps = dot2(k.c[j].x, qv.x, 0.0f);
            ps = dot2(k.c[j].y, qv.y, ps);
            ps = dot2(k.c[j].z, qv.z, ps);
            ps = dot2(k.c[j].w, qv.w, ps);
            ps = group_sum<16>(ps);
            s4[j] = (4 * j + tok_l < u.nvalid) ? ps * scale_log2 : -INFINITY;
            lmax = fmaxf(lmax, s4[j]);
        }
        rescale<G, REP>(st, r, wave_max(lmax), lane);
#pragma unroll
        for (int j = 0; j < 4; j++) {
            p4[r][j] = (s4[j] == -INFINITY) ? 0.0f : fast_exp2(s4[j] - st.m[r]);   // masked rows
            if (part == 0) st.lsum[r] += p4[r][j];
        }
    }
}
template <int G, int REP, int NWV>
__device__ __forceinline__ void fp16_values(const Unit &u, const VRegs<G> &v, int lane, int wave, AttnLds<G, REP, NWV> &L, WaveState<REP> &st, const float (&p1)[REP][4]) {
    const int tok_l = lane >> 4;
    const int nvalid = u.nvalid;
#pragma unroll
    for (int r = 0; r < REP; r++) {
        float acc8[8], p4[4];
        if constexpr (REP > 1) {
            const float4 p = *reinterpret_cast<const float4 *>(&L.sc[wave][0][tok_l * (4 * REP) + 4 * r]);
            p4[0] = p.x; p4[1] = p.y; p4[2] = p.z; p4[3] = p.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; j++) p4[j] = p1[0][j];
        }
#pragma unroll
        for (int e = 0; e < 8; e++) acc8[e] = 0.0f;
        // the packed halves feed the multiply-add directly (mixed-precision FMA), nothing is unpacked
        if (nvalid == 16) {
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const float p24 = p4[j] * kTwoM24;                 // accumulators carry a factor 2^-24
                const uint32_t w[4] = {v.c[j].x, v.c[j].y, v.c[j].z, v.c[j].w};
#pragma unroll
                for (int e = 0; e < 8; e++) {
                    const half2_t h = as_half2(w[e >> 1]);
                    acc8[e] = fmaf(p24, (float)((e & 1) ? h.y : h.x), acc8[e]);
                }
            }
        } else {                                                      // the last rows of the residual
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const float p24 = p4[j] * kTwoM24;
                const bool ok = 4 * j + tok_l < nvalid;               // rows past nvalid may hold NaN / Inf
                const uint32_t w[4] = {ok ? v.c[j].x : 0u, ok ? v.c[j].y : 0u, ok ? v.c[j].z : 0u, ok ? v.c[j].w : 0u};
#pragma unroll
                for (int e = 0; e < 8; e++) {
                    const half2_t h = as_half2(w[e >> 1]);
                    acc8[e] = fmaf(p24, (float)((e & 1) ? h.y : h.x), acc8[e]);
                }
            }
        }
        // sum over the four row groups (lanes l, l ^ 16, l ^ 32, l ^ 48), every exchange halving the dims a lane carries: lane l
        // ends up with dims 8 (l % 16) + 2 (l / 16), + 1.  (Through LDS: six accesses and two waits per head.)
        float t[4];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const auto x = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, acc8[e]), __builtin_bit_cast(uint32_t, acc8[e + 4]), false, false);
            t[e] = __builtin_bit_cast(float, (uint32_t)x[0]) + __builtin_bit_cast(float, (uint32_t)x[1]);
        }
#pragma unroll
        for (int e = 0; e < 2; e++) {
            const auto x = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, t[e]), __builtin_bit_cast(uint32_t, t[e + 2]), false, false);
            st.acc[r][e] += __builtin_bit_cast(float, (uint32_t)x[0]) + __builtin_bit_cast(float, (uint32_t)x[1]);
        }
    }
    if constexpr (REP > 1) wave_sync();                   // the weights are consumed
}

// ---- matrix-core path for grouped queries (REP > 1), quantised units -------------------------
// v_mfma_f32_16x16x32_f16 computes C[i][x] += sum_k A[i][k] B[k][x]; lane l = 16*qd + x holds
// A[x][8qd..8qd+7], B[8qd..8qd+7][x] and C[4qd..4qd+3][x].  Masked code words are valid B operands
// as they are (fp16 subnormals, which the matrix core keeps); the per-pair power of two and the
// 2^-24 are folded into A.  Tile rows carry (query head, group) pairs: row = head * NG + group.
//   scores: x = token of a 16-token tile, k = 32 dims (lane quarter qd holds dims 32qd + 8mi + 0..7 of
//           its token in pass mi = 0..3); A = q, zero outside the row's group.  The R = REP*NG rows in
//           use repeat 16/R times, so that many tiles are computed back to back and every lane keeps the
//           tile in which its own token lies: no lane is idle in the per-token arithmetic.
//   values: x = dim of a 16-dim column tile, k = 32 tokens (quarter qd holds its slice of the token
//           block); A = the softmax weights from LDS, rows >= R read zeros.
template <int G, int REP> struct MC {
    static constexpr int NG = kD / G;
    static constexpr int R = REP * NG;                   // tile rows in use
    static constexpr int F = 16 / (R < 16 ? R : 16);     // score tiles per pass
    static constexpr int HPL = 4 / NG;                   // query heads per lane (C register n: head n / NG)
    static constexpr int NSMAX = 8 / F;                  // passes of the largest unit (128 tokens, 8 tiles)
    __device__ static __forceinline__ int sel(int qd) { return F == 4 ? qd : (F == 2 ? (qd >> 1) : 0); }
    __device__ static __forceinline__ int slot0(int qd) { return (4 * qd) % R; }   // (head, group) slot of C register 0
};

template <int G, int REP> struct KRegsMC {
    uint4 c[4];
    uint32_t m[MC<G, REP>::NSMAX * (kD / G)];            // K meta words of the lane's own tokens
};

__device__ __forceinline__ v4f mfma16(v4u a, v4u b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b), c, 0, 0, 0);
}
__device__ __forceinline__ uint2 ld8(const uint8_t *sbase, uint32_t voff) {
    typedef uint32_t v2u __attribute__((ext_vector_type(2)));
    const v2u v = __builtin_nontemporal_load(reinterpret_cast<const v2u *>(sbase + voff));
    return uint2{v[0], v[1]};
}
// the k-th fp16 pair of a code word, left where it lies (scaled by 2^pair_exp(k))
template <int BITS> __device__ __forceinline__ uint32_t pair_reg(uint32_t w, int k) {
    using B = BW<BITS>;
    return k < B::KD ? (w & (B::MASK << (BITS * k))) : ((w >> B::SH) & (B::MASK << (BITS * (k - B::KD))));
}
template <int G, int REP>
__device__ __forceinline__ uint32_t kword(const KRegsMC<G, REP> &k, int i) {
    const uint4 &c = k.c[i >> 2];
    return (i & 3) == 0 ? c.x : ((i & 3) == 1 ? c.y : ((i & 3) == 2 ? c.z : c.w));
}
// pair index (inside its word) that feeds pair register pr of pass mi
template <int BITS> __device__ __forceinline__ constexpr int mc_pair(int mi, int pr) {
    return BITS == 2 ? 4 * (mi % 2) + pr : (BITS == 4 ? pr : pr % 2);
}
// B operand of score pass mi for token tile `tile`: the codes of dims 32qd + 8mi + 0..7
template <int BITS, int G, int REP>
__device__ __forceinline__ v4u mc_kcodes(const KRegsMC<G, REP> &k, int tile, int mi) {
    v4u b;
    if constexpr (BITS == 2) {
        const uint32_t w = kword(k, 2 * tile + mi / 2);
#pragma unroll
        for (int pr = 0; pr < 4; pr++) b[pr] = pair_reg<2>(w, mc_pair<2>(mi, pr));
    } else if constexpr (BITS == 4) {
        const uint32_t w = kword(k, 4 * tile + mi);
#pragma unroll
        for (int pr = 0; pr < 4; pr++) b[pr] = pair_reg<4>(w, pr);
    } else {
        const uint32_t w0 = kword(k, 8 * tile + 2 * mi), w1 = kword(k, 8 * tile + 2 * mi + 1);
        b[0] = pair_reg<8>(w0, 0); b[1] = pair_reg<8>(w0, 1); b[2] = pair_reg<8>(w1, 0); b[3] = pair_reg<8>(w1, 1);
    }
    return b;
}

// A operands of the score passes for the three quantised bit-widths, from the raw fp16 queries in LDS.
template <int G, int REP, typename LDS>
__device__ __forceinline__ void mc_build_q(const uint32_t *qraw32, int lane, int mi, LDS &L) {
    using M = MC<G, REP>;
    const int i = lane & 15, qd = lane >> 4;
    const int slot = i % M::R, r = slot / M::NG, g = slot % M::NG;
    const bool own = g == (32 * qd) / G;                 // the quarter's dims lie in the row's group
    {                                                    // pass mi: one wavefront per pass
        v4u ak[3];
#pragma unroll
        for (int pr = 0; pr < 4; pr++) {
            const uint32_t qq = qraw32[r * 64 + 16 * qd + 4 * mi + pr];          // dims 32qd + 8mi + 2pr, +1
            const float q0 = half_bits_to_float(qq & 0xffffu), q1 = half_bits_to_float(qq >> 16);
#pragma unroll
            for (int bi = 0; bi < 3; bi++) {
                const int kp = bi == 0 ? pair_exp<2>(mc_pair<2>(mi, pr)) : (bi == 1 ? pair_exp<4>(mc_pair<4>(mi, pr)) : 0);   // mi & 1 decides
                const float f = __builtin_bit_cast(float, (uint32_t)(127 - kp) << 23);
                const uint32_t v = float_to_half_bits(q0 * f) | (float_to_half_bits(q1 * f) << 16);
                ak[bi][pr] = own ? v : 0u;
            }
        }
#pragma unroll
        for (int bi = 0; bi < 3; bi++) L.qmc[bi][mi][lane] = ak[bi];
    }
}

// K side of a unit for grouped queries.  Quantised units: lane (x, qd) takes quarter qd of the code row
// of token 16*tile + x for every tile, and the meta words of its own tokens; raw fp16 units keep the
// slot order of load_k.  Eight 8-byte loads whatever the bit-width, branch-free like load_k.
template <int G, int REP, bool SMALL>
__device__ __forceinline__ void load_k_mc(const Unit &u, int lane, KRegsMC<G, REP> &k) {
    using M = MC<G, REP>;
    const int x = lane & 15, qd = lane >> 4;
    const bool raw = u.lgb == 4;
    const int rbsh = 4 + u.lgb;                           // log2(bytes of a code row)
    const uint32_t lane_off = raw ? (uint32_t)lane * 16u : (((uint32_t)x << rbsh) + ((uint32_t)qd << (rbsh - 2)));
    const int iptsh = raw ? 1 : u.lgb - 1;                // log2(loads per tile); raw: per KiB
    const int tbsh = raw ? 10 : rbsh + 4;                 // log2(bytes per tile); raw: a KiB
    // A streaming load drops its 128-byte line after use, so every line must be covered by ONE load instruction:
    // 8-byte pieces only at 2 bits (a quarter row is 8 bytes; the 16 lanes of a quarter cover whole lines together),
    // 16-byte pieces otherwise (a quarter row is 16 bytes at 4 bits, 32 bytes = two adjacent pieces at 8 bits).
    if (u.lgb == 1) {
        const int imax = 2 * u.nsub - 1;
#pragma unroll
        for (int i = 0; i < 8; i++) {
            const int ic = min(i, imax);
            const uint2 t = ld8(u.kb, u.kc + lane_off + (((uint32_t)(ic >> iptsh) << tbsh) + (uint32_t)(ic & ((1 << iptsh) - 1)) * 8u));
            if (i & 1) { k.c[i >> 1].z = t.x; k.c[i >> 1].w = t.y; } else { k.c[i >> 1].x = t.x; k.c[i >> 1].y = t.y; }
        }
    } else {
#pragma unroll
        for (int j = 0; j < 4; j++) {
            // 8 bits: a tile of 16 tokens is two pieces per lane, also when the chunk has only 8 tokens (1 KiB)
            const uint32_t jc = (uint32_t)min(j, (SMALL && u.lgb == 3 ? max(u.nsub, 2) : u.nsub) - 1);
            k.c[j] = ld16(u.kb, u.kc + lane_off + (u.lgb == 3 ? (jc >> 1) * 2048u + (jc & 1u) * 16u : jc * 1024u));
        }
    }
    const int TU = raw ? 16 : u.nvalid;                   // tokens of the unit
#pragma unroll
    for (int s = 0; s < M::NSMAX; s++) {
        const int t = min(16 * (s * M::F + M::sel(qd)) + x, TU - 1);
        if constexpr (M::NG == 2) {
            const uint2 mm = ld8(u.kb, u.km + (uint32_t)t * 8u);
            k.m[2 * s] = mm.x; k.m[2 * s + 1] = mm.y;
        } else {
            const uint4 mm = ld16(u.kb, u.km + (uint32_t)t * 16u);
            k.m[4 * s] = mm.x; k.m[4 * s + 1] = mm.y; k.m[4 * s + 2] = mm.z; k.m[4 * s + 3] = mm.w;
        }
    }
}

// Scores of a quantised unit -> L.sc (log2 domain), running maxima updated.
template <int BITS, int G, int REP, int NWV>
__device__ __forceinline__ void mc_scores(const Unit &u, const KRegsMC<G, REP> &k, const v4u (&ak)[4],
                                          const float (&qp)[4], int lane, int wave, float scale24,
                                          AttnLds<G, REP, NWV> &L, WaveState<REP> &st) {
    using M = MC<G, REP>;
    using B = BW<BITS>;
    constexpr int NG = M::NG, HPL = M::HPL, F = M::F;
    constexpr int TL = 16 / BITS;                         // tiles of a full unit: 8, 4, 2
    constexpr int NS = (TL + F - 1) / F;
    const int x = lane & 15, qd = lane >> 4, sel = M::sel(qd);
    const int TU = u.nvalid;
    float sv[NS][HPL], hmax[HPL];
#pragma unroll
    for (int h = 0; h < HPL; h++) hmax[h] = -INFINITY;
#pragma unroll
    for (int s = 0; s < NS; s++) {
        v4f own = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int f = 0; f < F; f++) {
            const int tile = s * F + f;
            if (tile < TL) {
                v4f c = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int mi = 0; mi < 4; mi++) c = mfma16(ak[mi], mc_kcodes<BITS, G, REP>(k, tile, mi), c);
                if (F == 1) own = c;
                else {
#pragma unroll
                    for (int n = 0; n < 4; n++) own[n] = (sel == f) ? c[n] : own[n];
                }
            }
        }
        const int t = 16 * (s * F + sel) + x;
        const bool valid = t < TU;
#pragma unroll
        for (int h = 0; h < HPL; h++) {
            float ps = 0.0f;
#pragma unroll
            for (int g = 0; g < NG; g++) {
                const uint32_t mw = k.m[s * NG + g];
                ps = fmaf(half_bits_to_float(mw & 0xffffu), own[h * NG + g], ps);
                ps = fmaf(half_bits_to_float(mw >> 16), qp[h * NG + g], ps);
            }
            sv[s][h] = valid ? ps * scale24 : -INFINITY;
            hmax[h] = fmaxf(hmax[h], sv[s][h]);
        }
    }
#pragma unroll
    for (int h = 0; h < HPL; h++) hmax[h] = group_max<16>(hmax[h]);
#pragma unroll
    for (int r = 0; r < REP; r++) {                       // the quarters whose rows hold head r
        float um = -INFINITY;
#pragma unroll
        for (int q4 = 0; q4 < 4; q4++) {
            const int r0q = ((4 * q4) % M::R) / NG;
            if (r0q <= r && r < r0q + HPL)
                um = fmaxf(um, __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, hmax[r - r0q]), 16 * q4)));
        }
        rescale<G, REP>(st, r, um, lane);
    }
    const int r0 = M::slot0(qd) / NG;
#pragma unroll
    for (int s = 0; s < NS; s++) {
        const int t = 16 * (s * F + sel) + x;
#pragma unroll
        for (int h = 0; h < HPL; h++) L.sc[wave][r0 + h][t] = sv[s][h];
    }
    wave_sync();
}

// Weighted value sum of a quantised unit on the matrix cores.
template <int BITS, int G, int REP, int NWV>
__device__ __forceinline__ void mc_value_dots(const VRegs<G> &v, int lane, int wave,
                                              AttnLds<G, REP, NWV> &L, WaveState<REP> &st) {
    using M = MC<G, REP>;
    constexpr int TW = 32 / BITS, TQ = TW > 8 ? TW : 8, WD = TQ / TW, CPK = 4 / WD, TB = 4 * TQ, KPB = 8 / CPK;
    constexpr int WLS = AttnLds<G, REP, NWV>::WLS;
    const int i = lane & 15, qd = lane >> 4;
    const uint16_t *arow = (i < M::R) ? &L.wl[wave][0][0][0] + i * WLS : &L.zrow[0];   // row = head * NG + group
    arow += qd * TQ;
    v4u a0 = {0, 0, 0, 0}, a1 = {0, 0, 0, 0};
#pragma unroll
    for (int jk = 0; jk < 4; jk++) {
        const int bu = jk / KPB, cg = jk % KPB;
        if (cg == 0) {                                    // the weights of this token block
            a0 = *reinterpret_cast<const v4u *>(arow + bu * TB);
            if constexpr (BITS == 2) a1 = *reinterpret_cast<const v4u *>(arow + bu * TB + 8);
        }
        const uint32_t wv[4] = {v.c[jk].x, v.c[jk].y, v.c[jk].z, v.c[jk].w};
        if constexpr (BITS == 8) {
#pragma unroll
            for (int nc = 0; nc < 2; nc++) {
                const int ct = cg * CPK + nc;
                v4u b;
                b[0] = pair_reg<8>(wv[2 * nc], 0); b[1] = pair_reg<8>(wv[2 * nc], 1);
                b[2] = pair_reg<8>(wv[2 * nc + 1], 0); b[3] = pair_reg<8>(wv[2 * nc + 1], 1);
                st.accA[ct] = mfma16(a0, b, st.accA[ct]);
            }
        } else {
#pragma unroll
            for (int nw = 0; nw < 4; nw++) {
                const int ct = cg * CPK + nw;
                v4u b;
#pragma unroll
                for (int pr = 0; pr < 4; pr++) b[pr] = pair_reg<BITS>(wv[nw], pr);
                st.accA[ct] = mfma16(a0, b, st.accA[ct]);
                if constexpr (BITS == 2) {
#pragma unroll
                    for (int pr = 0; pr < 4; pr++) b[pr] = pair_reg<2>(wv[nw], 4 + pr);
                    st.accA[ct] = mfma16(a1, b, st.accA[ct]);
                }
            }
        }
    }
    wave_sync();
}

// ---- integer matrix-core path (one query head per KV head), quantised units ------------------
// v_mfma_i32_16x16x64_i8 computes C[i][x] += sum_k A[i][k] B[k][x] on signed bytes; lane l = 16*xq + x
// holds A[x][16xq..16xq+15], B[16xq..16xq+15][x] and C[4xq..4xq+3][x].  The codes are the B operand:
// masking a code word byte-wise leaves one code per byte (2 bits: four planes, the code shifted left
// by 0, 2, 0, 2 bits; 4 bits: the low and the high nibbles; 8 bits: the bytes themselves, minus 128
// through a sign flip).  The other factor -- q for the scores, softmax weight * V scale for the values --
// is turned into a fixed-point integer, multiplied by the power of two that undoes its plane's shift,
// and split into four base-128 digits that sit in four rows of A; the four digit sums come back in the
// four C registers of a lane and are recombined exactly in integer / fp32 arithmetic.
//   scores: A is block diagonal (rows 4xq..4xq+3 are nonzero for k in quarter xq only), so that a lane's
//           C registers hold the dot product of its OWN 16 code bytes with the digits of q: the matrix
//           core serves as a per-lane 16-term integer dot product.  All lanes of a quarter must then hold
//           the same dims, which fixes the lane -> slot assignment of load_k_iq.
//   values: column x = dim of a 16-dim column tile, k = 64 tokens (quarter xq holds its slice of the token
//           block); rows 4g..4g+3 = digits of the weights of group g, so quarter g of the lanes ends up
//           with the sums for the column tiles whose dims lie in group g.
__device__ __forceinline__ v4i mfma_i8(v4i a, v4i b, v4i c) {
    return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
}
constexpr int kFix = 23;                                 // fixed-point numbers are below 2^(kFix + 1): four digits hold 28 bits, planes take 2
// sum_n 128^n C[n] as fp32 (the two halves are exact integers below 2^31)
__device__ __forceinline__ float iq_combine(v4i c) {
    const int hi = c[3] * 128 + c[2], lo = c[1] * 128 + c[0];
    return fmaf((float)hi, 16384.0f, (float)lo);
}
// The byte planes of a code word.  2 bits: byte y of plane p holds code 8*(y%2) + 2p + y/2 of the word, shifted left by
// {0, 2, 0, 2}[p] (five operations, as the shifts {0, 2, 4, 5} would take that leave three planes where they lie; but the
// factor that every product carries is 2^2 and not 2^6, so that q and the weights have room for 24 bits and not 21:
// the error of an attention output against binary64 went from 9.9e-6 to 1.3e-6 at 128k tokens); 4 bits: code 4*(y%2) + 2p + y/2; 8 bits: code 2*(y%2) + y/2, minus 128.
template <int BITS> struct IQ {
    static constexpr int NP = 8 / BITS;                  // planes of a word
    static constexpr int LGM = BITS == 2 ? 2 : 0;        // log2 of the factor every product carries
    static constexpr int BI = BITS == 2 ? 0 : (BITS == 4 ? 1 : 2);
    __device__ static __forceinline__ void planes(uint32_t w, int *m) {
        if constexpr (BITS == 2) {
            const uint32_t h = w >> 4;
            m[0] = (int)(w & 0x03030303u); m[1] = (int)(w & 0x0c0c0c0cu);
            m[2] = (int)(h & 0x03030303u); m[3] = (int)(h & 0x0c0c0c0cu);
        } else if constexpr (BITS == 4) {
            m[0] = (int)(w & 0x0f0f0f0fu); m[1] = (int)((w >> 4) & 0x0f0f0f0fu);
        } else {
            m[0] = (int)(w ^ 0x80808080u);
        }
    }
};
__device__ __forceinline__ uint32_t word_of(const uint4 &c, int i) {
    return i == 0 ? c.x : (i == 1 ? c.y : (i == 2 ? c.z : c.w));
}

// K side of a unit, one query head per KV head.  The codes are read in memory order (lane l takes the
// 16-byte slot 64j + l of KiB j, fully coalesced); iq_regroup then hands every lane the slot the matrix
// products want.  The meta words are read for the lane's final (token, group) directly:
//   2 bits: register j holds token 32j + 16*(xq/2) + c, half row xq%2 (64 dims);
//   4 bits: token 16j + c, quarter row xq (32 dims);
//   8 bits: token 16*(j/2) + c, eighth of a row 4*(j%2) + xq (16 dims);
// raw fp16 units keep the slot order and have no meta.
// KPC (keys quantised per channel): the meta words are [token group][dim]; lane l takes the words of dims 2l, 2l+1 of
// the (up to four) token groups the unit's tokens lie in.
template <int G, bool KPC, bool SMALL, typename LDS>
__device__ __forceinline__ void load_k_iq(const Unit &u, int lane, KRegs<G> &k, int N, const LDS &L) {
    constexpr int NG = kD / G;
    const uint32_t xq = (uint32_t)lane >> 4, c = (uint32_t)lane & 15u;
    if (SMALL && u.gath) {
        const Gather g(u, N);
        {
            const int s2 = g.lgnv + u.lgb;                                // log2 of the 16-byte slots of a chunk: at least 5
            const int lchunk = u.first + (lane >> s2);
            const uint32_t loff = (uint32_t)(lane & ((1 << s2) - 1)) * 16u;
#pragma unroll
            for (int j = 0; j < 4; j++)
                k.c[j] = ld16(g.block(L, min(lchunk + ((64 * j) >> s2), u.last)) + loff, (uint32_t)((64 * j) & ((1 << s2) - 1)) * 16u);
        }
        if constexpr (KPC) {                              // 32-token chunks in groups of 32: a token group per chunk
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const uint2 mm = ld8(g.block(L, min(u.first + j, u.last)) + g.code_bytes(), (uint32_t)lane * 8u);
                k.m[j][0] = mm.x; k.m[j][1] = mm.y;
            }
            return;
        }
        // token of register j: a part of the lane's, below 32, and 32j, 16j or 16 (j / 2)
        const uint32_t lt = u.lgb == 1 ? 16u * (xq >> 1) + c : c;
        const uint32_t grp = u.lgb == 1 ? (xq & 1u) * (NG / 2) : (u.lgb == 2 ? (NG == 2 ? (xq >> 1) : xq) : (NG == 2 ? 0u : (xq >> 1)));
        const uint32_t nv1 = (1u << g.lgnv) - 1u;
        const int lchunk = u.first + (int)(lt >> g.lgnv);
        const uint32_t loff = g.code_bytes() + ((lt & nv1) * NG + grp) * 4u;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const uint32_t tj = u.lgb == 1 ? 32u * j : (u.lgb == 2 ? 16u * j : 16u * (j >> 1));
            const uint32_t o = ((tj & nv1) * NG + (u.lgb == 3 ? (uint32_t)(j & 1) * (NG / 2) : 0u)) * 4u;
            const uint8_t *mb = g.block(L, min(lchunk + (int)(tj >> g.lgnv), u.last)) + loff;
            k.m[j][0] = ld4(mb, o);
            if constexpr (NG == 4) k.m[j][1] = ld4(mb, o + (u.lgb == 1 ? 4u : 0u));
        }
        return;
    }
    const uint32_t vk = u.kc + (uint32_t)lane * 16u;
#pragma unroll
    for (int j = 0; j < 4; j++) k.c[j] = ld16(u.kb, vk + (uint32_t)min(j, u.nsub - 1) * 1024u);   // short unit: the last KiB is read again (ignored)
    if constexpr (KPC) {                                  // four loads for every unit (a raw fp16 unit reads its own rows and ignores them)
        const int lgq = min(u.lgb, 3);
        const int t0 = (int)(u.kc >> (4 + lgq)), TU = u.nsub << (6 - lgq);
        const int ngu = u.lgb == 4 ? 1 : (t0 % G + TU + G - 1) / G;
        const uint32_t mbase = u.lgb == 4 ? u.kc : u.km;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const uint2 mm = ld8(u.kb, mbase + (uint32_t)min(j, ngu - 1) * (kD * 4u) + (uint32_t)lane * 8u);
            k.m[j][0] = mm.x; k.m[j][1] = mm.y;
        }
        return;
    }
    // The same number of loads whatever the unit (a raw fp16 unit reads four words of its rows and ignores them) and
    // no branch: the waits on everything requested after these loads can then be counted exactly.
    // word of the lane's (token, group) per bit-width, and the step from register j to j + 1 (8 bits: two steps)
    const uint32_t w1 = (16u * (xq >> 1) + c) * NG + (xq & 1u) * (NG / 2);
    const uint32_t w2 = c * NG + (NG == 2 ? (xq >> 1) : xq);
    const uint32_t w3 = c * NG + (NG == 2 ? 0u : (xq >> 1));
    const uint32_t vm = u.lgb == 4 ? u.kc + c * 4u : u.km + (u.lgb == 1 ? w1 : (u.lgb == 2 ? w2 : w3)) * 4u;
    const int jmax = u.lgb == 1 ? u.nsub - 1 : 3;              // a short unit's block ends early
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const uint32_t jc = (uint32_t)min(j, jmax);
        const uint32_t o1 = jc * (32u * NG * 4u), o2 = jc * (16u * NG * 4u);
        const uint32_t o3 = (uint32_t)(j >> 1) * (16u * NG * 4u) + (uint32_t)(j & 1) * ((NG / 2) * 4u);
        const uint32_t oj = u.lgb == 4 ? 0u : (u.lgb == 1 ? o1 : (u.lgb == 2 ? o2 : o3));
        k.m[j][0] = ld4(u.kb, vm + oj);
        if constexpr (NG == 4) k.m[j][1] = ld4(u.kb, vm + oj + (u.lgb == 1 ? 4u : 0u));
    }
}

// Hands every lane the code slots of its (token, part) through the wavefront's LDS buffer.  The slots
// are stored XOR-swizzled (and every KiB 128 bytes further than the last), so that both the writes in
// memory order and the regrouped reads touch every bank once.
template <int BITS, int G, int NWV>
__device__ __forceinline__ void iq_regroup(const KRegs<G> &k, int lane, int wave, AttnLds<G, 1, NWV> &L, uint4 (&kc)[4]) {
    constexpr int KS = 72;                                // slots between two KiBs
    uint4 *buf = &L.kx[wave][0];
    const int xq = lane >> 4, c = lane & 15;
    const int sw = BITS == 2 ? (lane >> 4) & 1 : (BITS == 4 ? (lane >> 4) & 3 : (lane >> 3) & 7);
#pragma unroll
    for (int j = 0; j < 4; j++) buf[j * KS + (lane ^ sw)] = k.c[j];
    wave_sync();
#pragma unroll
    for (int j = 0; j < 4; j++) {
        int pos;
        if constexpr (BITS == 2)      pos = j * KS + ((32 * (xq >> 1) + 2 * c + (xq & 1)) ^ (c >> 3));
        else if constexpr (BITS == 4) pos = j * KS + 4 * c + (xq ^ (c >> 2));
        else                          pos = (2 * (j >> 1) + (c >> 3)) * KS + 8 * (c & 7) + ((4 * (j & 1) + xq) ^ (c & 7));
        kc[j] = buf[pos];
    }
    wave_sync();
}

// Scores of a quantised unit -> L.sc (log2 domain), running maximum updated.
// SMALL: the unit may end inside a KiB of codes; the scores of the tokens past u.nvalid are masked one by one.
template <int BITS, int G, int NWV, bool SMALL>
__device__ __forceinline__ void iq_scores(const Unit &u, const KRegs<G> &k, int lane, int wave,
                                          AttnLds<G, 1, NWV> &L, WaveState<1> &st) {
    constexpr int NG = kD / G;
    const int xq = lane >> 4, c = lane & 15;
    const float sc = L.iqscale[IQ<BITS>::BI];
    const v4i zero = {0, 0, 0, 0};
    uint4 kc[4];
    iq_regroup<BITS, G, NWV>(k, lane, wave, L, kc);
    if constexpr (BITS == 2) {
        constexpr int GS = NG == 4 ? 2 : 1;              // groups inside a half row
        const int part = xq & 1;
        v4i A[4];
#pragma unroll
        for (int wd = 0; wd < 4; wd++) A[wd] = L.qa[wd][lane];
        float qp[GS];
#pragma unroll
        for (int gi = 0; gi < GS; gi++) qp[gi] = L.iqpart[0][part][gi];
        float s4[4], lmax = -INFINITY;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            v4i acc[GS];
#pragma unroll
            for (int gi = 0; gi < GS; gi++) acc[gi] = zero;
#pragma unroll
            for (int wd = 0; wd < 4; wd++) {
                int m[4];
                IQ<2>::planes(word_of(kc[j], wd), m);
                acc[wd / (4 / GS)] = mfma_i8(A[wd], v4i{m[0], m[1], m[2], m[3]}, acc[wd / (4 / GS)]);
            }
            float ps = 0.0f;
#pragma unroll
            for (int gi = 0; gi < GS; gi++) {
                ps = fmaf(half_bits_to_float(k.m[j][gi] & 0xffffu), iq_combine(acc[gi]), ps);
                ps = fmaf(half_bits_to_float(k.m[j][gi] >> 16), qp[gi], ps);
            }
            ps += __shfl_xor(ps, 16);
            const bool ok = SMALL ? 32 * j + 16 * (xq >> 1) + c < u.nvalid && !(u.half && (c & 8)) : j < u.nsub;   // KiB past a short unit: ignored
            s4[j] = ok ? ps * sc : -INFINITY;
            lmax = fmaxf(lmax, s4[j]);
        }
        rescale<G, 1>(st, 0, wave_max(lmax), lane);
        if (part == 0) {
#pragma unroll
            for (int j = 0; j < 4; j++) L.sc[wave][0][32 * j + 16 * (xq >> 1) + c] = s4[j];
        }
    } else if constexpr (BITS == 4) {
        const v4i A0 = L.qa[4][lane], A1 = L.qa[5][lane];
        const float qp = L.iqpart[1][xq][0];
        float s4[4], lmax = -INFINITY;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            int m0[2], m1[2], m2[2], m3[2];
            IQ<4>::planes(kc[j].x, m0); IQ<4>::planes(kc[j].y, m1);
            IQ<4>::planes(kc[j].z, m2); IQ<4>::planes(kc[j].w, m3);
            v4i acc = mfma_i8(A0, v4i{m0[0], m0[1], m1[0], m1[1]}, zero);
            acc = mfma_i8(A1, v4i{m2[0], m2[1], m3[0], m3[1]}, acc);
            float ps = half_bits_to_float(k.m[j][0] >> 16) * qp;
            ps = fmaf(half_bits_to_float(k.m[j][0] & 0xffffu), iq_combine(acc), ps);
            ps += __shfl_xor(ps, 16);
            ps += __shfl_xor(ps, 32);
            const bool ok = SMALL ? 16 * j + c < u.nvalid : j < u.nsub;   // KiB past a short unit: ignored
            s4[j] = ok ? ps * sc : -INFINITY;
            lmax = fmaxf(lmax, s4[j]);
        }
        rescale<G, 1>(st, 0, wave_max(lmax), lane);
        if (xq == 0) {
#pragma unroll
            for (int j = 0; j < 4; j++) L.sc[wave][0][16 * j + c] = s4[j];
        }
    } else {
        const v4i A[2] = {L.qa[6][lane], L.qa[7][lane]};
        const float qp[2] = {L.iqpart[2][xq][0], L.iqpart[2][4 + xq][0]};
        float s2[2], lmax = -INFINITY;
#pragma unroll
        for (int jj = 0; jj < 2; jj++) {
            float ps = 0.0f;
#pragma unroll
            for (int r = 0; r < 2; r++) {
                const uint4 &w = kc[2 * jj + r];
                const v4i b = {(int)(w.x ^ 0x80808080u), (int)(w.y ^ 0x80808080u), (int)(w.z ^ 0x80808080u), (int)(w.w ^ 0x80808080u)};
                const float isum = fmaf(128.0f, qp[r], iq_combine(mfma_i8(A[r], b, zero)));
                const uint32_t mw = k.m[2 * jj + r][0];
                ps = fmaf(half_bits_to_float(mw & 0xffffu), isum, ps);
                ps = fmaf(half_bits_to_float(mw >> 16), qp[r], ps);
            }
            ps += __shfl_xor(ps, 16);
            ps += __shfl_xor(ps, 32);
            s2[jj] = (!SMALL || 16 * jj + c < u.nvalid) ? ps * sc : -INFINITY;
            lmax = fmaxf(lmax, s2[jj]);
        }
        rescale<G, 1>(st, 0, wave_max(lmax), lane);
        if (xq == 0) { L.sc[wave][0][c] = s2[0]; L.sc[wave][0][16 + c] = s2[1]; }
    }
    wave_sync();
}

// Sums (or maxima) of P = 1, 2 or 4 values per lane over the wavefront, each wave-uniform.  Four at once: every exchange across
// half the lanes also halves the registers, 14 instructions against 40.
template <int P, bool MAX>
__device__ __forceinline__ void wave_fold(float (&v)[P]) {
    if constexpr (P == 4) {
        auto fold = [](float a, float b) { return MAX ? fmaxf(a, b) : a + b; };
        float t[2];
#pragma unroll
        for (int i = 0; i < 2; i++) {                    // lanes 32.. take values 2 and 3
            const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, v[i]), __builtin_bit_cast(uint32_t, v[i + 2]), false, false);
            t[i] = fold(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
        }
        const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, t[0]), __builtin_bit_cast(uint32_t, t[1]), false, false);
        float x = fold(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));   // row i of 16 lanes: value i
        x = MAX ? group_max<16>(x) : group_sum<16>(x);
#pragma unroll
        for (int i = 0; i < 4; i++) v[i] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 16 * i));
    } else {
#pragma unroll
        for (int i = 0; i < P; i++) v[i] = MAX ? wave_max(v[i]) : wave_sum(v[i]);
    }
}

// The pairs of a code word for products whose sums keep 24 bits: a subnormal number enters the matrix core's sum with the smallest
// normal exponent, so that of a code in the lowest bits of the mantissa little more than 12 bits of the product are left (sums of
// 128: error 5.6e-6 of the result at bit 0, 6.9e-7 at bit 2, 8.6e-8 at bit 4, 2e-8 from bit 6 on; normal numbers 2e-8).  Every pair
// is brought to the top of the mantissa: four instructions a word more than pair_reg at 2 bits, three at 4 bits, one at 8 bits.
template <int BITS> __device__ __forceinline__ constexpr int high_pair_exp(int k) {
    return BITS == 2 ? (k == 0 || k == 2 || k == 3 || k == 5 ? 6 : 8) : (BITS == 4 ? 6 : 2);
}
template <int BITS> __device__ __forceinline__ uint32_t high_pair(uint32_t w, int k) {
    const int to = high_pair_exp<BITS>(k), from = BITS * k;
    return (to >= from ? w << (to - from) : w >> (from - to)) & (BW<BITS>::MASK << to);
}

// Scores of a quantised unit whose keys are quantised per channel (a group = G consecutive tokens of one dim):
//   q . k^_t = sum_d (q_d * scale_{g,d}) * code_{t,d} + sum_d q_d * zero_{g,d},   g = the token group of t,
// so the scale folds into a copy of q per token group (built here from the unit's meta words and kept in LDS)
// and the zero-points into one number per group.  The code sums run on v_mfma_f32_16x16x32_f16, codes = the B operand (masked
// words, see mc_scores; column = token of a 16-token tile), the copy of q = A: scaled by a power of two of its group and split
// into two fp16 numbers, which hold the 22 bits that the product of two fp16 numbers has (down to 2^-28 of the group's largest),
// in the rows 2i and 2i + 1: every lane gets both sums of its column and keeps those of the tile its own token lies in.
// Result as iq_scores: L.sc (log2 domain), running maximum updated.
// What bounds it: instruction issue and LDS.  A multiply-add per code on the vector ALU takes 64 16-byte reads of the copy of q
// and 400 vector instructions for a 2-bit unit; this takes 4 writes and 8 half reads for the codes, 16 reads for q, and 280.
// 40 heads of 64k tokens in groups of 32: 84.6 -> 77.5 us a call; the error against binary64 stays at 1.3e-6.
template <int BITS, int G, int NWV>
__device__ __forceinline__ void pc_scores(const Unit &u, const KRegs<G> &k, int lane, int wave, float scale_log2,
                                          AttnLds<G, 1, NWV> &L, WaveState<1> &st) {
    constexpr int TL = 16 / BITS, NP = (TL + 3) / 4;      // 16-token tiles of a full unit, passes of four tiles
    constexpr int NGU = (256 / BITS) / G > 0 ? (256 / BITS) / G : 1;     // token groups a full unit spans: it starts at a group, or lies in one
    const int x = lane & 15, q = lane >> 4;
    // the codes of tile f: lane (x, q) takes 32 (8 bits: twice 16) dims of token 16f + x
    uint4 kc[4];
    uint2 kc2[TL];
    if constexpr (BITS == 2) {
        uint4 *buf = &L.kx[wave][0];
#pragma unroll
        for (int j = 0; j < 4; j++) buf[64 * j + lane] = k.c[j];
        wave_sync();
#pragma unroll
        for (int f = 0; f < TL; f++) kc2[f] = reinterpret_cast<const uint2 *>(buf)[64 * f + 4 * x + q];
        wave_sync();
    } else {
        iq_regroup<BITS, G, NWV>(k, lane, wave, L, kc);
    }
    const uint32_t qq = L.qraw[lane];
    const float q0 = half_bits_to_float(qq & 0xffffu), q1 = half_bits_to_float(qq >> 16);
    // dims 2l, 2l + 1 are one pair of their word: the power of two of its place rides in the copy of q
    const float unshift = __builtin_bit_cast(float, (uint32_t)(127 - high_pair_exp<BITS>(lane % (16 / BITS))) << 23);
    float v0[NGU], v1[NGU], big[NGU], bias[NGU], down[NGU];
#pragma unroll
    for (int j = 0; j < NGU; j++) {
        const uint32_t m0 = k.m[j][0], m1 = k.m[j][1];
        v0[j] = q0 * unshift * half_bits_to_float(m0 & 0xffffu); v1[j] = q1 * unshift * half_bits_to_float(m1 & 0xffffu);
        big[j] = fmaxf(fabsf(v0[j]), fabsf(v1[j]));
        bias[j] = fmaf(q0, half_bits_to_float(m0 >> 16), q1 * half_bits_to_float(m1 >> 16));
    }
    wave_fold<NGU, true>(big);
    wave_fold<NGU, false>(bias);
#pragma unroll
    for (int j = 0; j < NGU; j++) {
        // 2^ef <= the largest < 2^(ef+1): times 2^(14 - ef) it is below 2^15
        const int ef = min(max((int)((__builtin_bit_cast(uint32_t, big[j]) >> 23) & 255u) - 127, -100), 100);
        const float up = __builtin_bit_cast(float, (uint32_t)(127 + 14 - ef) << 23);
        down[j] = __builtin_bit_cast(float, (uint32_t)(127 + 24 - 14 + ef) << 23);       // the codes carry 2^-24
        const float a0 = v0[j] * up, a1 = v1[j] * up;
        const uint32_t h0 = float_to_half_bits(a0), h1 = float_to_half_bits(a1);
        const uint32_t l0 = float_to_half_bits((a0 - half_bits_to_float(h0)) * 2048.0f), l1 = float_to_half_bits((a1 - half_bits_to_float(h1)) * 2048.0f);
        L.pcq[wave][j][lane] = h0 | (h1 << 16);
        L.pcq[wave][j][64 + (lane ^ 4)] = l0 | (l1 << 16);   // 16-byte pieces swapped in pairs: a read of A touches every bank once
    }
    wave_sync();
    float own0[NP], own1[NP];
    v4u A[4];
#pragma unroll
    for (int f = 0; f < TL; f++) {
        if (NGU > 1 ? f % (G / 16) == 0 : f == 0) {       // the next token group
            const uint32_t *base = &L.pcq[wave][NGU > 1 ? f / (G / 16) : 0][(lane & 1) * 64];
#pragma unroll
            for (int mi = 0; mi < 4; mi++) {
                const int piece = BITS == 8 ? 8 * (mi >> 1) + 2 * q + (mi & 1) : 4 * q + mi;
                A[mi] = *reinterpret_cast<const v4u *>(base + ((piece ^ (lane & 1)) * 4));
            }
        }
        v4f c = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int mi = 0; mi < 4; mi++) {
            v4u b;
            if constexpr (BITS == 2) {
                const uint32_t w = (mi >> 1) ? kc2[f].y : kc2[f].x;
#pragma unroll
                for (int pr = 0; pr < 4; pr++) b[pr] = high_pair<2>(w, 4 * (mi & 1) + pr);
            } else if constexpr (BITS == 4) {
                const uint32_t w = word_of(kc[f], mi);
#pragma unroll
                for (int pr = 0; pr < 4; pr++) b[pr] = high_pair<4>(w, pr);
            } else {
                const uint4 &w = kc[2 * f + (mi >> 1)];
                const uint32_t w0 = (mi & 1) ? w.z : w.x, w1 = (mi & 1) ? w.w : w.y;
                b[0] = high_pair<8>(w0, 0); b[1] = high_pair<8>(w0, 1); b[2] = high_pair<8>(w1, 0); b[3] = high_pair<8>(w1, 1);
            }
            c = mfma16(A[mi], b, c);
        }
        own0[f / 4] = f % 4 == 0 || q == f % 4 ? c[0] : own0[f / 4];
        own1[f / 4] = f % 4 == 0 || q == f % 4 ? c[1] : own1[f / 4];
    }
    float s4[NP], lmax = -INFINITY;
    const int n_tok = u.nsub * (64 / BITS);
#pragma unroll
    for (int s = 0; s < NP; s++) {
        const int t = 64 * s + lane;
        float bz = bias[0], dn = down[0];
#pragma unroll
        for (int g = 1; g < NGU; g++) { bz = t >= g * G ? bias[g] : bz; dn = t >= g * G ? down[g] : dn; }
        const float dot = fmaf(own1[s], 1.0f / 2048.0f, own0[s]);
        s4[s] = t < n_tok && t < 16 * TL ? fmaf(dot, dn, bz) * scale_log2 : -INFINITY;       // past a short unit: ignored
        lmax = fmaxf(lmax, s4[s]);
    }
    rescale<G, 1>(st, 0, wave_max(lmax), lane);
#pragma unroll
    for (int s = 0; s < NP; s++)
        if (TL >= 4 || lane < 16 * TL) L.sc[wave][0][64 * s + lane] = s4[s];
    wave_sync();
}

// Softmax weights of a quantised unit as the A operand of the value products: one lane per V (token,
// group) meta word computes p * V scale, the wavefront agrees on a common power of two, and the four
// base-128 digits of the fixed-point weight go to the rows 4g..4g+3 of the operand image in LDS.
// Returns the factor that turns the recombined digit sums back into weights * codes.
template <int BITS, int G, int NWV>
__device__ __forceinline__ float iq_weights(const VRegs<G> &v, int lane, int wave,
                                            AttnLds<G, 1, NWV> &L, WaveState<1> &st) {
    constexpr int NG = kD / G;
    constexpr int MV = (256 / BITS) * NG / 64;           // meta words per lane: tokens of a unit * groups / 64
    float wv[MV], wmax = 0.0f;
#pragma unroll
    for (int jj = 0; jj < MV; jj++) {
        const int idx = 64 * jj + lane, tv = idx / NG, g = idx % NG;
        const float sV = half_bits_to_float(v.m[jj] & 0xffffu);
        const float zV = half_bits_to_float(v.m[jj] >> 16);
        const float p = fast_exp2(L.sc[wave][0][tv] - st.m[0]);       // tokens past a short unit: score -inf, p = 0
        if (g == 0) st.lsum[0] += p;
        st.z[0] = fmaf(p, BITS == 8 ? fmaf(128.0f, sV, zV) : zV, st.z[0]);   // 8 bits: the codes enter minus 128
        wv[jj] = p * sV;
        wmax = fmaxf(wmax, wv[jj]);
    }
    wmax = wave_max(wmax);
    // 2^ef <= wmax < 2^(ef+1) (ef >= -100): weight * 2^(23 - ef) < 2^24.  Rounded to the nearest integer: adding 0.5 and cutting
    // off would round twice, and from 2^23 on, where every binary32 number is an integer, make odd weights one larger
    const int ef = max((int)((__builtin_bit_cast(uint32_t, wmax) >> 23) & 255u) - 127, -100);
    const float up = __builtin_bit_cast(float, (uint32_t)(127 + kFix - ef) << 23);
    uint8_t *img = reinterpret_cast<uint8_t *>(&L.wa[wave][0][0]);
#pragma unroll
    for (int jj = 0; jj < MV; jj++) {
        const uint32_t pos = L.wpos[IQ<BITS>::BI][jj][lane];         // byte offset of digit 0 | plane shift << 16
        const uint32_t W = (uint32_t)rintf(wv[jj] * up) << (pos >> 16);
        uint8_t *dst = img + (pos & 0xffffu);
        dst[0] = (uint8_t)(W & 127u); dst[16] = (uint8_t)((W >> 7) & 127u);
        dst[32] = (uint8_t)((W >> 14) & 127u); dst[48] = (uint8_t)((W >> 21) & 127u);
    }
    wave_sync();
    return __builtin_bit_cast(float, (uint32_t)(127 + ef - kFix - IQ<BITS>::LGM) << 23);
}

// Weighted value sum of a quantised unit on the integer matrix cores.
template <int BITS, int G, int NWV>
__device__ __forceinline__ void iq_values(const VRegs<G> &v, int lane, int wave, float cw,
                                          AttnLds<G, 1, NWV> &L, WaveState<1> &st) {
    const v4i zero = {0, 0, 0, 0};
    const v4i A0 = L.wa[wave][0][lane];
    if constexpr (BITS == 2) {                           // two blocks of 64 tokens; KiB j: block j/2, column tiles 4*(j%2)..+3
        const v4i A1 = L.wa[wave][1][lane];
#pragma unroll
        for (int ct = 0; ct < 8; ct++) {
            int m[4];
            IQ<2>::planes(word_of(v.c[ct / 4], ct % 4), m);
            v4i acc = mfma_i8(A0, v4i{m[0], m[1], m[2], m[3]}, zero);
            IQ<2>::planes(word_of(v.c[2 + ct / 4], ct % 4), m);
            acc = mfma_i8(A1, v4i{m[0], m[1], m[2], m[3]}, acc);
            st.accq[0][ct] = fmaf(iq_combine(acc), cw, st.accq[0][ct]);
        }
    } else if constexpr (BITS == 4) {                    // two blocks of 32 tokens share one product
#pragma unroll
        for (int ct = 0; ct < 8; ct++) {
            int ma[2], mb[2];
            IQ<4>::planes(word_of(v.c[ct / 4], ct % 4), ma);
            IQ<4>::planes(word_of(v.c[2 + ct / 4], ct % 4), mb);
            const v4i acc = mfma_i8(A0, v4i{ma[0], ma[1], mb[0], mb[1]}, zero);
            st.accq[0][ct] = fmaf(iq_combine(acc), cw, st.accq[0][ct]);
        }
    } else {                                             // one block of 32 tokens: half of the k range is unused
#pragma unroll
        for (int ct = 0; ct < 8; ct++) {
            const uint32_t w0 = word_of(v.c[ct / 2], 2 * (ct % 2)), w1 = word_of(v.c[ct / 2], 2 * (ct % 2) + 1);
            const v4i acc = mfma_i8(A0, v4i{(int)(w0 ^ 0x80808080u), (int)(w1 ^ 0x80808080u), 0, 0}, zero);
            st.accq[0][ct] = fmaf(iq_combine(acc), cw, st.accq[0][ct]);
        }
    }
    wave_sync();
}

// Tables of the integer path for the queries of one row (REP == 1), built by the whole workgroup
// once L.qraw is in place:  iq[d] = q_d as a fixed-point integer below 2^24 in magnitude, qa = the
// eight A operands of the score products (2 bits: word 0..3 of a slot; 4 bits: word pair 0, 1;
// 8 bits: register parity 0, 1), iqpart = sum of iq over a lane's dims inside one group (times the
// common factor of the bit-width), iqscale = softmax scale (log2 domain) / fixed-point factors.
template <int G, int NWV>
__device__ __forceinline__ void iq_build_q(AttnLds<G, 1, NWV> &L, int tid, int lane, float scale_log2) {
    constexpr int NT = NWV * 64;
    const uint32_t pr = L.qraw[lane];
    float qm = fmaxf(fabsf(half_bits_to_float(pr & 0xffffu)), fabsf(half_bits_to_float(pr >> 16)));
    qm = wave_max(qm);
    const int ef = qm > 0.0f ? (int)((__builtin_bit_cast(uint32_t, qm) >> 23) & 255u) - 127 : 0;   // 2^ef <= max |q| < 2^(ef+1)
    const float up = __builtin_bit_cast(float, (uint32_t)(127 + kFix - ef) << 23);
    const uint16_t *qraw = reinterpret_cast<const uint16_t *>(L.qraw);
    if (tid < 3) L.iqscale[tid] = scale_log2 * __builtin_bit_cast(float, (uint32_t)(127 + ef - kFix - (tid == 0 ? IQ<2>::LGM : 0)) << 23);
    int s16 = 0;                                          // sums of iq over blocks of 16 dims (wavefronts 0 and 1)
    if (tid < kD) {
        s16 = L.iq[tid] = (int)rintf(half_bits_to_float(qraw[tid]) * up);
        s16 += (int)dpp_u<DPP_XOR1>((uint32_t)s16); s16 += (int)dpp_u<DPP_XOR2>((uint32_t)s16);
        s16 += (int)dpp_u<DPP_HALF_MIRROR>((uint32_t)s16); s16 += (int)dpp_u<DPP_MIRROR>((uint32_t)s16);
        if ((tid & 15) == 0) L.iqs16[tid >> 4] = s16;
    }
    __syncthreads();
    // the 16 lanes 20*xq + n of every operand are nonzero (the rest was zeroed once): one word per thread
    static_assert(NT == 512, "one operand word per thread");
    {
        const int t = tid >> 6, xq = (tid >> 4) & 3, n = (tid >> 2) & 3, m = tid & 3;
        uint32_t wd = 0u;
#pragma unroll
        for (int y = 0; y < 4; y++) {
            int d, sh = 0;                                // dim of byte 4m + y, power of two that undoes the plane's shift
            if (t < 4)      { d = (xq & 1) * 64 + t * 16 + 8 * (y & 1) + 2 * m + (y >> 1); sh = (m & 1) ? 0 : 2; }
            else if (t < 6) { d = xq * 32 + (2 * (t - 4) + (m >> 1)) * 8 + 4 * (y & 1) + 2 * (m & 1) + (y >> 1); }
            else            { d = (4 * (t - 6) + xq) * 16 + m * 4 + 2 * (y & 1) + (y >> 1); }
            const int Q = L.iq[d];
            const uint32_t mag = (uint32_t)(Q < 0 ? -Q : Q) << sh;
            int dg = (int)((mag >> (7 * n)) & 127u);
            if (Q < 0) dg = -dg;
            wd |= ((uint32_t)dg & 255u) << (8 * y);
        }
        reinterpret_cast<uint32_t *>(&L.qa[t][20 * xq + n])[m] = wd;
    }
    if (tid < 3 * 8 * 2) {
        const int bi = tid / 16, part = (tid / 2) % 8, gi = tid % 2;
        const int E = 64 >> bi;                           // codes of a slot
        const int gs = E > G ? E / G : 1;
        int sq = 0;
        if (part < (2 << bi) && gi < gs) {
            const int nb = E / gs / 16, b0 = (part * E + gi * (E / gs)) / 16;
            for (int k = 0; k < nb; k++) sq += L.iqs16[b0 + k];
        }
        L.iqpart[bi][part][gi] = (float)sq * (bi == 0 ? (float)(1 << IQ<2>::LGM) : 1.0f);
    }
}

// Positions of the weight digits in the operand image, per bit-width and (meta word, lane): byte
// offset of digit 0 (digit n follows 16n bytes later) | shift that undoes the plane's << 16.
template <int G, int NWV>
__device__ __forceinline__ void iq_build_wpos(AttnLds<G, 1, NWV> &L, int tid) {
    constexpr int NT = NWV * 64, NG = kD / G;
    for (int i = tid; i < 3 * 8 * 64; i += NT) {
        const int bi = i / 512, jj = (i / 64) % 8, l = i % 64;
        const int idx = 64 * jj + l, tv = idx / NG, g = idx % NG;
        uint32_t pos = 0;
        if (tv < (128 >> bi)) {
            int blk = 0, xq, b, sh = 0;
            if (bi == 0)      { blk = tv >> 6; const int tb = tv & 63, e = tb & 15, p = (e & 7) >> 1;
                                xq = tb >> 4; b = 4 * p + (e >> 3) + 2 * (e & 1); sh = (p & 1) ? 0 : 2; }
            else if (bi == 1) { const int tb = tv & 31, e = tb & 7, p = (e & 3) >> 1;
                                xq = tb >> 3; b = 8 * (tv >> 5) + 4 * p + (e >> 2) + 2 * (e & 1); }
            else              { const int e = tv & 3;
                                xq = tv >> 3; b = 4 * ((tv & 7) >> 2) + (e >> 1) + 2 * (e & 1); }
            pos = (uint32_t)(blk * 1024 + (16 * xq + 4 * g) * 16 + b) | ((uint32_t)sh << 16);
        }
        L.wpos[bi][jj][l] = pos;
    }
    // operand lanes / rows of the image that nobody writes stay zero
    for (int i = tid; i < 8 * 64; i += NT) L.qa[i / 64][i % 64] = v4i{0, 0, 0, 0};
    for (int i = tid; i < NWV * 2 * 64; i += NT) L.wa[i / 128][(i / 64) % 2][i % 64] = v4i{0, 0, 0, 0};
}

// ---- work distribution ----------------------------------------------------------------------
// One persistent workgroup per CU slot.  The rows are laid end to end on an axis measured in bytes to
// read (row u covers [U[u], U[u+1]): the cost of its units, added up by attn_prep_kernel from the routing
// decisions), and workgroup w of NW owns the interval [w*Utot/NW, (w+1)*Utot/NW): part of a row, or
// several rows, always the same amount of work whatever the rows' mixes of bit-widths.  With more than
// kMaxWeightedRows rows every row counts the same (U[u] = u * NW) and many rows average out.
// Short calls (a.row_wgs > 0) give every row the same number of workgroups instead, whose row is known without the costs: its
// queries and descriptors are requested first thing.  Where rows may differ (a.weigh) the costs are looked at while those are on
// their way, and intervals are taken after all if one row costs much more than the mean.
// Inside a row segment the workgroup's wavefronts draw tickets (one unit each) from counters shared by
// the workgroups of the row: a wavefront or workgroup that runs faster just takes more tickets, and
// all of them finish the row together.  The workgroup then folds its wavefronts' softmax states into
// ONE partial per row; partial slot of workgroup w in row u = w - (first workgroup that touches u).
constexpr int kMaxWeightedRows = 1024;
constexpr uint32_t kRowDone = 0xffffffffu;               // in the place of a row's workgroups: the output is written, nothing to merge
// Workgroup w's interval begins at floor(w * Utot / NW) (all 32-bit: w * (Utot % NW) < NW^2).
struct Axis {
    uint32_t Utot, NW, q, r;
    __device__ __forceinline__ Axis(uint32_t U, uint32_t nw) : Utot(U), NW(nw), q(U / nw), r(U % nw) {}
    __device__ __forceinline__ uint32_t begin(uint32_t w) const { return w * q + w * r / NW; }
    // largest w with begin(w) <= x, 0 <= x < Utot: an estimate, then exact
    __device__ __forceinline__ int owner(uint32_t x) const {
        int w = min((int)((float)x * ((float)NW / (float)Utot)), (int)NW - 1);
        while (begin((uint32_t)w) > x) w--;
        while (begin((uint32_t)w + 1u) <= x) w++;
        return w;
    }
};
// Partial slots per row.  A row's units are at most 8 times another's (16 against 2 bits), so a row
// holds at most 8/(BH+7) of all units and meets at most NW times that, plus two, intervals.
int attn_max_partials(int NW, int BH) {
    const int p = BH <= kMaxWeightedRows ? (8 * NW) / (BH + 7) + 3 : NW / BH + 2;
    return p < NW ? p : NW;
}
__device__ __forceinline__ int bits_of_expert(const AttnArgs &a, int e) {
    int b = 0;
#pragma unroll
    for (int k = 0; k < 8; k++) b = (e == k) ? a.bits_of[k] : b;
    return b;
}
__host__ __device__ __forceinline__ int lgb_of_bits(int bits) { return bits == 2 ? 1 : (bits == 4 ? 2 : (bits == 8 ? 3 : 4)); }
__host__ __device__ __forceinline__ uint32_t units_of_chunk(int N, int lgb) { return (uint32_t)((N + (256 >> lgb) - 1) >> (8 - lgb)); }

// Chunks shorter than 64 tokens share units (one query head per KV head).
__host__ __device__ inline bool gathers(int N, int rep) { return rep == 1 && N < 64; }

// Cost of a chunk: a unit costs its 8 KiB of codes plus its meta words, in steps of 512 bytes.
__host__ __device__ inline uint32_t chunk_cost(int N, int rep, int NG, int lgb) {
    const uint32_t cost = (uint32_t)(16 + (lgb < 4 ? (4 * NG) >> lgb : 0));
    if (!gathers(N, rep)) return units_of_chunk(N, lgb) * cost;
    const int sh = gather_shift(N, lgb);                 // a chunk's part of a unit, rounded
    if (sh >= 0) return cost << sh;
    const uint32_t part = (cost + (1u << (-sh - 1))) >> -sh;
    return part > 1u ? part : 1u;
}

// Chunks per row segment: at most kDescCap, and at most kUnitCap units if all of them were FP16.
__host__ __device__ inline int attn_segment_chunks(int N) { return min(kDescCap, kUnitCap / max(N / 16, 1)); }

// The costs of all rows, added up by every workgroup from the whole table of decisions (at most kWeighPieces 16-byte pieces per
// thread, in the second-level cache after the first workgroup), instead of by a kernel before this one.  A byte permute turns
// four decisions into their costs (a.cost_lut), a dot product adds them up.
constexpr int kWeighPieces = 2;
struct Weigh {
    int ppr, n;                                          // pieces per row and in all
    uint32_t magic;                                      // p / ppr = p * magic >> 20 for p < 1024
    __device__ __forceinline__ Weigh(const AttnArgs &a) : ppr((a.n_chunks + 15) / 16), n(a.BH * ppr), magic(a.weigh_magic) {}
    __device__ __forceinline__ int row(int p) const { return (int)((uint32_t)p * magic >> 20); }
};
template <int NT>
__device__ __forceinline__ void load_decisions(const AttnArgs &a, int tid, uint4 (&piece)[kWeighPieces]) {
    static_assert(kWeighPieces * NT <= 1024, "see Weigh::magic");
    const Weigh g(a);
#pragma unroll
    for (int k = 0; k < kWeighPieces; k++) {
        const int p = tid + k * NT, row = g.row(p);
        piece[k] = uint4{0u, 0u, 0u, 0u};
        if (p >= g.n) continue;
        const int c = (p - row * g.ppr) * 16;
        const uint8_t *src = a.expert + (int64_t)row * a.desc_stride + c;
        if (((reinterpret_cast<uintptr_t>(a.expert) | (uintptr_t)a.desc_stride) & 15u) == 0) piece[k] = *reinterpret_cast<const uint4 *>(src);
        else {                                           // rows that cannot be read in whole pieces
            uint32_t wv[4] = {0u, 0u, 0u, 0u};
            for (int i = 0; i < 16; i++) if (c + i < a.n_chunks) wv[i >> 2] |= (uint32_t)src[i] << (8 * (i & 3));
            piece[k] = uint4{wv[0], wv[1], wv[2], wv[3]};
        }
    }
}
// Fills cost[0 .. BH) (LDS, holding a.cost_base); true if the largest is at most a.weigh percent of the mean.
template <int NT>
__device__ __forceinline__ bool weigh_rows(const AttnArgs &a, int tid, int lane, const uint4 (&piece)[kWeighPieces], uint32_t *cost) {
    const Weigh g(a);
#pragma unroll
    for (int k = 0; k < kWeighPieces; k++) {
        const int p = tid + k * NT;
        if (p < g.n) {
            const int row = g.row(p), left = a.n_chunks - (p - row * g.ppr) * 16;   // chunks of the piece
            const uint32_t wv[4] = {piece[k].x, piece[k].y, piece[k].z, piece[k].w};
            uint32_t sum = 0u;
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const int nb = min(max(left - 4 * i, 0), 4);
                const uint32_t keep = nb == 4 ? ~0u : (1u << (8 * nb)) - 1u;
                const uint32_t sel = (wv[i] & 0x07070707u & keep) | (0x0c0c0c0cu & ~keep);      // selector 12: zero
                sum = __builtin_amdgcn_udot4(__builtin_amdgcn_perm(a.cost_lut[1], a.cost_lut[0], sel), 0x01010101u, sum, false);
            }
            atomicAdd(&cost[row], sum);
        }
    }
    __syncthreads();
    uint32_t total = 0u, most = 0u;                      // at most four rows per lane; every wavefront for itself
#pragma unroll
    for (int k = 0; k < 4; k++) { const uint32_t c = lane + 64 * k < a.BH ? cost[lane + 64 * k] : 0u; total += c; most = max(most, c); }
    return wave_max((float)most) * (float)a.BH * 100.0f <= wave_sum((float)total) * (float)a.weigh;
}

// RAGGED: the sequences of the batch have their own numbers of chunks and residual rows (a.seq_chunks,
// a.seq_tail, device arrays indexed by sequence); a.n_chunks is then the bound that sizes the segments.
// MODE: how the rows are split, a kernel each: intervals; fixed rows; fixed rows if the costs allow it, added up here or (Planned) in the
// workspace.  In one kernel every call held the registers of all of them (four heads: 39 spilled; intervals alone 30, fixed rows
// alone, which need no loop over rows, 2) and looked at its rows later: intervals, 2 x 32 ragged rows of up to 1152 tokens 24.4 ->
// 23.7 us, 40 heads of 128k tokens 114.7 -> 113.8, four sequences of 128k tokens on 8 heads x 4 queries 113.5 -> 111.6; fixed rows,
// 8 heads x 2k tokens 14.7 -> 12.8; weighed ones, 256 rows of 8k tokens in 32-token chunks 56.7 -> 56.3.  Grouped queries weigh in one
// kernel, and test a.weigh there although it is never 0: with a kernel for each way, or without the test, four heads spill 55
// registers and not 39 (four new tokens on 32 heads x 32k 48.1 us against 48.9).
// SMALL: chunks of 8, 16 or 32 tokens, see Gather (one query head per KV head) and load_v (grouped queries).  KPC: keys quantised per channel (REP == 1 only), see pc_scores.
constexpr int kIntervals = 0, kRows = 1, kRowsWeighed = 2, kRowsPlanned = 3;
template <int G, int REP, int NWV, bool RAGGED, int MODE, bool SMALL, bool KPC>
__global__ __launch_bounds__(NWV * 64) void attn_split_kernel(AttnArgs a) {
    constexpr bool ROWS = MODE != kIntervals, WEIGH = MODE == kRowsWeighed;
    static_assert(REP == 1 || MODE != kRowsPlanned, "grouped queries: kRowsWeighed, told apart by a.weigh_ws");
    static_assert(!RAGGED || !ROWS, "rows of different lengths: intervals");
    static_assert(!KPC || REP == 1, "per-channel keys: one query head per KV head");
    __shared__ AttnLds<G, REP, NWV> L;
    constexpr int NG = kD / G;
    constexpr int NT = NWV * 64;
    constexpr bool GATH = SMALL && REP == 1;             // units of several short chunks
    using KR = std::conditional_t<REP == 1, KRegs<G>, KRegsMC<G, REP>>;
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);           // wave-uniform, kept scalar
    const int w = (int)blockIdx.x, NW = (int)gridDim.x;
    const int N = a.N;

    auto bits_of = [&](int e) { return bits_of_expert(a, e); };

    const int seg_chunks = attn_segment_chunks(N);
    const int n_seg = max(1, (a.n_chunks + seg_chunks - 1) / seg_chunks);
    // ---- the workgroup's interval of the unit axis, or its part of a row (a.row_wgs workgroups per row, see AttnArgs)
    const int RW = ROWS ? a.row_wgs : 1;
    bool fixed = ROWS;
    uint32_t q_first = 0u;                               // a row's queries and the chunk descriptors of its first segment, as loaded
    uint8_t e_first[2] = {0, 0};
    uint64_t o_first[2] = {0ull, 0ull};
    const int KPT = (seg_chunks + NT - 1) / NT;          // chunks per thread of a segment (<= 2)
    auto request_row = [&](int u, int C) {
        static_assert(REP * 64 <= NT, "one query word per thread");
        // head r of the row = query r / rep_in, query head (u % Hkv) * rep_in + r % rep_in of q [B, nq, Hkv * rep_in, D]
        if (tid < REP * 64) {
            const int r = tid >> 6, bq = u / a.Hkv;
            const int64_t qrow = ((int64_t)bq * a.nq + r / a.rep_in) * (a.Hkv * a.rep_in) + (u % a.Hkv) * a.rep_in + r % a.rep_in;
            q_first = reinterpret_cast<const uint32_t *>(a.q)[qrow * 64 + (tid & 63)];
        }
        const uint8_t *erow = a.expert + (int64_t)u * a.desc_stride;
        const uint64_t *orow = a.chunk_off + (int64_t)u * a.desc_stride;
#pragma unroll
        for (int k = 0; k < 2; k++) {
            const int c = tid * KPT + k;
            if (k < KPT && c < min(C, seg_chunks)) { e_first[k] = erow[c]; o_first[k] = orow[c]; }
        }
    };
    const bool weigh = WEIGH && (REP == 1 || (a.weigh != 0 && !a.weigh_ws));    // the costs are added up here, see weigh_rows
    const bool by_counter = MODE == kIntervals || MODE == kRowsPlanned || (REP > 1 && WEIGH && a.weigh_ws);   // the workgroups of a row draw its tickets from a counter
    uint4 piece[kWeighPieces];
    if (weigh) {
        load_decisions<NT>(a, tid, piece);
        for (int i = tid; i < a.BH; i += NT) L.U[i + 1] = a.cost_base;
    }
    if (fixed) request_row(w / RW, a.n_chunks);
    bool weighted = by_counter && a.BH <= kMaxWeightedRows;
    uint32_t v0 = 0u, v1 = 0u;                           // costs of rows 2 * tid, 2 * tid + 1
    const int i0 = 2 * tid;
    if (weighted) {
        const uint32_t *row_units = a.counters + (size_t)a.BH * n_seg * kCounterStride;
        v0 = i0 < a.BH ? row_units[i0] : 0u; v1 = i0 + 1 < a.BH ? row_units[i0 + 1] : 0u;
    }
    if constexpr (REP == 1) iq_build_wpos<G, NWV>(L, tid);              // behind the loads
    if (weigh) {
        __syncthreads();
        if (!weigh_rows<NT>(a, tid, lane, piece, &L.U[1])) {            // too uneven: intervals of equal cost
            fixed = false; weighted = true;
            v0 = i0 < a.BH ? L.U[i0 + 1] : 0u; v1 = i0 + 1 < a.BH ? L.U[i0 + 2] : 0u;
            __syncthreads();
        }
    }
    if (weighted) {                                      // U = inclusive scan of the rows' unit counts, two rows per thread
        static_assert(kMaxWeightedRows <= 2 * NT, "two rows per thread");
        const uint32_t incl = wave_incl_scan(v0 + v1);
        if (lane == 63) L.wscan[wave] = incl;
        if (ROWS && tid == 0) L.uneven = 0u;
        __syncthreads();
        uint32_t excl = incl - (v0 + v1), total = 0u;
#pragma unroll
        for (int wv = 0; wv < NWV; wv++) { if (wv < wave) excl += L.wscan[wv]; total += L.wscan[wv]; }
        if (fixed && (float)max(v0, v1) * (float)a.BH * 100.0f > (float)total * (float)a.weigh) L.uneven = 1u;
        if (tid == 0) { L.U[0] = 0u; L.r0 = 0u; }
        if (i0 < a.BH) L.U[i0 + 1] = excl + v0;
        if (i0 + 1 < a.BH) L.U[i0 + 2] = excl + v0 + v1;
        __syncthreads();
        if (fixed) fixed = L.uneven == 0u;
    }
    auto Uof = [&](int u) -> uint32_t { return weighted ? L.U[u] : (uint32_t)u * (uint32_t)NW; };
    const Axis axis(Uof(a.BH), (uint32_t)NW);
    const uint32_t lo = axis.begin((uint32_t)w), hi = axis.begin((uint32_t)w + 1u);
    int r0 = fixed ? w / RW : (int)(lo / (uint32_t)NW);     // the row that holds unit lo
    if (weighted && !fixed) {
        for (int i = tid; i < a.BH; i += NT)
            if (L.U[i] <= lo && lo < L.U[i + 1]) L.r0 = (uint32_t)i;
        __syncthreads();
        r0 = (int)L.r0;
    }
    uint32_t *row_wgs = a.counters + (size_t)a.BH * n_seg * kCounterStride + a.BH;   // for the merge: workgroups per row
    const int u_end = fixed ? r0 + 1 : a.BH;
    for (int u = r0; u < u_end && (fixed || (lo < hi && Uof(u) < hi)); u++) {
        const uint32_t ub = Uof(u), ue = Uof(u + 1), ru = ue - ub;   // (fixed and not weighted: not used)
        if (ru == 0) continue;
        const uint8_t *erow = a.expert + (int64_t)u * a.desc_stride;
        const uint64_t *orow = a.chunk_off + (int64_t)u * a.desc_stride;
        int C = a.n_chunks, n_tail = a.n_tail;           // of this row
        if constexpr (RAGGED) {
            C = min(max(a.seq_chunks[u / a.Hkv], 0), a.n_chunks);
            n_tail = min(max(a.seq_tail[u / a.Hkv], 0), N - 1);
        }
        // workgroups that share this row's tickets, and the share of the row inside this workgroup's
        // interval: a workgroup whose interval covers only part of the row takes at most that part of
        // the tickets (it owes the rest of its time to the neighbouring row)
        const int wg_first = fixed ? u * RW : axis.owner(ub);
        const uint32_t P = fixed ? (uint32_t)RW : (uint32_t)(axis.owner(ue - 1u) - wg_first + 1);
        const uint32_t ov = min(hi, ue) - max(lo, ub);
        const bool whole = (lo >= ub && hi <= ue) || (ub >= lo && ue <= hi);   // the interval inside the row, or the row inside it
        if (MODE != kRows && (REP == 1 || !ROWS || a.weigh) && w == wg_first && tid == 0) row_wgs[u] = fixed && RW == 1 ? kRowDone : P;

        // ---- (a) row set-up.  One round trip to memory for everything the first units need: the raw
        //      queries, the chunk descriptors of the first segment and the first batch of tickets.  The
        //      tables derived from q are built later, while the first units' codes are on their way.
        // size of the first batch: a wavefront's worth each, but an even share of the row's tickets (estimated from its cost,
        // 16 a unit and more, without the set-up's) where the row has fewer: short rows then spread over all their compute units (not where the rows are too many to be weighted,
        // and ru is no cost)
        uint32_t b_first = (uint32_t)NWV;
        if (REP == 1 && !RAGGED && weighted && by_counter && ru < 16u * NWV * P + kRowSetupCost) {   // (grouped queries: the registers this takes are spilled in the unit loop; ragged batches of short rows: 32.0 -> 33.7 us)
            const uint32_t est = ru > kRowSetupCost ? (ru - kRowSetupCost) >> 4 : 1u;
            b_first = min((uint32_t)NWV, max(1u, (est + P - 1u) / P));
        }
        uint32_t g_first = 0u;
        {
            if (!fixed) request_row(u, C);
            const uint32_t q_row = q_first;
            if (by_counter && tid == 0) g_first = atomicAdd(a.counters + (size_t)u * n_seg * kCounterStride, b_first);
            __syncthreads();                             // LDS of the previous row is free
            if (tid < REP * 64) L.qraw[tid] = q_row;
            q_first = 0u;                                // not carried through the unit loop
        }
        constexpr bool kLateTables = REP == 1;           // grouped queries: the builders would not fit beside the loads in flight
        auto build_q_tables = [&]() {                    // by the whole workgroup; L.qraw is in place
            if (tid < REP * 64) L.qtab[tid / 64][tid % 64] = L.qraw[tid];   // raw fp16 rows: lane part = l%16 holds dims 8*part..+7
            if constexpr (REP == 1) iq_build_q<G, NWV>(L, tid, lane, a.scale_log2);
            if constexpr (REP > 1) {
                if (tid < REP * 64) {                     // a wavefront per head, its groups lie in whole rows of 16 lanes
                    const uint32_t qw = L.qraw[tid];
                    float sq = group_sum<16>(half_bits_to_float(qw & 0xffffu) + half_bits_to_float(qw >> 16));
                    if constexpr (G == 64) sq += __shfl_xor(sq, 16);
                    if ((tid & (G / 2 - 1)) == 0) L.qsumg[wave][lane / (G / 2)] = sq * kTwoM24;
                }
                for (int i = tid; i < AttnLds<G, REP, NWV>::WLS; i += NT) L.zrow[i] = 0;
                if (wave < 4) mc_build_q<G, REP>(L.qraw, lane, wave, L);
            }
            __syncthreads();
        };
        if constexpr (!kLateTables) { __syncthreads(); build_q_tables(); }

        WaveState<REP> st;
#pragma unroll
        for (int r = 0; r < REP; r++) {
            st.m[r] = -INFINITY; st.lsum[r] = 0.0f; st.z[r] = 0.0f; st.acc[r][0] = 0.0f; st.acc[r][1] = 0.0f;
#pragma unroll
            for (int ct = 0; ct < 8; ct++) st.accq[r][ct] = 0.0f;
        }
#pragma unroll
        for (int ct = 0; ct < 8; ct++) st.accA[ct] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        float qp[4];

        // ---- (b) the row in segments whose chunk descriptors (block offset | log2 bits) sit in LDS.
        //      A ticket is one unit (<= 4 KiB of K codes + 4 KiB of V codes: 128/64/32/16 tokens at
        //      2/4/8/16 bits, or 16 rows of the FP16 residual), so every ticket costs about the same.
        //      The tickets of a segment are shared by all workgroups of the row through a counter in
        //      global memory: a workgroup is granted batches of consecutive tickets (guided sizes: a
        //      share of what is left, so the last batches are small and everybody finishes together)
        //      and its wavefronts draw from the granted range through a counter in LDS.
        for (int seg = 0; seg < n_seg; seg++) {
            const int cs = seg * seg_chunks, ce = min(C, cs + seg_chunks);
            if (seg > 0) __syncthreads();                // previous segment's tables consumed
            // chunks [cs + tid*KPT, +KPT) per thread: descriptor, units per chunk, exclusive scan
            uint32_t ucnt[2] = {0u, 0u}, mine = 0u;
            unsigned long long dsc2[2] = {0ull, 0ull};    // GATH: the thread's descriptors, and its chunks per bit-width:
            uint32_t ca = 0u, cb = 0u;                    // 2 | 4 bits, 8 | 16 bits in half-words
            int cls[4] = {0, 0, 0, 0}, cpos[4], upos[5];  // GATH: chunks per bit-width, first place in desc, first unit
#pragma unroll
            for (int k = 0; k < 2; k++) {
                const int c = cs + tid * KPT + k;
                if constexpr (GATH) {
                    if (k < KPT && c < ce) {
                        const int lgb = lgb_of_bits(bits_of(seg == 0 ? e_first[k] : erow[c]));
                        dsc2[k] = (seg == 0 ? o_first[k] : orow[c]) | (unsigned long long)lgb;   // block offsets are multiples of 256
                        const uint32_t one = 1u << (16 * ((lgb - 1) & 1));
                        if (lgb <= 2) ca += one; else cb += one;
                    }
                } else if (k < KPT && c < ce) {
                    const int bits = bits_of(seg == 0 ? e_first[k] : erow[c]);
                    const int lgb = bits == 2 ? 1 : (bits == 4 ? 2 : (bits == 8 ? 3 : 4));
                    L.desc[c - cs] = (seg == 0 ? o_first[k] : orow[c]) | (unsigned long long)lgb;   // block offsets are multiples of 256
                    ucnt[k] = (uint32_t)((N + (256 >> lgb) - 1) >> (8 - lgb));
                    mine += ucnt[k];
                }
            }
            const uint32_t incl = wave_incl_scan(GATH ? ca : mine), incl_b = GATH ? wave_incl_scan(cb) : 0u;
            if (lane == 63) { L.wscan[wave] = incl; if constexpr (GATH) L.wscan2[wave] = incl_b; }
            if (tid == 0) { L.next = (uint32_t)NWV; L.limit = 0; L.done = 0; L.fetching = 0; L.g_seen = 0; L.nb = 0; }   // the first draws are fixed: wavefront v holds local ticket v
            __syncthreads();
            uint32_t pos = incl - mine, n_chunk_units = 0;
            if constexpr (GATH) {
                uint32_t pa = incl - ca, pb = incl_b - cb, ta = 0u, tb = 0u;
#pragma unroll
                for (int wv = 0; wv < NWV; wv++) {
                    if (wv < wave) { pa += L.wscan[wv]; pb += L.wscan2[wv]; }
                    ta += L.wscan[wv]; tb += L.wscan2[wv];
                }
                ta = (uint32_t)__builtin_amdgcn_readfirstlane((int)ta); tb = (uint32_t)__builtin_amdgcn_readfirstlane((int)tb);
                cls[0] = (int)(ta & 0xffffu); cls[1] = (int)(ta >> 16); cls[2] = (int)(tb & 0xffffu); cls[3] = (int)(tb >> 16);
                int at = 0, un = 0;
#pragma unroll
                for (int b = 0; b < 4; b++) {
                    const int sh = gather_shift(N, b + 1);
                    cpos[b] = at; upos[b] = un;
                    at += cls[b]; un += sh >= 0 ? cls[b] << sh : (cls[b] + (1 << -sh) - 1) >> -sh;
                }
                upos[4] = un; n_chunk_units = (uint32_t)un;
                // the block addresses ordered by bit-width
#pragma unroll
                for (int k = 0; k < 2; k++) {
                    const int lgb = (int)(dsc2[k] & 7u);
                    if (lgb) {
                        const uint32_t run = lgb <= 2 ? pa : pb;
                        const int place = (int)((run >> (16 * ((lgb - 1) & 1))) & 0xffffu)
                                        + of_width(lgb, cpos[0], cpos[1], cpos[2], cpos[3]);
                        L.desc[place] = dsc2[k] & ~7ull;
                        const uint32_t one = 1u << (16 * ((lgb - 1) & 1));
                        if (lgb <= 2) pa += one; else pb += one;
                    }
                }
            } else {
#pragma unroll
                for (int wv = 0; wv < NWV; wv++) { if (wv < wave) pos += L.wscan[wv]; n_chunk_units += L.wscan[wv]; }
                if constexpr (REP == 1) n_chunk_units = (uint32_t)__builtin_amdgcn_readfirstlane((int)n_chunk_units);
            }
            const uint32_t T = n_chunk_units + (uint32_t)(seg == n_seg - 1 ? (n_tail + 15) / 16 : 0);
            unsigned int *counter = a.counters + ((size_t)u * n_seg + seg) * kCounterStride;
            // no cap for a workgroup whose whole interval lies in this row, or that covers the whole row
            const uint32_t quota = whole || fixed || !by_counter ? 0xffffffffu : (uint32_t)((float)T * ((float)ov / (float)ru)) + 2u;   // never below T * ov / ru
            // static: nobody shares the row, or everybody's part of it is fixed; no counter in memory needed, and every wavefront
            // knows the tickets
            const bool fixed_part = REP == 1 && (P == 1u || !by_counter);
            // the latest batch of tickets that this wavefront has looked up: local tickets below c_hi are tickets c_off + t of the row;
            // no more have to be asked for as long as t + NWV < c_lim.  Looked up in LDS at every draw, the grant, the batch and a chunk's
            // first unit are reads that wait for one another before the next unit is known (256 rows of 8k tokens in 32-token chunks
            // 56.3 us a call against 54.1, 13B-shaped 128k caches no different: they wait for memory).  Grouped queries look everything
            // up, their kernels hold no register more: kept as here it is 1 to 2 % slower, with four heads in groups of 32 9 %.
            uint32_t c_hi = 0u, c_off = 0u, c_lim = 0u;
            if (P == 1u || !by_counter) {
                if (REP == 1 || tid == 0) {
                    uint32_t g0 = 0u, g1 = T;
                    if (GATH && fixed) {                 // ordered by bit-width, whose units differ by up to half in time: every P-th
                        g0 = (uint32_t)(w - wg_first); g1 = g0 + (T + P - 1u - g0) / P;
                    } else if (P > 1u && fixed) {
                        const uint32_t part = (uint32_t)(w - wg_first);
                        g0 = T * part / P; g1 = T * (part + 1u) / P;
                    } else if (P > 1u) {                 // the interval's part of the row; neighbours round the same number
                        if (lo > ub) g0 = (uint32_t)((float)T * ((float)(lo - ub) / (float)ru));
                        if (hi < ue) g1 = (uint32_t)((float)T * ((float)(hi - ub) / (float)ru));
                    }
                    if constexpr (REP == 1) { c_off = (uint32_t)__builtin_amdgcn_readfirstlane((int)g0); c_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(g1 - g0)); }
                    else { L.bl[0] = 0u; L.bg[0] = g0; L.nb = 1u; L.limit = g1 - g0; L.g_seen = T; L.done = 1u; }
                }
            } else if (seg == 0 && tid == 0) {           // the batch asked for during the row set-up
                const uint32_t granted = g_first < T ? min(b_first, T - g_first) : 0u;
                L.g_seen = g_first + b_first;
                if (granted) { L.bl[0] = 0u; L.bg[0] = g_first; L.nb = 1u; L.limit = granted; }
                if (g_first + b_first >= T || granted >= quota) L.done = 1u;
            }
#pragma unroll
            for (int k = 0; k < (GATH ? 0 : 2); k++) {
                const int c = cs + tid * KPT + k;
                if (k < KPT && c < ce) {
                    static_assert(kDescCap == 1024, "a chunk in ten bits, its units (at most 16) in six");
                    if constexpr (REP > 1) L.ustart[c - cs] = (uint16_t)pos;
                    for (uint32_t i = 0; i < ucnt[k]; i++) L.inv[pos + i] = (uint16_t)((uint32_t)(c - cs) | (REP == 1 ? i << 10 : 0u));
                    pos += ucnt[k];
                }
            }
            __syncthreads();

            if (ROWS && seg == 0) { e_first[0] = e_first[1] = 0; o_first[0] = o_first[1] = 0ull; }   // not carried through the unit loop

            // One wavefront at a time asks the row's counter for the next batch.
            auto fetch = [&]() {
                if (lane == 0) {
                    const uint32_t limit = __atomic_load_n(&L.limit, __ATOMIC_RELAXED);
                    if (!__atomic_load_n(&L.done, __ATOMIC_RELAXED)) {
                        const uint32_t seen = L.g_seen, nb = L.nb;
                        // guided batch size from the counter value seen at the previous grant (none yet:
                        // the smallest batch), so that nobody sits on a large batch when the row runs dry
                        uint32_t want = (uint32_t)NWV;
                        if (nb > 0 && T > seen) want = max(want, (T - seen) / (4u * P));
                        if (nb >= (uint32_t)kMaxBatches - 1) want = T;                 // table full: all that is left
                        want = min(want, quota - limit);                               // limit < quota here
                        const uint32_t g0 = atomicAdd(counter, want);
                        L.g_seen = g0 + want;
                        uint32_t granted = 0;
                        if (g0 < T) {
                            granted = min(want, T - g0);
                            L.bl[nb] = limit; L.bg[nb] = g0;
                            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");         // whoever sees the new nb may look at its batch before the limit grants it
                            __atomic_store_n(&L.nb, nb + 1, __ATOMIC_RELAXED);
                            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                            __atomic_store_n(&L.limit, limit + granted, __ATOMIC_RELAXED);
                        }
                        if (g0 + want >= T || limit + granted >= quota) {
                            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                            __atomic_store_n(&L.done, 1u, __ATOMIC_RELAXED);
                        }
                    }
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                    __atomic_store_n(&L.fetching, 0u, __ATOMIC_RELAXED);
                }
            };
            auto try_fetch = [&]() -> bool {             // true if this wavefront held the lock (and fetched)
                uint32_t won = 0;
                if (lane == 0) won = atomicCAS(&L.fetching, 0u, 1u) == 0u ? 1u : 0u;
                won = (uint32_t)__builtin_amdgcn_readfirstlane((int)won);
                if (won) {
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");                 // what the last holder wrote
                    fetch();
                }
                return won != 0;
            };

            // tickets: the draw for the next unit is issued when the current one is taken
            uint32_t pend = (uint32_t)wave;              // the first draw (L.next starts at NWV)
            // even shares of short chunks' units: workgroup p takes p, p + P, ..  (24 rows of 16k tokens, all bit-widths alike 42.0 -> 35.8 us
            // against shares of consecutive ones, some of them all raw rows; longer chunks lie in their order, mixed)
            const uint32_t stride = GATH && ROWS && fixed && !by_counter ? P : 1u;
            int bcur = 0;                                // batch of this wavefront's latest ticket
            // One head per KV head: the address comes from a vector register, as an atomic addition at a uniform address is combined over the
            // wavefront by the compiler, which then waits for its result on the spot.
            uint32_t *next = &L.next;
            if constexpr (REP == 1) { uint32_t vzero = 0u; asm volatile("" : "+v"(vzero)); next += vzero; }
            auto issue_draw = [&]() { if (lane == 0) pend = atomicAdd(REP == 1 ? next : &L.next, 1u); };
            constexpr uint32_t kNoTicket = 0xffffffffu;
            // one head per KV head: the row's ticket for local ticket t; waits until it is granted, or nothing is left
            auto ticket = [&](auto t) -> uint32_t {
              if constexpr (REP > 1) return kNoTicket;
              else {
                if (fixed_part) {
                    if (t >= c_hi) return kNoTicket;
                } else if (t >= c_hi || t + (uint32_t)NWV >= c_lim) {
                    uint32_t limit;
                    for (;;) {                           // wait until local ticket t is granted, or nothing is left
                        limit = (uint32_t)__builtin_amdgcn_readfirstlane((int)__atomic_load_n(&L.limit, __ATOMIC_RELAXED));
                        if (t < limit) break;
                        if (__builtin_amdgcn_readfirstlane((int)__atomic_load_n(&L.done, __ATOMIC_RELAXED))) {
                            limit = (uint32_t)__builtin_amdgcn_readfirstlane((int)__atomic_load_n(&L.limit, __ATOMIC_RELAXED));
                            if (t < limit) break;        // done is written after the last limit
                            return kNoTicket;
                        }
                        if (!try_fetch()) __builtin_amdgcn_s_sleep(2);
                    }
                    c_lim = limit;
                    if (t + (uint32_t)NWV >= limit) {
                        if (__builtin_amdgcn_readfirstlane((int)__atomic_load_n(&L.done, __ATOMIC_RELAXED))) c_lim = 0xffffffffu;   // there will be no more
                        else try_fetch();                // top up ahead of need; whoever gets the lock does it
                    }
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                    // the batch of ticket t ends where the next one begins, or at the limit read above (a batch is granted before the limit says so)
                    for (;;) {
                        const bool later = bcur + 1 < __builtin_amdgcn_readfirstlane((int)__atomic_load_n(&L.nb, __ATOMIC_RELAXED));
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");             // nb before its batch
                        c_hi = later ? (uint32_t)__builtin_amdgcn_readfirstlane((int)L.bl[bcur + 1]) : limit;
                        if (t < c_hi) break;
                        bcur++;
                    }
                    c_off = (uint32_t)__builtin_amdgcn_readfirstlane((int)(L.bg[bcur] - L.bl[bcur]));
                }
                return c_off + t * stride;
              }
            };
            auto next_unit = [&](Unit &un) -> bool {     // the pending draw becomes the next unit
                const uint32_t t = (uint32_t)__builtin_amdgcn_readfirstlane((int)pend);
                // grouped queries; one function for this wait and that of ticket() spills 141 registers and not 129 with four heads in
                // groups of 32 (32 rows of 64k tokens 206 -> 218 us)
                uint32_t limit;
                for (; REP > 1;) {                       // wait until local ticket t is granted, or nothing is left
                    limit = (uint32_t)__builtin_amdgcn_readfirstlane((int)__atomic_load_n(&L.limit, __ATOMIC_RELAXED));
                    if (t < limit) break;
                    if (__builtin_amdgcn_readfirstlane((int)__atomic_load_n(&L.done, __ATOMIC_RELAXED))) {
                        limit = (uint32_t)__builtin_amdgcn_readfirstlane((int)__atomic_load_n(&L.limit, __ATOMIC_RELAXED));
                        if (t < limit) break;            // done is written after the last limit
                        return false;
                    }
                    if (!try_fetch()) __builtin_amdgcn_s_sleep(2);
                }
                if (REP > 1 && t + (uint32_t)NWV >= limit && !__builtin_amdgcn_readfirstlane((int)__atomic_load_n(&L.done, __ATOMIC_RELAXED)))
                    try_fetch();                         // top up ahead of need; whoever gets the lock does it
                if (REP > 1) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                while (REP > 1 && bcur + 1 < __builtin_amdgcn_readfirstlane((int)__atomic_load_n(&L.nb, __ATOMIC_RELAXED))) {
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");                 // nb before its batch
                    if (t < (uint32_t)__builtin_amdgcn_readfirstlane((int)L.bl[bcur + 1])) break;
                    bcur++;
                }
                const uint32_t tk = REP == 1 ? ticket(t) : (uint32_t)__builtin_amdgcn_readfirstlane((int)(L.bg[bcur] + (t - L.bl[bcur]) * stride));
                if (REP == 1 && tk == kNoTicket) return false;
                issue_draw();
                Unit n;                                  // assigned as a whole: stores of single fields through the reference, merged across
                                                         // the branches, would keep the unit in memory
                if (GATH && tk < n_chunk_units) {
                    const int lgb = (int)tk < upos[1] ? 1 : ((int)tk < upos[2] ? 2 : ((int)tk < upos[3] ? 3 : 4));
                    const int idx = (int)tk - of_width(lgb, upos[0], upos[1], upos[2], upos[3]);
                    const int c0 = of_width(lgb, cpos[0], cpos[1], cpos[2], cpos[3]), nc = of_width(lgb, cls[0], cls[1], cls[2], cls[3]);
                    const int sh = gather_shift(N, lgb);
                    n.lgb = lgb; n.tail_rows = 1 << 20;
                    n.gath = sh < 0; n.half = lgb == 1 && N == 8; n.first = n.last = 0;
                    if (sh >= 0) {                       // a chunk is one unit, or at 16 bits one or two
                        const unsigned long long dsc = L.desc[c0 + (idx >> sh)];
                        n.kb = n.vb = a.arena + (((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(dsc >> 32)) << 32)
                                                   | (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)dsc));
                        const int t0 = (idx & ((1 << sh) - 1)) << (8 - lgb);
                        n.nvalid = min(N - t0, 256 >> lgb);
                        const uint32_t cb = (uint32_t)N << (4 + lgb), mb = lgb == 4 ? 0u : (uint32_t)N * NG * 4;
                        n.kc = (uint32_t)t0 << (4 + lgb); n.vc = n.kc + cb + mb;
                        n.km = lgb == 4 ? n.kc : cb; n.vm = lgb == 4 ? n.vc : n.vc + cb;
                    } else {
                        const int nch = min(1 << -sh, nc - (idx << -sh));
                        n.kb = n.vb = a.arena;
                        n.kc = n.km = n.vc = n.vm = 0u;
                        n.first = c0 + (idx << -sh); n.last = n.first + nch - 1;
                        n.nvalid = nch << (8 - lgb + sh);                 // NV tokens each
                    }
                    n.nsub = max((n.nvalid + (1 << (6 - lgb)) - 1) >> (6 - lgb), 1);
                } else if (!GATH && tk < n_chunk_units) {
                    const int cu = __builtin_amdgcn_readfirstlane((int)L.inv[tk]), cl = REP == 1 ? cu & (kDescCap - 1) : cu;
                    const unsigned long long dsc = L.desc[cl];
                    const uint32_t dlo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)dsc);
                    const uint32_t dhi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(dsc >> 32));
                    const int sidx = REP == 1 ? cu >> 10 : (int)tk - __builtin_amdgcn_readfirstlane((int)L.ustart[REP == 1 ? 0 : cl]);
                    const int lgb = (int)(dlo & 7u);
                    const uint8_t *blk = a.arena + (((unsigned long long)dhi << 32) | (dlo & ~0xffu));
                    const int t0 = sidx << (8 - lgb);
                    n.lgb = lgb;
                    n.nsub = max(min(4, (N - t0) >> (6 - lgb)), 1); n.nvalid = min(N - t0, 256 >> lgb); n.tail_rows = 1 << 20;
                    n.kb = blk; n.vb = blk;
                    if (lgb == 4) {
                        n.kc = (uint32_t)t0 << 8; n.vc = n.kc + ((uint32_t)N << 8);
                        n.km = n.kc; n.vm = n.kc;    // no meta: see load_k
                    } else {
                        const uint32_t cb = (uint32_t)N << (4 + lgb), mb = (uint32_t)N * NG * 4;
                        n.kc = (uint32_t)t0 << (4 + lgb);
                        n.km = KPC ? cb + (uint32_t)(t0 / G) * (kD * 4u) : cb + (uint32_t)t0 * NG * 4;
                        n.vc = n.kc + cb + mb;
                        n.vm = cb + mb + (SMALL ? (uint32_t)max(N, lgb == 1 ? 16 : 8) << (4 + lgb) : cb) + (uint32_t)t0 * NG * 4;   // 8 tokens at 2 bits: V codes of a whole slice
                    }
                } else {                                 // 16 rows of the FP16 residual
                    const int row0 = (int)(tk - n_chunk_units) * 16;
                    n.lgb = 4; n.nsub = SMALL ? min(4, N >> 2) : 4; n.nvalid = min(16, n_tail - row0); n.tail_rows = n_tail - row0;   // the buffers hold N rows
                    n.kb = reinterpret_cast<const uint8_t *>(a.K_tail) + (size_t)u * N * 256;
                    n.vb = reinterpret_cast<const uint8_t *>(a.V_tail) + (size_t)u * N * 256;
                    n.kc = n.vc = (uint32_t)row0 * 256u;
                    n.km = n.kc; n.vm = n.vc;
                    if constexpr (GATH) { n.gath = n.half = false; n.first = n.last = 0; }
                }
                un = n;
                return true;
            };

            // K is requested half a unit ahead (right after the scores of the current unit), V a
            // whole unit ahead into the buffer the current unit does not use.
            Unit cur, nxt;
            KR kr;
            VRegs<G> va, vb;
            bool have = next_unit(cur);
            auto load_keys = [&](const Unit &un) {
                if constexpr (REP == 1) load_k_iq<G, KPC, SMALL>(un, lane, kr, N, L); else load_k_mc<G, REP, SMALL>(un, lane, kr);
            };
            if (have) { load_keys(cur); load_v<G, SMALL, GATH>(cur, lane, va, N, L); }
            if (seg == 0) {                              // the q tables, behind the first units' loads
                if constexpr (kLateTables) build_q_tables();
                if constexpr (REP > 1) {
                    const int slot0 = MC<G, REP>::slot0(lane >> 4);
#pragma unroll
                    for (int n = 0; n < 4; n++) qp[n] = L.qsumg[(slot0 + n) / NG][(slot0 + n) % NG];
                }
            }
            const float scale24 = a.scale_log2 * kTwo24;
            auto step = [&](const VRegs<G> &vc, VRegs<G> &vn) {
                const bool have_next = next_unit(nxt);
                Unit picked;                              // nothing left: re-read the current unit (ignored)
                if constexpr (REP == 1) picked = either(have_next, nxt, cur);   // (grouped queries of two heads in groups of 32: 75 -> 87 us)
                const Unit &pf = REP == 1 ? picked : (have_next ? nxt : cur);
                const int lgb = cur.lgb;
                float p4[REP][4];                         // fp16 units: weights handed from scores to values
                v4u ak[4];                                // grouped queries: the score operands of this bit-width
                if constexpr (REP > 1) {
                    const int bi = min(lgb, 3) - 1;
#pragma unroll
                    for (int mi = 0; mi < 4; mi++) ak[mi] = L.qmc[bi][mi][lane];
                }
                load_v<G, SMALL, GATH>(pf, lane, vn, N, L);              // a whole unit ahead
                if constexpr (REP == 1 && KPC) {
                    if (lgb == 1)      pc_scores<2, G, NWV>(cur, kr, lane, wave, a.scale_log2, L, st);
                    else if (lgb == 2) pc_scores<4, G, NWV>(cur, kr, lane, wave, a.scale_log2, L, st);
                    else if (lgb == 3) pc_scores<8, G, NWV>(cur, kr, lane, wave, a.scale_log2, L, st);
                    else                fp16_scores<G, REP, NWV>(cur, kr, lane, wave, a.scale_log2, a.nq, a.rep_in, L, st, p4);
                    load_keys(pf);                        // half a unit ahead
                    if (lgb == 1)      iq_values<2, G, NWV>(vc, lane, wave, iq_weights<2, G, NWV>(vc, lane, wave, L, st), L, st);
                    else if (lgb == 2) iq_values<4, G, NWV>(vc, lane, wave, iq_weights<4, G, NWV>(vc, lane, wave, L, st), L, st);
                    else if (lgb == 3) iq_values<8, G, NWV>(vc, lane, wave, iq_weights<8, G, NWV>(vc, lane, wave, L, st), L, st);
                    else                fp16_values<G, REP, NWV>(cur, vc, lane, wave, L, st, p4);
                } else if constexpr (REP == 1) {
                    if (lgb == 1)      iq_scores<2, G, NWV, SMALL>(cur, kr, lane, wave, L, st);
                    else if (lgb == 2) iq_scores<4, G, NWV, SMALL>(cur, kr, lane, wave, L, st);
                    else if (lgb == 3) iq_scores<8, G, NWV, SMALL>(cur, kr, lane, wave, L, st);
                    else                fp16_scores<G, REP, NWV>(cur, kr, lane, wave, a.scale_log2, a.nq, a.rep_in, L, st, p4);
                    load_keys(pf);                        // half a unit ahead
                    if (lgb == 1)      iq_values<2, G, NWV>(vc, lane, wave, iq_weights<2, G, NWV>(vc, lane, wave, L, st), L, st);
                    else if (lgb == 2) iq_values<4, G, NWV>(vc, lane, wave, iq_weights<4, G, NWV>(vc, lane, wave, L, st), L, st);
                    else if (lgb == 3) iq_values<8, G, NWV>(vc, lane, wave, iq_weights<8, G, NWV>(vc, lane, wave, L, st), L, st);
                    else                fp16_values<G, REP, NWV>(cur, vc, lane, wave, L, st, p4);
                } else {
                    if (lgb == 1)      mc_scores<2, G, REP, NWV>(cur, kr, ak, qp, lane, wave, scale24, L, st);
                    else if (lgb == 2) mc_scores<4, G, REP, NWV>(cur, kr, ak, qp, lane, wave, scale24, L, st);
                    else if (lgb == 3) mc_scores<8, G, REP, NWV>(cur, kr, ak, qp, lane, wave, scale24, L, st);
                    else                fp16_scores<G, REP, NWV>(cur, kr, lane, wave, a.scale_log2, a.nq, a.rep_in, L, st, p4);
                    load_keys(pf);                        // half a unit ahead
                    if (lgb == 1)      value_weights<2, G, REP, NWV>(vc, lane, wave, L, st);
                    else if (lgb == 2) value_weights<4, G, REP, NWV>(vc, lane, wave, L, st);
                    else if (lgb == 3) value_weights<8, G, REP, NWV>(vc, lane, wave, L, st);
                    if (lgb == 1)      mc_value_dots<2, G, REP, NWV>(vc, lane, wave, L, st);
                    else if (lgb == 2) mc_value_dots<4, G, REP, NWV>(vc, lane, wave, L, st);
                    else if (lgb == 3) mc_value_dots<8, G, REP, NWV>(vc, lane, wave, L, st);
                    else                fp16_values<G, REP, NWV>(cur, vc, lane, wave, L, st, p4);
                }
                cur = nxt; have = have_next;
            };
            while (have) {
                step(va, vb);
                if (!have) break;
                step(vb, va);
            }
        }

        // ---- (c) fold the wavefronts' states: o[d] = acc[d] * 2^24 + sum_t p_t zero_{t,g(d)}.  The sums over lanes are DPP
        //      steps, and the matrix-core sums of a dim (held by one lane) are laid down in LDS first and picked up by the
        //      dim's lane in one read: adding them where they lie, one dependent read-modify-write per tile behind twelve
        //      dependent permutes per head, took 2.2 us of a call (one head per KV head) and 4 to 5 us (four).
        if constexpr (REP == 1) {
#pragma unroll
            for (int ct = 0; ct < 8; ct++)                // column tile ct: the lane quarter of its group holds the sums
                if ((lane >> 4) == (16 * ct) / G) L.comb[wave][0][16 * ct + (lane & 15)] = st.accq[0][ct];
        } else {
#pragma unroll
            for (int n = 0; n < 4; n++) {                 // tile row 4 * (l / 16) + n = head * NG + group
                const int slot = 4 * (lane >> 4) + n;
                if (slot < REP * NG) {
                    float *dst = &L.comb[wave][slot / NG][lane & 15];
#pragma unroll
                    for (int ct = 0; ct < 8; ct++)
                        if (slot % NG == (16 * ct) / G) dst[16 * ct] = st.accA[ct][n] * kTwo24;
                }
            }
        }
        wave_sync();
        const int d2 = 8 * (lane & 15) + 2 * (lane >> 4);        // the lane's dims of st.acc
#pragma unroll
        for (int r = 0; r < REP; r++) {
            float *dst = &L.comb[wave][r][0];
            const float lt = wave_sum(st.lsum[r]);
            float zg[NG];                                 // sums over the lanes with equal lane % NG
            strided_wave_sum<NG>(st.z[r], zg);
            float z = zg[0];
#pragma unroll
            for (int g = 1; g < NG; g++) z = d2 / G == g ? zg[g] : z;
            float2 o = *reinterpret_cast<const float2 *>(&dst[d2]);
            o.x += fmaf(st.acc[r][0], kTwo24, z); o.y += fmaf(st.acc[r][1], kTwo24, z);
            *reinterpret_cast<float2 *>(&dst[d2]) = o;
            if (lane == 0) { dst[kD] = st.m[r]; dst[kD + 1] = lt; }
        }
        __syncthreads();
        const int slot = w - wg_first;
        for (int i = tid; i < REP * kD; i += NT) {
            const int r = i / kD, d = i % kD;
            float M = -INFINITY;
#pragma unroll
            for (int wv = 0; wv < NWV; wv++) M = fmaxf(M, L.comb[wv][r][kD]);
            float num = 0.0f, den = 0.0f;
#pragma unroll
            for (int wv = 0; wv < NWV; wv++) {
                const float f = (L.comb[wv][r][kD] == -INFINITY) ? 0.0f : fast_exp2(L.comb[wv][r][kD] - M);
                num = fmaf(L.comb[wv][r][d], f, num);
                den = fmaf(L.comb[wv][r][kD + 1], f, den);
            }
            if (RW == 1 && fixed) {                       // the row's only workgroup: no merge
                const int64_t orow = ((int64_t)(u / a.Hkv) * a.nq + r / a.rep_in) * (a.Hkv * a.rep_in) + (u % a.Hkv) * a.rep_in + r % a.rep_in;
                a.out[orow * kD + d] = den > 0.0f ? num / den : 0.0f;
                continue;
            }
            float *dst = a.part + (((int64_t)u * REP + r) * a.max_partials + slot) * (kD + 2);
            dst[d] = num;
            if (d == 0) { dst[kD] = M; dst[kD + 1] = den; }
        }
    }
}

// Before the main kernel, one workgroup per row: zeroes the row's ticket counters (a kernel rather than a
// memset node, so that the call can be captured into a graph) and adds up the cost of the row's units.
__global__ __launch_bounds__(256) void attn_prep_kernel(AttnArgs a, int n_seg) {
    __shared__ uint32_t wsum[4];
    const int u = (int)blockIdx.x, tid = (int)threadIdx.x;
    for (int i = tid; i < n_seg; i += 256) a.counters[((size_t)u * n_seg + i) * kCounterStride] = 0u;
    uint32_t units = 0u;
    const uint8_t *erow = a.expert + (int64_t)u * a.desc_stride;
    const int NG = kD / a.G;
    int C = a.n_chunks, n_tail = a.n_tail;
    if (a.seq_chunks) {                                   // ragged batch: this row's own length
        C = min(max(a.seq_chunks[u / a.Hkv], 0), a.n_chunks);
        n_tail = min(max(a.seq_tail[u / a.Hkv], 0), a.N - 1);
    }
    for (int c = tid; c < C; c += 256) {
        const int lgb = lgb_of_bits(bits_of_expert(a, erow[c]));
        units += chunk_cost(a.N, a.rep, NG, lgb);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) units += __shfl_xor(units, o);
    if ((tid & 63) == 0) wsum[tid >> 6] = units;
    __syncthreads();
    if (tid == 0) {
        // plus what the set-up of a row costs a workgroup (three round trips to memory and the tables: about as long
        // as 27 units take its eight wavefronts; 40 measured best), so that many short rows are not all handed to one workgroup
        const uint32_t units_cost = wsum[0] + wsum[1] + wsum[2] + wsum[3] + 16u * (uint32_t)((n_tail + 15) / 16);
        a.counters[(size_t)a.BH * n_seg * kCounterStride + u] = units_cost ? units_cost + kRowSetupCost : 0u;
        a.counters[(size_t)a.BH * n_seg * kCounterStride + a.BH + u] = 0u;   // workgroups of the row: stays 0 for a row without tokens
    }
}
int attn_row_segments(int n_chunks, int N) {
    const int sc = attn_segment_chunks(N);
    return n_chunks > sc ? (n_chunks + sc - 1) / sc : 1;
}
size_t attn_counter_bytes(int BH, int n_chunks, int N) {
    // ticket counters, then the rows' unit counts and workgroup counts
    return ((size_t)BH * attn_row_segments(n_chunks, N) * kCounterStride + 2 * (size_t)BH) * sizeof(unsigned int);
}

// out[b, hq, :] = sum_p o_p 2^(m_p - M) / sum_p l_p 2^(m_p - M) over the partials of the row
// (one per workgroup that touched the row's KV head).  Thread (grp, d) takes the partials grp, grp + 8, ...:
// with the usual 6-8 partials per row every value is requested at once, one round trip to memory.
constexpr int kMergeGroups = 8;
__global__ __launch_bounds__(kD *kMergeGroups) void attn_merge_kernel(const float *__restrict__ part,
                                                                       float *__restrict__ out, int rep,
                                                                       const uint32_t *__restrict__ row_wgs, int fixed_wgs, int max_partials,
                                                                       unsigned int *zero_counters, int n_seg, int Hkv, int nq, int rep_in) {
    __shared__ float numl[kMergeGroups][kD];
    __shared__ float denl[kMergeGroups], ml[kMergeGroups];
    const int row = (int)blockIdx.x, tid = (int)threadIdx.x, d = tid & (kD - 1), grp = tid >> 7;
    const int u = row / rep;
    // calls that run on a plan (moqae_decode_plan) leave the ticket counters as they found them: zero
    if (zero_counters && row % rep == 0)
        for (int i = tid; i < n_seg; i += kD * kMergeGroups) zero_counters[((size_t)u * n_seg + i) * kCounterStride] = 0u;
    const uint32_t wgs = fixed_wgs ? (uint32_t)fixed_wgs : row_wgs[u];
    if (wgs == kRowDone) return;
    const int P = (int)wgs;
    const float *p0 = part + (int64_t)row * max_partials * (kD + 2);
    // this group's partials, merged on the way (online rescaling)
    float m = -INFINITY, num = 0.0f, den = 0.0f;
    for (int p = grp; p < P; p += kMergeGroups) {
        const float *pp = p0 + (int64_t)p * (kD + 2);
        const float mp = pp[kD], lp = pp[kD + 1], op = pp[d];
        const float mn = fmaxf(m, mp);
        const float fo = (m == -INFINITY) ? 0.0f : fast_exp2(m - mn), fp = (mp == -INFINITY) ? 0.0f : fast_exp2(mp - mn);   // empty partials
        num = fmaf(num, fo, op * fp);
        den = fmaf(den, fo, lp * fp);
        m = mn;
    }
    numl[grp][d] = num;
    if (d == 0) { denl[grp] = den; ml[grp] = m; }
    __syncthreads();
    if (grp == 0) {
        float M = -INFINITY;
#pragma unroll
        for (int g = 0; g < kMergeGroups; g++) M = fmaxf(M, ml[g]);
        float n = 0.0f, dn = 0.0f;
#pragma unroll
        for (int g = 0; g < kMergeGroups; g++) {
            const float f = (ml[g] == -INFINITY) ? 0.0f : fast_exp2(ml[g] - M);
            n = fmaf(numl[g][d], f, n); dn = fmaf(denl[g], f, dn);
        }
        const int rr = row % rep;                                       // out [B, nq, Hkv * rep_in, D]: head rr = query rr / rep_in
        const int64_t orow = ((int64_t)(u / Hkv) * nq + rr / rep_in) * (Hkv * rep_in) + (u % Hkv) * rep_in + rr % rep_in;
        out[orow * kD + d] = dn > 0.0f ? n / dn : 0.0f;                 // a sequence without tokens: zeros
    }
}

template <int REP> constexpr int waves_per_wg() { return 8; }

// The split kernel of a call: the instantiation for its batch shape (uniform / ragged) and chunk size.
template <int G, int REP, bool SMALL, bool KPC>
static void launch_split(const AttnArgs &a, dim3 grid, dim3 block, hipStream_t s) {
    constexpr int NWV = waves_per_wg<REP>();
    if (a.seq_chunks)         hipLaunchKernelGGL((attn_split_kernel<G, REP, NWV, true, kIntervals, SMALL, KPC>), grid, block, 0, s, a);
    else if (a.row_wgs == 0)  hipLaunchKernelGGL((attn_split_kernel<G, REP, NWV, false, kIntervals, SMALL, KPC>), grid, block, 0, s, a);
    else if (a.weigh == 0)    hipLaunchKernelGGL((attn_split_kernel<G, REP, NWV, false, kRows, SMALL, KPC>), grid, block, 0, s, a);
    else {
        if constexpr (REP == 1) {
            if (a.weigh_ws) { hipLaunchKernelGGL((attn_split_kernel<G, REP, NWV, false, kRowsPlanned, SMALL, KPC>), grid, block, 0, s, a); return; }
        }
        hipLaunchKernelGGL((attn_split_kernel<G, REP, NWV, false, kRowsWeighed, SMALL, KPC>), grid, block, 0, s, a);
    }
}
template <int G, int REP, bool KPC>
static void launch_split(const AttnArgs &a, dim3 grid, dim3 block, hipStream_t s) {
    if (a.N >= 64) launch_split<G, REP, false, KPC>(a, grid, block, s);
    else if constexpr (!(KPC && G == 64)) launch_split<G, REP, true, KPC>(a, grid, block, s);   // groups of 64 tokens do not fit a shorter chunk (checked by the caller)
}

template <int G, int REP>
static hipError_t launch_gr(const AttnArgs &a, hipStream_t s, hipEvent_t ev_begin, hipEvent_t ev_end) {
    constexpr int NWV = waves_per_wg<REP>();
    const int n_seg = attn_row_segments(a.n_chunks, a.N);
    if (a.kpc && REP != 1) return hipErrorInvalidValue;  // per-channel keys: one query head per KV head (checked by the caller)
    const bool by_counter = a.row_wgs == 0 || a.weigh_ws;   // else no costs, no counters are needed
    if (!a.planned && by_counter) {
        hipLaunchKernelGGL(attn_prep_kernel, dim3((unsigned)a.BH), dim3(256), 0, s, a, n_seg);
        hipError_t e0 = hipGetLastError();
        if (e0 != hipSuccess) return e0;
    }
    if (ev_begin && hipEventRecord(ev_begin, s) != hipSuccess) return hipErrorInvalidValue;
    const dim3 grid((unsigned)a.n_wg), block(NWV * 64);
    if constexpr (REP == 1) {
        if (a.kpc) launch_split<G, REP, true>(a, grid, block, s);
        else       launch_split<G, REP, false>(a, grid, block, s);
    } else {
        launch_split<G, REP, false>(a, grid, block, s);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (ev_end && hipEventRecord(ev_end, s) != hipSuccess) return hipErrorInvalidValue;
    if (a.row_wgs == 1 && !a.weigh) return hipSuccess;   // written by the rows' workgroups
    hipLaunchKernelGGL(attn_merge_kernel, dim3((unsigned)(a.BH * a.rep)), dim3(kD * kMergeGroups), 0, s,
                       (const float *)a.part, a.out, a.rep,
                       (const uint32_t *)(a.counters + (size_t)a.BH * n_seg * kCounterStride + a.BH), a.weigh ? 0 : a.row_wgs, a.max_partials,
                       a.planned && by_counter ? a.counters : (unsigned int *)nullptr, n_seg, a.Hkv, a.nq, a.rep_in);
    return hipGetLastError();
}

#define MOQAE_FOR_EACH_VARIANT(X) X(64, 1) X(64, 2) X(64, 4) X(64, 8) X(32, 1) X(32, 2) X(32, 4)

int attn_waves_per_wg(int rep) { (void)rep; return 8; }

// The first kernel of a decode call alone: ticket counters zeroed, the rows' costs (with a nominal residual of half
// a chunk, so that a row with any token has a cost) and zero workgroup counts left in the workspace.
hipError_t launch_attn_plan(const AttnArgs &a, hipStream_t s) {
    if (a.row_wgs > 0 && !a.weigh_ws) return hipSuccess; // calls on this cache use none of it
    hipLaunchKernelGGL(attn_prep_kernel, dim3((unsigned)a.BH), dim3(256), 0, s, a, attn_row_segments(a.n_chunks, a.N));
    return hipGetLastError();
}

bool attn_weigh(AttnArgs &a, int percent) {
    const int ppr = (a.n_chunks + 15) / 16;
    if ((int64_t)a.BH * ppr > kWeighPieces * waves_per_wg<1>() * 64 || a.BH > 4 * 64) return false;
    const int NG = kD / a.G;
    const uint32_t step = (chunk_cost(a.N, a.rep, NG, 4) + 254u) / 255u;       // costs that fit a byte
    a.weigh = percent; a.weigh_ws = 0;
    a.weigh_magic = ppr > 0 ? ((1u << 20) + (uint32_t)ppr - 1u) / (uint32_t)ppr : 0u;
    a.cost_base = (kRowSetupCost + 16u * (uint32_t)((a.n_tail + 15) / 16)) / step;
    a.cost_lut[0] = a.cost_lut[1] = 0u;
    for (int e = 0; e < 8; e++)
        a.cost_lut[e >> 2] |= ((chunk_cost(a.N, a.rep, NG, lgb_of_bits(a.bits_of[e])) + step - 1u) / step) << (8 * (e & 3));
    return true;
}

hipError_t launch_attn(const AttnArgs &a, hipStream_t s, hipEvent_t ev_begin, hipEvent_t ev_end) {
#define MOQAE_CASE(GV, RV) if (a.G == GV && a.rep == RV) return launch_gr<GV, RV>(a, s, ev_begin, ev_end);
    MOQAE_FOR_EACH_VARIANT(MOQAE_CASE)
#undef MOQAE_CASE
    return hipErrorInvalidValue;
}

}  // namespace moqae
