// moqae_quantize_pack: offset plan + group-wise quantisation and bit-packing of every chunk
// at its routed bit-width (Sec. 3.1-3.2 of the paper say only that a chunk is quantised with
// the configuration its router chose; the quantiser and the layout are defined in moqae.h).
//
//   plan_small_kernel / plan_rows_kernel / plan_kernel  block sizes -> exclusive scan in (b, h, c) order -> offsets and
//                capacity check: one thread per chunk up to 1024 chunks, then one workgroup per row when the table allows,
//                else one workgroup.
//   pack_kernel  two wavefronts per (K or V, 64 tokens, row), 32 rows each; chunks of 32 tokens and less: one (pack_wave_kernel).
//                The rows go from memory to LDS in whole lines, past the registers; then one lane per line of 64 dims takes
//                minimum and maximum with packed fp16 operations, computes scale and reciprocal once per group and then four
//                operations per code (no cross-lane step anywhere).  K words are assembled in registers (row-major layout);
//                V codes go through LDS as bytes and are gathered token-wise into the dimension-major tile layout.  Every
//                store of codes covers whole lines.
//                HBM-bound: reads 2*N*D*2 bytes, writes the block.  40 heads of 128k tokens (2.68 GB read, 0.69 GB written)
//                544 us, 6.2 TB/s, what a kernel that only moves such bytes reaches with streaming loads and stores (5.7 with
//                ordinary ones); a lane that loads its own line into registers, eight ordinary loads of 16 bytes: 588 to 595, and, where
//                8-bit codes leave in pieces of lines, 1024 against 693 for 8 bits alone.
#include "moqae_dev.hpp"
#include "moqae_kernels.hpp"
#include "pack_dev.hpp"

namespace moqae {

constexpr int kPlanThreads = 1024;

constexpr int kPlanRun = 8;                          // entries per thread and pass
constexpr int kPlanPass = kPlanThreads * kPlanRun;

// Sum over the workgroup (every thread gets it) and exclusive prefix of x over the threads.
__device__ __forceinline__ unsigned long long plan_block_scan(unsigned long long x, unsigned long long *wsum,
                                                              unsigned long long &total) {
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    unsigned long long incl = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long v = __shfl_up(incl, o);
        if (lane >= o) incl += v;
    }
    __syncthreads();                                  // wsum free
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    unsigned long long before = 0; total = 0;
#pragma unroll
    for (int wv = 0; wv < kPlanThreads / 64; wv++) { const unsigned long long v = wsum[wv]; if (wv < wave) before += v; total += v; }
    return before + incl - x;
}

// Tables of at most kPlanThreads chunks: one thread per chunk, everything read in one round trip.  A call is all latency here, a
// dependent read 1 to 2 us of it, and plan_kernel's two sweeps with their scans are five: the decode step that packs 32 chunks took
// 62.8 us with them and takes 56.5.
__global__ __launch_bounds__(kPlanThreads) void plan_small_kernel(PackArgs a) {
    __shared__ uint32_t wsum[kPlanThreads / 64];      // a wavefront's block bytes in units of 256 (below 2^20), bit 31: an expert out of range
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6, total = a.BH * a.n_chunks;
    const int u = min(tid, total - 1) / a.n_chunks, c = a.chunk_begin + min(tid, total - 1) % a.n_chunks;
    const int status = *a.status;
    const unsigned long long used = *a.arena_used;
    const int e = a.expert[(int64_t)u * a.expert_stride + c];
    int bits = 16;
#pragma unroll
    for (int k = 0; k < 8; k++) bits = e == k ? a.bits_of[k] : bits;
    const bool own = tid < total;
    const uint32_t size = own && e < a.M ? (uint32_t)((block_bytes(a.N, a.G, bits) + 255u) >> 8) : 0u;
    const uint32_t incl = wave_incl_scan(size);
    const bool wave_bad = __ballot(own && e >= a.M) != 0ull;
    if (lane == 63) wsum[wave] = incl | (wave_bad ? 0x80000000u : 0u);
    __syncthreads();
    uint32_t before = 0u, all = 0u, bad = 0u;
    for (int wv = 0; wv < (int)blockDim.x / 64; wv++) {
        const uint32_t v = wsum[wv];
        bad |= v >> 31; all += v & 0x7fffffffu;
        if (wv < wave) before += v & 0x7fffffffu;
    }
    if (status != 0) return;                          // sticky error: the call is a no-op
    if (bad) { if (tid == 0) *a.status = -1; return; }
    const unsigned long long start = (used + 255u) & ~255ull, end = start + ((unsigned long long)all << 8);
    if (end > a.capacity) { if (tid == 0) *a.status = -3; return; }
    if (own) a.chunk_off[(int64_t)u * a.off_stride + c] = start + ((unsigned long long)(before + incl - size) << 8);
    if (tid == 0) *a.arena_used = end;                // nobody else reads it: one kernel fewer than plan_rows_kernel
}

__global__ __launch_bounds__(kPlanThreads) void plan_kernel(PackArgs a) {
    __shared__ uint8_t ebuf[kPlanPass];               // a pass's expert indices, in (b, h, c) order
    __shared__ uint32_t obuf[kPlanPass];              // their block offsets relative to the pass, in units of 256 bytes
    __shared__ unsigned long long wsum[kPlanThreads / 64];
    __shared__ int bad;
    const int tid = (int)threadIdx.x;
    if (*a.status != 0) return;                       // sticky error: the call is a no-op
    if (tid == 0) bad = 0;
    __syncthreads();

    const int64_t total = (int64_t)a.BH * a.n_chunks;
    uint32_t size_of[8];                              // rounded block size per expert, in units of 256 bytes
#pragma unroll
    for (int e = 0; e < 8; e++) size_of[e] = (uint32_t)((block_bytes(a.N, a.G, a.bits_of[e]) + 255u) >> 8);
    auto size_at = [&](int e) {
        uint32_t v = 0;
#pragma unroll
        for (int k = 0; k < 8; k++) v = (e == k) ? size_of[k] : v;
        return v;
    };
    const unsigned long long start = (*a.arena_used + 255u) & ~255ull;
    // Entry j of the pass that begins at p0 is (row u, chunk cc) with u*n_chunks + cc = p0 + j; thread t
    // handles entries t, t + 1024, ... (coalesced), stepping (u, cc) without a division.
    const int step_u = kPlanThreads / a.n_chunks, step_c = kPlanThreads % a.n_chunks;

    // Sweep 1: the total size (capacity and expert check) -- nothing is written when the call fails.
    unsigned long long mine = 0, all = 0;
    {
        int64_t u = tid / a.n_chunks; int cc = tid - (int)u * a.n_chunks;
        for (int64_t i = tid; i < total; i += (int64_t)kPlanThreads * 16) {
            int e[16];
#pragma unroll
            for (int k = 0; k < 16; k++) {
                e[k] = (i + (int64_t)k * kPlanThreads < total) ? a.expert[u * a.expert_stride + a.chunk_begin + cc] : 0;
                u += step_u; cc += step_c;
                if (cc >= a.n_chunks) { cc -= a.n_chunks; u++; }
            }
#pragma unroll
            for (int k = 0; k < 16; k++)
                if (i + (int64_t)k * kPlanThreads < total) { if (e[k] >= a.M) bad = 1; else mine += size_at(e[k]); }
        }
    }
    plan_block_scan(mine, wsum, all);
    if (bad) { if (tid == 0) *a.status = -1; return; }
    if (start + (all << 8) > a.capacity) { if (tid == 0) *a.status = -3; return; }

    // Sweep 2: offsets, a pass of kPlanPass entries at a time: staged into LDS with coalesced loads,
    // thread t scans the run of kPlanRun entries from t*kPlanRun, offsets go back through LDS so
    // that the stores are coalesced too.
    unsigned long long carry = start;
    for (int64_t p0 = 0; p0 < total; p0 += kPlanPass) {
        const int n_pass = (int)min((int64_t)kPlanPass, total - p0);
        int64_t u = (p0 + tid) / a.n_chunks; int cc = (int)((p0 + tid) - u * a.n_chunks);
        int64_t at[kPlanRun];
#pragma unroll
        for (int k = 0; k < kPlanRun; k++) {
            const int j = k * kPlanThreads + tid;
            at[k] = u * a.off_stride + a.chunk_begin + cc;
            if (j < n_pass) ebuf[j] = a.expert[u * a.expert_stride + a.chunk_begin + cc];
            u += step_u; cc += step_c;
            if (cc >= a.n_chunks) { cc -= a.n_chunks; u++; }
        }
        __syncthreads();
        const int j0 = min(n_pass, tid * kPlanRun), j1 = min(n_pass, j0 + kPlanRun);
        uint32_t sz[kPlanRun], local = 0;
#pragma unroll
        for (int k = 0; k < kPlanRun; k++) { sz[k] = j0 + k < j1 ? size_at(ebuf[j0 + k]) : 0u; local += sz[k]; }
        unsigned long long pass_total;
        uint32_t pos = (uint32_t)plan_block_scan(local, wsum, pass_total);
#pragma unroll
        for (int k = 0; k < kPlanRun; k++) { if (j0 + k < j1) obuf[j0 + k] = pos; pos += sz[k]; }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPlanRun; k++) {
            const int j = k * kPlanThreads + tid;
            if (j < n_pass) a.chunk_off[at[k]] = carry + ((unsigned long long)obuf[j] << 8);
        }
        carry += pass_total << 8;
        __syncthreads();                              // ebuf, obuf free
    }
    if (tid == 0) *a.arena_used = carry;              // everybody has read it (barriers above); the end of the last block
}

// The same plan with one workgroup per (sequence, KV head) row, for tables whose rows can be read 16 bytes at a time.  Every
// workgroup adds up the sizes of the whole table (it is small and stays in L2), once as far as its own row and once in all, so that
// each knows the base of its row and the total for the capacity check without any exchange between workgroups; it then writes the
// offsets of its own row.  All latency: everything is requested at once, a byte permute turns four decisions into the low and one
// into the high bytes of their sizes and dot products add them up, and one barrier hands all sums over.  (Sizes looked up one by
// one and added to a sum per row in LDS, then scanned: 65536 chunks of 256 rows 15.4 us against 8.4, 40960 of 40 rows 11.5 against 5.8.)
constexpr int kPlanRowsMax = 1024;
// The pieces lie evenly over the wavefronts, so that a wavefront's 32-bit sum holds its share of the largest table (65535 chunks a row,
// as the entry point has it) of the largest blocks (256 raw tokens: 512 units).
static_assert((unsigned long long)kPlanRowsMax * 65535 * 512 / (kPlanThreads / 64) + 64 * 16 * 512 < (1ull << 32), "sums of the wavefronts");
__global__ __launch_bounds__(kPlanThreads) void plan_rows_kernel(PackArgs a) {
    constexpr int kWaves = kPlanThreads / 64, kBatch = 4;
    __shared__ uint32_t wall[kWaves], wbefore[kWaves], wown[2][kWaves];   // sums of the wavefronts, in units of 256 bytes
    __shared__ int wbad[kWaves], status_in;
    const int tid = (int)threadIdx.x, lane = tid & 63, u_own = (int)blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);            // wave-uniform, kept scalar
    const int C = a.n_chunks, ppr = (C + 15) / 16, n_pieces = a.BH * ppr;
    const uint8_t *own = a.expert + (int64_t)u_own * a.expert_stride + a.chunk_begin;
    uint32_t e_own = tid < C ? own[tid] : 0u;
    // One read of the status word per workgroup: workgroup 0 may set it while a workgroup that starts later is
    // reading it, and all wavefronts of a workgroup must take the same way out.  (A workgroup that still sees 0
    // reaches the same verdict as workgroup 0 by itself and writes nothing either.)
    if (tid == 0) status_in = *a.status;
    const unsigned long long start = (*a.arena_used + 255u) & ~255ull;
    auto size_at = [&](uint32_t e) {
        const uint32_t sel = 0x0c0c0c00u | (e & 7u);
        return __builtin_amdgcn_perm(a.size_lo[1], a.size_lo[0], sel) | (__builtin_amdgcn_perm(a.size_hi[1], a.size_hi[0], sel) << 8);
    };
    const uint32_t too_large = (128u - (uint32_t)a.M) * 0x01010101u;      // added to a decision >= M sets its top bit
    uint32_t all = 0u, before = 0u, bad = 0u;
    {
        int row = tid / ppr, at = tid - row * ppr;
        const int step_row = kPlanThreads / ppr, step_at = kPlanThreads % ppr;
        for (int p0 = 0; p0 < n_pieces; p0 += kPlanThreads * kBatch) {
            uint4 v[kBatch];
            int rw[kBatch], left[kBatch];
#pragma unroll
            for (int k = 0; k < kBatch; k++) {
                rw[k] = row; left[k] = row < a.BH ? C - at * 16 : 0;      // chunks of the piece
                v[k] = uint4{0u, 0u, 0u, 0u};
                const uint8_t *src = a.expert + (int64_t)row * a.expert_stride + a.chunk_begin + at * 16;
                if (left[k] >= 16) v[k] = *reinterpret_cast<const uint4 *>(src);
                else if (left[k] > 0) {                                   // the last chunks of a row
                    uint32_t wv[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                    for (int i = 0; i < 15; i++) if (i < left[k]) wv[i >> 2] |= (uint32_t)src[i] << (8 * (i & 3));
                    v[k] = uint4{wv[0], wv[1], wv[2], wv[3]};
                }
                row += step_row; at += step_at;
                if (at >= ppr) { at -= ppr; row++; }
            }
#pragma unroll
            for (int k = 0; k < kBatch; k++) {
                if (p0 + k * kPlanThreads + wave * 64 >= n_pieces) break;
                const uint32_t wv[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
                uint32_t lo = 0u, hi = 0u;
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const int nb = min(max(left[k] - 4 * i, 0), 4);
                    const uint32_t keep = nb == 4 ? ~0u : (1u << (8 * nb)) - 1u;
                    bad |= (wv[i] | (wv[i] + too_large)) & 0x80808080u & keep;
                    const uint32_t sel = (wv[i] & 0x07070707u & keep) | (0x0c0c0c0cu & ~keep);      // selector 12: zero
                    lo = __builtin_amdgcn_udot4(__builtin_amdgcn_perm(a.size_lo[1], a.size_lo[0], sel), 0x01010101u, lo, false);
                    hi = __builtin_amdgcn_udot4(__builtin_amdgcn_perm(a.size_hi[1], a.size_hi[0], sel), 0x01010101u, hi, false);
                }
                const uint32_t sum = lo + (hi << 8);
                all += sum; before += rw[k] < u_own ? sum : 0u;
            }
        }
    }
    uint32_t sz = tid < C ? size_at(e_own) : 0u;
    uint32_t incl = wave_incl_scan(sz);
    const uint32_t wave_all = wave_incl_scan(all), wave_before = wave_incl_scan(before);
    const bool wave_bad = __ballot(bad != 0u) != 0ull;
    if (lane == 63) { wall[wave] = wave_all; wbefore[wave] = wave_before; wown[0][wave] = incl; wbad[wave] = wave_bad; }
    __syncthreads();
    if (status_in != 0) return;                       // sticky error: the call is a no-op
    unsigned long long total = 0ull, carry = start;
    int any_bad = 0;
#pragma unroll
    for (int wv = 0; wv < kWaves; wv++) { total += wall[wv]; carry += (unsigned long long)wbefore[wv] << 8; any_bad |= wbad[wv]; }
    // the verdict is the same in every workgroup
    if (any_bad) { if (tid == 0 && u_own == 0) *a.status = -1; return; }
    if (start + (total << 8) > a.capacity) { if (tid == 0 && u_own == 0) *a.status = -3; return; }
    uint64_t *off = a.chunk_off + (int64_t)u_own * a.off_stride + a.chunk_begin;
    for (int c0 = 0, buf = 0;; buf ^= 1) {            // 1024 chunks a pass
        uint32_t pos = incl - sz, pass = 0u;
#pragma unroll
        for (int wv = 0; wv < kWaves; wv++) { const uint32_t v = wown[buf][wv]; if (wv < wave) pos += v; pass += v; }
        if (c0 + tid < C) off[c0 + tid] = carry + ((unsigned long long)pos << 8);
        carry += (unsigned long long)pass << 8;
        c0 += kPlanThreads;
        if (c0 >= C) break;
        sz = c0 + tid < C ? size_at(own[c0 + tid]) : 0u;
        incl = wave_incl_scan(sz);
        if (lane == 63) wown[buf ^ 1][wave] = incl;   // the pass before the last is read: see the barrier of the last
        __syncthreads();
    }
}

// ---- the pack kernels: 32 rows of K or V to a wavefront ----
// A row is two lines of 128 bytes, a lane owns a line: 64 dims, one group of 64 or two of 32.  A wavefront's lines go straight
// to its region of LDS (16 bytes per lane and load, no register holds them on their way), eight whole lines per load
// instruction: piece p of line l in slot 8 l + (p ^ l % 8), so that a lane that reads its line piece by piece shares no bank
// with the seven lanes beside it.
constexpr int kLine = 128, kRegionRows = 32, kRegion = kRegionRows * 2 * kLine;
// Where a call reads much (stream), a refused one requests nothing: lines_request then returns false.  The status word is read
// here, right before the loads, or by a caller that passes no pointer.  2.6 M rows in 128-token chunks: refused 38 us, 194 with the
// look behind the loads; accepted 264 and 279.  Below, the look comes when the lines are there: before them it would hold back accepted calls
// (524288 rows, 32-token chunks at 8 bits 68 -> 73 us), and a refused one takes 44 us (63 just below the line), 11 without its loads.
__device__ __forceinline__ bool lines_request(const uint16_t *rows, int64_t stride_s, int n_rows, bool stream, uint8_t *region, int lane,
                                              const int32_t *status = nullptr) {
    typedef const __attribute__((address_space(1))) uint32_t *global_p;
    typedef __attribute__((address_space(3))) uint32_t *lds_p;
    const uint16_t *p = rows + (int64_t)(lane >> 4) * stride_s + ((lane >> 3) & 1) * 64 + ((lane & 7) ^ (lane >> 3)) * 8;
    if (stream) {
        if (status != nullptr && *status != 0) return false;
#pragma unroll
        for (int j = 0; j < kRegionRows / 4; j++)         // four rows a load; the last argument 2: streaming
            if (4 * j < n_rows) __builtin_amdgcn_global_load_lds((global_p)(p + (int64_t)(4 * j) * stride_s), (lds_p)(region + j * 1024), 16, 0, 2);
    } else {
#pragma unroll
        for (int j = 0; j < kRegionRows / 4; j++)
            if (4 * j < n_rows) __builtin_amdgcn_global_load_lds((global_p)(p + (int64_t)(4 * j) * stride_s), (lds_p)(region + j * 1024), 16, 0, 0);
    }
    return true;
}
__device__ __forceinline__ void lines_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void line_read(const uint8_t *region, int lane, int n_lines, uint32_t (&w)[32]) {
    const uint4 *buf = reinterpret_cast<const uint4 *>(region) + min(lane, n_lines - 1) * 8;
#pragma unroll
    for (int p = 0; p < 8; p++) { const uint4 t = buf[p ^ (lane & 7)]; w[4 * p] = t.x; w[4 * p + 1] = t.y; w[4 * p + 2] = t.z; w[4 * p + 3] = t.w; }
}

// A lane's line at BITS bits: meta words to meta_w, V codes to the staging rows in the region (over the lines, which are in
// registers by now), K codes to kw.
template <int G, int BITS, bool isV>
__device__ __forceinline__ void pack_line(const uint32_t (&w)[32], int lane, uint32_t *meta_w, uint8_t *region, uint32_t (&kw)[2 * BITS]) {
    constexpr int NI = 64 / G;                            // groups of a line
    uint32_t mw[NI];
#pragma unroll
    for (int i = 0; i < NI; i++)
        pack_item<G, BITS, true>(&w[i * (G / 2)], isV, &mw[i], &kw[i * (2 * BITS / NI)],
                                 reinterpret_cast<uint32_t *>(region + (lane >> 1) * kVRow + (lane & 1) * 64 + i * G));
    if constexpr (NI == 1) nt_store(meta_w, mw[0]);
    else                   nt_store(reinterpret_cast<uint2 *>(meta_w), uint2{mw[0], mw[NI - 1]});
}
// The K codes of the wavefront's lines, consecutive bytes at dst: a lane's own 16, 32 or 64 of them go through LDS, from where they
// leave 1 KiB per store.  (Stored by their lanes in 16-byte pieces 64 bytes apart, 8-bit K codes took an all-8-bit call of 5.2 M rows
// to 1024 us, 693 so.)  Piece q of lane l in slot PPL l + (q ^ l / (8 / PPL) % PPL): both ways every bank once.
template <int BITS>
__device__ __forceinline__ int k_slot(int l, int q) {
    constexpr int PPL = BITS / 2;
    return l * PPL + (q ^ ((l / (8 / PPL)) & (PPL - 1)));
}
template <int BITS>
__device__ __forceinline__ void k_stage(const uint32_t (&kw)[2 * BITS], int lane, uint8_t *region) {
#pragma unroll
    for (int q = 0; q < BITS / 2; q++) reinterpret_cast<uint4 *>(region)[k_slot<BITS>(lane, q)] = uint4{kw[4 * q], kw[4 * q + 1], kw[4 * q + 2], kw[4 * q + 3]};
}
template <int G, int BITS>
__device__ __forceinline__ void pack_k_lines(const uint32_t (&w)[32], int lane, uint32_t *codes_w, uint32_t *meta_w, uint8_t *region) {
    uint32_t kw[2 * BITS];
    pack_line<G, BITS, false>(w, lane, meta_w + lane * (64 / G), region, kw);
    uint4 *dst = reinterpret_cast<uint4 *>(codes_w) + lane;
    if constexpr (BITS == 2) nt_store(dst, uint4{kw[0], kw[1], kw[2], kw[3]});
    else {
        k_stage<BITS>(kw, lane, region);
        wave_lds_sync();
        constexpr int PPL = BITS / 2;
#pragma unroll
        for (int k = 0; k < PPL; k++) nt_store(dst + 64 * k, reinterpret_cast<const uint4 *>(region)[k_slot<BITS>((64 * k + lane) / PPL, lane & (PPL - 1))]);
    }
}
template <int G, int BITS>
__device__ __forceinline__ void pack_v_lines(const uint32_t (&w)[32], int lane, uint32_t *meta_w, uint8_t *region) {
    uint32_t unused[2 * BITS];
    pack_line<G, BITS, true>(w, lane, meta_w + lane * (64 / G), region, unused);
}

// Keys quantised per channel: the wavefront's 32 rows, a group of 32 tokens or half of one of 64 (whose other half is the other
// wavefront's); codes_w and meta_w: those of the part's first row and group.  The lines come through LDS as the others do and the
// codes leave in whole lines: 40 heads of 64k tokens, groups of 64, routed and packed 382 us; a wavefront per group, its rows' words
// loaded into 64 registers and every code word stored by its lane, 416.
template <int G, int BITS>
__device__ __forceinline__ void pack_k_columns(int lane, int wave, uint8_t *region, uint8_t *lds, uint32_t *codes_w, uint32_t *meta_w) {
    uint32_t w[kRegionRows], mnp, mxp, metaw[2];
    float nmn[2], inv[2];
    const uint32_t *words = reinterpret_cast<const uint32_t *>(region);
#pragma unroll
    for (int r = 0; r < kRegionRows; r++) {               // word l of row r: piece l % 32 / 4 of line 2r + l / 32
        const int line = 2 * r + (lane >> 5);
        w[r] = words[(line * 8 + (((lane >> 2) & 7) ^ (line & 7))) * 4 + (lane & 3)];
    }
    column_range<kRegionRows>(w, mnp, mxp);
    if constexpr (G == 64) {
        __syncthreads();                                  // the lines are in registers
        uint2 *range = reinterpret_cast<uint2 *>(lds + kRegion / 2);     // behind the codes
        range[wave * 64 + lane] = uint2{mnp, mxp};
        __syncthreads();
        const uint2 other = range[(wave ^ 1) * 64 + lane];
        mnp = pk_min_f16(mnp, other.x); mxp = pk_max_f16(mxp, other.y);
    }
    column_scale<BITS>(mnp, mxp, nmn, inv, metaw);
    if (G == 32 || wave == 0) nt_store(reinterpret_cast<uint2 *>(meta_w + (G == 32 ? wave * kD : 0) + 2 * lane), uint2{metaw[0], metaw[1]});
    if constexpr (G == 32) wave_lds_sync();
    column_codes<BITS, kRegionRows, true>(w, nmn, inv, reinterpret_cast<uint32_t *>(region), lane);
    wave_lds_sync();
    uint4 *dst = reinterpret_cast<uint4 *>(codes_w + wave * kRegionRows * (kD * BITS / 32)) + lane;
#pragma unroll
    for (int k = 0; k < BITS / 2; k++) nt_store(dst + 64 * k, reinterpret_cast<const uint4 *>(region)[64 * k + lane]);
}

// Rows [r0, r0 + 32 n_waves) of K or V of a chunk -> its block, by n_waves wavefronts (1: a chunk of 32 tokens; 2) whose regions
// follow one another in `lds`; `wave` is this one's index.
template <int G, bool KPC>
__device__ __forceinline__ void pack_part(const PackArgs &a, int isV, int c, int u, int r0, int n_waves, int wave, int lane, uint8_t *lds) {
    constexpr int NG = kD / G;
    const int N = a.N;
    uint8_t *region = lds + wave * kRegion;
    const uint16_t *src = (isV ? a.V : a.K) + (int64_t)(u / a.Hkv) * a.stride_b + (int64_t)(u % a.Hkv) * a.stride_h + ((int64_t)c * N + r0) * a.stride_s;
    // on their way before the decision and the offset are looked at
    if (!lines_request(src + (int64_t)(wave * kRegionRows) * a.stride_s, a.stride_s, kRegionRows, a.stream, region, lane, a.status)) return;
    const int status = *a.status;
    const int bits = a.bits_of[a.expert[(int64_t)u * a.expert_stride + c] & 7];   // an expert out of range has set the status
    uint8_t *blk = a.arena + a.chunk_off[(int64_t)u * a.off_stride + c];
    lines_wait();                                         // also where the call is a no-op: LDS is not given back under a load
    if (status != 0) return;
    wave_lds_sync();

    const int row0 = r0 + wave * kRegionRows;
    if (bits == 16) {                                     // FP16 expert: rows copied verbatim
        uint4 *dst = reinterpret_cast<uint4 *>(blk + (isV ? (size_t)N * kD * 2 : 0)) + row0 * 16 + lane;
        const uint4 *buf = reinterpret_cast<const uint4 *>(region) + (lane ^ (lane >> 3));
#pragma unroll
        for (int j = 0; j < kRegionRows / 4; j++) nt_store(dst + 64 * j, buf[64 * j]);
        return;
    }
    uint8_t *area = blk + (isV ? (size_t)N * kD * bits / 8 + (size_t)N * NG * 4 : 0);
    uint32_t *codes_w = reinterpret_cast<uint32_t *>(area) + (size_t)r0 * (kD * bits / 32);
    uint32_t *meta_w = reinterpret_cast<uint32_t *>(area + (size_t)N * kD * bits / 8) + r0 * NG;
    if (KPC && !isV) {                                    // keys per channel: 32 rows of a group to a wavefront
        if (bits == 2)      pack_k_columns<G, 2>(lane, wave, region, lds, codes_w, meta_w);
        else if (bits == 4) pack_k_columns<G, 4>(lane, wave, region, lds, codes_w, meta_w);
        else                pack_k_columns<G, 8>(lane, wave, region, lds, codes_w, meta_w);
        return;
    }
    uint32_t w[32];
    line_read(region, lane, 64, w);
    wave_lds_sync();
    meta_w += wave * kRegionRows * NG;
    if (!isV) {
        codes_w += wave * kRegionRows * (kD * bits / 32);
        if (bits == 2)      pack_k_lines<G, 2>(w, lane, codes_w, meta_w, region);
        else if (bits == 4) pack_k_lines<G, 4>(w, lane, codes_w, meta_w, region);
        else                pack_k_lines<G, 8>(w, lane, codes_w, meta_w, region);
        return;
    }
    if (bits == 2)      pack_v_lines<G, 2>(w, lane, meta_w, region);
    else if (bits == 4) pack_v_lines<G, 4>(w, lane, meta_w, region);
    else                pack_v_lines<G, 8>(w, lane, meta_w, region);
    if (n_waves > 1) __syncthreads(); else wave_lds_sync();
    const int rows = n_waves * kRegionRows;               // whole token blocks of the V layout
    v_gather(rows, bits, rows, codes_w, lds, wave * 64 + lane, n_waves * 64, kRegion);
}

// 32 / N chunks of 8 or 16 tokens, one after the other in memory: K or V of the chunks [c, c + n) by one wavefront, every lane at its
// chunk's bit-width.  (A wavefront per chunk leaves half or three quarters of its lanes without a line.)  The codes of all widths are
// made in one pass, as bytes.  1.3 M rows of the usual mix, routed and packed: 8 tokens 227 us (343 with a wavefront per chunk), 16
// tokens 194 (217).  One chunk of 16 tokens a row, whose lanes then have 64 dims each and not 32, is slower: 32 rows 8.2 us (7.4).
template <int G>
__device__ __forceinline__ void pack_chunks(const PackArgs &a, int isV, int c, int n, int u, int lane, uint8_t *region) {
    constexpr int NG = kD / G;
    const int status = *a.status, N = a.N, lines = 2 * N, n_lines = n * lines;
    const uint16_t *src = (isV ? a.V : a.K) + (int64_t)(u / a.Hkv) * a.stride_b + (int64_t)(u % a.Hkv) * a.stride_h + (int64_t)c * N * a.stride_s;
    if (a.stream && status != 0) return;                  // early: lines_request's late look costs these kernels 2 %
    lines_request(src, a.stride_s, n * N, a.stream, region, lane);
    const int mine = min(lane / lines, n - 1);            // the lane's chunk
    const int e = a.expert[(int64_t)u * a.expert_stride + c + mine];
    const unsigned long long off = a.chunk_off[(int64_t)u * a.off_stride + c + mine];
    int bits = 16;
#pragma unroll
    for (int k = 0; k < 8; k++) bits = e == k ? a.bits_of[k] : bits;
    if (lane >= n_lines) bits = 0;
    lines_wait();
    if (status != 0) return;
    wave_lds_sync();
    auto area_of = [&](uint8_t *blk, int b) { return blk + (isV ? (size_t)N * kD * b / 8 + (size_t)N * NG * 4 : 0); };
    auto uniform = [&](int j, int &b, uint8_t *&blk) {    // of chunk j, on the scalar unit
        b = __builtin_amdgcn_readlane(bits, j * lines);
        blk = a.arena + (((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(off >> 32), j * lines) << 32)
                         | (uint32_t)__builtin_amdgcn_readlane((int)off, j * lines));
    };
    for (int j = 0; j < n; j++) {                         // FP16 expert: rows copied verbatim
        int b; uint8_t *blk;
        uniform(j, b, blk);
        if (b != 16) continue;
        uint4 *dst = reinterpret_cast<uint4 *>(blk + (isV ? (size_t)N * kD * 2 : 0)) + lane;
        const uint4 *buf = reinterpret_cast<const uint4 *>(region) + j * lines * 8 + (lane ^ (lane >> 3));
        for (int i = 0; i < N / 4; i++) nt_store(dst + 64 * i, buf[64 * i]);
    }
    if (__ballot(bits != 0 && bits != 16) == 0ull) return;   // raw chunks alone (32 rows of one chunk 7.4 -> 6.4 us a call)
    uint32_t w[32];
    line_read(region, lane, n_lines, w);
    wave_lds_sync();
    // the codes as bytes, whatever the width
    constexpr int NI = 64 / G;                            // groups of a line
    uint32_t bytes[16], mw[NI];
    const float qmax = (float)((1 << (bits & 15)) - 1);
#pragma unroll
    for (int i = 0; i < NI; i++) {
        float nmn, inv;
        mw[i] = group_scale<G>(&w[i * (G / 2)], qmax, nmn, inv);
#pragma unroll
        for (int k = 0; k < G / 4; k++) bytes[i * (G / 4) + k] = four_codes(&w[i * (G / 2)], 4 * k, nmn, inv);
    }
    uint8_t *own = area_of(a.arena + off, bits);
    const int line = lane - mine * lines;                 // in its chunk
    if (bits != 0 && bits != 16) {
        uint32_t *meta_w = reinterpret_cast<uint32_t *>(own + (size_t)(isV ? v_token_room(N, bits) : N) * kD * bits / 8) + line * NI;
        if constexpr (NI == 1) nt_store(meta_w, mw[0]);
        else                   nt_store(reinterpret_cast<uint2 *>(meta_w), uint2{mw[0], mw[NI - 1]});
    }
    if (isV) {
        if (lane < n_lines) {
            uint32_t *row = reinterpret_cast<uint32_t *>(region + (lane >> 1) * kVRow + (lane & 1) * 64);
#pragma unroll
            for (int k = 0; k < 16; k++) row[k] = bytes[k];
        }
    } else {
        // a code word from the bytes: the codes 2k and 2k + 1 share the shift bits * k
        auto pair = [&](int k) { return __builtin_amdgcn_perm(0u, bytes[k >> 1], (k & 1) ? 0x0c030c02u : 0x0c010c00u); };
        if (bits == 2) {
            uint32_t kw[4];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                kw[i] = pair(8 * i);
#pragma unroll
                for (int k = 1; k < 8; k++) kw[i] |= pair(8 * i + k) << (2 * k);
            }
            nt_store(reinterpret_cast<uint4 *>(own) + line, uint4{kw[0], kw[1], kw[2], kw[3]});
        } else if (bits == 4) {                           // lanes of different widths stage their codes in places that do not meet: 4 bits
            uint32_t kw[8];                               // the first 2 KiB, 8 bits the upper half
#pragma unroll
            for (int i = 0; i < 8; i++) {
                kw[i] = pair(4 * i);
#pragma unroll
                for (int k = 1; k < 4; k++) kw[i] |= pair(4 * i + k) << (4 * k);
            }
            k_stage<4>(kw, lane, region);
        } else if (bits == 8) {
            uint32_t kw[16];
#pragma unroll
            for (int i = 0; i < 16; i++) kw[i] = pair(2 * i) | (pair(2 * i + 1) << 8);
            k_stage<8>(kw, lane, region + kRegion / 2);
        }
    }
    wave_lds_sync();
    for (int j = 0; j < n; j++) {
        int b; uint8_t *blk;
        uniform(j, b, blk);
        if (b == 16 || (!isV && b == 2)) continue;
        uint8_t *area = area_of(blk, b);
        if (isV) v_gather(N, b, v_token_room(N, b), reinterpret_cast<uint32_t *>(area), region + j * N * kVRow, lane, 64);
        else {
            uint4 *dst = reinterpret_cast<uint4 *>(area) + lane;
            if (b == 4) { if (lane < lines * 2) nt_store(dst, reinterpret_cast<const uint4 *>(region)[k_slot<4>(j * lines + lane / 2, lane & 1)]); }
            else for (int k = 0; k * 64 < lines * 4; k++)
                nt_store(dst + 64 * k, reinterpret_cast<const uint4 *>(region + kRegion / 2)[k_slot<8>(j * lines + (64 * k + lane) / 4, lane & 3)]);
        }
    }
}

// The new end of the arena = the end of the last block in (b, h, c) order.  plan_rows_kernel cannot move the counter, its
// workgroups read it at different times; nobody reads it here.
__device__ __forceinline__ void move_arena_end(const PackArgs &a) {
    if (*a.status != 0) return;
    const int64_t lu = a.BH - 1, lc = a.chunk_begin + a.n_chunks - 1;
    const unsigned long long sz = (block_bytes(a.N, a.G, a.bits_of[a.expert[lu * a.expert_stride + lc]]) + 255u) & ~255ull;
    *a.arena_used = a.chunk_off[lu * a.off_stride + lc] + sz;
}

// Chunks of 64 tokens and more: a workgroup of two wavefronts per (K or V, 64 tokens, chunk, row).
constexpr int kPartRows = 2 * kRegionRows;
template <int G, bool KPC>
__global__ __launch_bounds__(kPartRows * 2) void pack_kernel(PackArgs a) {
    __shared__ uint4 lds[2 * kRegion / 16];
    const int isV = (int)blockIdx.x & 1;              // K and V of a chunk side by side in launch order
    const int c = a.chunk_begin + (int)blockIdx.y, u = (int)blockIdx.z, tid = (int)threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (blockIdx.x + blockIdx.y + blockIdx.z == 0 && tid == 0) move_arena_end(a);
    pack_part<G, KPC>(a, isV, c, u, ((int)blockIdx.x >> 1) * kPartRows, 2, wave, tid & 63, reinterpret_cast<uint8_t *>(lds));
}

// Short chunks: a wavefront per (K or V, 32 tokens, row), four of them in a workgroup.  SEVERAL: chunks of 8 and 16 tokens.
template <int G, bool KPC, bool SEVERAL>
__global__ __launch_bounds__(kPackThreads) void pack_wave_kernel(PackArgs a) {
    __shared__ uint4 lds[kPackThreads / 64][kRegion / 16];
    const int lane = (int)threadIdx.x & 63, u = (int)blockIdx.y;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int side = (int)blockIdx.x * (kPackThreads / 64) + wave, isV = side & 1;       // K and V side by side
    const int per = SEVERAL ? kRegionRows / a.N : 1, c0 = (side >> 1) * per;
    if (blockIdx.x + blockIdx.y == 0 && threadIdx.x == 0) move_arena_end(a);
    if (c0 >= a.n_chunks) return;
    uint8_t *region = reinterpret_cast<uint8_t *>(&lds[wave][0]);
    if constexpr (!SEVERAL) pack_part<G, KPC>(a, isV, a.chunk_begin + c0, u, 0, 1, 0, lane, region);
    else                    pack_chunks<G>(a, isV, a.chunk_begin + c0, min(per, a.n_chunks - c0), u, lane, region);
}

// The new token's K and V rows (fp16 [B*Hkv, D]) into row n_tail of the FP16 residual buffers ([B*Hkv, N, D]): one
// kernel for both, one 16-byte piece per thread.
__global__ __launch_bounds__(32) void append_tail_kernel(const uint4 *__restrict__ k_new, const uint4 *__restrict__ v_new,
                                                         uint4 *__restrict__ K_tail, uint4 *__restrict__ V_tail, int N, int n_tail) {
    const int u = (int)blockIdx.x, t = (int)threadIdx.x;   // 16 pieces of K, 16 of V
    const size_t dst = ((size_t)u * N + n_tail) * (kD / 8) + (t & 15);
    if (t < 16) K_tail[dst] = k_new[(size_t)u * (kD / 8) + t];
    else        V_tail[dst] = v_new[(size_t)u * (kD / 8) + (t & 15)];
}
hipError_t launch_append_tail(const void *k_new, const void *v_new, void *K_tail, void *V_tail, int BH, int N, int n_tail,
                              hipStream_t s) {
    hipLaunchKernelGGL(append_tail_kernel, dim3((unsigned)BH), dim3(32), 0, s, static_cast<const uint4 *>(k_new),
                       static_cast<const uint4 *>(v_new), static_cast<uint4 *>(K_tail), static_cast<uint4 *>(V_tail), N, n_tail);
    return hipGetLastError();
}

hipError_t launch_pack(PackArgs a, hipStream_t s) {
    if (a.n_chunks <= 0 || a.BH <= 0) return hipSuccess;
    a.size_lo[0] = a.size_lo[1] = a.size_hi[0] = a.size_hi[1] = 0u;
    for (int e = 0; e < 8; e++) {
        const uint32_t size = (uint32_t)((block_bytes(a.N, a.G, a.bits_of[e]) + 255u) >> 8);
        a.size_lo[e >> 2] |= (size & 255u) << (8 * (e & 3)); a.size_hi[e >> 2] |= (size >> 8) << (8 * (e & 3));
    }
    // Streaming loads from 384 MiB of K and V on: 419 MB (40 heads x 20k tokens, 128-token chunks) routed and packed 124 us against 130, 503 MB 145
    // against 156, 1342 MB 364 against 394.  Below, ordinary loads keep what the last-level cache (256 MiB) holds of K from the routing,
    // and of both from whoever wrote them: 336 MB 98 us against 101, 252 MB 76 against 79.  (Given decisions and keys that nobody has
    // just read: 336 MB 78 against 72, 252 MB 53 against 56.)
    a.stream = (int64_t)a.BH * a.n_chunks * a.N * (2 * kD * 2) > (384ll << 20);
    const bool rows_ok = a.BH <= kPlanRowsMax &&
                         ((reinterpret_cast<uintptr_t>(a.expert + a.chunk_begin) | (uintptr_t)a.expert_stride) & 15u) == 0;
    const int64_t total = (int64_t)a.BH * a.n_chunks;
    const bool small = total <= kPlanThreads, rows = rows_ok && !small;
    if (small)     hipLaunchKernelGGL(plan_small_kernel, dim3(1), dim3((unsigned)((total + 63) / 64 * 64)), 0, s, a);
    else if (rows) hipLaunchKernelGGL(plan_rows_kernel, dim3((unsigned)a.BH), dim3(kPlanThreads), 0, s, a);
    else           hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(kPlanThreads), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (a.N < 64) {
        const int per = kRegionRows / a.N, sides = 2 * ((a.n_chunks + per - 1) / per), waves = kPackThreads / 64;
        const dim3 grid((unsigned)((sides + waves - 1) / waves), (unsigned)a.BH), block(kPackThreads);
        if (a.kpc)            hipLaunchKernelGGL((pack_wave_kernel<32, true, false>), grid, block, 0, s, a);   // groups of 64 tokens do not fit
        else if (a.G == 32) {
            if (per > 1)      hipLaunchKernelGGL((pack_wave_kernel<32, false, true>), grid, block, 0, s, a);
            else              hipLaunchKernelGGL((pack_wave_kernel<32, false, false>), grid, block, 0, s, a);
        } else {
            if (per > 1)      hipLaunchKernelGGL((pack_wave_kernel<64, false, true>), grid, block, 0, s, a);
            else              hipLaunchKernelGGL((pack_wave_kernel<64, false, false>), grid, block, 0, s, a);
        }
        return hipGetLastError();
    }
    const dim3 grid((unsigned)(2 * a.N / kPartRows), (unsigned)a.n_chunks, (unsigned)a.BH), block(kPartRows * 2);
    if (a.kpc) {
        if (a.G == 32) hipLaunchKernelGGL((pack_kernel<32, true>), grid, block, 0, s, a);
        else           hipLaunchKernelGGL((pack_kernel<64, true>), grid, block, 0, s, a);
    } else {
        if (a.G == 32) hipLaunchKernelGGL((pack_kernel<32, false>), grid, block, 0, s, a);
        else           hipLaunchKernelGGL((pack_kernel<64, false>), grid, block, 0, s, a);
    }
    return hipGetLastError();
}

}  // namespace moqae
