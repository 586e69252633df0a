// Influence scores and per-query top-k (Sec. 2 Eq. (2) step (2); top-k most
// valuable training data, Sec. 4.1).
//
//   s[q][j] = sum_d te[q][d] * tr[j][d]      (fp32 result)
//
// Score GEMM (bf16, fp32 accumulation; launches with few or padded tiles take
// the smaller tiles of k_scores_small): one workgroup per 256 x 256 output tile; 4 waves, each
// owning a 128 x 128 quadrant as 4 x 4 blocks of 32x32x16 bf16 MFMAs (256
// fp32 accumulators per lane), 64 contraction columns (one slab) per step.
// Tiles are ordered so that the workgroups sharing one 256-row train slab are
// dispatched together onto the same XCD (dispatch round-robins workgroups
// over the 8 XCDs), so the slab is fetched from HBM once into that XCD's L2.
// Operands are copied straight from memory into an LDS ring with gfx950's
// buffer_load ... lds (no register staging); the issue order of MFMAs,
// copies and fragment reads is fixed by hand.  fp32 / fp64 operands take two
// float64-accumulating kernels.
//
// Top-k: one workgroup per query row.  An exact radix select (four 8-bit
// passes over order-preserving keys) finds the k-th largest score; when more
// scores tie at it than are needed, a second radix select over the
// (complemented) indices keeps the lowest-indexed ones.  The selected
// entries are sorted by (value desc, index asc), each by counting the larger
// ones, and, with merge, merged with the caller's running list.  For long chunks the GEMM
// epilogue filters: only scores at or above a per-query threshold (the k-th
// value of a running list that already covers a prefix of the chunk, hence
// a lower bound on the final k-th value) are appended to candidate lists, and
// the selection runs over those; a list that overflows falls back to the
// query's full score row.
#include <type_traits>

#include "common.h"
#include "internal.h"

namespace logra {
namespace {

constexpr int BM = 256, BN = 256, BK = 64;
constexpr int GT = 256;           // GEMM threads
constexpr int kXcd = 8;

// Epilogue of a 256 x 256 tile: the fp32 scores, times the optional row and
// column scales (s * row_scale[q] * col_scale[j], for normalised scores), go
// to s (rows past Q and columns past N are skipped).  With a filter, scores at
// or above the row's threshold are also appended to the row's top-k candidate
// list; the count keeps growing past the capacity so that an overflow is
// visible.  Each half-wave of one (i, r) step holds one row, so candidates
// are counted with ballots: a first pass writes the scores and each (row,
// column half)'s count to LDS, one global atomic per row reserves the tile's
// space, and a second pass places each candidate at its reserved base plus its
// ballot prefix (in column order within a column half).  `lds` is 5 KB of free
// LDS (thresholds, counts and bases).
__device__ __forceinline__ void store_scores(const f32x16 (&acc)[4][4], float *lds, float *__restrict__ s,
                                             int64_t ld_s, int m0, int64_t n0, int rows_a, int rows_b,
                                             int wm, int wn, int tid, int lane, const ScoreFilter &filt,
                                             const ScoreScale &scale) {
    const bool filter = filt.thr != nullptr;
    float *ths = lds;                                        // [256] row thresholds
    int *cnt = reinterpret_cast<int *>(lds + 256);           // [2][256] candidates per column half
    int *base = reinterpret_cast<int *>(lds + 768);          // [2][256] first slot per column half
    if (filter) {
        ths[tid] = tid < rows_a ? filt.thr[m0 + tid] : __builtin_inff();
        __syncthreads();
    }
    const uint64_t half = lane < 32 ? 0xffffffffull : 0xffffffff00000000ull;   // the lanes of this row
    auto value = [&](int i, int r, int j, float rs, int col) {   // the same in both passes
        float v = acc[i][j][r];
        if (scale.row) v *= rs;
        if (scale.col && col < rows_b) v *= scale.col[n0 + col];
        return v;
    };
    // result register r of block (i, j): row 8*(r/4) + 4*(lane/32) + r%4, column lane%32
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = wm * 128 + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
            if (row >= rows_a) continue;
            const int64_t q = m0 + row;
            float *srow_p = s + q * ld_s + n0;
            const float t = filter ? ths[row] : 0.f;
            const float rs = scale.row ? scale.row[q] : 1.f;
            int hits = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int col = wn * 128 + j * 32 + (lane & 31);
                const float v = value(i, r, j, rs, col);
                if (col < rows_b) srow_p[col] = v;
                if (filter) hits += __popcll(__builtin_amdgcn_ballot_w64(col < rows_b && v >= t) & half);
            }
            if (filter && (lane & 31) == 0) cnt[wn * 256 + row] = hits;
        }
    if (!filter) return;
    __syncthreads();
    if (tid < rows_a) {
        const int c0 = cnt[tid], c1 = cnt[256 + tid];
        const int b = c0 + c1 > 0 ? atomicAdd(filt.cnt + m0 + tid, c0 + c1) : 0;
        base[tid] = b;
        base[256 + tid] = b + c0;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = wm * 128 + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
            if (row >= rows_a) continue;
            const int64_t q = m0 + row;
            const float t = ths[row];
            const float rs = scale.row ? scale.row[q] : 1.f;
            int pos = base[wn * 256 + row];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int col = wn * 128 + j * 32 + (lane & 31);
                const float v = value(i, r, j, rs, col);
                const bool hit = col < rows_b && v >= t;
                const uint64_t m = __builtin_amdgcn_ballot_w64(hit) & half;
                if (hit) {
                    const int p = pos + static_cast<int>(__builtin_amdgcn_mbcnt_hi(
                                            static_cast<uint32_t>(m >> 32),
                                            __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u)));
                    if (p < filt.cap) {
                        filt.val[q * filt.cap + p] = v;
                        filt.idx[q * filt.cap + p] = static_cast<int>(n0) + col;
                    }
                }
                pos += __popcll(m);
            }
        }
}

// ------------------------------------------------------------------------
// Score GEMM with asynchronous global->LDS copies (gfx950 buffer_load ... lds).
// The operands travel from memory straight into LDS (no register staging, no
// LDS store instructions).  The LDS ring holds three slabs of the train operand, which
// streams from HBM and is copied two slabs ahead, and two slabs of the test
// operand, which the L2 mostly serves and is copied one slab ahead
// (3 x 32 KB + 2 x 32 KB = 160 KB).  The train copies carry the
// non-temporal hint: the streamed rows are evicted first, so the test operand
// (re-read by every train tile) stays in the caches longer.  One barrier per slab: each wave waits
// for its own copies of the slab, the barrier makes every wave's copies
// visible and frees the stages of the previous slab, and the next copies are
// issued before the slab is multiplied.
//
// LDS layout of an operand slab: 256 rows of 128 bytes (8 chunks of 16 B);
// chunk c of row r is stored at position c ^ ((r >> 1) & 7), which makes the
// 16 lanes of each quarter-wave fragment read (16 consecutive rows, one chunk)
// hit 16 different 16-byte bank groups.  A copy instruction writes a
// contiguous 1 KB (8 whole rows, so every request is a full 128-byte line):
// lane l stores row (l >> 3), position (l & 7).
constexpr int kSlabOp = BM * BK * 2;         // bytes of one operand slab (32 KB)
constexpr int kStagesA = 2, kStagesB = 3;
constexpr int kLdsB = kStagesA * kSlabOp;    // B stages follow the A stages
constexpr int kLdsBytes = (kStagesA + kStagesB) * kSlabOp;
constexpr int kCopies = kSlabOp / 1024 / 4;  // 1 KB copies per wave and operand per slab (8)

__global__ __launch_bounds__(GT, 1) void k_scores_dma(const bf16_bits *__restrict__ te, int64_t ld_te,
                                                      int Q, const bf16_bits *__restrict__ tr,
                                                      int64_t ld_tr, int64_t N, int D,
                                                      float *__restrict__ s, int64_t ld_s,
                                                      int m_tiles, int n_tiles, ScoreFilter filt,
                                                       ScoreScale scale) {
    __shared__ __attribute__((aligned(1024))) uint8_t smem[kLdsBytes];

    const int bid = blockIdx.x;
    const int xcd = bid % kXcd, local = bid / kXcd;
    const int mt = local % m_tiles;
    const int nt = (local / m_tiles) * kXcd + xcd;
    if (nt >= n_tiles) return;
    const int m0 = mt * BM;
    const int64_t n0 = static_cast<int64_t>(nt) * BN;
    const int rows_a = Q - m0 < BM ? Q - m0 : BM;
    const int rows_b = N - n0 < BN ? static_cast<int>(N - n0) : BN;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    // LDS byte address of the ring (the address-space cast yields the 32-bit LDS offset)
    const uint32_t lds0 = static_cast<uint32_t>(
        reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint8_t *)smem));

    const auto rsa = buf_rsrc_uniform(te + static_cast<int64_t>(m0) * ld_te,
                                      static_cast<uint32_t>(rows_a * ld_te * 2));
    const auto rsb = buf_rsrc_uniform(tr + n0 * ld_tr, static_cast<uint32_t>(rows_b * ld_tr * 2));
    // copy i of this wave covers rows (8 wave + i) * 8 .. +8 of an operand slab;
    // lane l loads chunk (l & 7) ^ (((8 wave + i) * 4 + (l >> 4)) & 7) of its row
    uint32_t oa[kCopies], ob[kCopies];
    int ccol[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) ccol[h] = 8 * ((lane & 7) ^ ((4 * h + (lane >> 4)) & 7));
#pragma unroll
    for (int i = 0; i < kCopies; ++i) {
        const int r = (wave * kCopies + i) * 8 + (lane >> 3);
        oa[i] = r < rows_a ? static_cast<uint32_t>((r * ld_te + ccol[i & 1]) * 2) : kBufOOB;
        ob[i] = r < rows_b ? static_cast<uint32_t>((r * ld_tr + ccol[i & 1]) * 2) : kBufOOB;
    }
    auto issue = [&](const __amdgpu_buffer_rsrc_t &rs, const uint32_t(&o)[kCopies], int slab, uint32_t lds) {
        const int k0 = slab * BK;
        const uint32_t dk = static_cast<uint32_t>(k0) * 2u;
        const bool kin0 = k0 + ccol[0] < D, kin1 = k0 + ccol[1] < D;
        const uint32_t la = lds + wave * kCopies * 1024;
#pragma unroll
        for (int i = 0; i < kCopies; ++i)
            copy_to_lds(rs, ((i & 1) ? kin1 : kin0) ? o[i] + dk : kBufOOB, la + i * 1024);
    };

    // fragment byte offsets inside an operand slab: lane l reads row (l % 32) of
    // each 32-row block, logical chunk 2 ks + (l / 32) at position chunk ^ sw
    const int sw = (lane >> 1) & 7;
    const uint32_t fa0 = (wm * 128 + (lane & 31)) * 128, fb0 = (wn * 128 + (lane & 31)) * 128;
    uint32_t fo[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) fo[ks] = static_cast<uint32_t>(((2 * ks + (lane >> 5)) ^ sw) * 16);

    f32x16 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    bf16x8 fa[2][4], fb[2][4];
    // fragment read g (0..7) of a 16-wide step: A block g/2 for even g, B block g/2 for odd g
    auto ldfrag1 = [&](int f, const uint8_t *abase, const uint8_t *bbase, int ks, int g) {
        const int i = g >> 1;
        if (g & 1)
            fb[f][i] = as_bf16x8(*reinterpret_cast<const u32x4 *>(bbase + fb0 + fo[ks] + i * 4096));
        else
            fa[f][i] = as_bf16x8(*reinterpret_cast<const u32x4 *>(abase + fa0 + fo[ks] + i * 4096));
    };
    auto mfma1 = [&](int f, int idx) {
        const int i = idx >> 2, j = idx & 3;
        acc[i][j] = mfma32_bf16(fa[f][i], fb[f][j], acc[i][j]);
    };

    // Slab kt lives in A stage kt % 2 and B stage kt % 3.  Before slab kt
    // is read, the copies in flight are (A kt, B kt+1), issued during slab
    // kt-1, and B kt from before; waiting until at most kCopies remain leaves
    // only B kt+1 (issued last).  The wait and the barrier sit in the middle
    // of the previous slab's last 16-wide step: its first 8 MFMAs cover the
    // barrier, its last 8 cover the reads of the new slab's first fragments.
    // (lgkmcnt(0) first: this wave's reads of the stages that the next copies
    // overwrite are complete before any wave passes the barrier.)  The step
    // is issued in a fixed order (scheduling barriers): groups of two MFMAs
    // with one copy of the next slabs and one fragment read of the next
    // 16-wide step.
    const int nk = (D + BK - 1) / BK;
    issue(rsa, oa, 0, lds0);
    issue(rsb, ob, 0, lds0 + kLdsB);
    issue(rsb, ob, 1, lds0 + kLdsB + kSlabOp);
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"(kCopies) : "memory");
#pragma unroll
    for (int g = 0; g < 8; ++g) ldfrag1(0, smem, smem + kLdsB, 0, g);
    int sa = 0, sb = 0;   // stages of slab kt
    for (int kt = 0; kt < nk; ++kt) {
        const int na = sa ^ 1, nb2 = sb == 0 ? 2 : sb - 1;   // stages of A kt+1 and B kt+2
        const int nb1 = sb == 2 ? 0 : sb + 1;                // stage of B kt+1
        const uint8_t *abase = smem + sa * kSlabOp, *bbase = smem + kLdsB + sb * kSlabOp;
        const uint32_t dka = static_cast<uint32_t>((kt + 1) * BK) * 2u, dkb = dka + BK * 2u;
        const bool ka0 = (kt + 1) * BK + ccol[0] < D, ka1 = (kt + 1) * BK + ccol[1] < D;
        const bool kb0 = (kt + 2) * BK + ccol[0] < D, kb1 = (kt + 2) * BK + ccol[1] < D;
        const uint32_t la = lds0 + na * kSlabOp + wave * kCopies * 1024;
        const uint32_t lb = lds0 + kLdsB + nb2 * kSlabOp + wave * kCopies * 1024;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < 3; ++ks) {
            const int f = ks & 1;
#pragma unroll
            for (int g = 0; g < 8; ++g) {
                mfma1(f, 2 * g);
                mfma1(f, 2 * g + 1);
                if (ks == 0)
                    copy_to_lds(rsa, ((g & 1) ? ka1 : ka0) ? oa[g] + dka : kBufOOB, la + g * 1024);
                else if (ks == 1)
                    copy_to_lds_nt(rsb, ((g & 1) ? kb1 : kb0) ? ob[g] + dkb : kBufOOB, lb + g * 1024);
                ldfrag1(f ^ 1, abase, bbase, ks + 1, g);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int m = 0; m < 8; ++m) mfma1(1, m);
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(kCopies) : "memory");
        const uint8_t *nabase = smem + na * kSlabOp, *nbbase = smem + kLdsB + nb1 * kSlabOp;
#pragma unroll
        for (int g = 0; g < 8; ++g) {
            ldfrag1(0, nabase, nbbase, 0, g);
            mfma1(1, 8 + g);
            __builtin_amdgcn_sched_barrier(0);
        }
        sa = na;
        sb = nb1;
    }
    // the copies of the slabs past the end are still in flight
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    store_scores(acc, reinterpret_cast<float *>(smem), s, ld_s, m0, n0, rows_a, rows_b, wm, wn, tid,
                 lane, filt, scale);
}

// ------------------------------------------------------------------------
// Small output tiles, for launches whose 256 x 256 tiles are too few for the
// chip or mostly padding (few queries or few train rows).  A workgroup owns
// 16 MT queries x 16 NT train rows; its four waves split the contraction into
// four contiguous bands of 64-column steps, so a 57,344-wide dot product is
// four chains side by side instead of one.  Each wave copies its own operand
// rows into a ring of ST stages in LDS (gfx950 buffer_load ... lds, whole
// 128-byte rows, ST - 1 steps ahead), waits only for its own copies, and
// multiplies 16x16x32 MFMA fragments read from the ring: no barrier before the
// final fold, which adds the four partial tiles in fixed order through LDS.
// The workgroups of one train slab go to one XCD, as in k_scores_dma.
// Bound by HBM where few queries meet many rows.  Otherwise every workgroup's
// copies arrive at 50 to 56 GB/s (256 x 256 rows: 3.67 MB in 66 us), far from the
// HBM and MFMA rates of the chip; what holds them there has not been found.
// Measured, D = 57,344, against the 256 x 256 tiles: 256 x 256 rows 954 -> 68 us,
// 4 queries x 4,096 rows 887 -> 87, 4 x 65,536 1256 -> 1099 (6.8 TB/s), 32 x
// 65,536 1261 -> 1185, 256 x 4,096 956 -> 290.
//
// LDS slab: rows of 128 bytes, chunk c of row r at position c ^ ((r >> 1) & 7),
// so that the 16 rows read by a quarter-wave hit 16 different 16-byte banks.
template <int MT, int NT, int ST>
__global__ __launch_bounds__(GT, 1) void k_scores_small(const bf16_bits *__restrict__ te, int64_t ld_te, int Q,
                                                        const bf16_bits *__restrict__ tr, int64_t ld_tr, int64_t N,
                                                        int D, float *__restrict__ s, int64_t ld_s, int m_tiles,
                                                        int n_tiles, ScoreFilter filt, ScoreScale scale) {
    constexpr int TM = 16 * MT, TN = 16 * NT;
    constexpr int kRowsBytes = (TM + TN) * 128;        // one stage of one wave
    constexpr int kCp = (TM + TN) / 8;                 // 1 KB copies per stage
    static_assert(4 * ST * kRowsBytes <= 160 * 1024, "ring fits in LDS");
    static_assert((ST - 1) * kCp < 64, "vmcnt range");
    __shared__ __attribute__((aligned(1024))) uint8_t smem[4 * ST * kRowsBytes];

    const int bid = blockIdx.x;
    const int xcd = bid % kXcd, local = bid / kXcd;
    const int mt = local % m_tiles;
    const int64_t nt = static_cast<int64_t>(local / m_tiles) * kXcd + xcd;
    if (nt >= n_tiles) return;
    const int m0 = mt * TM;
    const int64_t n0 = nt * TN;
    const int rows_a = Q - m0 < TM ? Q - m0 : TM;
    const int rows_b = N - n0 < TN ? static_cast<int>(N - n0) : TN;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t ring = lds_addr(smem) + wave * ST * kRowsBytes;
    uint8_t *ring_p = smem + wave * ST * kRowsBytes;

    const auto rsa = buf_rsrc_uniform(te + static_cast<int64_t>(m0) * ld_te, static_cast<uint32_t>(rows_a * ld_te * 2));
    const auto rsb = buf_rsrc_uniform(tr + n0 * ld_tr, static_cast<uint32_t>(rows_b * ld_tr * 2));
    // copy i covers rows 8 i .. 8 i + 7: lane l brings chunk (l & 7) ^ ((row >> 1) & 7) of row 8 i + (l >> 3)
    int ccol[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) ccol[h] = 8 * ((lane & 7) ^ ((4 * h + (lane >> 4)) & 7));
    uint32_t oa[2 * MT], ob[2 * NT];
#pragma unroll
    for (int i = 0; i < 2 * MT; ++i) {
        const int r = 8 * i + (lane >> 3);
        oa[i] = r < rows_a ? static_cast<uint32_t>((r * ld_te + ccol[i & 1]) * 2) : kBufOOB;
    }
#pragma unroll
    for (int i = 0; i < 2 * NT; ++i) {
        const int r = 8 * i + (lane >> 3);
        ob[i] = r < rows_b ? static_cast<uint32_t>((r * ld_tr + ccol[i & 1]) * 2) : kBufOOB;
    }
    const int nk = (D + BK - 1) / BK, per = (nk + 3) / 4;
    const int k_lo = wave * per, k_hi = k_lo + per < nk ? k_lo + per : nk;   // this wave's steps
    // step t of the band into stage t % ST; columns past D and steps past the
    // band read as zeros, without a memory access
    auto issue = [&](int t, int stage) {
        const int k0 = (k_lo + t) * BK;
        const bool live = k_lo + t < k_hi;
        const bool in0 = live && k0 + ccol[0] < D, in1 = live && k0 + ccol[1] < D;
        const uint32_t dk = static_cast<uint32_t>(k0) * 2u, l0 = ring + stage * kRowsBytes;
#pragma unroll
        for (int i = 0; i < 2 * MT; ++i)
            copy_to_lds(rsa, ((i & 1) ? in1 : in0) ? oa[i] + dk : kBufOOB, l0 + i * 1024);
#pragma unroll
        for (int i = 0; i < 2 * NT; ++i)
            copy_to_lds_nt(rsb, ((i & 1) ? in1 : in0) ? ob[i] + dk : kBufOOB, l0 + (2 * MT + i) * 1024);
    };
    const int frow = lane & 15, sw = (frow >> 1) & 7;
    uint32_t fo[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) fo[h] = static_cast<uint32_t>(frow * 128 + (((lane >> 4) + 4 * h) ^ sw) * 16);

    f32x4 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < ST - 1; ++t) issue(t, t);
    int cur = 0, nxt = ST - 1;
    for (int t = 0; t < per; ++t) {
        // step t's copies are done once only those of the ST - 2 later steps remain; this wave's
        // fragment reads of step t - 1, whose stage the next copies overwrite, are done too
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"((ST - 2) * kCp) : "memory");
        issue(t + ST - 1, nxt);
        const uint8_t *st = ring_p + cur * kRowsBytes;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            bf16x8 fa[MT], fb[NT];
#pragma unroll
            for (int i = 0; i < MT; ++i) fa[i] = as_bf16x8(*reinterpret_cast<const u32x4 *>(st + fo[h] + i * 2048));
#pragma unroll
            for (int j = 0; j < NT; ++j)
                fb[j] = as_bf16x8(*reinterpret_cast<const u32x4 *>(st + fo[h] + (MT + j) * 2048));
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[i][j] = mfma16_bf16(fa[i], fb[j], acc[i][j]);
        }
        cur = cur == ST - 1 ? 0 : cur + 1;
        nxt = nxt == ST - 1 ? 0 : nxt + 1;
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

    // fold: part[w][m][n] (rows padded by 4 floats), then one output per thread and round
    constexpr int kPad = TN + 4, kOut = TM * TN / GT;
    static_assert(4 * TM * kPad * 4 + TM * 4 <= 4 * ST * kRowsBytes, "the partial tiles and the counts fit in the ring");
    float *part = reinterpret_cast<float *>(smem);
    int *slot = reinterpret_cast<int *>(part + 4 * TM * kPad);   // a row's candidates, then the first one's place
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                part[(wave * TM + 16 * i + 4 * (lane >> 4) + r) * kPad + 16 * j + (lane & 15)] = acc[i][j][r];
    __syncthreads();
    const bool filter = filt.thr != nullptr;
    float v[kOut];
    uint64_t hits[kOut];   // the lanes of this one's row (TN neighbours in one round) that hold candidates
    const uint64_t row_lanes = (TN == 64 ? ~uint64_t{0} : (uint64_t{1} << (TN & 63)) - 1) << (lane & ~(TN - 1));
#pragma unroll
    for (int u = 0; u < kOut; ++u) {
        const int m = (tid + GT * u) / TN, c = (tid + GT * u) % TN;
        const bool in = m < rows_a && c < rows_b;
        const int64_t q = m0 + m, j = n0 + c;
        v[u] = (part[m * kPad + c] + part[(TM + m) * kPad + c]) +
               (part[(2 * TM + m) * kPad + c] + part[(3 * TM + m) * kPad + c]);
        if (in && scale.row) v[u] *= scale.row[q];
        if (in && scale.col) v[u] *= scale.col[j];
        if (in) s[q * ld_s + j] = v[u];
        if (filter) {
            hits[u] = __builtin_amdgcn_ballot_w64(in && v[u] >= filt.thr[q]) & row_lanes;
            if ((lane & (TN - 1)) == 0) slot[m] = __popcll(hits[u]);
        }
    }
    if (!filter) return;
    // one atomic a row takes its candidates' places: one for each of them would queue up at the
    // 4 B counter (64 x 32,768 scores of 64 columns, k = 100: 384-411 us against 86; every score tied: 16.1 ms against 0.33)
    __syncthreads();
    if (tid < rows_a) slot[tid] = slot[tid] > 0 ? atomicAdd(filt.cnt + m0 + tid, slot[tid]) : 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kOut; ++u) {
        const int m = (tid + GT * u) / TN, c = (tid + GT * u) % TN;
        if (!(hits[u] >> lane & 1)) continue;
        const int64_t q = m0 + m;
        const int p = slot[m] + static_cast<int>(__builtin_amdgcn_mbcnt_hi(
                                    static_cast<uint32_t>(hits[u] >> 32),
                                    __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(hits[u]), 0u)));
        if (p < filt.cap) {
            filt.val[q * filt.cap + p] = v[u];
            filt.idx[q * filt.cap + p] = static_cast<int>(n0) + c;
        }
    }
}

// fp32 / fp64 operands: every product and sum in float64 (a product of two
// fp32 values is exact there), on the fp64 matrix cores, the result rounded
// once to fp32.  A workgroup owns 16 F queries x 16 F train rows; its four waves
// split the columns into contiguous bands of 16-column units, loaded one unit
// ahead (lane (r, q) reads columns 2 q, 2 q + 1, 2 q + 8, 2 q + 9 of a unit of
// row r, for the four MFMAs of the unit, of both operands), and the four
// partial tiles are added in fixed order through LDS.  Scales (normalised
// scores) multiply in float64 before the rounding.  Bound by latency at the sizes
// of fp32 workloads: a call of 8 x 32 rows of 1,024 columns 22 us (the kernel 14); 116
// in k_scores_f64_chain.
template <int F, typename TA, typename TB>
__global__ __launch_bounds__(256) void k_scores_f64acc(const TA *te, int64_t ld_te, int Q, const TB *tr,
                                                       int64_t ld_tr, int64_t N, int D, float *s, int64_t ld_s,
                                                       ScoreScale scale) {
    constexpr int FT = 16 * F;
    __shared__ double part[4][FT][FT + 1];
    const int q0 = blockIdx.y * FT;
    const int64_t j0 = static_cast<int64_t>(blockIdx.x) * FT;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, q = lane >> 4;
    const int nu = (D + 15) / 16, per = (nu + 3) / 4;
    const int u0 = wave * per, u1 = min(nu, u0 + per);
    const TA *pa[F];
    const TB *pb[F];
#pragma unroll
    for (int x = 0; x < F; ++x) {   // rows past the end: the last one, not stored
        pa[x] = te + static_cast<int64_t>(min(q0 + 16 * x + r, Q - 1)) * ld_te;
        const int64_t j = j0 + 16 * x + r;
        pb[x] = tr + (j < N ? j : N - 1) * ld_tr;
    }
    f64x4 acc[F][F];
#pragma unroll
    for (int x = 0; x < F; ++x)
#pragma unroll
        for (int y = 0; y < F; ++y) acc[x][y] = f64x4{0.0, 0.0, 0.0, 0.0};
    TA a[2][F][4];
    TB b[2][F][4];
    auto load = [&](int buf, int u) {
        const int k0 = 16 * u + 2 * q;
        const bool whole = 16 * u + 16 <= D;   // the last unit reads its missing columns from the last one
#pragma unroll
        for (int x = 0; x < F; ++x)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int k = k0 + 8 * (t >> 1) + (t & 1), kc = whole || k < D ? k : D - 1;
                a[buf][x][t] = pa[x][kc];
                b[buf][x][t] = pb[x][kc];
            }
    };
    auto mul = [&](int buf, int u) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const bool in = 16 * u + 2 * q + 8 * (t >> 1) + (t & 1) < D;   // and counts them as zero
            double av[F], bv[F];
#pragma unroll
            for (int x = 0; x < F; ++x) {
                av[x] = in ? static_cast<double>(a[buf][x][t]) : 0.0;
                bv[x] = in ? static_cast<double>(b[buf][x][t]) : 0.0;
            }
#pragma unroll
            for (int x = 0; x < F; ++x)
#pragma unroll
                for (int y = 0; y < F; ++y) acc[x][y] = mfma16_f64(av[x], bv[y], acc[x][y]);
        }
    };
    if (u0 < u1) load(0, u0);
    for (int u = u0; u < u1; u += 2) {
        if (u + 1 < u1) load(1, u + 1);
        mul(0, u);
        if (u + 2 < u1) load(0, u + 2);
        if (u + 1 < u1) mul(1, u + 1);
    }
#pragma unroll
    for (int x = 0; x < F; ++x)
#pragma unroll
        for (int y = 0; y < F; ++y)
#pragma unroll
            for (int t = 0; t < 4; ++t) part[wave][16 * x + q + 4 * t][16 * y + r] = acc[x][y][t];
    __syncthreads();
    for (int e = tid; e < FT * FT; e += 256) {
        const int m = e / FT, c = e % FT;   // consecutive threads: consecutive columns
        const int64_t j = j0 + c;
        if (q0 + m >= Q || j >= N) continue;
        double val = ((part[0][m][c] + part[1][m][c]) + part[2][m][c]) + part[3][m][c];
        if (scale.row) val *= static_cast<double>(scale.row[q0 + m]);
        if (scale.col) val *= static_cast<double>(scale.col[j]);
        s[static_cast<int64_t>(q0 + m) * ld_s + j] = static_cast<float>(val);
    }
}

// The same scores in one chain of FMAs over the columns, for many scores of few
// columns: one 64 x 64 output tile per workgroup, 16-column slabs of both
// operands staged through LDS as float64 (coalesced row reads, transposed
// stores), 4 x 4 outputs a thread.  Bound by the fp64 FMAs and their LDS reads,
// with nothing to fold at the end.  Measured against the bands in 64 x 64 tiles
// (fp32 operands): 1,024 x 16,384 scores of 16 columns 36 us against 113, of 64
// 78 against 154, of 256 266 against 388, of 768 787 against 842, of 1,024 1,050
// against 1,057 (1,024 x 4,096: 287 against 272).
constexpr int kChainTile = 64, kChainCols = 16;
template <typename TA, typename TB>
__global__ __launch_bounds__(256) void k_scores_f64_chain(const TA *te, int64_t ld_te, int Q, const TB *tr,
                                                          int64_t ld_tr, int64_t N, int D, float *s, int64_t ld_s,
                                                          ScoreScale scale) {
    __shared__ double As[kChainCols][kChainTile + 1];   // [column][query]
    __shared__ double Bs[kChainCols][kChainTile + 1];   // [column][train row]
    const int q0 = blockIdx.y * kChainTile;
    const int64_t j0 = static_cast<int64_t>(blockIdx.x) * kChainTile;
    const int tid = threadIdx.x, ta = tid >> 4, tb = tid & 15;
    double acc[4][4] = {};
    for (int k0 = 0; k0 < D; k0 += kChainCols) {
#pragma unroll
        for (int u = 0; u < kChainTile * kChainCols / 256; ++u) {
            const int e = tid + 256 * u, r = e / kChainCols, c = e % kChainCols, d = k0 + c;
            const int q = q0 + r;
            const int64_t j = j0 + r;
            As[c][r] = (q < Q && d < D) ? load_in_d<TA>(te + static_cast<int64_t>(q) * ld_te + d) : 0.0;
            Bs[c][r] = (j < N && d < D) ? load_in_d<TB>(tr + j * ld_tr + d) : 0.0;
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < kChainCols; ++c) {
            double x[4], y[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                x[u] = As[c][4 * ta + u];
                y[u] = Bs[c][tb + 16 * u];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[u][v] = fma(x[u], y[v], acc[u][v]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int q = q0 + 4 * ta + u;
        if (q >= Q) continue;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t j = j0 + tb + 16 * v;   // consecutive threads: consecutive columns
            if (j >= N) continue;
            double val = acc[u][v];
            if (scale.row) val *= static_cast<double>(scale.row[q]);
            if (scale.col) val *= static_cast<double>(scale.col[j]);
            s[static_cast<int64_t>(q) * ld_s + j] = static_cast<float>(val);
        }
    }
}

// ---------------------------------------------------------------- top-k --
constexpr int KT_THREADS = 256;

// Order-preserving map float -> uint32 (larger float <=> larger key); -0.0
// maps to the key of +0.0 so that equal values tie.
__device__ __forceinline__ uint32_t fkey(float f) {
    uint32_t u = __float_as_uint(f);
    if (u == 0x80000000u) u = 0u;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float unkey(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// (key a, idx a) ranks before (key b, idx b); idx < 0 is padding, ranks last.
__device__ __forceinline__ bool before(uint32_t ka, int64_t ia, uint32_t kb, int64_t ib) {
    if (ia < 0) return false;
    if (ib < 0) return true;
    if (ka != kb) return ka > kb;
    return ia < ib;
}

// Sources of a selection: a row of scores (local index = column), or a
// row's candidate list (local index = the candidate's column).  Global index
// = base + local index.
struct RowSrc {
    const float *row;
    int64_t n;
    int64_t base;
    __device__ int64_t size() const { return n; }
    __device__ float value(int64_t j) const { return row[j]; }
    __device__ uint32_t local(int64_t j) const { return static_cast<uint32_t>(j); }
};
struct CandSrc {
    const float *v;
    const int *c;
    int64_t n;
    int64_t base;
    __device__ int64_t size() const { return n; }
    __device__ float value(int64_t j) const { return v[j]; }
    __device__ uint32_t local(int64_t j) const { return static_cast<uint32_t>(c[j]); }
};

// Working memory of one row's selection (36 KB: four rows of 256 threads per
// CU).  `keys` holds the row's keys during the selection, where they fit, and
// the caller's running list afterwards.
constexpr int kTopkWaves = KT_THREADS / 64;
constexpr int kTopkKeys = 4096;
struct TopkShared {
    uint32_t hist[kTopkWaves][256];
    uint64_t sel[kMaxTopk];      // the selected elements, key << 32 | ~local index
    uint64_t sorted[kMaxTopk];   // the same in descending order
    union {
        uint32_t keys[kTopkKeys];
        struct {
            int64_t idx[kMaxTopk];
            uint32_t key[kMaxTopk];
        } old;
    };
    uint32_t wsum[kTopkWaves];
    uint32_t prefix;
    int rem;
    uint32_t neq;
    int count;
};

// Radix select (four 8-bit digits, most significant first) of the `want`-th
// largest key(j) over the j < n with in(j) (at least `want` of them).
// Returns that key; *rem = how many elements equal to it belong to the `want`
// largest, *neq = how many exist.  Every wave counts in a histogram of its
// own; thread d sums digit d over the waves, and the digits above it are
// added by a scan across lanes, so no thread walks the histogram.
template <class KeyFn, class InFn>
__device__ uint32_t radix_select(int64_t n, KeyFn key, InFn in, int want, TopkShared &sh, int *rem,
                                 uint32_t *neq) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t prefix = 0, pmask = 0;
    uint32_t r = static_cast<uint32_t>(want);
    uint32_t eq = 0;
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
#pragma unroll
        for (int w = 0; w < kTopkWaves; ++w) sh.hist[w][tid] = 0;
        __syncthreads();
        for (int64_t j = tid; j < n; j += KT_THREADS) {
            if (!in(j)) continue;
            const uint32_t kk = key(j);
            if ((kk & pmask) == prefix) atomicAdd(&sh.hist[wave][(kk >> shift) & 255u], 1u);
        }
        __syncthreads();
        uint32_t v = 0;
#pragma unroll
        for (int w = 0; w < kTopkWaves; ++w) v += sh.hist[w][tid];
        uint32_t above = v;   // elements of digits >= tid
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_down(above, o, 64);
            if (lane + o < 64) above += y;
        }
        if (lane == 0) sh.wsum[wave] = above;
        __syncthreads();
#pragma unroll
        for (int w = 1; w < kTopkWaves; ++w)
            if (w > wave) above += sh.wsum[w];
        if (above >= r && above - v < r) {   // the digit of the want-th largest
            sh.prefix = prefix | (static_cast<uint32_t>(tid) << shift);
            sh.rem = static_cast<int>(r - (above - v));
            sh.neq = v;
        }
        __syncthreads();
        prefix = sh.prefix;
        r = static_cast<uint32_t>(sh.rem);
        eq = sh.neq;
        pmask |= 255u << shift;
        __syncthreads();
    }
    *rem = static_cast<int>(r);
    *neq = eq;
    return prefix;
}

// sorted[] = the m elements of sel[] in descending order.  Every element is
// different (its low half is its index), so its place is the number of larger
// ones: each thread counts for up to four elements while the list goes past
// once as LDS broadcasts, and no step waits for another.
__device__ __forceinline__ void rank_sort(TopkShared &sh, int m) {
    constexpr int kPer = kMaxTopk / KT_THREADS;
    const int tid = threadIdx.x;
    uint64_t x[kPer];
    int rank[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int i = tid + KT_THREADS * u;
        x[u] = i < m ? sh.sel[i] : ~uint64_t{0};
        rank[u] = 0;
    }
    auto count = [&](auto per) {
        for (int j = 0; j < m; ++j) {
            const uint64_t y = sh.sel[j];
#pragma unroll
            for (int u = 0; u < decltype(per)::value; ++u) rank[u] += y > x[u] ? 1 : 0;
        }
    };
    if (m <= KT_THREADS)
        count(std::integral_constant<int, 1>{});
    else
        count(std::integral_constant<int, kPer>{});
#pragma unroll
    for (int u = 0; u < kPer; ++u)
        if (tid + KT_THREADS * u < m) sh.sorted[rank[u]] = x[u];
}

// Top-k of one source, merged with the running list (vo, io) when `merge`.
// At most kMaxTopk elements are taken whole.  Otherwise the k-th largest key
// is found by radix select (over keys kept in LDS where they fit); when more
// elements tie at it than are needed, a second radix select over the
// complemented local index keeps the lowest-indexed ones, and exactly k
// elements are collected.  The elements are then sorted by (value descending,
// index ascending), and merged by rank: an element's place in the merged list
// is its place in its own list plus the number of elements of the other list
// that go before it (a binary search).
// Bound by its chain of passes and barriers.  Measured, k = 100, against one
// thread walking the histogram and the merge and a bitonic sort: 4 rows of
// 4,096 scores 53 -> 20 us, 4 lists of 1,500 candidates 80 -> 16, 1,024 lists
// 117 -> 37; 8 rows of 32 scores, k = 10: 46 -> 5.
template <class Src>
__device__ void topk_row(const Src &src, int k, float *vo, int64_t *io, bool merge, TopkShared &sh) {
    const int tid = threadIdx.x;
    const int64_t n = src.size();
    int m;   // selected elements
    auto packed = [&](uint32_t key, int64_t j) {
        return (static_cast<uint64_t>(key) << 32) | static_cast<uint32_t>(~src.local(j));
    };
    if (n <= kMaxTopk) {
        m = static_cast<int>(n);
        for (int j = tid; j < m; j += KT_THREADS) sh.sel[j] = packed(fkey(src.value(j)), j);
        __syncthreads();
    } else {
        m = k;   // k <= kMaxTopk < n
        const bool staged = n <= kTopkKeys;
        if (staged) {
            for (int j = tid; j < static_cast<int>(n); j += KT_THREADS) sh.keys[j] = fkey(src.value(j));
            __syncthreads();
        }
        auto key = [&](int64_t j) { return staged ? sh.keys[j] : fkey(src.value(j)); };
        int rem;
        uint32_t neq, idx_limit = 0xffffffffu;
        const uint32_t kth = radix_select(n, key, [](int64_t) { return true; }, k, sh, &rem, &neq);
        if (neq > static_cast<uint32_t>(rem)) {
            int rem2;
            uint32_t neq2;
            const uint32_t c = radix_select(
                n, [&](int64_t j) { return ~src.local(j); }, [&](int64_t j) { return key(j) == kth; }, rem, sh,
                &rem2, &neq2);
            idx_limit = ~c;
        }
        if (tid == 0) sh.count = 0;
        __syncthreads();
        for (int64_t j = tid; j < n; j += KT_THREADS) {
            const uint32_t kk = key(j);
            if (kk > kth || (kk == kth && src.local(j) <= idx_limit)) sh.sel[atomicAdd(&sh.count, 1)] = packed(kk, j);
        }
        __syncthreads();
    }
    rank_sort(sh, m);
    auto new_key = [&](int r) { return r < m ? static_cast<uint32_t>(sh.sorted[r] >> 32) : 0u; };
    auto new_idx = [&](int r) {
        return r < m ? src.base + static_cast<int64_t>(static_cast<uint32_t>(~sh.sorted[r])) : int64_t{-1};
    };
    auto put = [&](int r, uint32_t key, int64_t idx) {
        vo[r] = idx >= 0 ? unkey(key) : -__builtin_huge_valf();
        io[r] = idx >= 0 ? idx : -1;
    };
    if (!merge) {
        __syncthreads();
        for (int r = tid; r < k; r += KT_THREADS) put(r, new_key(r), new_idx(r));
        return;
    }
    for (int r = tid; r < k; r += KT_THREADS) {   // the keys are no longer needed
        sh.old.key[r] = fkey(vo[r]);
        sh.old.idx[r] = io[r];
    }
    __syncthreads();   // the running list is read completely before it is overwritten
    auto old_first = [&](int a, int b) {   // old element a goes before new element b
        return before(sh.old.key[a], sh.old.idx[a], new_key(b), new_idx(b));
    };
    for (int r = tid; r < k; r += KT_THREADS) {
        int lo = 0, hi = k;   // old element r: the new elements that go before it
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (old_first(r, mid))
                hi = mid;
            else
                lo = mid + 1;
        }
        if (r + lo < k) put(r + lo, sh.old.key[r], sh.old.idx[r]);
        lo = 0, hi = k;       // new element r: the old elements that go before it
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (old_first(mid, r))
                lo = mid + 1;
            else
                hi = mid;
        }
        if (r + lo < k) put(r + lo, new_key(r), new_idx(r));
    }
}

// One workgroup per query row over a full row of scores.
__global__ __launch_bounds__(KT_THREADS) void k_topk(const float *__restrict__ S, int64_t ld_s,
                                                     int64_t N, int64_t base, int k,
                                                     float *__restrict__ val,
                                                     int64_t *__restrict__ idx, int merge) {
    __shared__ TopkShared sh;
    const int q = blockIdx.x;
    const RowSrc src{S + static_cast<int64_t>(q) * ld_s, N, base};
    topk_row(src, k, val + static_cast<int64_t>(q) * k, idx + static_cast<int64_t>(q) * k, merge != 0,
             sh);
}

// Threshold of each row for candidate filtering: the k-th value of the
// running list (-inf while it holds fewer than k entries); clears the row's
// candidate count.
__global__ __launch_bounds__(256) void k_topk_threshold(const float *__restrict__ val,
                                                        const int64_t *__restrict__ idx, int Q, int k,
                                                        float *__restrict__ thr, int *__restrict__ cnt) {
    const int q = blockIdx.x * 256 + threadIdx.x;
    if (q >= Q) return;
    const int64_t last = static_cast<int64_t>(q) * k + k - 1;
    thr[q] = idx[last] >= 0 ? val[last] : -__builtin_huge_valf();
    cnt[q] = 0;
}

// Merge of each row's candidates into its running list; a row whose
// candidates overflowed the capacity is selected from its full score row.
__global__ __launch_bounds__(KT_THREADS) void k_topk_filtered(
    const float *__restrict__ S, int64_t ld_s, int64_t N, int64_t base, int k, float *__restrict__ val,
    int64_t *__restrict__ idx, const int *__restrict__ cnt, const float *__restrict__ cval,
    const int *__restrict__ cidx, int cap) {
    __shared__ TopkShared sh;
    const int q = blockIdx.x;
    float *vo = val + static_cast<int64_t>(q) * k;
    int64_t *io = idx + static_cast<int64_t>(q) * k;
    const int c = cnt[q];
    if (c <= cap) {
        const CandSrc src{cval + static_cast<int64_t>(q) * cap, cidx + static_cast<int64_t>(q) * cap, c,
                          base};
        topk_row(src, k, vo, io, true, sh);
    } else {
        const RowSrc src{S + static_cast<int64_t>(q) * ld_s, N, base};
        topk_row(src, k, vo, io, true, sh);
    }
}

}  // namespace

namespace {
// bf16 score kernels, by output tile: the largest first.  One workgroup fills
// a CU in each, so a launch takes as many rounds as tiles fall to the busiest
// XCD's 32 CUs.  A round costs `fixed` plus `per_k` us for every 1,024 columns,
// measured with all CUs busy (a 256 x 256 tile: 920 us at 57,344 columns and
// about 30 more for its epilogue; 64 x 64: 265; 16 x 16: 68).  The smallest
// product of the two is taken: small tiles while they fill an idle chip or
// spare padding, large ones as soon as their operand reuse counts (256 queries
// x 4,096 rows: 290 us in 64 x 64 tiles against 956; x 16,384: 1185 against
// 959).
struct ScoreTile {
    int m, n;
    double fixed, per_k;
};
constexpr ScoreTile kScoreTiles[] = {{256, 256, 30., 16.4}, {64, 64, 5., 4.7}, {32, 64, 4., 3.5},
                                     {16, 64, 4., 2.8},     {32, 32, 3., 2.4}, {16, 16, 3., 1.15}};

// The cheapest of the tiles first .. last whose grid can be launched (small
// tiles of very many rows cannot), or `first`.
constexpr int kLastTile = static_cast<int>(sizeof kScoreTiles / sizeof kScoreTiles[0]) - 1;
int score_tile(int Q, int64_t N, int D, int first, int last) {
    int best = -1;
    double cost = 0.;
    for (int v = first; v <= last; ++v) {
        const ScoreTile &t = kScoreTiles[v];
        const int64_t m_tiles = (Q + t.m - 1) / t.m, n_tiles = (N + t.n - 1) / t.n;
        const int64_t per_xcd = (n_tiles + kXcd - 1) / kXcd * m_tiles, rounds = (per_xcd + 31) / 32;
        if (per_xcd * kXcd * GT >= kMaxGridThreads) continue;
        const double c = static_cast<double>(rounds) * (t.fixed + t.per_k * D / 1024.);
        if (best < 0 || c < cost) {
            best = v;
            cost = c;
        }
    }
    return best < 0 ? first : best;
}

int64_t square_tiles(int Q, int64_t N, int64_t edge) { return (N + edge - 1) / edge * ((Q + edge - 1) / edge); }
}  // namespace

// fp32 / fp64: one chain where two 64 x 64 tiles or more fall to every CU and
// the rows are short (times at k_scores_f64_chain: the bands win from about
// 1,000 columns on), but not of 32 rows or fewer, which fill half of such a
// tile (16 x 60,000 scores of 256 columns: 80 us, 57 in 32 x 32 tiles of bands).
ScoreOrder score_order(bool bf16, int Q, int64_t N, int D) {
    if (bf16) return score_tile(Q, N, D, 0, kLastTile) == 0 ? kOneChain : kFourBands;
    return Q > 32 && N > 32 && D <= 768 && square_tiles(Q, N, 64) >= 512 ? kOneChain : kFourBands;
}

hipError_t launch_scores(const void *te, int te_dt, int64_t ld_te, int Q, const void *tr, int tr_dt,
                         int64_t ld_tr, int64_t N, int D, float *s, int64_t ld_s, const ScoreFilter *filt,
                         const ScoreScale &scale, ScoreOrder order, hipStream_t st) {
    if (Q == 0 || N == 0) return hipSuccess;
    if (te_dt == kBF16 && tr_dt == kBF16) {
        const int tile = order == kOneChain ? 0 : score_tile(Q, N, D, 1, kLastTile);
        const int m_tiles = (Q + kScoreTiles[tile].m - 1) / kScoreTiles[tile].m;
        const int n_tiles = static_cast<int>((N + kScoreTiles[tile].n - 1) / kScoreTiles[tile].n);
        const int n_groups = (n_tiles + kXcd - 1) / kXcd;
        const unsigned grid = static_cast<unsigned>(kXcd) * n_groups * m_tiles;
        const ScoreFilter none{nullptr, nullptr, nullptr, nullptr, 0};
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(grid), dim3(GT), 0, st, static_cast<const bf16_bits *>(te), ld_te, Q,
                               static_cast<const bf16_bits *>(tr), ld_tr, N, D, s, ld_s, m_tiles, n_tiles,
                               filt ? *filt : none, scale);
            return hipGetLastError();
        };
        switch (tile) {
            case 1: return go(k_scores_small<4, 4, 2>);
            case 2: return go(k_scores_small<2, 4, 3>);
            case 3: return go(k_scores_small<1, 4, 3>);
            case 4: return go(k_scores_small<2, 2, 4>);
            case 5: return go(k_scores_small<1, 1, 8>);
            default: return go(k_scores_dma);
        }
    }
    if (filt || te_dt == kBF16 || tr_dt == kBF16) return hipErrorInvalidValue;   // bf16 pairs only with bf16
    // bands: the largest tile that gives every CU a workgroup; 64 x 64 neither for 32 rows or fewer (above)
    // nor for rows so short that its fold outlasts its products (64 x 16,384 scores of 16 columns 17 us, 14.5
    // in 32 x 32 tiles; of 96 the same; of 256 35 against 41)
    const bool wide = square_tiles(Q, N, 64) >= 256 && Q > 32 && N > 32 && D > 96;
    const int f = order == kOneChain || wide ? 4 : square_tiles(Q, N, 32) >= 256 ? 2 : 1;
    const dim3 grid(static_cast<unsigned>((N + 16 * f - 1) / (16 * f)), static_cast<unsigned>((Q + 16 * f - 1) / (16 * f)));
    auto go = [&](auto a, auto b) {
        using TA = decltype(a);
        using TB = decltype(b);
        auto run = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, static_cast<const TA *>(te), ld_te, Q,
                               static_cast<const TB *>(tr), ld_tr, N, D, s, ld_s, scale);
            return hipGetLastError();
        };
        if (order == kOneChain) return run(k_scores_f64_chain<TA, TB>);   // 64 x 64 tiles
        return f == 4 ? run(k_scores_f64acc<4, TA, TB>) : f == 2 ? run(k_scores_f64acc<2, TA, TB>) : run(k_scores_f64acc<1, TA, TB>);
    };
    if (te_dt == kF64) return tr_dt == kF64 ? go(double{}, double{}) : go(double{}, float{});
    return tr_dt == kF64 ? go(float{}, double{}) : go(float{}, float{});
}

int64_t topk_prefix_rows(int64_t N, int k) {
    // Expected candidates past a prefix of P rows: about k (N - P) / P; aim
    // for at most half the capacity.
    int64_t P = (2 * static_cast<int64_t>(k) * N + kCandCap - 1) / kCandCap;
    if (P < 4096) P = 4096;
    P = (P + 255) / 256 * 256;
    return 2 * P <= N ? P : 0;
}

hipError_t launch_topk(const float *s, int64_t ld_s, int Q, int64_t N, int64_t base, int k,
                       float *val, int64_t *idx, bool merge, hipStream_t st) {
    if (Q == 0) return hipSuccess;
    hipLaunchKernelGGL(k_topk, dim3(Q), dim3(KT_THREADS), 0, st, s, ld_s, N, base, k, val, idx,
                       merge ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_topk_threshold(const float *val, const int64_t *idx, int Q, int k, float *thr,
                                 int *cnt, hipStream_t st) {
    if (Q == 0) return hipSuccess;
    hipLaunchKernelGGL(k_topk_threshold, dim3((Q + 255) / 256), dim3(256), 0, st, val, idx, Q, k, thr,
                       cnt);
    return hipGetLastError();
}

hipError_t launch_topk_filtered(const float *s, int64_t ld_s, int Q, int64_t N, int64_t base, int k,
                                float *val, int64_t *idx, const int *cnt, const float *cval,
                                const int *cidx, int cap, hipStream_t st) {
    if (Q == 0) return hipSuccess;
    hipLaunchKernelGGL(k_topk_filtered, dim3(Q), dim3(KT_THREADS), 0, st, s, ld_s, N, base, k, val, idx,
                       cnt, cval, cidx, cap);
    return hipGetLastError();
}

}  // namespace logra
