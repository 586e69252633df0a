// Self-influence of gradients, the normaliser of l-RelatIF (Sec. 4.2: each
// influence score is divided by the training example's own influence, which
// penalises outliers with large gradient norms):
//
//   self_j = sum_l g_jl^T (C_l + lambda_l I)^{-1} g_jl = sum_l |W_l g_jl|^2,
//   W_l = L_l^{-1},  C_l + lambda_l I = L_l L_l^T
//
// for a block-diagonal (per-layer) Hessian.  W_l comes from the damped
// Cholesky factor in float64 and is held as two bf16 arrays hi + lo (about
// 16 significant bits together), so the products run on the bf16 matrix
// cores with fp32 accumulation: y = g W_hi^T + g W_lo^T.
//
// bf16 gradients: one workgroup per 256 gradients and range of blocks, 256 output
// dimensions per pass as 4 waves x (4 x 4 32x32x16 MFMA blocks), operands
// copied straight into an LDS ring; W is lower triangular and the MFMAs above
// its diagonal are left out.  After the last slab of a pass the squares of the
// outputs are summed over the wave's columns (registers, then DPP lane
// permutations inside rows of 16 lanes) into the gradients' running sums; at
// the end the partial sums are added through LDS, in a fixed order.
#include <type_traits>

#include "common.h"
#include "internal.h"


namespace logra {
namespace {

constexpr int SR = 256;                    // gradients per workgroup
constexpr int SO = 256;                    // output dimensions per pass
constexpr int STH = 256;                   // threads

// DPP lane permutations within rows of 16 lanes (dpp_ctrl encodings)
constexpr int kDppXor1 = 0xB1;             // quad_perm [1, 0, 3, 2]
constexpr int kDppXor2 = 0x4E;             // quad_perm [2, 3, 0, 1]
constexpr int kDppRowHalfMirror = 0x141;   // lane i <-> 7 - i within 8
constexpr int kDppRowMirror = 0x140;       // lane i <-> 15 - i within 16

template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}

typedef f32x16 Acc[4][4];   // one wave's 128 x 128 result quadrant (4 x 4 blocks of 32 x 32)

__device__ __forceinline__ void zero_acc(Acc &acc) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
}

// After the last slab of an output pass: the squared outputs, summed over
// the lane's four column blocks, then reduce-scattered over the 16 lanes of
// each DPP row in four halvings (partners l ^ 15, l ^ 7, l ^ 2, l ^ 1, all
// within the row; each lane keeps the half selected by the bit in which it
// differs from its partner), so that each lane ends with 4 of the 64 row
// entries e = 16 i + r (block i, register r) summed over the row's 16
// columns: psum[s] += entry 4 (lane % 16) + s.  Lanes l and l ^ 16 hold the
// two halves of the same rows' sums.  Clears the accumulators.
__device__ __forceinline__ void fold_rows(Acc &acc, float (&psum)[4], int lane) {
    const bool b3 = lane & 8, b2 = lane & 4, b1 = lane & 2, b0 = lane & 1;
    auto sq = [&](int e) {
        const int i = e >> 4, r = e & 15;
        float v = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j) v = __builtin_fmaf(acc[i][j][r], acc[i][j][r], v);
        return v;
    };
    float u[32], w[16], x[8];
#pragma unroll
    for (int k = 0; k < 32; ++k) {
        const float lo = sq(k), hi = sq(32 + k);
        u[k] = (b3 ? hi : lo) + dpp_f<kDppRowMirror>(b3 ? lo : hi);
        __builtin_amdgcn_sched_barrier(0);   // a few accumulators in VGPRs at a time
    }
#pragma unroll
    for (int k = 0; k < 16; ++k)
        w[k] = (b2 ? u[16 + k] : u[k]) + dpp_f<kDppRowHalfMirror>(b2 ? u[k] : u[16 + k]);
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = (b1 ? w[8 + k] : w[k]) + dpp_f<kDppXor2>(b1 ? w[k] : w[8 + k]);
#pragma unroll
    for (int k = 0; k < 4; ++k) psum[k] += (b0 ? x[4 + k] : x[k]) + dpp_f<kDppXor1>(b0 ? x[k] : x[4 + k]);
    zero_acc(acc);
}

// Adds the partial row sums of the workgroup's 256 gradients -- two column
// halves (waves wn = 0, 1) x the two 16-lane rows of each half-wave --
// through LDS (rowsum: 4 x 256 floats) in a fixed order and writes the
// results.  Ends with the workgroup's last barrier.
__device__ __forceinline__ void finish_rows(const float (&psum)[4], float *rowsum, int tid, int lane, int wm,
                                            int wn, int nrows, int64_t r0, float *self_out, float *rsqrt_out) {
    const int h16 = (lane >> 4) & 1;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int e = 4 * (lane & 15) + k, i = e >> 4, r = e & 15;
        rowsum[(2 * wn + h16) * 256 + wm * 128 + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)] = psum[k];
    }
    __syncthreads();
    if (tid < nrows) {
        const float sv = (rowsum[tid] + rowsum[256 + tid]) + (rowsum[512 + tid] + rowsum[768 + tid]);
        if (self_out) self_out[r0 + tid] = sv;
        if (rsqrt_out) rsqrt_out[r0 + tid] = sv > 0.f ? 1.0f / sqrtf(sv) : 0.f;
    }
}

// ------------------------------------------------------------------------
// bf16 gradients: a 256 x 256 tile per pass (gradients x outputs), 4 waves x
// (4 x 4 32x32x16 MFMA blocks), with the operands copied straight from memory
// into an LDS ring (gfx950 buffer_load ... lds), as in the score GEMM.  The
// contraction of a pass runs over the interleaved W (per 64-column chunk c: hi,
// then lo), one 64-column step at a time; the gradients' 64 columns of chunk c
// serve both steps of the chunk, so a gradient slab is copied once per two
// steps.  Ring: 2 gradient stages, 3 W stages of 32 KB (256 rows of 128 bytes,
// chunk c of row r at position c ^ ((r >> 1) & 7)).  Copies run two steps
// ahead: during the first step of a chunk, the next chunk's gradient slab and
// the W slab two steps ahead; during the second, the W slab two steps ahead.
// One barrier per step, in the middle of its last 16-wide MFMA group, after
// each wave has waited for its own copies of the next step's slabs (vmcnt,
// which counts the copies).
//
// W is lower triangular: pass ot needs chunks up to 4 ot + 3, and of its eight
// 32-output blocks chunk 4 ot + d meets only those from 2 d on.  Wave column
// wn takes blocks 0, 3, 4, 7 (wn = 0) or 1, 2, 5, 6, so that both have 4 - d of
// them, the last ones: at D = 256, 20 of 32 products are formed.  The last
// chunk of a D that is not a multiple of 64 is narrower; columns past it read
// as zeros on both sides.
//
// blockIdx.y: one of gridDim.y ranges of blocks, whose sums go to
// part[range][gradient] when there are several (k_self_influence_fold adds
// them).  32,768 gradients are 128 workgroups, half the chip, without ranges.
// Measured, 32,768 gradients of 224 blocks of 256: 1.25 to 1.43 ms by run; 2,645 us
// with all products and one range.
constexpr int DBK = 64;                          // columns per step
constexpr int kDSlab = 256 * DBK * 2;            // bytes of one operand slab
constexpr int kDStA = 2, kDStB = 3;
constexpr int kDLdsB = kDStA * kDSlab;
constexpr int kDLds = (kDStA + kDStB) * kDSlab;  // 160 KB
constexpr int kDCopies = kDSlab / 1024 / 4;      // 1 KB copies per wave and operand slab (8)

__global__ __launch_bounds__(STH, 1) void k_self_influence_dma(const bf16_bits *__restrict__ g, int64_t ld,
                                                               int64_t rows, int D, int n_blocks,
                                                               const bf16_bits *__restrict__ w, float *part,
                                                               float *__restrict__ self_out,
                                                               float *__restrict__ rsqrt_out) {
    __shared__ __attribute__((aligned(1024))) uint8_t smem[kDLds];

    const int64_t r0 = static_cast<int64_t>(blockIdx.x) * SR;
    const int nrows = rows - r0 < SR ? static_cast<int>(rows - r0) : SR;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const uint32_t lds0 = lds_addr(smem);
    const int n_ot = (D + SO - 1) / SO;
    const int Dp = n_ot * SO;
    const int n_chunks = (D + DBK - 1) / DBK;
    const uint32_t w_row = 2u * D * 2u;      // bytes per row of the interleaved W
    // this workgroup's blocks
    const uint32_t nb = n_blocks, range = blockIdx.y, ranges = gridDim.y;   // nb * ranges < 2^24
    const int l0 = __builtin_amdgcn_readfirstlane(static_cast<int>(nb * range / ranges));
    const int l1 = __builtin_amdgcn_readfirstlane(static_cast<int>(nb * (range + 1) / ranges));
    auto chunks_of = [&](int ot) { return min(n_chunks, 4 * (ot + 1)); };

    // copy i of this wave covers rows rb + 8 i, rb = 64 wave + (l >> 3), of a
    // slab; lane l loads chunk (l & 7) ^ (((8 wave + i) * 4 + (l >> 4)) & 7) of
    // its row.  Byte offsets are va[i & 1] + i * (8 rows), plus the slab's
    // column offset: two per-lane bases per operand.  Rows at or past nrows
    // lie past the gradient buffer's range and read zeros; so does every copy
    // past the last block, through a descriptor of size 0.
    const int rb = 64 * wave + (lane >> 3);
    uint32_t va[2], vb[2];
    int cc[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        cc[h] = 8 * ((lane & 7) ^ ((4 * h + (lane >> 4)) & 7));
        va[h] = static_cast<uint32_t>((rb * ld + cc[h]) * 2);
        vb[h] = static_cast<uint32_t>(rb) * w_row + static_cast<uint32_t>(cc[h]) * 2u;
    }
    const uint32_t a_bytes = static_cast<uint32_t>(nrows * ld * 2);
    const uint32_t a_step8 = static_cast<uint32_t>(8 * ld * 2), b_step8 = 8u * w_row;
    // issue cursors, advanced in the order the slabs are consumed: gradient
    // slab (al, aot, aj) and W step (bl, bot, bt) = (block, output pass, chunk
    // or step within the pass)
    int al = l0, aot = 0, aj = 0, bl = l0, bot = 0, bt = 0;
    auto rsrc_a = [&]() { return buf_rsrc_uniform(g + r0 * ld, al < l1 ? a_bytes : 0u); };
    auto issue_a = [&](const __amdgpu_buffer_rsrc_t &rsa, uint32_t lds, int i) {
        uint32_t dk = static_cast<uint32_t>((al * D + aj * DBK) * 2) + i * a_step8;
        asm volatile("" : "+s"(dk));   // stays scalar: 16 hoisted vector sums would spill
        // the streamed gradients carry the non-temporal hint (1% faster on a 200,000-row
        // store; the same hint on the inverse-factor copies was slower)
        copy_to_lds_nt(rsa, cc[i & 1] < D - aj * DBK ? va[i & 1] + dk : kBufOOB, lds + wave * kDCopies * 1024 + i * 1024);
    };
    auto next_a = [&]() {
        if (++aj == chunks_of(aot)) {
            aj = 0;
            if (++aot == n_ot) {
                aot = 0;
                ++al;
            }
        }
    };
    auto rsrc_b = [&]() {   // nothing past the last block, nor of rows whose outputs the step leaves out
        const bool live = bl < l1 && wave >= (bt >> 1) - 4 * bot;
        const size_t blk = static_cast<size_t>(bl < l1 ? bl : l0) * Dp * 2 * D;
        return buf_rsrc_uniform(w + blk, live ? static_cast<uint32_t>(Dp) * w_row : 0u);
    };
    auto issue_b = [&](const __amdgpu_buffer_rsrc_t &rsb, uint32_t lds, int i) {
        const int width = min(DBK, D - (bt >> 1) * DBK);   // of the chunk
        const uint32_t col = static_cast<uint32_t>((bt >> 1) * 2 * DBK + (bt & 1) * width);
        uint32_t dk = static_cast<uint32_t>(bot * SO) * w_row + col * 2u + i * b_step8;
        asm volatile("" : "+s"(dk));
        copy_to_lds(rsb, cc[i & 1] < width ? vb[i & 1] + dk : kBufOOB, lds + wave * kDCopies * 1024 + i * 1024);
    };
    auto next_b = [&]() {
        if (++bt == 2 * chunks_of(bot)) {
            bt = 0;
            if (++bot == n_ot) {
                bot = 0;
                ++bl;
            }
        }
    };

    // fragment byte offsets inside a slab: lane l reads row (l % 32) of each
    // 32-row block, logical chunk 2 ks + (l / 32) at position chunk ^ sw; the
    // wave's output block j is 2 j + (j & 1 ^ wn)
    const int sw = (lane >> 1) & 7;
    uint32_t fo[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
        fo[ks] = static_cast<uint32_t>((lane & 31) * 128 + ((2 * ks + (lane >> 5)) ^ sw) * 16);
    const int ua = wm * 128 * 128, ub[2] = {wn * 4096, (1 - wn) * 4096};   // wave-uniform parts

    Acc acc;
    float psum[4] = {0.f, 0.f, 0.f, 0.f};
    zero_acc(acc);
    bf16x8 fa[2][4], fb[2][4];
    // fragment read q (0..7) of a 16-wide step: A block q/2 for even q, B block q/2 for odd q
    auto ldfrag1 = [&](int f, const uint8_t *abase, const uint8_t *bbase, int ks, int q) {
        const int i = q >> 1;
        if (q & 1)
            fb[f][i] = as_bf16x8(*reinterpret_cast<const u32x4 *>(bbase + ub[i & 1] + fo[ks] + 2 * i * 4096));
        else
            fa[f][i] = as_bf16x8(*reinterpret_cast<const u32x4 *>(abase + ua + fo[ks] + i * 4096));
    };

    // One step: W slab t (stage sb) against the gradient slab of its chunk
    // (stage sa).  FIRST (first step of a chunk): also copies the next
    // gradient slab, into the other A stage, whose previous slab was last
    // read in the step before this one.  J0: the first of the wave's output
    // blocks that the chunk meets.
    int sa = 0, sb = 0;
    auto step = [&](auto first_tag, auto j0_tag) {
        constexpr bool FIRST = decltype(first_tag)::value;
        constexpr int J0 = decltype(j0_tag)::value;
        auto mfma1 = [&](int f, int idx) {
            const int i = idx >> 2, j = idx & 3;
            if (j >= J0) acc[i][j] = mfma32_bf16(fa[f][i], fb[f][j], acc[i][j]);
        };
        const uint8_t *abase = smem + sa * kDSlab, *bbase = smem + kDLdsB + sb * kDSlab;
        const int nb1 = sb == 2 ? 0 : sb + 1;   // stage of W step t + 1
        const int nb2 = sb == 0 ? 2 : sb - 1;   // stage of W step t + 2 (held step t - 1)
        const int na = FIRST ? sa : sa ^ 1;     // gradient stage of step t + 1
        const uint32_t la = lds0 + (sa ^ 1) * kDSlab, lb = lds0 + kDLdsB + nb2 * kDSlab;
        const auto rsa = rsrc_a();
        const auto rsb = rsrc_b();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < 3; ++ks) {
            const int f = ks & 1;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                mfma1(f, 2 * q);
                mfma1(f, 2 * q + 1);
                if (ks == 0 && FIRST) issue_a(rsa, la, q);
                if (ks == 1) issue_b(rsb, lb, q);
                ldfrag1(f ^ 1, abase, bbase, ks + 1, q);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (FIRST) next_a();
        next_b();
#pragma unroll
        for (int m = 0; m < 8; ++m) mfma1(1, m);
        __builtin_amdgcn_sched_barrier(0);
        // outstanding copies allowed: this step's (A + B after a FIRST step, B after a second)
        if (FIRST)
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(2 * kDCopies) : "memory");
        else
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(kDCopies) : "memory");
        const uint8_t *nabase = smem + na * kDSlab, *nbbase = smem + kDLdsB + nb1 * kDSlab;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            ldfrag1(0, nabase, nbbase, 0, q);
            mfma1(1, 8 + q);
            __builtin_amdgcn_sched_barrier(0);
        }
        sa = na;
        sb = nb1;
    };
    auto chunk = [&](auto j0_tag) {
        step(std::integral_constant<bool, true>(), j0_tag);
        step(std::integral_constant<bool, false>(), j0_tag);
    };

    {   // prologue: gradient slab 0, W steps 0 and 1
        const auto rsa0 = rsrc_a();
        const auto rsb0 = rsrc_b();
#pragma unroll
        for (int q = 0; q < 8; ++q) issue_a(rsa0, lds0, q);
        next_a();
#pragma unroll
        for (int q = 0; q < 8; ++q) issue_b(rsb0, lds0 + kDLdsB, q);
        next_b();
        const auto rsb1 = rsrc_b();
#pragma unroll
        for (int q = 0; q < 8; ++q) issue_b(rsb1, lds0 + kDLdsB + kDSlab, q);
        next_b();
    }
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"(kDCopies) : "memory");
#pragma unroll
    for (int q = 0; q < 8; ++q) ldfrag1(0, smem, smem + kDLdsB, 0, q);
    for (int l = l0; l < l1; ++l)
        for (int ot = 0; ot < n_ot; ++ot) {
            // as loops of 0 or 1 passes: branches around the steps would copy the accumulators
            const int diag = chunks_of(ot) - 4 * ot;   // 1 .. 4
            const int n0 = 4 * ot + 1, n1 = min(diag / 2, 1), n2 = min(diag / 3, 1), n3 = diag / 4;
            for (int c = 0; c < n0; ++c) chunk(std::integral_constant<int, 0>());
            for (int c = 0; c < n1; ++c) chunk(std::integral_constant<int, 1>());
            for (int c = 0; c < n2; ++c) chunk(std::integral_constant<int, 2>());
            for (int c = 0; c < n3; ++c) chunk(std::integral_constant<int, 3>());
            fold_rows(acc, psum, lane);
        }
    // the copies past the last block are still in flight
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    if (gridDim.y > 1)
        finish_rows(psum, reinterpret_cast<float *>(smem), tid, lane, wm, wn, nrows, r0, part + blockIdx.y * rows, nullptr);
    else
        finish_rows(psum, reinterpret_cast<float *>(smem), tid, lane, wm, wn, nrows, r0, self_out, rsqrt_out);
}

// The sums of the ranges of blocks, in order.
__global__ __launch_bounds__(256) void k_self_influence_fold(const float *__restrict__ part, int64_t rows, int ranges,
                                                             float *__restrict__ self_out, float *__restrict__ rsqrt_out) {
    const int64_t j = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (j >= rows) return;
    float sv = part[j];
    for (int r = 1; r < ranges; ++r) sv += part[r * rows + j];
    if (self_out) self_out[j] = sv;
    if (rsqrt_out) rsqrt_out[j] = sv > 0.f ? 1.0f / sqrtf(sv) : 0.f;
}

// fp32 gradients: one workgroup per gradient; thread d forms output d of W_l g_l
// with the hi + lo halves (all D columns), a fixed-order block sum adds the
// squares, blocks in order.  For small problems.
__global__ __launch_bounds__(256) void k_self_influence_rows(const float *__restrict__ g, int64_t ld, int D,
                                                             int n_blocks, const bf16_bits *__restrict__ w_hi,
                                                             const bf16_bits *__restrict__ w_lo,
                                                             float *__restrict__ self_out,
                                                             float *__restrict__ rsqrt_out) {
    __shared__ float red[256];
    const int64_t j = blockIdx.x;
    const int tid = threadIdx.x;
    const int Dp = (D + 255) / 256 * 256;
    float total = 0.f;
    for (int l = 0; l < n_blocks; ++l) {
        const float *gl = g + j * ld + static_cast<int64_t>(l) * D;
        float part = 0.f;
        for (int d = tid; d < D; d += 256) {
            const bf16_bits *h = w_hi + (static_cast<size_t>(l) * Dp + d) * D;
            const bf16_bits *lo = w_lo + (static_cast<size_t>(l) * Dp + d) * D;
            float y = 0.f;
            for (int k = 0; k < D; ++k)
                y = __builtin_fmaf(bf16_to_f32(h[k]) + bf16_to_f32(lo[k]), gl[k], y);
            part = __builtin_fmaf(y, y, part);
        }
        red[tid] = part;
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if (tid < w) red[tid] += red[tid + w];
            __syncthreads();
        }
        if (tid == 0) total += red[0];
        __syncthreads();
    }
    if (tid == 0) {
        if (self_out) self_out[j] = total;
        if (rsqrt_out) rsqrt_out[j] = total > 0.f ? 1.0f / sqrtf(total) : 0.f;
    }
}

}  // namespace

hipError_t launch_self_influence(const void *g, bool bf16, int64_t ld, int64_t rows, int D, int n_blocks,
                                 const void *ws, float *self_out, float *rsqrt_out, hipStream_t s) {
    if (rows == 0) return hipSuccess;
    void *w = const_cast<void *>(ws);
    const bf16_bits *hi = self_influence_w(w, D, n_blocks, false), *lo = self_influence_w(w, D, n_blocks, true);
    if (self_influence_interleaved(bf16)) {
        // Ranges of blocks, so that the last round of workgroups is full: the
        // rounds times the blocks of a range plus one (the fill and the fold),
        // at its least; as many as fit in the preconditioner's solutions, which
        // are no longer needed.
        const int64_t wgs = (rows + SR - 1) / SR;
        size_t room = 0;
        float *part = self_influence_part(w, D, n_blocks, &room);
        int ranges = 1;
        int64_t best = 0;
        for (int r = 1; r <= n_blocks && r <= 256; ++r) {
            if (r > 1 && static_cast<size_t>(r) * rows * sizeof(float) > room) break;
            const int64_t cost = ((wgs * r + 255) / 256) * ((n_blocks + r - 1) / r + 1);
            if (r == 1 || cost < best) {
                best = cost;
                ranges = r;
            }
        }
        hipLaunchKernelGGL(k_self_influence_dma, dim3(static_cast<unsigned>(wgs), static_cast<unsigned>(ranges)), dim3(STH),
                           0, s, static_cast<const bf16_bits *>(g), ld, rows, D, n_blocks, hi, part, self_out, rsqrt_out);
        if (ranges > 1)
            hipLaunchKernelGGL(k_self_influence_fold, dim3(static_cast<unsigned>((rows + 255) / 256)), dim3(256), 0, s, part,
                               rows, ranges, self_out, rsqrt_out);
    } else {
        hipLaunchKernelGGL(k_self_influence_rows, dim3(static_cast<unsigned>(rows)), dim3(256), 0, s,
                           static_cast<const float *>(g), ld, D, n_blocks, hi, lo, self_out, rsqrt_out);
    }
    return hipGetLastError();
}

}  // namespace logra
