// Damped inverse applied to test gradients, per layer block (the iHVP step of
// the influence function, Sec. 2 Eq. (2), in the projected space of Eq. (3)):
//
//   C = S / N,  lambda = r * tr(C) / D   (r x mean eigenvalue, App. C)
//   out_q = (C + lambda I)^{-1} g_q
//
// All arithmetic is float64, the products on the fp64 matrix cores; S may be
// given in fp32 or fp64.  C + lambda I = L L^T is factored in column panels of
// 256 (one workgroup per layer block factors a panel's diagonal block and
// inverts its factor at the same time, W = L_II^{-1}, in registers):
//
//   D <= 256    k_factor reads S itself and leaves W; k_solve applies W, then
//               W^T, to 16 or 32 right-hand sides per workgroup out of LDS.
//   wider       k_lambda and k_form write A = C + lambda I (lower triangle);
//               for each panel I: its factor (W_II over A's diagonal block),
//               k_panel (L_JI = A_JI W_II^T), k_trail_next (A_JK -= L_JI L_KI^T for
//               the columns K of the next panel), k_trail_factor (the other
//               columns, and the next factor beside them).
//               Solve, forward: Y_I = W_II R_I (k_solve), R_J -= L_JI Y_I
//               (k_solve_gemm) for J > I; backward: Z_I = W_II^T Y_I, then
//               Y_J -= L_IJ^T Z_I for J < I.
//
// So no step is a row-by-row recurrence except the 16 x 16 diagonal blocks
// inside k_factor.
//
// Fragments.  A 16x16x4 fp64 MFMA takes from lane l row (column) l % 16 of each
// operand and contraction index l / 16.  Four of them contract 16 indices
// ("a unit"); index 2 (l / 16) + kx(i) goes to the i-th, for both operands, so
// that a row's 16 values are two loads, in each of which four lanes read 64
// contiguous bytes.
#include <type_traits>

#include "common.h"
#include "internal.h"

namespace logra {
namespace {

constexpr int PB = 256;   // column panel width
constexpr int FB = 16;    // block edge inside a panel
constexpr int kFactorThreads = 512;

__host__ __device__ constexpr int kx(int i) { return 8 * (i >> 1) + (i & 1); }   // 0, 1, 8, 9

struct WsLayout {
    double *A;      // [n_blocks][D][D] panel columns of L below the diagonal blocks, W_II in those
    double *lam;    // [n_blocks]
    int *info;      // [n_blocks] 0 or 1 + first non-positive pivot
    double *Y;      // [n_blocks][D][Qp] solutions (D > 256)
};

inline int padded_q(int Q) { return (Q + 63) / 64 * 64; }

inline WsLayout ws_layout(void *ws, int D, int n_blocks) {
    char *p = static_cast<char *>(ws);
    const size_t nb = static_cast<size_t>(n_blocks);
    WsLayout w;
    w.A = reinterpret_cast<double *>(p);
    p += align256(sizeof(double) * nb * D * D);
    w.lam = reinterpret_cast<double *>(p);
    p += align256(sizeof(double) * nb);
    w.info = reinterpret_cast<int *>(p);
    p += align256(sizeof(int) * nb);
    w.Y = reinterpret_cast<double *>(p);
    return w;
}

// An element of a gradient array of dtype `dt` (a DtypeCode).
__device__ __forceinline__ double load_any(const void *p, int dt, int64_t i) {
    if (dt == kBF16) return load_in_d<bf16_bits>(static_cast<const bf16_bits *>(p) + i);
    if (dt == kF64) return static_cast<const double *>(p)[i];
    return load_in_d<float>(static_cast<const float *>(p) + i);
}
// f(a value of the element type of dtype `dt`)
template <typename F>
__device__ __forceinline__ void with_dtype(int dt, F f) {
    if (dt == kBF16)
        f(bf16_bits{});
    else if (dt == kF64)
        f(double{});
    else
        f(float{});
}

template <typename TS>
__global__ __launch_bounds__(256) void k_lambda(const TS *S, int D, int64_t N, double r,
                                                double *lam) {
    __shared__ double part[256];
    const int blk = blockIdx.x;
    const TS *Sb = S + static_cast<size_t>(blk) * D * D;
    double s = 0.0;
    for (int d = threadIdx.x; d < D; d += 256) s += load_in_d<TS>(Sb + static_cast<size_t>(d) * D + d);
    part[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) lam[blk] = r * (part[0] / static_cast<double>(N)) / static_cast<double>(D);
}

template <typename TS>
__global__ __launch_bounds__(256) void k_form(const TS *S, int D, int64_t N, const double *lam,
                                              double *A, int *info) {
    const int blk = blockIdx.y, i = blockIdx.x;
    const TS *Sr = S + (static_cast<size_t>(blk) * D + i) * D;
    double *Ar = A + (static_cast<size_t>(blk) * D + i) * D;
    const double inv = 1.0 / static_cast<double>(N);
    for (int j = threadIdx.x; j <= i; j += 256) {
        double v = load_in_d<TS>(Sr + j) * inv;
        if (j == i) v += lam[blk];
        Ar[j] = v;
    }
    if (i == 0 && threadIdx.x == 0) info[blk] = 0;
}

__device__ __forceinline__ f64x4 mma_unit(const double (&a)[4], const double (&b)[4], f64x4 c) {
#pragma unroll
    for (int i = 0; i < 4; ++i) c = mfma16_f64(a[i], b[i], c);
    return c;
}
// acc[x][y] += a[x] b[y] over a unit, the four products of one block apart
template <int FX, int FY>
__device__ __forceinline__ void mma_units(const double (&a)[FX][4], const double (&b)[FY][4], f64x4 (&acc)[FX][FY]) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int x = 0; x < FX; ++x)
#pragma unroll
            for (int y = 0; y < FY; ++y) acc[x][y] = mfma16_f64(a[x][i], b[y][i], acc[x][y]);
}

// Barrier for data in LDS alone: memory operations in flight stay in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Factor of the (at most) 256 x 256 diagonal block at c0 of each layer block and
// the inverse W of that factor, whose lower triangle replaces the block's in A.
// (The factor itself is not needed again.)  One workgroup of 8 waves.
//
// Seven waves hold the block as 16 x 16 blocks (hi, lo), lo <= hi, in MFMA
// accumulators, up to 20 each, transposed and negated.  Step s eliminates block column s
// of [A; I]: the rows of A below (blocks (i, s)) and the rows of I above
// (X = L^{-T}, nonzero in blocks (t, s), t <= s) take the same operations.  A
// block (i, s) of A is final after step s, and X's block (s, i) starts there,
// so accumulator (hi, lo) holds A(hi, lo) up to step lo and X(lo, hi) from then
// to step hi.  A step:
//   1  the owner of (s, s) brings it up to date and hands it over in LDS;
//   2  the eighth wave factors it, a row per lane, with the rows of I below it
//      in the next 16 lanes, which end as X_ss = L_ss^{-T}; meanwhile the others
//      bring their open blocks up to date with step s - 1: acc += P P^T;
//   3  column s: the owners multiply their blocks by X_ss (a transposed
//      accumulator is the B operand as it stands) into P, 256 rows of 16 in LDS,
//      and store those of X, which are rows of W.
// Rows and columns past the block are identity rows.  With FROM_S (D <= 256)
// the block is read from S: S / N + lambda I, lambda formed here.
// Bound by fp64 MFMA issue on one CU (11 MFLOP) and by the chain of the 16
// pivots of a diagonal block (a SIMD that issues fp64 MFMAs lets one vector
// instruction of another wave through per MFMA, so the eighth wave's partner
// has to run dry first).  Measured: 224 blocks of 256 119 to 125 us, one 111; with the
// factor, panel, update and tile-inverse kernels of 64-wide steps before it:
// 790 us.  All 128 products of panel and pivots in every wave, publication of
// each column through LDS and both triangles of W stored: 185.
constexpr int kPRow = FB + 2;   // LDS row in doubles: 144 bytes, the 64 lanes of a fragment read spread evenly
template <typename TS, bool FROM_S>
__device__ __forceinline__ void factor_block(const TS *S_all, int64_t N, double r, double *A_all, int D, int c0, int *info,
                                             int blk) {
    constexpr int kOwners = 7, kSlots = 20;
    __shared__ __attribute__((aligned(16))) double P[PB * kPRow];
    __shared__ __attribute__((aligned(16))) double Dg[FB * kPRow];   // the diagonal block of the step
    __shared__ __attribute__((aligned(16))) double Xs[FB * kPRow];   // X_ss
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = lane & 15, kg = lane >> 4;
    double *A = A_all + static_cast<size_t>(blk) * D * D + static_cast<size_t>(c0) * D + c0;
    const TS *S = FROM_S ? S_all + static_cast<size_t>(blk) * D * D : nullptr;
    const int w = D - c0 < PB ? D - c0 : PB, nblk = (w + FB - 1) / FB;

    double inv_n = 1.0, lam = 0.0;
    if (FROM_S) {
        if (tid < PB) P[tid] = tid < w ? load_in_d<TS>(S + static_cast<size_t>(tid) * D + tid) : 0.0;
        __syncthreads();
        for (int o = PB / 2; o > 0; o >>= 1) {
            if (tid < o) P[tid] += P[tid + o];
            __syncthreads();
        }
        lam = r * (P[0] / static_cast<double>(N)) / static_cast<double>(D);
        inv_n = 1.0 / static_cast<double>(N);
        __syncthreads();
    }

    if (wave == kOwners) {   // the eighth wave; its barriers pair with the owners' below
        int bad = 0;         // 1 + first non-positive pivot
        for (int s = 0; s < nblk; ++s) {
            lds_barrier();
            double x[FB];
#pragma unroll
            for (int k = 0; k < FB; ++k) x[k] = Dg[row * kPRow + k];
#pragma unroll
            for (int k = 0; k < FB; ++k) x[k] = lane < FB ? x[k] : (k == row ? 1.0 : 0.0);
            // Pivot j's column, then the one update that the next pivot waits for,
            // then the others beside the next reciprocal root (the order is fixed:
            // left alone, each column's updates move into the chain of its pivot).
            double piv = readlane_d(x[0], 0), mine = piv;   // lane j keeps pivot j
            double inv = rsqrt_d<true>(piv);
#pragma unroll
            for (int j = 0; j < FB; ++j) {
                x[j] *= inv;
                __builtin_amdgcn_sched_barrier(0);
                if (j + 1 < FB) {
                    x[j + 1] = fma(-x[j], readlane_d(x[j], j + 1), x[j + 1]);
                    piv = readlane_d(x[j + 1], j + 1);
                    mine = lane == j + 1 ? piv : mine;
                    __builtin_amdgcn_sched_barrier(0);
                    inv = rsqrt_d<true>(piv);
#pragma unroll
                    for (int k = j + 2; k < FB; ++k) x[k] = fma(-x[j], readlane_d(x[j], k), x[k]);
                }
            }
            // a non-positive pivot spoils what follows it (the call then fails); the first one is kept
            const uint64_t neg = __builtin_amdgcn_ballot_w64(lane < FB && !(mine > 0.0));
            if (neg != 0 && bad == 0) bad = c0 + FB * s + 1 + __builtin_ctzll(neg);
            if (kg == 1) {   // lanes 16-31: rows of X_ss, which are columns of W_ss
#pragma unroll
                for (int k = 0; k < FB; ++k) Xs[row * kPRow + k] = x[k];
#pragma unroll
                for (int k = 0; k < FB; ++k)
                    if (k >= row && FB * s + k < w) A[static_cast<size_t>(FB * s + k) * D + FB * s + row] = x[k];
            }
            lds_barrier();
            if (kg == 1) {   // block s of P; the owners are past their reads of the old one
#pragma unroll
                for (int k = 0; k < FB; ++k) P[(FB * s + row) * kPRow + k] = x[k];
            }
            lds_barrier();
        }
        if (lane == 0 && (FROM_S || bad)) {
            if (FROM_S)
                info[blk] = bad;
            else if (info[blk] == 0)
                info[blk] = bad;
        }
        return;
    }

    // Slot u of a wave is block number wave + 7 u of the lower triangle, row by
    // row.  Lane u keeps its (hi, lo) (PB: past the last one), so that a step
    // finds the slots it meets with one ballot.
    int my_hi = PB, my_lo = PB;
    {
        const int b = wave + kOwners * lane;
        int h = 0;
        while ((h + 1) * (h + 2) / 2 <= b) ++h;
        if (lane < kSlots && h < nblk) {
            my_hi = h;
            my_lo = b - h * (h + 1) / 2;
        }
    }
    f64x4 acc[kSlots];
    TS raw[kSlots][4];
#pragma unroll
    for (int u = 0; u < kSlots; ++u) {
        const int h = __builtin_amdgcn_readlane(my_hi, u), l = __builtin_amdgcn_readlane(my_lo, u);
#pragma unroll
        for (int q = 0; q < 4; ++q) {   // -block^T: row kg + 4 q, column `row`
            const int i = FB * h + row, j = FB * l + kg + 4 * q;
            const int rr = i > j ? i : j, cc = i > j ? j : i;   // only the lower triangle is read
            const uint32_t at = rr < w ? static_cast<uint32_t>(rr) * D + cc : 0u;   // past the block: any element
            raw[u][q] = FROM_S ? S[at] : static_cast<TS>(A[at]);
        }
    }
#pragma unroll
    for (int u = 0; u < kSlots; ++u) {
        const int h = __builtin_amdgcn_readlane(my_hi, u), l = __builtin_amdgcn_readlane(my_lo, u);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = FB * h + row, j = FB * l + kg + 4 * q;
            double v = static_cast<double>(raw[u][q]);
            if (FROM_S) v = i == j ? v * inv_n + lam : v * inv_n;
            acc[u][q] = -((i > j ? i : j) < w ? v : (i == j ? 1.0 : 0.0));
        }
    }
    // LDS byte offsets of the fragments of block rows: uniform part in a register
    const uint32_t frag0 = static_cast<uint32_t>((row * kPRow + 2 * kg) * 8);
    constexpr uint32_t kBlkBytes = FB * kPRow * 8;
    auto load4 = [&](double (&v)[4], int blk_row) {
        const double *src = reinterpret_cast<const double *>(reinterpret_cast<const char *>(P) + blk_row * kBlkBytes + frag0);
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = src[kx(i)];
    };
    for (int s = 0; s < nblk; ++s) {
        const int diag = s * (s + 3) / 2 - wave;   // number of block (s, s) less the wave's first
        const uint32_t own = diag >= 0 && diag % kOwners == 0 ? 1u << (diag / kOwners) : 0u;
        if (own) {
#pragma unroll
            for (int u = 0; u < kSlots; ++u)
                if (own & (1u << u)) {
                    if (s > 0) {
                        double f[4];
                        load4(f, s);
                        acc[u] = mma_unit(f, f, acc[u]);
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) Dg[row * kPRow + kg + 4 * q] = -acc[u][q];
                }
        }
        lds_barrier();
        if (s > 0) {
            const uint32_t open = static_cast<uint32_t>(__builtin_amdgcn_ballot_w64(my_hi >= s && my_hi < PB)) & ~own;
            const bool low = my_lo >= s;   // still a block of A
            const int my_rb = low ? my_hi : my_lo, my_cb = low ? my_lo : my_hi;
#pragma unroll
            for (int u = 0; u < kSlots; u += 2) {   // two slots' fragments at a time
                if (!(open & (3u << u))) continue;
                double pr[2][4], pc[2][4];
#pragma unroll
                for (int v = 0; v < 2; ++v) {   // a slot that is not open reads some block in range
                    load4(pr[v], __builtin_amdgcn_readlane(my_rb, u + v) & 15);
                    load4(pc[v], __builtin_amdgcn_readlane(my_cb, u + v) & 15);
                }
                if (open & (1u << u)) acc[u] = mma_unit(pc[0], pr[0], acc[u]);
                if (open & (2u << u)) acc[u + 1] = mma_unit(pc[1], pr[1], acc[u + 1]);
            }
        }
        lds_barrier();
        const uint32_t col = static_cast<uint32_t>(__builtin_amdgcn_ballot_w64((my_lo == s) != (my_hi == s)));
        double xs[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) xs[q] = -Xs[(kg + 4 * q) * kPRow + row];   // contraction index kg + 4 q
#pragma unroll
        for (int u = 0; u < kSlots; ++u)
            if (col & (1u << u)) {
                const int h = __builtin_amdgcn_readlane(my_hi, u), l = __builtin_amdgcn_readlane(my_lo, u);
                const bool low = l == s;
                const int rb = low ? h : l;
                double y[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) y[q] = acc[u][q];
                const f64x4 v = mma_unit(xs, y, f64x4{0.0, 0.0, 0.0, 0.0});
#pragma unroll
                for (int q = 0; q < 4; ++q) P[(rb * FB + row) * kPRow + kg + 4 * q] = v[q];
                if (!low) {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (FB * s + kg + 4 * q < w)
                            A[static_cast<size_t>(FB * s + kg + 4 * q) * D + FB * rb + row] = v[q];
                }
                acc[u] = f64x4{0.0, 0.0, 0.0, 0.0};
            }
        lds_barrier();
    }
}

template <typename TS, bool FROM_S>
__global__ __launch_bounds__(kFactorThreads, 2) void k_factor(const TS *S_all, int64_t N, double r, double *A_all, int D,
                                                              int c0, int *info) {
    factor_block<TS, FROM_S>(S_all, N, r, A_all, D, c0, info, blockIdx.x);
}

// Y = W R and / or Z = W^T Y for the diagonal block at c0 (width w <= 256, the
// lower triangle of W in A): one workgroup per 16 NC right-hand sides, which it keeps in LDS ([row][query],
// padded by 4); 8 waves.  Block rows of 16 are dealt so that waves do equal
// work on the triangles: wave v takes rows v and 15 - v (NBK = 16 block rows;
// 8: row v; 4: row v % 4 and half of the columns).  A wave streams its rows (or
// columns) of W from memory, mostly the L2, four units ahead, and reads the
// right-hand sides as LDS fragments.  Measured, 224 blocks of 256, 1,024
// right-hand sides (30 GFLOP): 650 to 740 us by run (675 in the benchmark's trace) in
// workgroups of 32, 885 in workgroups of 64, whose loads and stores no second workgroup of the CU covers; blocked
// substitution in 64-wide steps took 1,200.
enum SolveSrc { kFromG = 0, kFromY = 1, kFromIdent = 2 };
struct SolveArgs {
    const double *A;       // [n_blocks][D][D]
    double *Y;             // [n_blocks][D][Qp]
    const void *g;         // right-hand sides (kFromG)
    void *out;             // results, or NULL
    int64_t ld_in, ld_out;
    int D, c0, Q, Qp, in_dt, out_dt;
    int src;               // where the right-hand sides come from
    int fwd, bwd;          // apply W, then W^T
    int to_y;              // write the result to Y
    int wg0;               // number of the launch's first workgroup
};

template <int NBK, int NC>
__global__ __launch_bounds__(512, 4) void k_solve(SolveArgs p) {
    constexpr int kLd = 16 * NC + 4;   // fragment reads spread evenly over the banks
    constexpr int kGroups = NBK == 16 ? 2 : 1;
    constexpr int kHalves = NBK == 4 && NC > 1 ? 2 : 1;
    constexpr int kCols = NC / kHalves;
    constexpr int kBat = NBK == 4 ? 2 : 4;
    __shared__ __attribute__((aligned(16))) double R[NBK * FB * kLd];
    const int blk = blockIdx.y, q0 = (p.wg0 + static_cast<int>(blockIdx.x)) * 16 * NC, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = lane & 15, kg = lane >> 4;
    const int D = p.D, w = D - p.c0 < NBK * FB ? D - p.c0 : NBK * FB, nblk = (w + FB - 1) / FB;
    const double *M = p.A + static_cast<size_t>(blk) * D * D + static_cast<size_t>(p.c0) * D + p.c0;
    double *Y = p.Y ? p.Y + (static_cast<size_t>(blk) * D + p.c0) * p.Qp : nullptr;
    const int64_t col0 = static_cast<int64_t>(blk) * D + p.c0;

    // the right-hand sides, eight loads of a thread in flight
    if (p.src == kFromG) {   // a wave per row of g, consecutive lanes on consecutive elements
        const int per = (nblk * FB + 63) / 64, all = 2 * NC * per;   // 64-element pieces of the wave's 2 NC rows
        with_dtype(p.in_dt, [&](auto tag) {
            using T = decltype(tag);
            const T *src = static_cast<const T *>(p.g);
            for (int e0 = 0; e0 < all; e0 += 8) {
                T v[8];
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const int e = e0 + t, q = wave + 8 * (e / per), d = lane + 64 * (e % per);
                    v[t] = src[e < all && q0 + q < p.Q && d < w ? (q0 + q) * p.ld_in + col0 + d : col0];
                }
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const int e = e0 + t, q = wave + 8 * (e / per), d = lane + 64 * (e % per);
                    if (e < all && d < nblk * FB) R[d * kLd + q] = q0 + q < p.Q && d < w ? load_in_d<T>(&v[t]) : 0.0;
                }
            }
        });
    } else {
        const int all = 16 * NC * nblk * FB;
        for (int e0 = tid; e0 < all; e0 += 8 * 512) {
            double v[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const int e = e0 + 512 * t, d = e / (16 * NC), q = e % (16 * NC);
                const bool ident = p.src == kFromIdent && q0 + q >= p.c0, in = e < all && d < w && !ident;
                v[t] = Y[in ? static_cast<size_t>(d) * p.Qp + q0 + q : q0];
                v[t] = in ? v[t] : ident && p.c0 + d == q0 + q ? 1.0 : 0.0;
            }
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const int e = e0 + 512 * t, d = e / (16 * NC), q = e % (16 * NC);
                if (e < all) R[d * kLd + q] = v[t];
            }
        }
    }
    __syncthreads();

    const int ch = kHalves == 2 ? wave >> 2 : 0;   // column half
    int g[kGroups];
    g[0] = NBK == 4 ? wave & 3 : wave;
    if (kGroups == 2) g[kGroups - 1] = 15 - wave;
    if (NBK == 4 && kHalves == 1 && wave >= 4) g[0] = NBK;   // no rows left
    // Four values of unit u for row i = 16 gr + row: of W (indices up to i), or of
    // W^T (indices from i on: a column of W), a wave-uniform base and a lane's
    // offset.  In the diagonal unit the others are made zero; so are, in the
    // backward direction, indices past w, which read the workspace behind A
    // (at most 15 rows; Y alone has 64).  Forward, those lie in diagonal units.
    const bool ragged = w % FB != 0;
    auto frag = [&](double (&a)[4], uint32_t off, int u, bool back) {
        const char *base = reinterpret_cast<const char *>(back ? M + static_cast<size_t>(FB * u) * D : M + FB * u);
#pragma unroll
        for (int t = 0; t < 4; ++t)
            a[t] = *reinterpret_cast<const double *>(base + (back ? static_cast<size_t>(kx(t)) * D : kx(t)) * sizeof(double) + off);
    };
    auto mask = [&](double (&a)[4], int gr, int u, bool back) {
        const int i = FB * gr + row, k0 = FB * u + 2 * kg;
        const int from = back && u == gr ? i : 0, to = !back && u == gr ? i : w - 1;
#pragma unroll
        for (int t = 0; t < 4; ++t) a[t] = k0 + kx(t) >= from && k0 + kx(t) <= to ? a[t] : 0.0;
    };
    f64x4 acc[kGroups][kCols];
    // Units of a block row go in batches of kBat: one is on its way while the
    // one before it is multiplied.  (Next to fp64 MFMAs, vector instructions of
    // the other waves issue one per MFMA, so there are few: addresses are
    // scalar and only diagonal units are masked.)
    auto pass = [&](bool back) {
#pragma unroll
        for (int x = 0; x < kGroups; ++x) {
#pragma unroll
            for (int c = 0; c < kCols; ++c) acc[x][c] = f64x4{0.0, 0.0, 0.0, 0.0};
            const int gr = g[x];
            if (gr >= nblk) continue;
            const int i = FB * gr + row, ic = i < w ? i : 0;
            const uint32_t off = 8u * (back ? 2u * kg * D + ic : static_cast<uint32_t>(ic) * D + 2u * kg);
            const int u0 = back ? gr : 0, end = back ? nblk : gr + 1;
            double a[2][kBat][4];
#pragma unroll
            for (int v = 0; v < kBat; ++v)
                if (u0 + v < end) frag(a[0][v], off, u0 + v, back);
#pragma unroll
            for (int t = 0; t < NBK / kBat; ++t) {
                const int u = u0 + t * kBat;
                if (u >= end) break;
#pragma unroll
                for (int v = 0; v < kBat; ++v)
                    if (u + kBat + v < end) frag(a[(t + 1) & 1][v], off, u + kBat + v, back);
#pragma unroll
                for (int v = 0; v < kBat; ++v) {
                    if (u + v >= end) break;
                    double b[kCols][4];
#pragma unroll
                    for (int c = 0; c < kCols; ++c)
#pragma unroll
                        for (int i4 = 0; i4 < 4; ++i4)
                            b[c][i4] = R[(FB * (u + v) + 2 * kg + kx(i4)) * kLd + 16 * (kCols * ch + c) + row];
                    if (u + v == gr || (ragged && back && u + v == nblk - 1)) mask(a[t & 1][v], gr, u + v, back);
#pragma unroll
                    for (int i4 = 0; i4 < 4; ++i4)
#pragma unroll
                        for (int c = 0; c < kCols; ++c) acc[x][c] = mfma16_f64(a[t & 1][v][i4], b[c][i4], acc[x][c]);
                }
            }
        }
    };
    // f(row, column, value) over the wave's results (of no meaning in rows past w)
    auto each = [&](auto f) {
#pragma unroll
        for (int x = 0; x < kGroups; ++x)
            if (g[x] < nblk) {
#pragma unroll
                for (int c = 0; c < kCols; ++c)
#pragma unroll
                    for (int q = 0; q < 4; ++q) f(FB * g[x] + kg + 4 * q, 16 * (kCols * ch + c) + row, acc[x][c][q]);
            }
    };
    auto to_lds = [&]() {
        __syncthreads();
        each([&](int d, int q, double v) { R[d * kLd + q] = d < w ? v : 0.0; });
        __syncthreads();
    };
    if (p.fwd) pass(false);
    if (p.bwd) {
        if (p.fwd) to_lds();
        pass(true);
    }
    if (p.to_y)
        each([&](int d, int q, double v) {
            if (d < w) Y[static_cast<size_t>(d) * p.Qp + q0 + q] = v;
        });
    if (p.out) {   // whole rows, through LDS
        to_lds();
        with_dtype(p.out_dt, [&](auto tag) {
            using T = decltype(tag);
            for (int q = wave; q < 16 * NC && q0 + q < p.Q; q += 8) {
                T *dst = static_cast<T *>(p.out) + (q0 + q) * p.ld_out + col0;
#pragma unroll 4
                for (int d = lane; d < w; d += 64) store_out_d<T>(dst + d, R[d * kLd + q]);
            }
        });
    }
}

// Panel below the diagonal block at c0: L_J = A_J W^T in place, 32 rows per
// workgroup, two workgroups a CU.  Wave (rh, ch) has rows 16 rh.., held in
// registers, and the 16-column blocks c % 2 == ch, which need indices up to
// their own column only: 72 products of a unit.  W's rows go through a ring of
// eight stages in LDS, one of 32 rows (both halves' block) x two units, seven
// ahead, so that a CU fetches W once per workgroup: fetched by each wave into
// registers it is four times that, at about 50 GB/s a CU.
// Measured: seven 4,096-wide layer blocks' panels 0.54 ms (0.76 from registers).
__global__ __launch_bounds__(256, 2) void k_panel(double *A_all, int D, int c0) {
    constexpr int kUnits = PB / FB, kPairs = kUnits / 2, kSteps = kPairs * (kPairs + 1) / 2;
    constexpr int kStages = 8, kStage = 32 * 2 * 128;
    __shared__ __attribute__((aligned(1024))) uint8_t ring[kStages * kStage];
    const int blk = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rh = wave >> 1, ch = wave & 1, row = lane & 15, kg = lane >> 4;
    double *A = A_all + static_cast<size_t>(blk) * D * D;
    const int r0 = c0 + PB + blockIdx.x * 32 + 16 * rh;
    const int ir = r0 + row < D ? r0 + row : D - 1;

    // Step s is units 2 k and 2 k + 1 of the blocks 2 c and 2 c + 1, c (c + 1) / 2 + k = s, k <= c (for block
    // 2 c the last unit lies above the diagonal and is masked whole).  Copy i of a wave: unit (wave >> 1) of
    // the step, rows 16 (wave & 1) + 8 i .. + 7, lane l chunk (l & 7) ^ ((row >> 1) & 7) of row l / 8.
    auto pair_of = [](int s) { return (s >= 1) + (s >= 3) + (s >= 6) + (s >= 10) + (s >= 15) + (s >= 21) + (s >= 28); };
    const auto rs = buf_rsrc_uniform(A, static_cast<uint32_t>(D) * D * 8u);
    uint32_t off[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = 16 * (wave & 1) + 8 * i + (lane >> 3);
        off[i] = 8u * (static_cast<uint32_t>(c0 + r) * D + c0) + 128u * (wave >> 1) + 16u * ((lane & 7) ^ ((r >> 1) & 7));
    }
    const uint32_t lds0 = lds_addr(ring) + wave * 2048;
    auto issue = [&](int s) {
        const int c = pair_of(s), k = s - c * (c + 1) / 2;
        const uint32_t d = 8u * 32u * c * static_cast<uint32_t>(D) + 256u * k;
#pragma unroll
        for (int i = 0; i < 2; ++i) copy_to_lds(rs, off[i] + d, lds0 + s % kStages * kStage + i * 1024);
    };
    auto wait = [](int stages) {   // until only the copies of that many stages are under way
        switch (stages) {
            case 0: asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); break;
            case 1: asm volatile("s_waitcnt vmcnt(2) lgkmcnt(0)\n\ts_barrier" ::: "memory"); break;
            case 2: asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier" ::: "memory"); break;
            case 3: asm volatile("s_waitcnt vmcnt(6) lgkmcnt(0)\n\ts_barrier" ::: "memory"); break;
            case 4: asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)\n\ts_barrier" ::: "memory"); break;
            case 5: asm volatile("s_waitcnt vmcnt(10) lgkmcnt(0)\n\ts_barrier" ::: "memory"); break;
            default: asm volatile("s_waitcnt vmcnt(12) lgkmcnt(0)\n\ts_barrier" ::: "memory"); break;
        }
    };
#pragma unroll
    for (int s = 0; s < kStages - 1; ++s) issue(s);
    const double *src = A + static_cast<size_t>(ir) * D + c0 + 2 * kg;
    double a[kUnits][4];
#pragma unroll
    for (int u = 0; u < kUnits; ++u)
#pragma unroll
        for (int t = 0; t < 4; ++t) a[u][t] = src[FB * u + kx(t)];
#pragma unroll
    for (int u = 0; u < kUnits; ++u)
#pragma unroll
        for (int t = 0; t < 4; ++t) asm volatile("" : "+v"(a[u][t]));   // here, so that no step waits for its rows
    uint32_t fo[2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
        fo[h] = static_cast<uint32_t>((16 * ch + row) * 128 + ((kg + 4 * h) ^ ((row >> 1) & 7)) * 16);
    f64x4 acc[kPairs];
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
        const int c = pair_of(s), k = s - c * (c + 1) / 2;
        // (stores come at the end, when every wave has long had its rows)
        wait(kSteps - 1 - s < kStages - 2 ? kSteps - 1 - s : kStages - 2);
        if (s + kStages - 1 < kSteps) issue(s + kStages - 1);   // the stage that step s - 1 read
        if (k == 0) acc[c] = f64x4{0.0, 0.0, 0.0, 0.0};
        double b[2][4];
#pragma unroll
        for (int v = 0; v < 2; ++v)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const double2 d = *reinterpret_cast<const double2 *>(ring + s % kStages * kStage + v * 4096 + fo[h]);
                b[v][2 * h] = d.x;
                b[v][2 * h + 1] = d.y;
            }
        if (k == c) {   // on or past the diagonal: index 16 u + 2 kg + kx(t) up to column 16 (2 c + ch) + row
#pragma unroll
            for (int v = 0; v < 2; ++v)
#pragma unroll
                for (int t = 0; t < 4; ++t) b[v][t] = FB * (v - ch) + 2 * kg + kx(t) <= row ? b[v][t] : 0.0;
        }
#pragma unroll
        for (int v = 0; v < 2; ++v) acc[c] = mma_unit(a[2 * k + v], b[v], acc[c]);
    }
#pragma unroll
    for (int c = 0; c < kPairs; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = r0 + kg + 4 * q;
            if (i < D) A[static_cast<size_t>(i) * D + c0 + FB * (2 * c + ch) + row] = acc[c][q];
        }
}

// C -= A_op B_op over the indices of the panel at c0: the trailing updates of
// the factor and the block steps of the solves.
constexpr int kTrailGroup = 6;
enum GemmMode { kTrailNext, kTrailRest, kForward, kBackward };   // A_JK -= L_JI L_KI^T (two parts), the solves
struct GemmArgs {
    double *A;
    double *Y;
    const void *g;    // first forward step: the right-hand sides are still here
    int64_t ld_in;
    int D, c0, Q, Qp, in_dt;
    int src;          // forward: where C's columns are (kFromIdent: zero from column c0 on)
};

// Trailing update, A_JK -= L_JI L_KI^T for the tile `tile` of 16 FX WX rows and as
// many columns.  A wave has FX x FY blocks of 16 x 16, a workgroup WX x WY waves.
// A unit of the operands (16 contiguous indices of the tile's rows, then of its
// columns' rows: 128 bytes each) is copied straight into a ring of three stages
// in LDS, two units ahead, chunk c of row r at position c ^ ((r >> 1) & 7), so
// that 16 lanes reading one chunk of 16 rows hit 16 banks; one barrier a unit.
// (Fragments loaded from memory by each wave instead ask the CU for three times
// the bytes, and it takes about 50 GB/s of such loads: 54 us a tile of 128 x 128
// where its MFMAs take 32.)  C is read beside the last products.
// Measured: seven 4,096-wide layer blocks' trailing updates 4.0 ms with the
// factors beside them (5.1 with fragments from memory, 13.6 in 64-wide steps of
// scalar fp64 FMAs).
template <int FX, int FY, int WX, int WY, int MODE>
__device__ __forceinline__ void trail_tile(const GemmArgs &p, int tile, int blk) {
    constexpr int kTx = 16 * FX * WX, kWaves = WX * WY, kStages = 3;
    constexpr int kStage = 2 * kTx * 128, kCopies = 2 * kTx / 8 / kWaves;   // bytes; 1 KB copies per wave and unit
    static_assert(FX * WX == FY * WY, "the triangle is cut into squares");
    __shared__ __attribute__((aligned(1024))) uint8_t ring[kStages * kStage];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = lane & 15, kg = lane >> 4;
    const int D = p.D, base = p.c0 + PB;   // first row updated
    double *A = p.A + static_cast<size_t>(blk) * D * D;
    int ti, tj;
    constexpr int kW = PB / kTx;   // the next panel's columns are the first kW tile columns
    if (MODE == kTrailNext) {      // of the lower triangle of tiles, row by row
        constexpr int kTri = kW * (kW + 1) / 2;
        ti = tile < kTri ? 0 : kW + (tile - kTri) / kW;
        if (tile < kTri)
            while ((ti + 1) * (ti + 2) / 2 <= tile) ++ti;
        tj = tile < kTri ? tile - ti * (ti + 1) / 2 : (tile - kTri) % kW;
    } else {
        // The other tile columns: tile rows in groups of kTrailGroup, column by
        // column within a group, so that the 32 tiles an XCD has in hand at a
        // time share about 12 operand panels (3 MB, its L2) instead of 33.
        int g = 0;
        while (kTrailGroup * kTrailGroup * (g + 1) * (g + 2) / 2 <= tile) ++g;
        const int rest = tile - kTrailGroup * kTrailGroup * g * (g + 1) / 2;
        ti = kTrailGroup * g + rest % kTrailGroup;
        tj = rest / kTrailGroup;
        if (tj > ti) return;   // a slot above the diagonal
        ti += kW;
        tj += kW;
        if (base + ti * kTx >= D) return;
    }
    const int it = base + ti * kTx, jt = base + tj * kTx;   // the tile's first row and column
    const int wx = wave / WY, wy = wave % WY;

    // copy i of this wave: stage rows 8 (kCopies wave + i) .. + 7, lane l chunk (l & 7) ^ ((row >> 1) & 7) of row l / 8
    const auto rs = buf_rsrc_uniform(A, static_cast<uint32_t>(D) * D * 8u);
    uint32_t off[kCopies];
#pragma unroll
    for (int i = 0; i < kCopies; ++i) {
        const int r = 8 * (kCopies * wave + i) + (lane >> 3);
        const int m = r < kTx ? it + r : jt + r - kTx;   // past D: the last row, not stored
        off[i] = 8u * (static_cast<uint32_t>(m < D ? m : D - 1) * D + p.c0) + 16u * ((lane & 7) ^ ((r >> 1) & 7));
    }
    const uint32_t lds0 = lds_addr(ring) + kCopies * wave * 1024;
    auto issue = [&](int u, int stage) {   // past the panel: a unit of the panel again, not used
        const uint32_t du = 128u * (u < PB / FB ? u : 0);
#pragma unroll
        for (int i = 0; i < kCopies; ++i) copy_to_lds(rs, off[i] + du, lds0 + stage * kStage + i * 1024);
    };
    // a lane's two 16-byte chunks of a fragment row (rows 16 apart share the swizzle)
    uint32_t fo[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) fo[h] = static_cast<uint32_t>(row * 128 + ((kg + 4 * h) ^ ((row >> 1) & 7)) * 16);
    auto frag = [&](double (&v)[4], const uint8_t *blk16) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const double2 d = *reinterpret_cast<const double2 *>(blk16 + fo[h]);
            v[2 * h] = d.x;
            v[2 * h + 1] = d.y;
        }
    };
    f64x4 acc[FX][FY];
#pragma unroll
    for (int x = 0; x < FX; ++x)
#pragma unroll
        for (int y = 0; y < FY; ++y) acc[x][y] = f64x4{0.0, 0.0, 0.0, 0.0};
    issue(0, 0);
    issue(1, 1);
    int cur = 0;
    f64x4 c[FX][FY];
    auto step = [&](int u) {
        // this wave's copies of unit u are done when only the next unit's remain; after the barrier every
        // wave's are, and every wave has read unit u - 1, whose stage the next copies refill
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(kCopies) : "memory");
        issue(u + 2, cur == 0 ? 2 : cur - 1);
        const uint8_t *st = ring + cur * kStage;
        double a[FX][4], b[FY][4];
#pragma unroll
        for (int x = 0; x < FX; ++x) frag(a[x], st + (16 * FX * wx + 16 * x) * 128);
#pragma unroll
        for (int y = 0; y < FY; ++y) frag(b[y], st + (kTx + 16 * FY * wy + 16 * y) * 128);
        mma_units(a, b, acc);
        cur = cur == 2 ? 0 : cur + 1;
    };
    for (int u = 0; u < PB / FB - 1; ++u) step(u);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the compiler's own loads follow
    const int i0 = it + 16 * FX * wx, j0 = jt + 16 * FY * wy;
#pragma unroll
    for (int x = 0; x < FX; ++x)
#pragma unroll
        for (int y = 0; y < FY; ++y)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = i0 + 16 * x + kg + 4 * q, j = j0 + 16 * y + row;
                c[x][y][q] = A[static_cast<size_t>(i < D ? i : D - 1) * D + (j < D ? j : D - 1)];
            }
    {   // the last unit: no more copies
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        const uint8_t *st = ring + cur * kStage;
        double a[FX][4], b[FY][4];
#pragma unroll
        for (int x = 0; x < FX; ++x) frag(a[x], st + (16 * FX * wx + 16 * x) * 128);
#pragma unroll
        for (int y = 0; y < FY; ++y) frag(b[y], st + (kTx + 16 * FY * wy + 16 * y) * 128);
        mma_units(a, b, acc);
    }
#pragma unroll
    for (int x = 0; x < FX; ++x)
#pragma unroll
        for (int y = 0; y < FY; ++y)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = i0 + 16 * x + kg + 4 * q, j = j0 + 16 * y + row;
                if (i < D && j < D) A[static_cast<size_t>(i) * D + j] = c[x][y][q] - acc[x][y][q];
            }
}

template <int FX, int FY, int WX, int WY>
__global__ __launch_bounds__(64 * WX * WY, 2) void k_trail_next(GemmArgs p) {
    trail_tile<FX, FY, WX, WY, kTrailNext>(p, blockIdx.x, blockIdx.y);
}

// Block step of a solve in tiles of 64 rows x 64 right-hand sides, four waves of
// 2 x 2 blocks of 16 x 16 (TAIL: a backward step from a panel narrower than 256).
// The ring of trail_tile, of units of 16 KB, three workgroups a CU: forward L's
// rows as there, backward (L^T) and for the right-hand sides 16 rows of the
// contraction, 64 columns each, whose two 128-byte halves of each 256 change
// places in every other pair of rows (lanes 16 apart read rows two apart).
// C is read beside the last products.
// Measured: seven 4,096-wide layer blocks, 256 right-hand sides: 1.38 ms for the
// 30 steps (1.59 with each wave's operands fetched into registers).
template <int MODE, bool TAIL>
__global__ __launch_bounds__(256, 3) void k_solve_gemm(GemmArgs p) {
    constexpr int F = 2, kT = 64, kStages = 3, kStage = 2 * 8192;
    __shared__ __attribute__((aligned(1024))) uint8_t ring[kStages * kStage];
    const int blk = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = lane & 15, kg = lane >> 4;
    const int D = p.D;
    const double *A = p.A + static_cast<size_t>(blk) * D * D;
    double *Y = p.Y + static_cast<size_t>(blk) * D * p.Qp;
    const int base = MODE == kBackward ? 0 : p.c0 + PB;   // first row updated
    const int rows_end = MODE == kBackward ? p.c0 : D;    // backward: a multiple of kT
    const int nq = p.src == kFromIdent && p.c0 + PB < p.Qp ? p.c0 + PB : p.Qp, ntq = (nq + kT - 1) / kT;
    const int it = base + static_cast<int>(blockIdx.x / ntq) * kT, jt = static_cast<int>(blockIdx.x % ntq) * kT;
    const int i0 = it + 32 * (wave >> 1), j0 = jt + 32 * (wave & 1);
    const int kn = TAIL ? D - p.c0 : PB;   // indices of the panel
    const int nu = TAIL ? (kn + FB - 1) / FB : PB / FB;

    // A wave's copies of a unit, 1 KB each: two of either operand.  Rows of the contraction: its rows 2 n and
    // 2 n + 1, n = 2 wave + i, of 64 columns from `from`; past D the last row, which is masked (TAIL).
    const uint32_t lds0 = lds_addr(ring) + wave * 2048;
    auto copy_rows = [&](const double *from, int ld, int u, uint32_t lds) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int k = FB * u + 4 * wave + 2 * i, kc = TAIL && k >= kn ? kn - 1 : k;
            const int second = TAIL && kc + 1 >= kn ? 0 : lane >> 5;
            const auto rs = buf_rsrc_uniform(from + static_cast<size_t>(kc) * ld, 8u * ld + 512u);
            copy_to_lds(rs, 8u * ld * second + 16u * ((lane & 31) ^ (8 * i)), lds + i * 1024);
        }
    };
    const auto rs_l = buf_rsrc_uniform(A, static_cast<uint32_t>(D) * D * 8u);
    uint32_t off[2];   // forward: rows of L, 128 bytes each, as in trail_tile
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = 16 * wave + 8 * i + (lane >> 3), m = it + r < D ? it + r : D - 1;
        off[i] = 8u * (static_cast<uint32_t>(m) * D + p.c0) + 16u * ((lane & 7) ^ ((r >> 1) & 7));
    }
    auto issue = [&](int u, int stage) {   // past the panel: a unit of the panel again, not used
        u = u < nu ? u : 0;
        const uint32_t lds = lds0 + stage * kStage;
        if (MODE == kBackward) {
            copy_rows(A + static_cast<size_t>(p.c0) * D + it, D, u, lds);
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i) copy_to_lds(rs_l, off[i] + 128u * u, lds + i * 1024);
        }
        copy_rows(Y + static_cast<size_t>(p.c0) * p.Qp + jt, p.Qp, u, lds + 8192);
    };
    uint32_t fo[2];   // a lane's two chunks of a fragment row of L
#pragma unroll
    for (int h = 0; h < 2; ++h)
        fo[h] = static_cast<uint32_t>((32 * (wave >> 1) + row) * 128 + ((kg + 4 * h) ^ ((row >> 1) & 7)) * 16);
    auto frag_rows = [&](double (&v)[4], const uint8_t *op, int n, int left) {   // columns n.., of which `left` indices count
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const double d = *reinterpret_cast<const double *>(op + kg * 1024 + kx(t) * 512 + ((8 * (n + row)) ^ (128 * (kg & 1))));
            v[t] = 2 * kg + kx(t) < left ? d : 0.0;
        }
    };
    f64x4 acc[F][F], c[F][F];
#pragma unroll
    for (int x = 0; x < F; ++x)
#pragma unroll
        for (int y = 0; y < F; ++y) acc[x][y] = f64x4{0.0, 0.0, 0.0, 0.0};
    int cur = 0;
    auto products = [&](int left) {
        const uint8_t *st = ring + cur * kStage;
        double a[F][4], b[F][4];
#pragma unroll
        for (int x = 0; x < F; ++x) {
            if (MODE == kBackward) {
                frag_rows(a[x], st, 32 * (wave >> 1) + 16 * x, left);
            } else {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const double2 d = *reinterpret_cast<const double2 *>(st + fo[h] + 2048 * x);
                    a[x][2 * h] = d.x;
                    a[x][2 * h + 1] = d.y;
                }
            }
            frag_rows(b[x], st + 8192, 32 * (wave & 1) + 16 * x, left);
        }
        mma_units(a, b, acc);
    };
    issue(0, 0);
    issue(1, 1);
    for (int u = 0; u < nu - 1; ++u) {
        asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier" ::: "memory");   // as in trail_tile
        issue(u + 2, cur == 0 ? 2 : cur - 1);
        products(FB);
        cur = cur == 2 ? 0 : cur + 1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the compiler's own loads follow
    auto c_value = [&](int x, int y, int q) {   // rows and columns past the end: the last one's
        const int i = i0 + 16 * x + kg + 4 * q, j = j0 + 16 * y + row;
        const int ic = i < rows_end ? i : rows_end - 1, jc = j < p.Qp ? j : p.Qp - 1;
        if (MODE == kForward && p.src == kFromG)
            return j < p.Q ? load_any(p.g, p.in_dt, j * p.ld_in + static_cast<int64_t>(blk) * D + ic) : 0.0;
        if (MODE == kForward && p.src == kFromIdent && j >= p.c0) return 0.0;
        return Y[static_cast<size_t>(ic) * p.Qp + jc];
    };
#pragma unroll
    for (int x = 0; x < F; ++x)
#pragma unroll
        for (int y = 0; y < F; ++y)
#pragma unroll
            for (int q = 0; q < 4; ++q) c[x][y][q] = c_value(x, y, q);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    products(TAIL ? kn - FB * (nu - 1) : FB);
#pragma unroll
    for (int x = 0; x < F; ++x)
#pragma unroll
        for (int y = 0; y < F; ++y)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = i0 + 16 * x + kg + 4 * q, j = j0 + 16 * y + row;
                if (i < rows_end && j < p.Qp) Y[static_cast<size_t>(i) * p.Qp + j] = c[x][y][q] - acc[x][y][q];
            }
}

// The rest of a trailing update beside the factor of the next panel, which only
// needs the tiles that are done (kTrailNext): the first n_blocks workgroups
// factor, so that this chain of pivots, on one CU each, is hidden.  The tiles of
// all layer blocks follow in one list, of which each XCD (workgroups are dealt
// to the 8 in turn) takes a contiguous eighth.
__global__ __launch_bounds__(kFactorThreads, 2) void k_trail_factor(GemmArgs p, int n_blocks, int slots, int *info) {
    const int b = static_cast<int>(blockIdx.x) - n_blocks;
    if (b < 0) {
        factor_block<double, false>(nullptr, 1, 0.0, p.A, p.D, p.c0 + PB, info, blockIdx.x);
        return;
    }
    const int per = (n_blocks * slots + 7) / 8, n = (b & 7) * per + (b >> 3);
    if ((b >> 3) >= per || n >= n_blocks * slots) return;
    trail_tile<4, 2, 2, 4, kTrailRest>(p, n % slots, n / slots);
}

__global__ __launch_bounds__(256) void k_clear_info(int *info, int n) {
    for (int i = threadIdx.x; i < n; i += 256) info[i] = 0;
}

// W = L^{-1} (fp64, row d at src + d * ld, zero past the diagonal) as two bf16
// arrays whose sum carries about 16 significant bits: hi = RNE(W), lo =
// RNE(W - hi); rows d past D (up to Dp = gridDim.x) are zero.  Split layout:
// hi [blk][Dp][D] then lo; interleaved: [blk][Dp][2D], the 64 columns of
// chunk c at 128 c (hi) and behind them (lo).  With `ident`, W = I.
__global__ __launch_bounds__(256) void k_split_w(const double *src_all, int D, int ld, bool ident,
                                                  bool interleaved, bf16_bits *w_hi, bf16_bits *w_lo) {
    const int blk = blockIdx.y, d = blockIdx.x;
    const size_t row = static_cast<size_t>(blk) * gridDim.x + d;
    bf16_bits *h = interleaved ? w_hi + row * 2 * D : w_hi + row * D;
    bf16_bits *l = interleaved ? h : w_lo + row * D;
    for (int q = threadIdx.x; q < D; q += 256) {
        const int c0 = q & ~63;
        const int at = interleaved ? q + c0 : q;   // 128 (q / 64) + q % 64
        const int at_lo = interleaved ? at + min(64, D - c0) : q;
        if (d >= D || (!ident && q > d)) {
            h[at] = l[at_lo] = 0;
            continue;
        }
        const double y = ident ? (q == d ? 1.0 : 0.0)
                               : src_all[static_cast<size_t>(blk) * D * ld + static_cast<size_t>(d) * ld + q];
        const bf16_bits hb = f32_to_bf16_rne(static_cast<float>(y));
        h[at] = hb;
        l[at_lo] = f32_to_bf16_rne(static_cast<float>(y - static_cast<double>(bf16_to_f32(hb))));
    }
}

template <typename TIn, typename TOut>
__global__ __launch_bounds__(256) void k_copy_rows(const TIn *src, int64_t ld_in, int cols,
                                                   TOut *dst, int64_t ld_out) {
    const int r = blockIdx.y;
    for (int c = blockIdx.x * 256 + threadIdx.x; c < cols; c += gridDim.x * 256)
        store_out_d<TOut>(dst + static_cast<int64_t>(r) * ld_out + c, load_in_d<TIn>(src + static_cast<int64_t>(r) * ld_in + c));
}

// k_solve over the first `cols` right-hand sides, 32 of them per workgroup (two
// workgroups share a CU), or 16 where that would leave CUs idle; one launch, but
// for more workgroups than a launch takes.
hipError_t launch_solve_block(SolveArgs p, int cols, int n_blocks, hipStream_t s) {
    auto wgs = [&](int nc) { return (cols + 16 * nc - 1) / (16 * nc) * static_cast<int64_t>(n_blocks); };
    const int nc = wgs(2) >= 256 ? 2 : 1;
    const int all = (cols + 16 * nc - 1) / (16 * nc), most = static_cast<int>(kMaxGridThreads / 512 - 1);
    const int w = p.D - p.c0 < PB ? p.D - p.c0 : PB;
    auto go = [&](auto k) {
        hipError_t e = hipSuccess;
        for (p.wg0 = 0; p.wg0 < all && e == hipSuccess; p.wg0 += most) {
            const dim3 grid(static_cast<unsigned>(min(most, all - p.wg0)), static_cast<unsigned>(n_blocks));
            hipLaunchKernelGGL(k, grid, dim3(512), 0, s, p);
            e = hipGetLastError();
        }
        return e;
    };
    if (w <= 64) return nc == 2 ? go(k_solve<4, 2>) : go(k_solve<4, 1>);
    if (w <= 128) return nc == 2 ? go(k_solve<8, 2>) : go(k_solve<8, 1>);
    return nc == 2 ? go(k_solve<16, 2>) : go(k_solve<16, 1>);
}

// One k_solve_gemm launch, in 64 x 64 tiles.
template <int MODE>
hipError_t launch_solve_gemm(const GemmArgs &p, int rows, int cols, int n_blocks, hipStream_t s) {
    const int64_t tiles = static_cast<int64_t>((rows + 63) / 64) * ((cols + 63) / 64);
    const dim3 grid(static_cast<unsigned>(tiles), static_cast<unsigned>(n_blocks));
    if (MODE == kBackward && p.D - p.c0 < PB)
        hipLaunchKernelGGL((k_solve_gemm<MODE, MODE == kBackward>), grid, dim3(256), 0, s, p);
    else
        hipLaunchKernelGGL((k_solve_gemm<MODE, false>), grid, dim3(256), 0, s, p);
    return hipGetLastError();
}

// The trailing update of the panel at c0 and the factor of the next one: first
// the next panel's columns, in 64 x 64 tiles while 128 x 128 ones would leave
// CUs idle, then the rest (128 x 128 tiles) beside the factor.
hipError_t launch_trail(const GemmArgs &p, int rest, int n_blocks, int *info, hipStream_t s) {
    auto next = [&](int t) {   // tiles of the next panel's columns
        const int r = (rest + t - 1) / t, w = PB / t;
        return r < w ? r * (r + 1) / 2 : w * (w + 1) / 2 + (r - w) * w;
    };
    if (next(128) * n_blocks >= 256)
        hipLaunchKernelGGL((k_trail_next<4, 2, 2, 4>), dim3(next(128), n_blocks), dim3(512), 0, s, p);
    else
        hipLaunchKernelGGL((k_trail_next<2, 2, 2, 2>), dim3(next(64), n_blocks), dim3(256), 0, s, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int r = (rest + 127) / 128 - PB / 128, groups = r > 0 ? (r + kTrailGroup - 1) / kTrailGroup : 0;
    const int slots = kTrailGroup * kTrailGroup * groups * (groups + 1) / 2;
    hipLaunchKernelGGL(k_trail_factor, dim3(n_blocks + (n_blocks * slots + 7) / 8 * 8), dim3(kFactorThreads), 0, s, p, n_blocks,
                       slots, info);
    return hipGetLastError();
}

// W (D <= 256), or the panels of L and every W_II: the factorisation.
hipError_t launch_factor(const void *S, bool s_f64, int D, int n_blocks, int64_t N, double damp_ratio,
                         const WsLayout &w, hipStream_t s) {
    const double *Sd = static_cast<const double *>(S);
    const float *Sf = static_cast<const float *>(S);
    if (D <= PB) {
        if (s_f64)
            hipLaunchKernelGGL((k_factor<double, true>), dim3(n_blocks), dim3(kFactorThreads), 0, s, Sd, N, damp_ratio,
                               w.A, D, 0, w.info);
        else
            hipLaunchKernelGGL((k_factor<float, true>), dim3(n_blocks), dim3(kFactorThreads), 0, s, Sf, N, damp_ratio,
                               w.A, D, 0, w.info);
        return hipGetLastError();
    }
    if (s_f64) {
        hipLaunchKernelGGL(k_lambda<double>, dim3(n_blocks), dim3(256), 0, s, Sd, D, N, damp_ratio, w.lam);
        hipLaunchKernelGGL(k_form<double>, dim3(D, n_blocks), dim3(256), 0, s, Sd, D, N, w.lam, w.A, w.info);
    } else {
        hipLaunchKernelGGL(k_lambda<float>, dim3(n_blocks), dim3(256), 0, s, Sf, D, N, damp_ratio, w.lam);
        hipLaunchKernelGGL(k_form<float>, dim3(D, n_blocks), dim3(256), 0, s, Sf, D, N, w.lam, w.A, w.info);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_factor<double, false>), dim3(n_blocks), dim3(kFactorThreads), 0, s,
                       static_cast<const double *>(nullptr), N, damp_ratio, w.A, D, 0, w.info);
    e = hipGetLastError();
    for (int c0 = 0; c0 + PB < D && e == hipSuccess; c0 += PB) {
        const int rest = D - c0 - PB;
        hipLaunchKernelGGL(k_panel, dim3((rest + 31) / 32, n_blocks), dim3(256), 0, s, w.A, D, c0);
        if ((e = hipGetLastError()) != hipSuccess) break;
        e = launch_trail(GemmArgs{w.A, nullptr, nullptr, 0, D, c0, 0, 0, kF32, kFromY}, rest, n_blocks, w.info, s);
    }
    return e;
}

// Forward solve, D > 256: Y = L^{-1} g (src kFromG) or L^{-1} (kFromIdent, Q = D:
// only the columns up to each block are formed).
hipError_t launch_forward(const WsLayout &w, int D, int n_blocks, const void *g, int in_dt, int64_t ld_in, int Q, int src,
                          hipStream_t s) {
    const int Qp = padded_q(Q);
    hipError_t e = hipSuccess;
    for (int c0 = 0; c0 < D && e == hipSuccess; c0 += PB) {
        const int from = src == kFromG && c0 > 0 ? static_cast<int>(kFromY) : src;
        const int cols = src == kFromIdent && c0 + PB < Qp ? c0 + PB : Qp;
        e = launch_solve_block(SolveArgs{w.A, w.Y, g, nullptr, ld_in, 0, D, c0, Q, Qp, in_dt, kF32, from, 1, 0, 1, 0}, cols,
                               n_blocks, s);
        const int rest = D - c0 - PB;
        if (rest <= 0 || e != hipSuccess) continue;
        e = launch_solve_gemm<kForward>(GemmArgs{w.A, w.Y, g, ld_in, D, c0, Q, Qp, in_dt, from}, rest, cols, n_blocks, s);
    }
    return e;
}

}  // namespace

inline size_t w_half_bytes(int D, int n_blocks) {
    const size_t Dp = static_cast<size_t>(D + 255) / 256 * 256;
    return align256(sizeof(bf16_bits) * static_cast<size_t>(n_blocks) * Dp * D);
}

size_t self_influence_ws_bytes(int D, int n_blocks) {
    return precond_ws_bytes(D, n_blocks, D) + 2 * w_half_bytes(D, n_blocks);
}

bf16_bits *self_influence_w(void *ws, int D, int n_blocks, bool lo) {
    char *p = static_cast<char *>(ws) + precond_ws_bytes(D, n_blocks, D);
    if (lo) p += w_half_bytes(D, n_blocks);
    return reinterpret_cast<bf16_bits *>(p);
}

float *self_influence_part(void *ws, int D, int n_blocks, size_t *bytes) {
    *bytes = sizeof(double) * static_cast<size_t>(n_blocks) * D * padded_q(D);
    return reinterpret_cast<float *>(ws_layout(ws, D, n_blocks).Y);
}

size_t precond_ws_bytes(int D, int n_blocks, int Q) {
    const size_t nb = static_cast<size_t>(n_blocks);
    return align256(sizeof(double) * nb * D * D) + align256(sizeof(double) * nb) + align256(sizeof(int) * nb) +
           align256(sizeof(double) * nb * D * padded_q(Q));
}

int *precond_info_ptr(void *ws, int D, int n_blocks) { return ws_layout(ws, D, n_blocks).info; }

namespace {
// Dispatch over the element types of an input and an output (dtype codes).
template <typename F>
hipError_t with_types(int in_dt, int out_dt, F &&f) {
    auto out = [&](auto in_tag) -> hipError_t {
        using TI = decltype(in_tag);
        if (out_dt == kBF16) return f(TI{}, bf16_bits{});
        if (out_dt == kF64) return f(TI{}, double{});
        return f(TI{}, float{});
    };
    if (in_dt == kBF16) return out(bf16_bits{});
    if (in_dt == kF64) return out(double{});
    return out(float{});
}
}  // namespace

hipError_t launch_copy_rows(const void *src, int in_dt, int64_t ld_in, int rows, int cols,
                            void *dst, int out_dt, int64_t ld_out, hipStream_t s) {
    if (rows == 0 || cols == 0) return hipSuccess;
    const dim3 grid(static_cast<unsigned>(min((cols + 255) / 256, 64)), static_cast<unsigned>(rows));
    return with_types(in_dt, out_dt, [&](auto ti, auto to) {
        using TI = decltype(ti);
        using TO = decltype(to);
        hipLaunchKernelGGL((k_copy_rows<TI, TO>), grid, dim3(256), 0, s, static_cast<const TI *>(src), ld_in,
                           cols, static_cast<TO *>(dst), ld_out);
        return hipGetLastError();
    });
}

hipError_t launch_precondition(const void *S, bool s_f64, int D, int n_blocks, int64_t N, double damp_ratio,
                               const void *g_test, int in_dt, int64_t ld_in, int Q, void *g_out, int out_dt,
                               int64_t ld_out, void *ws, hipStream_t s) {
    const WsLayout w = ws_layout(ws, D, n_blocks);
    hipError_t e = launch_factor(S, s_f64, D, n_blocks, N, damp_ratio, w, s);
    if (e != hipSuccess || Q == 0) return e;
    const int Qp = padded_q(Q);
    if (D <= PB)
        return launch_solve_block(SolveArgs{w.A, nullptr, g_test, g_out, ld_in, ld_out, D, 0, Q, Qp, in_dt, out_dt, kFromG,
                                            1, 1, 0, 0},
                                  Q, n_blocks, s);
    e = launch_forward(w, D, n_blocks, g_test, in_dt, ld_in, Q, kFromG, s);
    for (int c0 = (D - 1) / PB * PB; c0 >= 0 && e == hipSuccess; c0 -= PB) {
        e = launch_solve_block(SolveArgs{w.A, w.Y, nullptr, g_out, 0, ld_out, D, c0, Q, Qp, kF32, out_dt, kFromY, 0, 1, 1, 0},
                               Qp, n_blocks, s);
        if (c0 == 0 || e != hipSuccess) continue;
        e = launch_solve_gemm<kBackward>(GemmArgs{w.A, w.Y, nullptr, 0, D, c0, Q, Qp, kF32, kFromY}, c0, Qp, n_blocks, s);
    }
    return e;
}

hipError_t launch_inverse_factor(const float *S, int D, int n_blocks, int64_t N, double damp_ratio,
                                 bool interleaved, void *ws, hipStream_t s) {
    const WsLayout w = ws_layout(ws, D, n_blocks);
    bf16_bits *hi = self_influence_w(ws, D, n_blocks, false), *lo = self_influence_w(ws, D, n_blocks, true);
    const bool ident = damp_ratio < 0;
    const double *src = w.A;   // D <= 256: W itself
    int ld = D;
    if (!ident) {
        hipError_t e = launch_factor(S, false, D, n_blocks, N, damp_ratio, w, s);
        if (e == hipSuccess && D > PB) {   // L^{-1}: forward solve of the identity
            e = launch_forward(w, D, n_blocks, nullptr, kF32, 0, D, kFromIdent, s);
            src = w.Y;
            ld = padded_q(D);
        }
        if (e != hipSuccess) return e;
    } else {
        hipLaunchKernelGGL(k_clear_info, dim3(1), dim3(256), 0, s, w.info, n_blocks);
    }
    hipLaunchKernelGGL(k_split_w, dim3((D + 255) / 256 * 256, n_blocks), dim3(256), 0, s, src, D, ld, ident, interleaved, hi,
                       lo);
    return hipGetLastError();
}

}  // namespace logra
