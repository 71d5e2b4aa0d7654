// Algebraic compression of a symmetric H^2 matrix with orthonormal nested
// bases (Sec. 5.2 and 5.3), FP64.
//
// Basis generation, top-down: node i of level l stacks
//     Sbar_i = [R_i+ E_i^T; S_ij1^T; ...; S_ijb^T]
// (i+ its parent, S_ij the coupling blocks of its block row; when the blocks
// are not symmetric, the blocks S_ji of its block column follow, since the
// one basis tree serves the columns too) and keeps the triangular factor R_i
// of its QR factorization.  The stack is not formed
// whole: a workgroup holds 512 x 64 in registers, so blocks are appended
// under the current factor and folded into it with a QR of the stack
// whenever the next block would not fit (the same R up to row signs, which
// the truncation does not see: it uses R only through R^T R).
//
// A matrix with a row and a column tree of their own runs basis generation
// and truncation once per tree (the column tree from the block columns,
// through V_j^T and F_c^T read transposed), a level taking the larger rank.
//
// Truncation, bottom-up: leaves decompose W_i = U_i R_i^T; as U_i has
// orthonormal columns, the left singular vectors of W_i are U_i times those
// of R_i^T, so the SVD runs on the k x k matrix R_i^T.  Parents decompose
// W_p = Z_p R_p^T with Z_p = [T_c1 E_c1; T_c2 E_c2]; a tall W_p is first
// reduced to its triangular factor by a Householder QR (W_p = Q R_w), and
// the left singular vectors are Q times those of R_w.  The SVD is the
// one-sided Jacobi method with accumulated rotations, so the kept vectors
// are orthonormal also past the numerical rank of a node.  The rotations act
// on the rows of a triangular factor: R_i^T = Q_2 R_2 at the leaves, and
// W_p^T = Q_1 R_1, R_1^T = Q_2 R_2 where W_p is not tall, the rotations then
// starting from Q_2.  Rows of such a factor are nearly orthogonal where the
// columns R_i and R_1 come with are not: 6-7 sweeps instead of 20-25 (the
// 2^16-point 2-D workload at 1e-7: leaves 6.0 -> 1.65 ms, levels 11.9 -> 3.9 ms).  A node keeps the
// singular values at least eps times its largest; the host takes the
// largest count of a level as its new rank.
//
// One workgroup per node: 1024 threads with the stack in registers for the
// basis generation, 256 threads with every matrix staged column-major in LDS
// for the truncation.

#include <hip/hip_runtime.h>

#include <cstdint>

#include "h2_device.h"
#include "h2_lds_la.h"

namespace h2 {
namespace {

using namespace lds;

typedef double f64x2 __attribute__((ext_vector_type(2)));

constexpr int GEN_LD = QR_MAXM + QR_PAD;   // LDS matrices of up to 128 rows (+ pad) x 64 columns
constexpr int SQ_LD = 64 + QR_PAD;         // LDS square matrices: 64 x 64 (+ pad)
constexpr double JACOBI_TOL = 64 * 2.220446049250313e-16;
constexpr int JACOBI_SWEEPS = 30;

__device__ inline int64_t level_first(int l) { return (int64_t(1) << l) - 1; }

// Basis generation of one node, a 512 x k stack held in registers of a
// 1024-thread workgroup: wave w owns columns w, w + 16, w + 32, w + 48 (NS of
// them; a[s] = column w + 16 s) and lane l of it rows l + 64 i (a[s][i]).
// Rows 0 .. 63 hold the current triangular factor (first: the parent term),
// rows 64 .. 511 the coupling blocks appended since (as many k-row blocks as
// fit).  A fold is a Householder QR without Q over these rows: step c reads
// reflector c from LDS (double buffered, one barrier per step), and the wave
// of column c + 1 applies it to that column first and publishes reflector
// c + 1 while the others still apply reflector c.  Entries below the diagonal
// are set to zero as they are eliminated, so after a fold rows k .. 511 are
// zero.  Register arrays are indexed statically only.
//
// Bound by the serial chain of a step (reduction over the wave, square root,
// division, barrier), so steps are few and short: 448 new rows share one
// pass over the columns, a reflector's LDS read serves four columns, and
// their four sums go through one reduction (the halves of two columns are
// exchanged, then the 16-lane rows, so that each row of 16 lanes ends with
// one column).  Columns are dealt in turn, so every wave has work until the
// last ones.  A 2^16-point 2-D build at rank 64: 9.3 -> 4.1 ms over its
// levels (before: 192 new rows per pass, four adjacent columns per wave with
// 16 rows per lane, a reflector read whole by every wave: LDS-bound).
constexpr int BG_THREADS = 1024, BG_ROWS = 8, BG_FIT = 64 * (BG_ROWS - 1), BG_STAGE = 128, BG_TLD = 65;

struct StackLds {
    double v[2][64 * BG_ROWS], tau[2];
    int64_t off[BG_FIT];             // the appended blocks' offsets
    double tile[BG_STAGE * BG_TLD];  // staged blocks, row-major; first R_parent and E_i
};

// x of one half of the wave added to the other half, y likewise: lanes 0 ..
// 31 get x, lanes 32 .. 63 y (WIDTH 32); even 16-lane rows x, odd rows y
// (WIDTH 16).
template <int WIDTH>
__device__ inline double swap_add(double x, double y) {
    const uint64_t xb = uint64_t(__double_as_longlong(x)), yb = uint64_t(__double_as_longlong(y));
    uint64_t p, q;
    if constexpr (WIDTH == 32) {
        const auto lo = __builtin_amdgcn_permlane32_swap(uint32_t(xb), uint32_t(yb), false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap(uint32_t(xb >> 32), uint32_t(yb >> 32), false, false);
        p = (uint64_t(hi[0]) << 32) | lo[0];
        q = (uint64_t(hi[1]) << 32) | lo[1];
    } else {
        const auto lo = __builtin_amdgcn_permlane16_swap(uint32_t(xb), uint32_t(yb), false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap(uint32_t(xb >> 32), uint32_t(yb >> 32), false, false);
        p = (uint64_t(hi[0]) << 32) | lo[0];
        q = (uint64_t(hi[1]) << 32) | lo[1];
    }
    return __longlong_as_double(int64_t(p)) + __longlong_as_double(int64_t(q));
}

__device__ inline double lane_value(double x, int l) {   // lane l's x, l uniform
    const int64_t b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readlane(int(b), l), hi = __builtin_amdgcn_readlane(int(b >> 32), l);
    return __longlong_as_double((int64_t(hi) << 32) | uint32_t(lo));
}

// The sums over the wave of N <= 4 values, in every lane.
template <int N>
__device__ __forceinline__ void wave_sums(double (&d)[N]) {
    const double e = swap_add<32>(d[0], d[N > 1 ? 1 : 0]);
    if constexpr (N <= 2) {   // rows of 16 lanes: 0 0 1 1
        const double f = dpp_sum16(swap_add<16>(e, e));
        if constexpr (N == 1) {
            d[0] = f;
        } else {
            d[0] = lane_value(f, 0);
            d[1] = lane_value(f, 32);
        }
    } else {                  // rows of 16 lanes: 0 2 1 3
        const double f = dpp_sum16(swap_add<16>(e, swap_add<32>(d[2], d[N - 1])));
        d[0] = lane_value(f, 0);
        d[1] = lane_value(f, 32);
        d[2] = lane_value(f, 16);
        if constexpr (N == 4) d[3] = lane_value(f, 48);
    }
}

// The reflector of column c (x, the wave's rows of it), left in v and tau.
template <int NI>
__device__ __forceinline__ void publish(double (&x)[BG_ROWS], int c, int lane, double *v, double *tau) {
    double sq[1] = {lane > c ? x[0] * x[0] : 0.0};
#pragma unroll
    for (int i = 1; i < NI; ++i) sq[0] += x[i] * x[i];
    wave_sums<1>(sq);
    const double al = lane_value(x[0], c), nrm = sqrt(sq[0] + al * al);
    double beta = al, tc = 0.0, sc = 0.0;
    if (sq[0] > 0.0) {
        beta = al >= 0.0 ? -nrm : nrm;
        tc = (beta - al) / beta;
        sc = 1.0 / (al - beta);
    }
    v[lane] = lane > c ? x[0] * sc : (lane == c ? 1.0 : 0.0);
    x[0] = lane > c ? 0.0 : (lane == c ? beta : x[0]);
#pragma unroll
    for (int i = 1; i < NI; ++i) {
        v[lane + 64 * i] = x[i] * sc;
        x[i] = 0.0;
    }
    if (lane == 0) *tau = tc;
}

// Steps c = 16 S .. 16 S + 15 of a fold, then those of the next slot.
template <int NS, int NI, int S>
__device__ __forceinline__ void fold_slot(double (&a)[NS][BG_ROWS], int k, int wv, int lane, StackLds &s) {
    if constexpr (S < NS) {
#pragma unroll 1
        for (int cc = 0; cc < 16 && 16 * S + cc < k; ++cc) {
            const int c = 16 * S + cc;
            __syncthreads();   // reflector c is published; reflector c - 1 has been read
            double v[NI], d[NS - S];
#pragma unroll
            for (int i = 0; i < NI; ++i) v[i] = s.v[c & 1][lane + 64 * i];
            const double tc = s.tau[c & 1];
#pragma unroll
            for (int n = S; n < NS; ++n) {
                d[n - S] = 0.0;
                if (n > S || wv > cc) {   // the wave's columns to the right of c
#pragma unroll
                    for (int i = 0; i < NI; ++i) d[n - S] += v[i] * a[n][i];
                }
            }
            wave_sums<NS - S>(d);
#pragma unroll
            for (int n = S; n < NS; ++n) {
                if (n > S || wv > cc) {
                    d[n - S] *= tc;
#pragma unroll
                    for (int i = 0; i < NI; ++i) a[n][i] -= d[n - S] * v[i];
                    if (n <= S + 1 && 16 * n + wv == c + 1 && c + 1 < k)
                        publish<NI>(a[n], c + 1, lane, s.v[(c + 1) & 1], &s.tau[(c + 1) & 1]);
                }
            }
        }
        fold_slot<NS, NI, S + 1>(a, k, wv, lane, s);
    }
}

template <int NS, int NI>
__device__ __forceinline__ void fold_r(double (&a)[NS][BG_ROWS], int k, int wv, int lane, StackLds &s) {
    if (wv == 0) publish<NI>(a[0], 0, lane, s.v[0], &s.tau[0]);
    fold_slot<NS, NI, 0>(a, k, wv, lane, s);
    __syncthreads();   // the last reflectors are read before they are overwritten
}

template <int NS>
__global__ __launch_bounds__(BG_THREADS) void basis_generation_kernel(CompLaunch L, int level, int k, int kp,
                                                                      int parent_term) {
    __shared__ StackLds s;
    const int t = threadIdx.x, lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int64_t node = level_first(level) + blockIdx.x;
    double a[NS][BG_ROWS];
#pragma unroll
    for (int n = 0; n < NS; ++n)
#pragma unroll
        for (int i = 0; i < BG_ROWS; ++i) a[n][i] = 0.0;
    bool dirty = false;   // rows hold entries not yet folded into a triangular factor
    if (parent_term) {    // rows 0 .. kp-1: P = R_parent E_i^T (kp x k), R_parent upper triangular
        const double *Rp = L.R + ((node - 1) >> 1) * L.kmax * L.kmax;   // zero below its diagonal
        const double *E = L.basis + L.off_E[node];                      // k x kp (or its transpose)
        double *Et = s.tile + 64 * BG_TLD;
        for (int i = t; i < 64 * kp; i += BG_THREADS) {
            const int u = i >> 6, r = i & 63;
            s.tile[u * BG_TLD + r] = r < kp ? Rp[int64_t(u) * L.kmax + r] : 0.0;
            if (r < k) Et[u * BG_TLD + r] = L.x_t ? E[at2(kp, u, r)] : E[at2(k, r, u)];
        }
        __syncthreads();
        for (int u = 0; u < kp; ++u) {
            const double x = s.tile[u * BG_TLD + lane];
#pragma unroll
            for (int n = 0; n < NS; ++n)
                if (wv + 16 * n < k) a[n][0] += x * Et[u * BG_TLD + wv + 16 * n];
        }
        dirty = true;
    }
    // the stack's blocks: those of block row i, transposed, then (when the
    // coupling blocks are not symmetric) those of block column i as they are
    const int64_t nrow = L.use_rows ? L.row_start[node + 1] - L.row_start[node] : 0;
    const int64_t nb = nrow + (L.columns ? L.col_start[node + 1] - L.col_start[node] : 0);
    const int ng = (k + 1) >> 1, items = ng * k, stage = BG_STAGE / k;   // stage: blocks staged at a time
    const float per_k = 1.0f / float(k);   // (x + 1/2) / k is at least 1/128 away from a whole number
    const float per_items = 1.0f / float(items);
    for (int64_t b = 0;;) {   // append as many blocks as fit under the factor, then fold
        const int fit = int(nb - b < BG_FIT / k ? nb - b : BG_FIT / k);
        __syncthreads();   // the previous offsets and tile are consumed
        if (t < fit) {
            const int64_t e = b + t;
            s.off[t] = e < nrow ? L.blk[L.row_start[node] + e].off : L.col_blk[L.col_start[node] + (e - nrow)];
        }
        __syncthreads();
        for (int f = 0; f < fit; f += stage) {
            const int cnt = fit - f < stage ? fit - f : stage;
            int e0 = t;
            asm volatile("" : "+v"(e0));   // the items' places are computed here each time, not kept across folds
            f64x2 x[BG_STAGE * 32 / BG_THREADS];   // cnt items <= stage ng k <= 128 * 32 (k = 1: 128)
            int at[BG_STAGE * 32 / BG_THREADS];
#pragma unroll
            for (int m = 0; m < BG_STAGE * 32 / BG_THREADS; ++m) {   // S(r, 2g .. 2g+1) is one 16-byte item
                const int e = e0 + BG_THREADS * m;
                at[m] = -1;
                if (e < cnt * items) {
                    const int bi = int((float(e) + 0.5f) * per_items), w = e - bi * items;
                    const int g = int((float(w) + 0.5f) * per_k), r = w - g * k;
                    x[m] = *reinterpret_cast<const f64x2 *>(L.blocks + s.off[f + bi] + (int64_t(g) * k + r) * 2);
                    at[m] = (bi * k + r) * BG_TLD + 2 * g;
                }
            }
            if (f > 0) __syncthreads();   // the tile's previous contents are consumed
#pragma unroll
            for (int m = 0; m < BG_STAGE * 32 / BG_THREADS; ++m)
                if (at[m] >= 0) {
                    s.tile[at[m]] = x[m].x;
                    s.tile[at[m] + 1] = x[m].y;   // column k when k is odd: padding, never read
                }
            __syncthreads();
            // row 64 + f k + y k + rr, column col is S(col, rr) of block y for a row block (S^T) and
            // S(rr, col) for a column block
#pragma unroll
            for (int i = 1; i < BG_ROWS; ++i) {
                const int q = lane + 64 * (i - 1) - f * k;
                if (q >= 0 && q < cnt * k) {
                    const int y = int((float(q) + 0.5f) * per_k), rr = q - y * k;
                    const bool from_row = b + f + y < nrow;
                    const double *S = s.tile + y * k * BG_TLD + (from_row ? rr : rr * BG_TLD);
                    const int step = from_row ? BG_TLD : 1;
#pragma unroll
                    for (int n = 0; n < NS; ++n)
                        if (wv + 16 * n < k) a[n][i] = S[(wv + 16 * n) * step];
                }
            }
        }
        b += fit;
        if (fit == 0 && !dirty) break;
        if (fit * k <= 192) fold_r<NS, 4>(a, k, wv, lane, s);
        else fold_r<NS, BG_ROWS>(a, k, wv, lane, s);
        dirty = false;
        if (b >= nb) break;
    }
    double *R = L.R + node * L.kmax * L.kmax;   // rows 0 .. k-1 (zero below the diagonal)
#pragma unroll
    for (int n = 0; n < NS; ++n) {
        const int col = wv + 16 * n;
        if (col < k && lane < k) R[int64_t(col) * L.kmax + lane] = a[n][0];
    }
}

// After jacobi_svd: the singular values s (column norms of G, n columns of
// length Lrows), rank[j] = position of column j in descending order (ties by
// index), sigma (n values, descending) and the count kept for eps.
__device__ inline void sort_and_count(const double *G, int ldg, int Lrows, int n, double eps, double *s, int *rank,
                                      double *sigma, int32_t *count) {
    const int t = threadIdx.x;
    if (t < n) {
        double a = 0.0;
        for (int r = 0; r < Lrows; ++r) a += G[t * ldg + r] * G[t * ldg + r];
        s[t] = sqrt(a);
    }
    __syncthreads();
    if (t < n) {
        const double v = s[t];
        int rk = 0;
        for (int i = 0; i < n; ++i) rk += (s[i] > v) || (s[i] == v && i < t);
        rank[t] = rk;
        sigma[rk] = v;
    }
    if (t == 0) {
        double smax = 0.0;
        for (int i = 0; i < n; ++i) smax = s[i] > smax ? s[i] : smax;
        int cnt = 0;
        if (smax > 0.0)
            for (int i = 0; i < n; ++i) cnt += s[i] >= eps * smax;
        *count = cnt;
    }
    __syncthreads();
}

__global__ __launch_bounds__(256) void truncate_leaves_kernel(CompLaunch L, int k, double eps) {
    __shared__ double G[64 * SQ_LD], Y[64 * SQ_LD], tau[64], s[64];
    __shared__ int rank[64], flag;
    const int t = threadIdx.x, ldy = k + QR_PAD;   // the leading dimension householder_qr uses
    const int64_t j = blockIdx.x, node = L.first_leaf + j;
    const double *R = L.R + node * L.kmax * L.kmax;
    for (int i = t; i < k * k; i += 256) {
        const int c = i / k, r = i - c * k;
        Y[r * ldy + c] = R[int64_t(c) * L.kmax + r];   // R_j^T
    }
    __syncthreads();
    householder_qr<64>(Y, tau, s, k, k, G, SQ_LD);   // R_j^T = Y R_2
    __syncthreads();
    transpose_square(G, SQ_LD, k);   // the rows of R_2
    jacobi_svd(G, SQ_LD, k, Y, ldy, k, JACOBI_TOL, JACOBI_SWEEPS, &flag, s);
    sort_and_count(G, SQ_LD, k, k, eps, s, rank, L.sigma + j * 64, L.count + j);
    double *X = L.X + j * COMP_XSLOT;
    for (int i = t; i < k * k; i += 256) {
        const int c = i / k, r = i - c * k;
        X[int64_t(rank[c]) * COMP_XLD + r] = Y[c * ldy + r];
    }
}

__global__ __launch_bounds__(256) void truncate_leaves_apply_kernel(CompLaunch L, int k, int kt) {
    __shared__ double Uo[64 * SQ_LD], Xs[64 * SQ_LD];
    const int t = threadIdx.x;
    const int64_t j = blockIdx.x, node = L.first_leaf + j;
    const int m = int(L.leaf_end[j] - L.leaf_begin[j]);
    const double *U = L.basis + L.off_U[j];   // m x k (or its transpose)
    const double *X = L.X + j * COMP_XSLOT;
    for (int i = t; i < m * k; i += 256) {
        const int c = i / m, r = i - c * m;
        Uo[c * SQ_LD + r] = L.b_t ? U[at2(k, c, r)] : U[at2(m, r, c)];
    }
    for (int i = t; i < k * kt; i += 256) {
        const int c = i / k, r = i - c * k;
        Xs[c * SQ_LD + r] = X[int64_t(c) * COMP_XLD + r];
    }
    __syncthreads();
    double *Un = L.Unew + j * COMP_USLOT;
    for (int i = t; i < m * kt; i += 256) {   // U_new = U X(:, 0:kt)
        const int c = i / m, r = i - c * m;
        double acc = 0.0;
        for (int u = 0; u < k; ++u) acc += Uo[u * SQ_LD + r] * Xs[c * SQ_LD + u];
        Un[c * 64 + r] = acc;
    }
    double *T = L.T + node * L.kmax * L.kmax;   // T_j = X(:, 0:kt)^T (kt x k)
    for (int i = t; i < kt * k; i += 256) {
        const int c = i / kt, r = i - c * kt;
        T[int64_t(c) * L.kmax + r] = Xs[r * SQ_LD + c];
    }
}

// Z_p = [T_c1 E_c1; T_c2 E_c2] (2 kt x kp) into Z (leading dimension ldz);
// Ts and Es are 64 x 64 LDS staging buffers.
__device__ inline void form_z(const CompLaunch &L, int64_t p, int kc, int kt, int kp, double *Z, int ldz, double *Ts,
                              double *Es) {
    const int t = threadIdx.x;
    for (int h = 0; h < 2; ++h) {
        const int64_t ch = 2 * p + 1 + h;
        const double *Tc = L.T + ch * L.kmax * L.kmax;   // kt x kc
        const double *E = L.basis + L.off_E[ch];        // kc x kp (or its transpose)
        for (int i = t; i < kt * kc; i += 256) {
            const int c = i / kt, r = i - c * kt;
            Ts[c * SQ_LD + r] = Tc[int64_t(c) * L.kmax + r];
        }
        for (int i = t; i < kc * kp; i += 256) {
            const int c = i / kc, r = i - c * kc;
            Es[c * SQ_LD + r] = L.x_t ? E[at2(kp, c, r)] : E[at2(kc, r, c)];
        }
        __syncthreads();
        for (int i = t; i < kt * kp; i += 256) {
            const int c = i / kt, r = i - c * kt;
            double acc = 0.0;
            for (int u = 0; u < kc; ++u) acc += Ts[u * SQ_LD + r] * Es[c * SQ_LD + u];
            Z[c * ldz + h * kt + r] = acc;
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void truncate_level_kernel(CompLaunch L, int l, int kc, int kt, int kp, double eps) {
    __shared__ double A[GEN_LD * QR_MAXN], G[64 * SQ_LD], Y[64 * SQ_LD];
    __shared__ double tau[QR_MAXN], sgn[QR_MAXN], s[64];
    __shared__ int rank[64], flag;
    const int t = threadIdx.x;
    const int64_t i0 = blockIdx.x, p = level_first(l - 1) + i0;
    const int M = 2 * kt, ldz = M + QR_PAD;   // the leading dimension householder_qr uses
    form_z(L, p, kc, kt, kp, A, ldz, G, Y);
    // W = Z R_p^T (M x kp): R_p staged in G, the products held in registers
    const double *Rp = L.R + p * L.kmax * L.kmax;
    for (int i = t; i < kp * kp; i += 256) {
        const int c = i / kp, r = i - c * kp;
        G[c * SQ_LD + r] = Rp[int64_t(c) * L.kmax + r];
    }
    __syncthreads();
    double w[32];
#pragma unroll
    for (int q = 0; q < 32; ++q) {
        const int i = t + 256 * q, c = i / M, r = i - c * M;
        double acc = 0.0;
        if (c < kp)
            for (int u = c; u < kp; ++u) acc += A[u * ldz + r] * G[u * SQ_LD + c];   // Z(r, u) R_p(c, u)
        w[q] = acc;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 32; ++q) {
        const int i = t + 256 * q, c = i / M, r = i - c * M;
        if (c < kp) A[c * ldz + r] = w[q];
    }
    __syncthreads();
    const bool tall = M > kp;
    int n;
    double *Yj = Y;      // the rotations' matrix, leading dimension ldy
    int ldy = SQ_LD;
    if (tall) {   // W = Q R_w: Q in A, R_w in Y, then G = R_w^T (its rows as columns)
        householder_qr(A, tau, sgn, M, kp, Y, SQ_LD);
        n = kp;
        for (int i = t; i < kp * kp; i += 256) {
            const int c = i / kp, r = i - c * kp;
            G[c * SQ_LD + r] = Y[r * SQ_LD + c];
        }
        __syncthreads();
        for (int i = t; i < kp * kp; i += 256) {
            const int c = i / kp, r = i - c * kp;
            Y[c * SQ_LD + r] = r == c ? 1.0 : 0.0;
        }
        __syncthreads();
    } else {      // W^T = Q_1 R_1, R_1^T = Q_2 R_2: G = R_2^T, starting from Q_2 (in A)
        n = M;
        for (int i = t; i < kp * M; i += 256) {
            const int c = i / kp, r = i - c * kp;
            G[c * SQ_LD + r] = A[r * ldz + c];
        }
        __syncthreads();
        for (int i = t; i < kp * M; i += 256) {
            const int c = i / kp, r = i - c * kp;
            A[c * (kp + QR_PAD) + r] = G[c * SQ_LD + r];
        }
        __syncthreads();
        householder_qr<64, false>(A, tau, sgn, kp, M, Y, SQ_LD);
        __syncthreads();
        ldy = M + QR_PAD;
        for (int i = t; i < M * M; i += 256) {
            const int c = i / M, r = i - c * M;
            A[r * ldy + c] = Y[c * SQ_LD + r];
        }
        __syncthreads();
        householder_qr<64>(A, tau, sgn, M, M, G, SQ_LD);
        __syncthreads();
        transpose_square(G, SQ_LD, M);
        Yj = A;
    }
    const int Lrows = n;
    jacobi_svd(G, SQ_LD, Lrows, Yj, ldy, n, JACOBI_TOL, JACOBI_SWEEPS, &flag, s);
    sort_and_count(G, SQ_LD, Lrows, n, eps, s, rank, L.sigma + i0 * 64, L.count + i0);
    double *X = L.X + i0 * COMP_XSLOT;   // left singular vectors of W: M x n
    if (tall) {
        for (int i = t; i < M * n; i += 256) {
            const int c = i / M, r = i - c * M;
            double acc = 0.0;
            for (int u = 0; u < kp; ++u) acc += A[u * ldz + r] * Y[c * SQ_LD + u];
            X[int64_t(rank[c]) * COMP_XLD + r] = acc;
        }
    } else {
        for (int i = t; i < M * n; i += 256) {
            const int c = i / M, r = i - c * M;
            X[int64_t(rank[c]) * COMP_XLD + r] = A[c * ldy + r];
        }
    }
}

__global__ __launch_bounds__(256) void truncate_level_apply_kernel(CompLaunch L, int l, int kc, int kt, int kp,
                                                                   int ktp) {
    __shared__ double A[GEN_LD * QR_MAXN], G[64 * SQ_LD], Y[64 * SQ_LD];
    const int t = threadIdx.x;
    const int64_t i0 = blockIdx.x, p = level_first(l - 1) + i0;
    const int M = 2 * kt, ldz = M + QR_PAD;
    const double *X = L.X + i0 * COMP_XSLOT;   // M x ktp used
    for (int h = 0; h < 2; ++h) {              // new transfers: the two kt x ktp blocks of X
        double *En = L.Enew + (2 * p + 1 + h) * L.kmax * L.kmax;
        for (int i = t; i < kt * ktp; i += 256) {
            const int c = i / kt, r = i - c * kt;
            En[int64_t(c) * L.kmax + r] = X[int64_t(c) * COMP_XLD + h * kt + r];
        }
    }
    form_z(L, p, kc, kt, kp, A, ldz, G, Y);
    double *T = L.T + p * L.kmax * L.kmax;     // T_p = X(:, 0:ktp)^T Z_p (ktp x kp)
    for (int i = t; i < ktp * kp; i += 256) {
        const int c = i / ktp, r = i - c * ktp;
        double acc = 0.0;
        for (int u = 0; u < M; ++u) acc += X[int64_t(r) * COMP_XLD + u] * A[c * ldz + u];
        T[int64_t(c) * L.kmax + r] = acc;
    }
}

__global__ __launch_bounds__(256) void symmetry_check_kernel(const double *blocks, const MirrorDesc *desc, int64_t n,
                                                             int32_t *flag) {
    for (int64_t p = blockIdx.x; p < n; p += gridDim.x) {
        const MirrorDesc d = desc[p];
        int diff = 0;
        for (int e = threadIdx.x; e < d.k * d.k; e += 256) {
            const int c = e / d.k, r = e - c * d.k;
            diff |= blocks[d.a + at2(d.k, r, c)] != blocks[d.b + at2(d.k, c, r)];
        }
        if (__syncthreads_or(diff) && threadIdx.x == 0) *flag = 1;
    }
}

__global__ __launch_bounds__(256) void place_kernel(const double *src, double *dst, const PlaceDesc *desc, int64_t n) {
    for (int64_t b = blockIdx.x; b < n; b += gridDim.x) {
        const PlaceDesc d = desc[b];
        const int64_t ne = int64_t((d.C + 1) >> 1) * d.R * 2;
        for (int64_t e = threadIdx.x; e < ne; e += 256) {
            const int w = int(e & 1);
            const int64_t g = e >> 1;
            const int r = int(g % d.R), c = int(g / d.R) * 2 + w;
            double v = 0.0;
            if (c < d.C) v = d.transpose ? src[d.src + int64_t(r) * d.ld + c] : src[d.src + int64_t(c) * d.ld + r];
            dst[d.dst + e] = v;
        }
    }
}

}  // namespace

hipError_t launch_basis_generation(const CompLaunch &L, int level, int k, int kp, bool parent_term, hipStream_t st) {
    if (k < 1 || k > QR_MAXN || kp > QR_MAXN || (parent_term && kp < 1)) return hipErrorInvalidValue;
    auto *kernel = k <= 16 ? basis_generation_kernel<1>
                 : k <= 32 ? basis_generation_kernel<2>
                 : k <= 48 ? basis_generation_kernel<3> : basis_generation_kernel<4>;
    hipLaunchKernelGGL(kernel, dim3(unsigned(int64_t(1) << level)), dim3(BG_THREADS), 0, st, L,
                       level, k, kp, parent_term ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_truncate_leaves(const CompLaunch &L, int k, double eps, hipStream_t st) {
    if (k < 1 || k > QR_MAXN) return hipErrorInvalidValue;
    hipLaunchKernelGGL(truncate_leaves_kernel, dim3(unsigned(L.nleaves)), dim3(256), 0, st, L, k, eps);
    return hipGetLastError();
}

hipError_t launch_truncate_leaves_apply(const CompLaunch &L, int k, int kt, hipStream_t st) {
    if (k < 1 || k > QR_MAXN || kt < 1 || kt > k) return hipErrorInvalidValue;
    hipLaunchKernelGGL(truncate_leaves_apply_kernel, dim3(unsigned(L.nleaves)), dim3(256), 0, st, L, k, kt);
    return hipGetLastError();
}

hipError_t launch_truncate_level(const CompLaunch &L, int l, int kc, int kt, int kp, double eps, hipStream_t st) {
    if (l < 1 || kc < 1 || kc > QR_MAXN || kt < 1 || kt > kc || 2 * kt > QR_MAXM || kp < 1 || kp > QR_MAXN)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(truncate_level_kernel, dim3(unsigned(int64_t(1) << (l - 1))), dim3(256), 0, st, L, l, kc, kt,
                       kp, eps);
    return hipGetLastError();
}

hipError_t launch_truncate_level_apply(const CompLaunch &L, int l, int kc, int kt, int kp, int ktp, hipStream_t st) {
    if (l < 1 || kc < 1 || kc > QR_MAXN || kt < 1 || kt > kc || 2 * kt > QR_MAXM || kp < 1 || kp > QR_MAXN ||
        ktp < 1 || ktp > kp || ktp > 2 * kt)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(truncate_level_apply_kernel, dim3(unsigned(int64_t(1) << (l - 1))), dim3(256), 0, st, L, l, kc,
                       kt, kp, ktp);
    return hipGetLastError();
}

hipError_t launch_symmetry_check(const double *blocks, const MirrorDesc *desc, int64_t n, int32_t *flag,
                                 hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const int64_t grid = n < 65536 ? n : 65536;
    hipLaunchKernelGGL(symmetry_check_kernel, dim3(unsigned(grid)), dim3(256), 0, st, blocks, desc, n, flag);
    return hipGetLastError();
}

hipError_t launch_place(const double *src, double *dst, const PlaceDesc *desc, int64_t n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const int64_t grid = n < 65536 ? n : 65536;
    hipLaunchKernelGGL(place_kernel, dim3(unsigned(grid)), dim3(256), 0, st, src, dst, desc, n);
    return hipGetLastError();
}

}  // namespace h2
