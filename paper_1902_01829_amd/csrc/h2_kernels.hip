// HIP kernels of libh2mv for gfx950 (MI355X): generation of the H^2
// representation on the device, and the phases of the single-vector product
// (Sec. 4): leaf projection and upsweep (Sec. 4.2), tree multiplication with
// all levels in one launch together with the dense near field (Sec. 4.3,
// Sec. 4.1), downsweep and leaf expansion (Sec. 4.4).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "h2_device.h"

namespace h2 {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------- geometry
// 1-D Lagrange polynomial a over the Chebyshev nodes t, at s.
__device__ double lagrange_1d(const double *t, int p, int a, double s) {
    double v = 1.0;
    for (int b = 0; b < p; ++b)
        if (b != a) v *= (s - t[b]) / (t[a] - t[b]);
    return v;
}

// Tensor Lagrange polynomial nu (axis 0 fastest) of node v's box at x.
__device__ double lagrange_box(const Geometry &g, int64_t v, int nu, const double *x) {
    double val = 1.0;
    for (int ax = 0; ax < g.dim; ++ax) {
        const int a = nu % g.cheb_p;
        nu /= g.cheb_p;
        const double lo = g.lo[v * g.dim + ax], hi = g.hi[v * g.dim + ax];
        const double c = 0.5 * (lo + hi), h = 0.5 * (hi - lo);
        val *= lagrange_1d(g.cheb, g.cheb_p, a, (x[ax] - c) / h);
    }
    return val;
}

// Chebyshev interpolation node nu of node v's box.
__device__ void cheb_point(const Geometry &g, int64_t v, int nu, double *xi) {
    for (int ax = 0; ax < g.dim; ++ax) {
        const int a = nu % g.cheb_p;
        nu /= g.cheb_p;
        const double lo = g.lo[v * g.dim + ax], hi = g.hi[v * g.dim + ax];
        xi[ax] = 0.5 * (lo + hi) + 0.5 * (hi - lo) * g.cheb[a];
    }
}

// Exponential covariance exp(-|a - b| / corr_len) (Sec. 4.6).
__device__ double kernel_exp(const double *a, const double *b, int dim, double corr_len) {
    double r2 = 0.0;
    for (int i = 0; i < dim; ++i) r2 += (a[i] - b[i]) * (a[i] - b[i]);
    return exp(-sqrt(r2) / corr_len);
}

// Round-to-nearest-even of an FP32 value to its upper 16 bits (BF16 code).
__device__ uint16_t bf16_rne(float f) {
    const uint32_t u = __float_as_uint(f);
    return uint16_t((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Element kinds: storage type T, the 16-byte item type V holding W elements,
// and the arithmetic type P of a block's partial sums.
template <int KIND> struct Elem;
template <> struct Elem<ELEM_F64> {
    using T = double;
    using V = f64x2;
    using P = double;
    static constexpr int W = 2;
    __device__ static void unpack(const V &r, double *v) {
        v[0] = r.x;
        v[1] = r.y;
    }
    __device__ static T store(double v) { return v; }
};
template <> struct Elem<ELEM_F32> {
    using T = float;
    using V = f32x4;
    using P = float;
    static constexpr int W = 4;
    __device__ static void unpack(const V &r, float *v) {
        v[0] = r.x;
        v[1] = r.y;
        v[2] = r.z;
        v[3] = r.w;
    }
    __device__ static T store(double v) { return float(v); }
};
template <> struct Elem<ELEM_BF16> {
    using T = uint16_t;
    using V = u32x4;
    using P = float;
    static constexpr int W = 8;
    __device__ static void unpack(const V &r, float *v) {
        v[0] = __uint_as_float(r.x << 16);
        v[1] = __uint_as_float(r.x & 0xffff0000u);
        v[2] = __uint_as_float(r.y << 16);
        v[3] = __uint_as_float(r.y & 0xffff0000u);
        v[4] = __uint_as_float(r.z << 16);
        v[5] = __uint_as_float(r.z & 0xffff0000u);
        v[6] = __uint_as_float(r.w << 16);
        v[7] = __uint_as_float(r.w & 0xffff0000u);
    }
};

__device__ inline int64_t readlane64(int64_t v, int j) {
    const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(uint64_t(v))), j));
    const uint32_t hi = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(uint64_t(v) >> 32)), j));
    return int64_t((uint64_t(hi) << 32) | lo);
}

// Decodes element index e of an R-row block in 16-byte column groups of W.
__device__ inline void decode(int e, int R, int W, int &r, int &c) {
    const int w = e % W, t = e / W;
    r = t % R;
    c = (t / R) * W + w;
}

// ---------------------------------------------------------------- fill kernels
// Leaf bases: U_j (m_j x k) with U[r, nu] = L^(j)_nu(point r), and V_j^T
// (k x m_j), the same values transposed (V = U: one tree for rows and columns,
// the symmetric case of Sec. 2.2).
template <int KIND>
__global__ __launch_bounds__(256) void fill_leaf_bases_kernel(
    Geometry g, typename Elem<KIND>::T *basis, const int64_t *leaf_node, const int64_t *off_U,
    const int64_t *off_VT, int64_t nleaves) {
    using E = Elem<KIND>;
    constexpr int W = E::W;
    const int64_t j = blockIdx.x;
    if (j >= nleaves) return;
    const int64_t v = leaf_node[j], b = g.begin[v];
    const int m = int(g.end[v] - b), k = g.rank;
    const int nU = m * ((k + W - 1) / W) * W, nVT = k * ((m + W - 1) / W) * W;
    for (int e = threadIdx.x; e < nU; e += blockDim.x) {
        int r, c;
        decode(e, m, W, r, c);
        const double val = c < k ? lagrange_box(g, v, c, g.pts + (b + r) * g.dim) : 0.0;
        basis[off_U[j] + e] = E::store(val);
    }
    for (int e = threadIdx.x; e < nVT; e += blockDim.x) {
        int r, c;
        decode(e, k, W, r, c);
        const double val = c < m ? lagrange_box(g, v, r, g.pts + (b + c) * g.dim) : 0.0;
        basis[off_VT[j] + e] = E::store(val);
    }
}

// Transfers (Eq. (1) of Sec. 2.2): E_c[mu, nu] = L^(parent)_nu(xi^(c)_mu), a
// k x k block with U_parent = [U_c1 E_c1; U_c2 E_c2]; F_c^T = E_c^T is stored
// next to it for the upsweep.
template <int KIND>
__global__ __launch_bounds__(256) void fill_transfers_kernel(
    Geometry g, typename Elem<KIND>::T *basis, const int64_t *off_E, const int64_t *off_FT,
    int64_t nnodes) {
    using E = Elem<KIND>;
    constexpr int W = E::W;
    const int64_t c = int64_t(blockIdx.x) + 1;
    if (c >= nnodes || off_E[c] < 0) return;
    const int64_t par = (c - 1) / 2;
    const int k = g.rank, nE = k * ((k + W - 1) / W) * W;
    for (int e = threadIdx.x; e < nE; e += blockDim.x) {
        int r, col;
        decode(e, k, W, r, col);
        double xi[3];
        double ev = 0.0, fv = 0.0;
        if (col < k) {
            cheb_point(g, c, r, xi);               // E[r, col]
            ev = lagrange_box(g, par, col, xi);
            cheb_point(g, c, col, xi);             // F^T[r, col] = E[col, r]
            fv = lagrange_box(g, par, r, xi);
        }
        basis[off_E[c] + e] = E::store(ev);
        basis[off_FT[c] + e] = E::store(fv);
    }
}

// Coupling blocks S_st[mu, nu] = K(xi^(s)_mu, xi^(t)_nu) and dense blocks
// D_st[a, b] = K(p_a, p_b) (Sec. 4.6), stored as FP64 / FP32 values.
template <int KIND>
__global__ __launch_bounds__(256) void fill_blocks_kernel(Geometry g, typename Elem<KIND>::T *out,
                                                           const FillDesc *desc, int64_t nblocks) {
    using E = Elem<KIND>;
    constexpr int W = E::W;
    const int64_t blk = blockIdx.x;
    if (blk >= nblocks) return;
    const FillDesc d = desc[blk];
    const bool dense = d.kind == FILL_DENSE;
    const int R = dense ? int(g.end[d.s] - g.begin[d.s]) : g.rank;
    const int C = dense ? int(g.end[d.t] - g.begin[d.t]) : g.rank;
    const int ne = R * ((C + W - 1) / W) * W;
    for (int e = threadIdx.x; e < ne; e += blockDim.x) {
        int r, c;
        decode(e, R, W, r, c);
        double val = 0.0;
        if (c < C) {
            if (dense) {
                val = kernel_exp(g.pts + (g.begin[d.s] + r) * g.dim, g.pts + (g.begin[d.t] + c) * g.dim,
                                 g.dim, g.corr_len);
            } else {
                double xs[3], xt[3];
                cheb_point(g, d.s, r, xs);
                cheb_point(g, d.t, c, xt);
                val = kernel_exp(xs, xt, g.dim, g.corr_len);
            }
        }
        out[d.a + e] = E::store(val);
    }
}

// BF16 with one FP32 scale per block: s = max |fp32(a)|, code = bf16(fp32(a) / s).
__global__ __launch_bounds__(256) void fill_blocks_bf16_kernel(Geometry g, uint16_t *out, float *scales,
                                                                const FillDesc *desc, int64_t nblocks) {
    constexpr int W = 8;
    __shared__ float vals[64 * 64];
    __shared__ float wmax[4];
    const int64_t blk = blockIdx.x;
    if (blk >= nblocks) return;
    const FillDesc d = desc[blk];
    const bool dense = d.kind == FILL_DENSE;
    const int R = dense ? int(g.end[d.s] - g.begin[d.s]) : g.rank;
    const int C = dense ? int(g.end[d.t] - g.begin[d.t]) : g.rank;
    const int ne = R * ((C + W - 1) / W) * W;
    float mx = 0.0f;
    for (int e = threadIdx.x; e < ne; e += blockDim.x) {
        int r, c;
        decode(e, R, W, r, c);
        double val = 0.0;
        if (c < C) {
            if (dense) {
                val = kernel_exp(g.pts + (g.begin[d.s] + r) * g.dim, g.pts + (g.begin[d.t] + c) * g.dim,
                                 g.dim, g.corr_len);
            } else {
                double xs[3], xt[3];
                cheb_point(g, d.s, r, xs);
                cheb_point(g, d.t, c, xt);
                val = kernel_exp(xs, xt, g.dim, g.corr_len);
            }
        }
        const float f = float(val);
        vals[e] = f;
        mx = fmaxf(mx, fabsf(f));
    }
    for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = mx;
    __syncthreads();
    const float s = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
    for (int e = threadIdx.x; e < ne; e += blockDim.x)
        out[d.a + e] = s == 0.0f ? uint16_t(0) : bf16_rne(vals[e] / s);
    if (threadIdx.x == 0) scales[d.sidx] = s;
}

// ---------------------------------------------------------------- slot sums
// One wavefront per segment: lane r adds partials[c * 64 + r] over the
// segment's slots in order, in FP64, to the segment's element r.
template <typename TV>
__global__ __launch_bounds__(256) void reduce_chunks_kernel(const ReduceDesc *__restrict__ desc, int64_t n,
                                                            const TV *__restrict__ partials, TV *__restrict__ out0,
                                                            TV *__restrict__ out1) {
    const int64_t i = int64_t(blockIdx.x) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = threadIdx.x & 63;
    if (i >= n) return;
    const ReduceDesc d = desc[i];
    if (r >= d.R) return;
    TV *dst = (d.point ? out1 : out0) + d.out + r;
    double acc = double(*dst);
    int c = d.c0;
    for (; c + 8 <= d.c1; c += 8) {   // eight loads in flight, added in order
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = double(partials[int64_t(c + u) * 64 + r]);
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += v[u];
    }
    for (; c < d.c1; ++c) acc += double(partials[int64_t(c) * 64 + r]);
    *dst = TV(acc);
}

// ---------------------------------------------------------------- transposed copies
// One workgroup per block (grid-strided over the list): destination element
// e = ((r / W) * C + c) * W + r % W of the C x R transpose takes source element
// (r, c) at ((c / W) * R + r) * W + c % W; padding columns of the destination's
// last group are written as zero.
template <typename T, int W>
__global__ __launch_bounds__(256) void transpose_blocks_kernel(const T *__restrict__ src, T *__restrict__ dst,
                                                               const TransDesc *__restrict__ desc, int64_t n) {
    for (int64_t b = blockIdx.x; b < n; b += gridDim.x) {
        const TransDesc d = desc[b];
        const int R = d.R, C = d.C;                       // source R x C, destination C x R
        const int64_t ne = int64_t((R + W - 1) / W) * C * W;
        for (int64_t e = threadIdx.x; e < ne; e += blockDim.x) {
            const int w = int(e % W);
            const int64_t g = e / W;
            const int c = int(g % C), r = int(g / C) * W + w;   // destination (c, r) = source (r, c)
            T v = T(0);
            if (r < R) v = src[d.src + (int64_t(c / W) * R + r) * W + c % W];
            dst[d.dst + e] = v;
        }
    }
}

// ---------------------------------------------------------------- tree sweeps
// A launch takes up to SWEEP_MAX_DEPTH levels of the tree: one workgroup per
// subtree of 2^depth bottom nodes, 2^depth 2^split wavefronts, the subtree's
// vectors in LDS.  Every level is then that many equal pieces of work -- 2^p
// nodes at depth p, their blocks' columns split over the wavefronts -- and
// costs one exchange through LDS instead of a launch and its chain of memory
// round trips: a piece's items (at most 8 per lane by the choice of split) are
// requested before the level above is summed, behind barriers that order LDS
// only.  Partial sums are added in a fixed order; FP32 bases keep a block's FP32
// sum whole (pieces are blocks, split = 0), as splitting it would round it
// differently.  Bound by latency for small
// matrices -- the code is kept short, with one copy of each step, as its first
// fetch is part of it -- and by the blocks' bytes near the leaves of large ones.
// Against one launch per level, a launch for the leaves and one for the chunk
// sums: 4,096 points of rank 16 FP64 41 -> 31 us (12 -> 3 launches), 16,384
// points of rank 64 FP64 153 -> 122 us, FP32 98 -> 81, BF16 80 -> 63 us; 60,000
// points of rank 49 FP32 262 -> 205 us; 2^20 points of rank 64 6.93 -> 6.85 ms.

// Barrier of a workgroup that exchanges data through LDS alone: unlike
// __syncthreads, it does not wait for the global loads in flight.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// One wavefront's piece of a block: lane = grp * R + r takes the column groups
// c0 + grp, c0 + grp + G, ... below c1 of row r (G = 64 / R lane groups); the
// first N are requested ahead of their use.
template <int KIND>
struct Piece {
    using E = Elem<KIND>;
    using V = typename E::V;
    using P = typename E::P;
    static constexpr int W = E::W;
    static constexpr int N = KIND == ELEM_F64 ? 8 : 16;
    const char *base;
    uint32_t row;            // the lane's byte offset of column group 0
    int R, G, first, c1, cw_last, n;   // n: items per lane, wave-uniform
    bool live;
    V raw[N];

    // part k of ks of the R x C block at base
    __device__ __forceinline__ void request(const typename E::T *block, int rows, int C, int k, int ks, int lane) {
        base = reinterpret_cast<const char *>(block);
        R = rows;
        G = 64 / R;
        const int grp = lane / R, CW = (C + W - 1) / W, c0 = CW * k / ks;
        live = grp < G;
        row = uint32_t(lane - grp * R) * 16u;
        first = c0 + (live ? grp : 0);
        c1 = CW * (k + 1) / ks;
        cw_last = CW - 1;
        n = (c1 - c0 + G - 1) / G;
        // (four at a time; the addresses past the piece are clamped into the block)
#pragma unroll
        for (int u = 0; u < N; u += 4) {
            if (u >= n) continue;   // wave-uniform
#pragma unroll
            for (int t = u; t < u + 4; ++t) raw[t] = item(first + t * G);
        }
    }
    __device__ __forceinline__ V item(int cw) const {
        return __builtin_nontemporal_load(
            reinterpret_cast<const V *>(base + (__umul24(cw < cw_last ? cw : cw_last, R) * 16u + row)));
    }
    // its products with the input x (LDS, zero past the block's columns)
    __device__ __forceinline__ double products(const P *x) const {
        P s = P(0);
        // four items: the inputs read together, items past the piece left out
        auto add = [&](const V *r, int cw0) __attribute__((always_inline)) {
            P xi[4][W];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int cw = cw0 + t * G, cl = cw < cw_last ? cw : cw_last;
#pragma unroll
                for (int w = 0; w < W; ++w) xi[t][w] = x[cl * W + w];
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                P v[W], q = s;
                E::unpack(r[t], v);
#pragma unroll
                for (int w = 0; w < W; ++w) q = fma(v[w], xi[t][w], q);
                s = cw0 + t * G < c1 ? q : s;
            }
        };
#pragma unroll
        for (int u = 0; u < N; u += 4)
            if (u < n) add(raw + u, first + u * G);
#pragma unroll 1
        for (int u = N; u < n; u += 4) {
            V r[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) r[t] = item(first + (u + t) * G);
            add(r, first + u * G);
        }
        return double(s);
    }
};

// The np pieces of one node are stored one after the other, G R values each
// (64 reserved).  Row r: lane group by lane group the sum of the pieces' values
// for FP32 bases (at most two pieces, whole blocks), piece by piece for FP64;
// added in order, the loads of eight values at a time.
template <int KIND>
__device__ __forceinline__ double add_pieces(const double *part, int np, int R, int r) {
    const int G = 64 / R, n = np * G;
    double t = 0.0;
    if constexpr (KIND == ELEM_F64) {
#pragma unroll 1
        for (int c = 0; c < n; c += 8) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = part[(c + u < n ? c + u : c) * R + r];
#pragma unroll
            for (int u = 0; u < 8; ++u) t += c + u < n ? v[u] : 0.0;
        }
    } else {
#pragma unroll 1
        for (int g = 0; g < G; g += 4) {
            double v[2][4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = g + u < G ? g + u : g;
                v[0][u] = part[c * R + r];
                v[1][u] = np > 1 ? part[(G + c) * R + r] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) t += g + u < G ? v[0][u] + v[1][u] : 0.0;
        }
    }
    return t;
}

// log2 of the wavefronts that share the 2^d blocks of a level, 2^ws in all.
template <int KIND>
__device__ __forceinline__ int sharing(int ws, int d) { return KIND == ELEM_F64 ? ws : d; }

// Leaf projection x^_j = V_j^T x(j) (with a.leaf) and
// x^_p = F_c1^T x^_c1 + F_c2^T x^_c2 for the depths above the bottom one.
template <int KIND>
__global__ __launch_bounds__(1024) void upsweep_kernel(const SweepLaunch a, const int64_t *__restrict__ off_leaf,
                                                       const int64_t *__restrict__ off_tr,
                                                       const int64_t *__restrict__ leaf_begin,
                                                       const int64_t *__restrict__ leaf_end) {
    using P = typename Elem<KIND>::P;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int T = a.depth, S = a.split, WS = T + S, NB = 1 << T;   // NB bottom nodes
    double *part = reinterpret_cast<double *>(lds);                // (1 << WS) x 64
    P *xs = reinterpret_cast<P *>(part + (64 << WS));              // leaf inputs: NB x 64
    P *xv = xs + (a.leaf ? NB * 64 : 0);                           // the subtree's x^, heap order: (2 NB - 1) x 64
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t b = blockIdx.x;
    const auto *basis = static_cast<const typename Elem<KIND>::T *>(a.basis);
    P *tree = static_cast<P *>(a.tree);
    auto node = [&](int p, int i) { return (int64_t(1) << (a.level + p)) - 1 + (b << p) + i; };
    // depths a.leaf ? T : T - 1 down to 0, this wavefront's piece of each: of the
    // leaf basis (depth T) or of a child's transfer
    Piece<KIND> piece;
    if (!a.leaf) {
        if (wv < NB) xv[(NB - 1 + wv) * 64 + lane] = lane < a.rank[T] ? tree[node(T, wv) * a.stride + lane] : P(0);
    } else if (wv < NB) {
        const int64_t j = (b << T) + wv, x0 = leaf_begin[j];
        xs[wv * 64 + lane] = lane < int(leaf_end[j] - x0) ? P(a.x[x0 + lane]) : P(0);
    }
    const P *in = nullptr;   // the piece's input
    bool active = false;     // whether this wavefront has a piece
#pragma unroll 1
    for (int p = a.leaf ? T : T - 1, have = 0; p >= -1; --p, have = 1) {
        if (have) {
            lds_barrier();
            // piece `sub` of its node of depth p + 1, whose blocks are those of depth p + 1 (leaf) or p + 2
            const int sub = wv & ((1 << (sharing<KIND>(WS, p + 1 == T ? T : p + 2) - p - 1)) - 1);
            const double v = active ? piece.products(in) : 0.0;
            if (active && piece.live) part[(wv - sub) * 64 + sub * piece.G * piece.R + lane] = v;
        }
        const int shared = have ? sharing<KIND>(WS, p + 1 == T ? T : p + 2) : 0;
        if (p >= 0) {
            const bool at_leaf = p == T;
            const int d = at_leaf ? T : p + 1, w = sharing<KIND>(WS, d), ks = 1 << (w - d), i = wv >> (w - d);   // input node i of depth d
            active = wv < (1 << w);   // wave-uniform
            if (active) {
                const int64_t j = (b << T) + i;
                const int64_t off = at_leaf ? off_leaf[j] : off_tr[node(d, i)];
                const int C = at_leaf ? int(leaf_end[j] - leaf_begin[j]) : a.rank[d];
                in = at_leaf ? xs + i * 64 : xv + ((1 << d) - 1 + i) * 64;
                piece.request(basis + off, a.rank[p], C, wv & (ks - 1), ks, lane);
            }
        }
        if (have) {   // sums of depth p + 1: wavefront i adds node i's pieces, in order
            lds_barrier();
            const int d = p + 1;
            if (wv < (1 << d)) {
                const int R = a.rank[d], nw = 1 << (shared - d);
                const P v = lane < R ? P(add_pieces<KIND>(part + wv * nw * 64, nw, R, lane)) : P(0);
                xv[((1 << d) - 1 + wv) * 64 + lane] = v;
                if (lane < R) tree[node(d, wv) * a.stride + lane] = v;
            }
        }
    }
}

// y^_c = (its tree multiplication's sum) + E_c y^_parent for the depths below
// the root, and with a.leaf y(j) = y_near(j) + U_j y^_j (FP64).  The sums come
// from the stream launch's chunks where its list was cut (a.partials), in
// order, else from the tree and the near-field vector.
template <int KIND>
__global__ __launch_bounds__(1024) void downsweep_kernel(const SweepLaunch a, const int64_t *__restrict__ off_leaf,
                                                         const int64_t *__restrict__ off_tr,
                                                         const int64_t *__restrict__ leaf_begin,
                                                         const int64_t *__restrict__ leaf_end,
                                                         const SumRange *__restrict__ tree_sums,
                                                         const SumRange *__restrict__ near_sums) {
    using P = typename Elem<KIND>::P;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int T = a.depth, S = a.split, WS = T + S, NB = 1 << T;
    double *part = reinterpret_cast<double *>(lds);          // (1 << WS) x 64
    double *iv = part + (64 << WS);          // sums of the subtree's nodes, heap order, then near fields: (3 NB - 1) x 64
    P *yv = reinterpret_cast<P *>(iv + (3 * NB - 1) * 64);   // its y^: (2 NB - 1) x 64
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t b = blockIdx.x;
    const auto *basis = static_cast<const typename Elem<KIND>::T *>(a.basis);
    P *tree = static_cast<P *>(a.tree);
    auto node = [&](int p, int i) { return (int64_t(1) << (a.level + p)) - 1 + (b << p) + i; };
    const bool lowrank = !a.leaf || off_leaf != nullptr;
    const int last = !lowrank ? 0 : a.leaf ? T + 1 : T;   // depths 1 .. T: transfers, T + 1: the leaf basis
    Piece<KIND> piece;
    const P *in = nullptr;   // the piece's input
    bool active = false;     // whether this wavefront has a piece
#pragma unroll 1
    for (int p = 1, have = 0; p <= last + 1; ++p, have = 1) {
        if (have) {
            lds_barrier();
            const int d = p - 1 <= T ? p - 1 : T, sub = wv & ((1 << (sharing<KIND>(WS, d) - d)) - 1);   // piece `sub` of its node
            const double v = active ? piece.products(in) : 0.0;
            if (active && piece.live) part[(wv - sub) * 64 + sub * piece.G * piece.R + lane] = v;
        }
        if (p <= last) {
            const bool at_leaf = p > T;
            const int d = at_leaf ? T : p, w = sharing<KIND>(WS, d), ks = 1 << (w - d), i = wv >> (w - d);   // output node i of depth d
            active = wv < (1 << w);   // wave-uniform
            if (active) {
                const int64_t j = (b << T) + i;
                const int64_t off = at_leaf ? off_leaf[j] : off_tr[node(d, i)];
                const int R = at_leaf ? int(leaf_end[j] - leaf_begin[j]) : a.rank[d];
                in = yv + (at_leaf ? (1 << T) - 1 + i : (1 << (d - 1)) - 1 + (i >> 1)) * 64;
                piece.request(basis + off, R, a.rank[p - 1], wv & (ks - 1), ks, lane);
            }
        }
        if (!have) {   // the starting sums of the subtree's nodes and of its leaves' near fields
#pragma unroll 1
            for (int h = lowrank ? wv : 2 * NB - 1 + wv; h < (a.leaf ? 3 : 2) * NB - 1; h += 1 << WS) {
                const bool leaf = h >= 2 * NB - 1;
                const int d = leaf ? T : 31 - __builtin_clz(unsigned(h + 1)), i = leaf ? h - (2 * NB - 1) : h + 1 - (1 << d);
                const int64_t v = leaf ? (b << T) + i : node(d, i);
                const int64_t y0 = leaf ? leaf_begin[v] : v * a.stride;
                const int n = leaf ? int(leaf_end[v] - y0) : a.rank[d];
                double t = 0.0;
                if (!a.partials || (h == 0 && a.root_done)) {
                    if (lane < n) t = double((leaf ? static_cast<const P *>(a.near) : tree)[y0 + lane]);
                } else {
                    const SumRange r = (leaf ? near_sums : tree_sums)[v];
#pragma unroll 1
                    for (int c = r.c0; c < r.c1; c += 8) {   // eight loads in flight, added in order
                        double w[8];
#pragma unroll
                        for (int u = 0; u < 8; ++u)
                            w[u] = a.partials[int64_t(c + u < r.c1 ? c + u : c) * 64 + (lane < n ? lane : 0)];
#pragma unroll
                        for (int u = 0; u < 8; ++u) t += c + u < r.c1 ? w[u] : 0.0;
                    }
                    if (lane >= n) t = 0.0;
                }
                // (rounded to the vectors' type, as the stream launch stores a sum that is not cut)
                if (h > 0 || leaf) iv[h * 64 + lane] = double(P(t));
                else yv[lane] = P(t);
            }
            if (last == 0) lds_barrier();
        } else {       // sums of depth p - 1: wavefront i adds node i's pieces, in order
            lds_barrier();
            const int d = p - 1;
            if (d <= T && wv < (1 << d)) {
                const int R = a.rank[d], nw = 1 << (sharing<KIND>(WS, d) - d), h = (1 << d) - 1 + wv;
                const P v = lane < R ? P(iv[h * 64 + lane] + add_pieces<KIND>(part + wv * nw * 64, nw, R, lane)) : P(0);
                yv[h * 64 + lane] = v;
                if (d == T && !a.leaf && lane < R) tree[node(d, wv) * a.stride + lane] = v;
            }
        }
    }
    if (a.leaf && wv < NB) {
        const int64_t j = (b << T) + wv, y0 = leaf_begin[j];
        const int m = int(leaf_end[j] - y0);
        if (lane < m)
            a.y[y0 + lane] = iv[(2 * NB - 1 + wv) * 64 + lane] + (lowrank ? add_pieces<KIND>(part + (wv << (sharing<KIND>(WS, T) - T)) * 64, 1 << (sharing<KIND>(WS, T) - T), m, lane) : 0.0);
    }
}

// ---------------------------------------------------------------- streaming launch
// One wavefront per row (or chunk of a row), lane = grp * R + r: lane group
// grp < G = 64 / R takes the block's column groups grp, grp + G, ... of row r.
// A row is walked as one sequence of steps -- in step t of a block every lane
// takes item t of its column groups -- through a ring of D steps held in
// registers, refilled as they are used, so D steps' loads stay in flight
// across block boundaries.  (Waiting at every block's end for its input, then
// for its items eight at a time, left blocks of a few KiB latency-bound: three
// dependent round trips each.)  Of the input segment a step loads only the
// G W values it multiplies, one per lane, and shares them through the
// wavefront's LDS slot.  Bound by the HBM for large matrices (2^20 points: 6.9
// TB/s as before); the product of 50,000 3-D points of rank 27 with leaves of
// 24-25 points went from 1239 to 610 us in FP64, 745 to 350 in FP32 and 559 to
// 240 in BF16.  The loads carry no condition (addresses are clamped
// into the block, past the last step it is loaded again), so the compiler's
// waits count them exactly.  One block's partial sum is kept in the block
// arithmetic type, sums over blocks in FP64, in block order.
template <int KIND, typename TV, typename TO1, int D>
__device__ __forceinline__ void stream_body(
    const RowDesc *__restrict__ rows, int64_t nrows, const BlkDesc *__restrict__ blks,
    const typename Elem<KIND>::T *__restrict__ data, const float *__restrict__ scales,
    const TV *__restrict__ in0, const double *__restrict__ in1, TV *__restrict__ out0, TO1 *__restrict__ out1) {
    using E = Elem<KIND>;
    using P = typename E::P;
    using V = typename E::V;
    constexpr int W = E::W;
    __shared__ __attribute__((aligned(16))) P xs[4][64];
    __shared__ double red[4][64];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t row = int64_t(blockIdx.x) * 4 + wv;
    if (row >= nrows) return;
    const RowDesc rd = rows[row];
    const int R = rd.R, G = 64 / R, g0 = lane / R, rr = lane - g0 * R;
    const int grp = g0 < G ? g0 : 0;   // lanes past the last group repeat the first one's loads; their sums are not used
    const int nb = rd.b1 - rd.b0;
    double acc = 0.0;
    if (nb > 0) {   // wave-uniform
        const BlkDesc first = blks[rd.b0];
        BlkDesc my = blks[rd.b0 + (lane < nb ? lane : nb - 1)];   // descriptors of 64 blocks, one per lane
        float sc = 1.0f;
        if constexpr (KIND == ELEM_BF16) sc = scales[my.sidx];
        const int gw = G * W;
        int nsteps = rd.sel >> 8;
        if (nsteps == 0) {
            for (int k = lane; k < nb; k += 64) nsteps += (blks[rd.b0 + k].C + gw - 1) / gw;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) nsteps += __shfl_xor(nsteps, o);
            nsteps = __builtin_amdgcn_readfirstlane(nsteps);
        }
        const double *in64 = in1;   // the FP64 input: x, or x^ of an FP64 matrix
        if constexpr (std::is_same<TV, double>::value) {
            if (!(rd.sel & ROW_IN_X)) in64 = in0;
        }
        auto steps = [&](auto input_is_x) __attribute__((always_inline)) {
            constexpr bool IN_X = decltype(input_is_x)::value;
            using TX = std::conditional_t<IN_X, double, TV>;
            const TX *xbase;
            if constexpr (IN_X) xbase = in64;
            else xbase = in0;
            struct Step {
                V a;
                TX x;
                int left;     // columns of the block from this step on
                float scale;  // BF16
            };
            // the next step to load: its block and input segment, the lane's byte
            // offsets in them with their last valid values, the columns left
            const char *pa = nullptr, *px = nullptr;
            uint32_t oa = 0, oa_last = 0, ox = 0, ox_last = 0;
            int left = 0, k = 0;
            float scale = 1.0f;
            const uint32_t oa0 = uint32_t(grp * R + rr) * 16u, oa_step = uint32_t(G * R) * 16u;
            const uint32_t ox0 = uint32_t(min(lane, gw - 1)) * uint32_t(sizeof(TX));
            auto start = [&](int64_t a, int64_t in, int C) __attribute__((always_inline)) {
                pa = reinterpret_cast<const char *>(data + a);
                px = reinterpret_cast<const char *>(xbase + in);
                left = C;
                oa = oa0;
                ox = ox0;
                oa_last = uint32_t((((C + W - 1) / W) - 1) * R + rr) * 16u;
                ox_last = uint32_t(C - 1) * uint32_t(sizeof(TX));
            };
            auto open = [&](int kk) __attribute__((always_inline)) {   // block kk of the row, 64 descriptors at a time
                const int j = kk & 63;
                if (j == 0) {
                    my = blks[rd.b0 + (kk + lane < nb ? kk + lane : nb - 1)];
                    if constexpr (KIND == ELEM_BF16) sc = scales[my.sidx];
                    // used here, so that the wait for these loads stays on this path
                    asm volatile("" : "+v"(my.a), "+v"(my.in), "+v"(my.C), "+v"(sc));
                }
                start(readlane64(my.a, j), readlane64(my.in, j), __builtin_amdgcn_readlane(my.C, j));
                if constexpr (KIND == ELEM_BF16)
                    scale = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(sc), j));
            };
            auto load = [&](Step &st) __attribute__((always_inline)) {
                st.left = left;
                st.scale = scale;
                st.a = __builtin_nontemporal_load(reinterpret_cast<const V *>(pa + min(oa, oa_last)));
                st.x = *reinterpret_cast<const TX *>(px + min(ox, ox_last));
                if (k < nb) {   // wave-uniform
                    if (left > gw) {
                        left -= gw;
                        oa += oa_step;
                        ox += uint32_t(gw) * uint32_t(sizeof(TX));
                    } else if (++k < nb) {
                        open(k);
                    }
                }
            };
            P part = P(0);
            auto use = [&](const Step &st) __attribute__((always_inline)) {
                const bool whole = st.left >= gw;   // wave-uniform: the step's columns all exist
                P xv = P(st.x);
                if (!whole) xv = lane < st.left ? xv : P(0);
                xs[wv][lane] = xv;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
                P v[W], x[W];
                E::unpack(st.a, v);
#pragma unroll
                for (int w = 0; w < W; ++w) x[w] = xs[wv][grp * W + w];
                if (whole || grp * W < st.left) {
#pragma unroll
                    for (int w = 0; w < W; ++w) part = fma(v[w], x[w], part);
                }
                if (st.left <= gw) {   // wave-uniform: the block's last step
                    if constexpr (KIND == ELEM_BF16) acc += double(part) * double(st.scale);
                    else acc += double(part);
                    part = P(0);
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
            };
            // the first block's descriptor by itself: a scalar load returns sooner
            start(first.a, first.in, first.C);
            if constexpr (KIND == ELEM_BF16) scale = scales[first.sidx];
            Step ring[D];
#pragma unroll
            for (int s = 0; s < D; ++s) load(ring[s]);
            int i = 0;
            for (; i + D <= nsteps; i += D) {
#pragma unroll
                for (int s = 0; s < D; ++s) {
                    use(ring[s]);
                    load(ring[s]);
                }
            }
#pragma unroll
            for (int s = 0; s < D - 1; ++s)
                if (i + s < nsteps) use(ring[s]);
        };
        if constexpr (std::is_same<TV, double>::value) {
            steps(std::true_type{});   // either input is FP64
        } else {
            if (rd.sel & ROW_IN_X) steps(std::true_type{});
            else steps(std::false_type{});
        }
    }
    if (G > 1) {
        red[wv][lane] = acc;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (lane < R)
            for (int g2 = 1; g2 < G; ++g2) acc += red[wv][g2 * R + lane];
    }
    if (lane < R) {
        if (rd.sel & ROW_OUT_P)
            out1[rd.out + lane] = TO1(acc);
        else
            out0[rd.out + lane] = TV(acc);
    }
}

// Steps in flight per wavefront (8: 84 registers at most, 5 wavefronts per SIMD;
// 6 and 12 measured within 5 % of it over 5,000 to 2^18 points).
constexpr int kStreamDepth = 8;

template <int KIND, typename TV, typename TO1>
__global__ __launch_bounds__(256) void stream_kernel(
    const RowDesc *__restrict__ rows, int64_t nrows, const BlkDesc *__restrict__ blks,
    const typename Elem<KIND>::T *__restrict__ data, const float *__restrict__ scales, const TV *__restrict__ in0,
    const double *__restrict__ in1, TV *__restrict__ out0, TO1 *__restrict__ out1) {
    stream_body<KIND, TV, TO1, kStreamDepth>(rows, nrows, blks, data, scales, in0, in1, out0, out1);
}

// ---------------------------------------------------------------- half storage
// Sums of N values per lane across the N lanes that differ in the lane bits
// MASK, MASK / 2, ..., MASK / (N / 2) (v[k] = the lane's value number k): each
// fold pairs lanes across one bit, each partner keeps the half of its live
// values named by that bit and adds the other's copy of it; lane l ends with
// value number (those bits of l, highest first) summed over its N lanes.
template <int H, int MASK, int N, typename P>
__device__ __forceinline__ void fold_half(P (&v)[N], int lane) {
    const bool up = (lane & MASK) != 0;
#pragma unroll
    for (int k = 0; k < H; ++k) {
        const P keep = up ? v[k + H] : v[k];
        const P send = up ? v[k] : v[k + H];
        v[k] = keep + __shfl_xor(send, MASK);
    }
}
template <int N, int MASK, int LIVE = N, typename P>
__device__ __forceinline__ P fold_lanes(P (&v)[N], int lane) {
    if constexpr (LIVE == 1) {
        return v[0];
    } else {
        fold_half<LIVE / 2, MASK>(v, lane);
        return fold_lanes<N, MASK / 2, LIVE / 2>(v, lane);
    }
}

// Stream phase of a matrix stored by halves: block row i holds only its
// blocks with j >= i (S_ji = S_ij^T, D_ji = D_ij^T).  One wavefront per group
// of consecutive block rows (at most HALF_GROUP_ROWS, taken one after the
// other); with TR lanes per column strip, lane l = TR g + a holds, of every
// block, the tile of rows a + TR k (k < 64 / TR) and columns TR g + c
// (c < TR), so each stored block is read once (all of a lane's 16-byte items
// issued together; each load reads 64 / TR runs of TR consecutive rows) and
// gives both of its products from registers: the lane's partial sums of
// S_ij x_j for its rows, accumulated over the row's blocks (FP64 across
// blocks), and of S_ij^T x_i for its columns, summed over the TR lanes of its
// strip (log2 TR folds), after which lane l holds column l of the transposed
// product.  The group's transposed products of one column segment are added
// in the wavefront's LDS slot for that segment, rows in order (slot[b] >= 0;
// lane l only ever touches element l of a slot, so no barrier), and each LDS
// slot is written once, at the end of the group, to its partial slot
// (gslot): adjacent block rows share many columns, so this writes fewer
// partials, whose cost on the read stream exceeds their share of the bytes.
// A block whose column found no LDS slot writes its own partial slot
// -(slot[b] + 2); slot[b] == -1 marks a diagonal block (no transposed
// product).  Partials are in the vector type (FP64, or FP32 in the reduced
// modes).  At the end of each row the row sums are folded over the strip
// bits (lane l: row l).  A second launch adds each segment's slots to its row
// sum.  The row's own input segment has the offset of its output segment
// (x^ and y^ share the node layout, x and y_near the point layout).
template <int KIND, typename TV, int TR>
__global__ __launch_bounds__(256) void stream_half_kernel(
    const HalfGroup *__restrict__ groups, int64_t ngroups, const RowDesc *__restrict__ rows,
    const BlkDesc *__restrict__ blks, const int32_t *__restrict__ slot, const int32_t *__restrict__ gslot,
    const typename Elem<KIND>::T *__restrict__ data, const float *__restrict__ scales, const TV *__restrict__ in0,
    const double *__restrict__ in1, TV *__restrict__ out0, TV *__restrict__ out1, TV *__restrict__ partials) {
    using E = Elem<KIND>;
    using P = typename E::P;
    using V = typename E::V;
    constexpr int W = E::W;
    constexpr int NS = 64 / TR;    // strips, and rows per lane
    constexpr int IPR = TR / W;    // 16-byte items per row of a strip
    static_assert(IPR >= 1 && TR * NS == 64, "strip of whole 16-byte items");
    __shared__ __attribute__((aligned(16))) P xs[4][64];
    __shared__ TV acc[4][HALF_LDS_SLOTS][64];
    // the wave index made uniform: group, row and block descriptors come through scalar loads
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int a = lane % TR, g = lane / TR;
    const int64_t gi = int64_t(blockIdx.x) * 4 + wv;
    if (gi >= ngroups) return;
    const HalfGroup gd = groups[gi];
    const int ns = gd.s1 - gd.s0;
    for (int s = 0; s < ns; ++s) acc[wv][s][lane] = TV(0);
    for (int32_t row = gd.r0; row < gd.r1; ++row) {
        const RowDesc rd = rows[row];
        const int R = rd.R;
        double rp[NS] = {};   // partial sums of the lane's rows, over the row's blocks
        // The block loop is pipelined: block b + 1's descriptor, slot and input
        // are loaded while block b's items are in flight, the next block's
        // input is staged before block b's transposed product is stored, the
        // LDS fences order LDS only, and the input vector is chosen once per
        // row (the row is uniform, so one of two instantiations runs).
        auto blocks = [&](auto input_is_x) {
            constexpr bool IN_X = decltype(input_is_x)::value;
            // element e of the input segment at off, zero from element n on (the
            // load is clamped into the segment, so the loads issue back to back)
            auto input = [&](int64_t off, int e, int n) {
                const int ec = e < n ? e : n - 1;
                P v;
                if constexpr (IN_X) v = P(in1[off + ec]);
                else v = P(in0[off + ec]);
                return e < n ? v : P(0);
            };
            P xi[NS];   // the row's own input at the lane's rows
#pragma unroll
            for (int k = 0; k < NS; ++k) xi[k] = input(rd.out, a + TR * k, R);
            if (rd.b0 >= rd.b1) return;
            P xj[TR];   // the input at the lane's columns of the current block
            auto stage = [&](const P xv) {
                xs[wv][lane] = xv;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
#pragma unroll
                for (int c = 0; c < TR; ++c) xj[c] = xs[wv][TR * g + c];
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
            };
            BlkDesc bd = blks[rd.b0];
            int32_t sl = slot[rd.b0];
            stage(input(bd.in, lane, bd.C));
            for (int b = rd.b0; b < rd.b1; ++b) {
                const int C = bd.C, CW = (C + W - 1) / W;
                const V *p = reinterpret_cast<const V *>(data + bd.a);   // item (cw, r) at cw * R + r
                V raw[NS][IPR];
#pragma unroll
                for (int k = 0; k < NS; ++k)
#pragma unroll
                    for (int i = 0; i < IPR; ++i) {
                        const int r = a + TR * k, cw = g * IPR + i;
                        raw[k][i] = V{};
                        if (r < R && cw < CW) raw[k][i] = __builtin_nontemporal_load(p + cw * R + r);
                    }
                const bool more = b + 1 < rd.b1;
                const BlkDesc nbd = blks[more ? b + 1 : b];
                const int32_t nsl = slot[more ? b + 1 : b];
                const P nxv = input(nbd.in, lane, nbd.C);   // unused after the last block
                double scale = 1.0;
                if constexpr (KIND == ELEM_BF16) scale = double(scales[bd.sidx]);
                P cp[TR] = {};
#pragma unroll
                for (int k = 0; k < NS; ++k) {
                    P v[TR];
#pragma unroll
                    for (int i = 0; i < IPR; ++i) E::unpack(raw[k][i], v + i * W);
                    P s = P(0);
#pragma unroll
                    for (int c = 0; c < TR; ++c) {
                        s = fma(v[c], xj[c], s);
                        cp[c] = fma(v[c], xi[k], cp[c]);
                    }
                    rp[k] += double(s) * scale;
                }
                P t = P(0);
                if (sl != -1) t = fold_lanes<TR, TR / 2>(cp, lane);   // column TR g + a = lane
                if (more) stage(nxv);
                if (lane < C) {
                    if (sl >= 0)
                        acc[wv][sl][lane] += TV(double(t) * scale);
                    else if (sl <= -2)
                        partials[int64_t(-(sl + 2)) * 64 + lane] = TV(double(t) * scale);
                }
                bd = nbd;
                sl = nsl;
            }
        };
        if (rd.sel & ROW_IN_X)
            blocks(std::true_type{});
        else
            blocks(std::false_type{});
        const double t = fold_lanes<NS, 32>(rp, lane);   // row a + TR g = lane
        if (lane < R) ((rd.sel & ROW_OUT_P) ? out1 : out0)[rd.out + lane] = TV(t);
    }
    for (int s = 0; s < ns; ++s) partials[int64_t(gslot[gd.s0 + s]) * 64 + lane] = acc[wv][s][lane];
}

constexpr int kRowsPerBlock = 4;

template <int KIND, typename TV, typename TO1>
hipError_t run_stream(const RowLaunch &L, hipStream_t st) {
    if (L.nrows <= 0) return hipSuccess;
    const dim3 grid(unsigned((L.nrows + kRowsPerBlock - 1) / kRowsPerBlock)), block(256);
    hipLaunchKernelGGL((stream_kernel<KIND, TV, TO1>), grid, block, L.lds_bytes, st, L.rows, L.nrows, L.blks,
                       static_cast<const typename Elem<KIND>::T *>(L.data), L.scales, static_cast<const TV *>(L.in0),
                       L.in1, static_cast<TV *>(L.out0), static_cast<TO1 *>(L.out1));
    return hipGetLastError();
}

}  // namespace

hipError_t launch_fill_bases(const Geometry &g, int basis_kind, void *basis, const int64_t *leaf_node,
                             const int64_t *off_U, const int64_t *off_VT, int64_t nleaves,
                             const int64_t *off_E, const int64_t *off_FT, int64_t nnodes, hipStream_t st) {
    if (nleaves > 0) {
        if (basis_kind == ELEM_F64)
            hipLaunchKernelGGL(fill_leaf_bases_kernel<ELEM_F64>, dim3(unsigned(nleaves)), dim3(256), 0, st, g,
                               static_cast<double *>(basis), leaf_node, off_U, off_VT, nleaves);
        else
            hipLaunchKernelGGL(fill_leaf_bases_kernel<ELEM_F32>, dim3(unsigned(nleaves)), dim3(256), 0, st, g,
                               static_cast<float *>(basis), leaf_node, off_U, off_VT, nleaves);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (nnodes > 1) {
        if (basis_kind == ELEM_F64)
            hipLaunchKernelGGL(fill_transfers_kernel<ELEM_F64>, dim3(unsigned(nnodes - 1)), dim3(256), 0, st, g,
                               static_cast<double *>(basis), off_E, off_FT, nnodes);
        else
            hipLaunchKernelGGL(fill_transfers_kernel<ELEM_F32>, dim3(unsigned(nnodes - 1)), dim3(256), 0, st, g,
                               static_cast<float *>(basis), off_E, off_FT, nnodes);
        return hipGetLastError();
    }
    return hipSuccess;
}

hipError_t launch_fill_blocks(const Geometry &g, int block_kind, void *blocks, float *scales,
                              const FillDesc *desc, int64_t nblocks, hipStream_t st) {
    if (nblocks <= 0) return hipSuccess;
    // launch in chunks: a grid dimension times the block size must stay below 2^32
    const int64_t chunk = int64_t(1) << 22;
    for (int64_t b0 = 0; b0 < nblocks; b0 += chunk) {
        const int64_t nb = nblocks - b0 < chunk ? nblocks - b0 : chunk;
        if (block_kind == ELEM_F64)
            hipLaunchKernelGGL(fill_blocks_kernel<ELEM_F64>, dim3(unsigned(nb)), dim3(256), 0, st, g,
                               static_cast<double *>(blocks), desc + b0, nb);
        else if (block_kind == ELEM_F32)
            hipLaunchKernelGGL(fill_blocks_kernel<ELEM_F32>, dim3(unsigned(nb)), dim3(256), 0, st, g,
                               static_cast<float *>(blocks), desc + b0, nb);
        else
            hipLaunchKernelGGL(fill_blocks_bf16_kernel, dim3(unsigned(nb)), dim3(256), 0, st, g,
                               static_cast<uint16_t *>(blocks), scales, desc + b0, nb);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_reduce_chunks(const ReduceDesc *desc, int64_t n, const void *partials, void *out0, void *out1,
                                bool vec_f64, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const dim3 grid(unsigned((n + 3) / 4)), block(256);
    if (vec_f64)
        hipLaunchKernelGGL(reduce_chunks_kernel<double>, grid, block, 0, st, desc, n, static_cast<const double *>(partials),
                           static_cast<double *>(out0), static_cast<double *>(out1));
    else
        hipLaunchKernelGGL(reduce_chunks_kernel<float>, grid, block, 0, st, desc, n, static_cast<const float *>(partials),
                           static_cast<float *>(out0), static_cast<float *>(out1));
    return hipGetLastError();
}

// Lanes per column strip of the half-storage kernel, per element kind (16 and
// 32 measured no faster: 8 x 8 tiles in every storage mode).
constexpr int kHalfStripF64 = 8, kHalfStripF32 = 8, kHalfStripBF16 = 8;

hipError_t stream_half_workgroups_per_cu(int kind, bool vec_f64, int *n) {
    if (vec_f64)
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(n, stream_half_kernel<ELEM_F64, double, kHalfStripF64>, 256, 0);
    if (kind == ELEM_F32)
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(n, stream_half_kernel<ELEM_F32, float, kHalfStripF32>, 256, 0);
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(n, stream_half_kernel<ELEM_BF16, float, kHalfStripBF16>, 256, 0);
}

hipError_t launch_stream_half(const RowLaunch &L, const HalfGroup *groups, int64_t ngroups, const int32_t *slot,
                              const int32_t *gslot, void *partials, int kind, bool vec_f64, hipStream_t st) {
    if (ngroups <= 0) return hipSuccess;
    const dim3 grid(unsigned((ngroups + kRowsPerBlock - 1) / kRowsPerBlock)), block(256);
    if (vec_f64) {
        hipLaunchKernelGGL((stream_half_kernel<ELEM_F64, double, kHalfStripF64>), grid, block, 0, st, groups, ngroups,
                           L.rows, L.blks, slot, gslot, static_cast<const double *>(L.data), L.scales,
                           static_cast<const double *>(L.in0), L.in1, static_cast<double *>(L.out0),
                           static_cast<double *>(L.out1), static_cast<double *>(partials));
    } else if (kind == ELEM_F32) {
        hipLaunchKernelGGL((stream_half_kernel<ELEM_F32, float, kHalfStripF32>), grid, block, 0, st, groups, ngroups,
                           L.rows, L.blks, slot, gslot, static_cast<const float *>(L.data), L.scales,
                           static_cast<const float *>(L.in0), L.in1, static_cast<float *>(L.out0),
                           static_cast<float *>(L.out1), static_cast<float *>(partials));
    } else {
        hipLaunchKernelGGL((stream_half_kernel<ELEM_BF16, float, kHalfStripBF16>), grid, block, 0, st, groups,
                           ngroups, L.rows, L.blks, slot, gslot, static_cast<const uint16_t *>(L.data), L.scales,
                           static_cast<const float *>(L.in0), L.in1, static_cast<float *>(L.out0),
                           static_cast<float *>(L.out1), static_cast<float *>(partials));
    }
    return hipGetLastError();
}

hipError_t launch_transpose_blocks(int kind, const void *src, void *dst, const TransDesc *desc, int64_t n,
                                   hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const dim3 grid(unsigned(n < 65536 ? n : 65536)), block(256);
    if (kind == ELEM_F64)
        hipLaunchKernelGGL((transpose_blocks_kernel<double, 2>), grid, block, 0, st, static_cast<const double *>(src),
                           static_cast<double *>(dst), desc, n);
    else if (kind == ELEM_F32)
        hipLaunchKernelGGL((transpose_blocks_kernel<float, 4>), grid, block, 0, st, static_cast<const float *>(src),
                           static_cast<float *>(dst), desc, n);
    else
        hipLaunchKernelGGL((transpose_blocks_kernel<uint16_t, 8>), grid, block, 0, st,
                           static_cast<const uint16_t *>(src), static_cast<uint16_t *>(dst), desc, n);
    return hipGetLastError();
}

hipError_t launch_stream(const RowLaunch &L, int kind, bool vec_f64, bool out1_f64, hipStream_t st) {
    if (vec_f64) return run_stream<ELEM_F64, double, double>(L, st);
    if (kind == ELEM_F32)
        return out1_f64 ? run_stream<ELEM_F32, float, double>(L, st) : run_stream<ELEM_F32, float, float>(L, st);
    return out1_f64 ? run_stream<ELEM_BF16, float, double>(L, st) : run_stream<ELEM_BF16, float, float>(L, st);
}

hipError_t launch_sweep(const SweepLaunch &L, bool up, bool vec_f64, hipStream_t st) {
    if (L.depth < 0 || L.split < 0 || L.depth + L.split > SWEEP_MAX_DEPTH || (L.depth == 0 && !L.leaf)) return hipErrorInvalidValue;
    const int nb = 1 << L.depth, nw = nb << L.split, vb = vec_f64 ? 8 : 4;
    const dim3 grid(1u << L.level), block(64u * unsigned(nw));
    const int slots = 2 * nb - 1;
    const size_t lds = 64 * size_t(up ? nw * 8 + (L.leaf ? nb : 0) * vb + slots * vb : nw * 8 + (slots + nb) * 8 + slots * vb);
    if (up) {
        if (vec_f64)
            hipLaunchKernelGGL(upsweep_kernel<ELEM_F64>, grid, block, lds, st, L, L.off_leaf, L.off_tr, L.leaf_begin, L.leaf_end);
        else
            hipLaunchKernelGGL(upsweep_kernel<ELEM_F32>, grid, block, lds, st, L, L.off_leaf, L.off_tr, L.leaf_begin, L.leaf_end);
    } else {
        if (vec_f64)
            hipLaunchKernelGGL(downsweep_kernel<ELEM_F64>, grid, block, lds, st, L, L.off_leaf, L.off_tr, L.leaf_begin,
                               L.leaf_end, L.tree_sums, L.near_sums);
        else
            hipLaunchKernelGGL(downsweep_kernel<ELEM_F32>, grid, block, lds, st, L, L.off_leaf, L.off_tr, L.leaf_begin,
                               L.leaf_end, L.tree_sums, L.near_sums);
    }
    return hipGetLastError();
}

namespace {

// A plain streaming read: consecutive lanes take consecutive 16-byte items
// (each wavefront load is one contiguous kilobyte, like the product kernels'),
// non-temporal, eight in flight per lane, grid-strided; one XOR per workgroup
// reaches sink so that the loads stay.
typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
__global__ __launch_bounds__(256) void read_probe_kernel(const u64x2 *__restrict__ p, int64_t n16,
                                                         unsigned long long *__restrict__ sink) {
    __shared__ unsigned long long part[256];
    const int64_t stride = int64_t(gridDim.x) * 256;
    int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    unsigned long long acc = 0;
    for (; i + 7 * stride < n16; i += 8 * stride) {
        u64x2 v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = __builtin_nontemporal_load(p + i + k * stride);
#pragma unroll
        for (int k = 0; k < 8; ++k) acc ^= v[k].x ^ v[k].y;
    }
    for (; i < n16; i += stride) {
        const u64x2 v = __builtin_nontemporal_load(p + i);
        acc ^= v.x ^ v.y;
    }
    part[threadIdx.x] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0;
        for (int k = 0; k < 256; ++k) t ^= part[k];
        sink[blockIdx.x] = t;
    }
}

}  // namespace

hipError_t launch_read_probe(const void *buf, int64_t bytes, int grid, void *sink, hipStream_t st) {
    hipLaunchKernelGGL(read_probe_kernel, dim3(unsigned(grid)), dim3(256), 0, st, static_cast<const u64x2 *>(buf),
                       bytes / 16, static_cast<unsigned long long *>(sink));
    return hipGetLastError();
}

}  // namespace h2
