// Many right-hand sides of an FP64 matrix on the FP64 matrix cores (gfx950).
//
// Same phases and work lists as the FP32 tiles of h2_mm.hip: every per-node
// vector is a tile of up to MM_TILE right-hand sides, a block product is an
// (R x C block) x (C x NR tile) contraction with v_mfma_f64_16x16x4_f64.
// Within a tile, row r holds its NR right-hand sides in consecutive doubles
// (NR = 16 or 32, the width of the pass), rows padded with zeros to a
// multiple of 16, so a lane's operand is one 8- or 16-byte load and each
// quarter-wavefront reads one contiguous run.
//
// What bounds it: the blocks' bytes, and at 32 right-hand sides nearly as much
// the matrix cores (2 x 32 flops per 8 stored bytes at 78.6 TFLOP/s take 0.7
// of the time the bytes take at 7 TB/s).  2-D, 2^18 points, rank 64: 32
// right-hand sides 58.1 ms as single-vector products -> 2.8 ms (10.4 GB of
// blocks; the streaming launch 2.35 ms, 4.4 TB/s, L1 address units 93 % busy,
// matrix cores 51 %), 8 right-hand sides 14.0 -> 2.2 ms.  The block reads alone, without the result tiles' stores, run at
// 7.0 TB/s (6.27 ms for the 43.7 GB of the 2^20-point matrix) and the whole
// launch without its stores takes 6.7 ms (16 right-hand sides) and 7.6 ms
// (32): the 0.4 and 0.8 GB of tiles written while the HBM is read at its
// limit cost 1.5 and 1.9 ms, whatever the rows' order, the loads' shape (256-byte
// or 1-KiB runs) and the depth of the ring.
//
// Included by h2_mm.hip only (round16 and readlane64 are defined there).
#pragma once

namespace h2 {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

// A tile row's operand of one lane: right-hand sides 2n and 2n + 1 (NR = 32)
// or n (NR = 16), n = lane % 16.
template <int NR> struct Rhs;
template <> struct Rhs<32> {
    typedef f64x2 V;
    __device__ static double get(const V &v, int t) { return t ? v.y : v.x; }
};
template <> struct Rhs<16> {
    typedef double V;
    __device__ static double get(const V &v, int) { return v; }
};

// One chunk of a row's work: 8 columns of a block, 32 rows.  Lane (g, n)
// = (lane / 16, lane % 16) holds the 16-byte block items of column pair g of
// the chunk at rows 16 t + n (t = 0, 1), and the tile rows of its two columns:
// the K = 4 operands of two MFMA steps (the pairs' first, then second columns).
template <int NR>
struct Chunk {
    f64x2 a[2];
    typename Rhs<NR>::V b[2];
    int left;   // columns of the block from this chunk on
    int tr;     // HALF: the block is the transpose of the stored one
};

// HALF (streaming launch of a matrix stored by halves): blocks with sidx = 1
// are the transposes of the stored ones.  A 16-byte item then holds two rows
// of the product's block at one column, where otherwise it holds two columns
// at one row, so the item's two row tiles take the even and the odd rows for
// either kind, and a chunk's two loads per lane are the items of columns
// 4 u + g (transposed) or of rows 2 n + t (as stored).  Every stored block is
// read twice, as itself and as its mirror: writing the mirror's product out
// instead would cost as many bytes in partial tiles as the second read.
// (60,000 2-D points of rank 49, 6 right-hand sides 1.98 -> 0.75 ms against
// single-vector products; 2^18 points of rank 64, 32 of them 37.1 -> 3.4 ms.)
//
// SPLIT = 4: the four wavefronts of a workgroup take a quarter of one item's
// chunks each, and the first adds the others' sums in order through LDS.
//
// One work item: rows 32 mt .. 32 mt + 31 of an output segment, all NR
// right-hand sides.  The row's blocks are walked as one sequence of 8-column
// chunks through a ring of D chunk registers sets: each is refilled as soon as
// its products are issued, so D chunks (4 KiB of block and tile loads each)
// stay in flight across block boundaries whatever the blocks' widths.  The
// loads carry no condition (past the last chunk they re-read it), which keeps
// the compiler's wait counts exact.  Sums run in FP64 accumulators over all
// blocks of the row, in block order.
template <int NR, bool LEAF, int D, int SPLIT, bool HALF>
__device__ __forceinline__ void mm64_item(const Mm64Launch &L, const RowDesc *__restrict__ rows,
                                          const BlkDesc *__restrict__ blks, int32_t item, int wv, int lane) {
    constexpr int NN = NR / 16;   // MFMA column tiles
    using B = typename Rhs<NR>::V;
    const RowDesc rd = rows[item >> 1];
    const int R = rd.R, mt = item & 1, n = lane & 15, g = lane >> 4;
    if (32 * mt >= R) return;
    const bool two = HALF ? 32 * mt + 1 < R : 32 * mt + 16 < R;   // wave-uniform: the item has a second row tile
    int rc[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int r = 32 * mt + (HALF ? 2 * n + t : 16 * t + n);
        rc[t] = r < R ? r : R - 1;   // rows past the segment read its last row; their sums are not used
    }
    const double *xbase = (rd.sel & ROW_IN_X) ? L.in_pts : L.in_tree;
    f64x4 acc[2][NN] = {};

    const int nb = rd.b1 - rd.b0;
    if (nb > 0) {
        const BlkDesc my = blks[rd.b0 + (lane < nb ? lane : nb - 1)];   // one descriptor per lane
        const char *pa = nullptr, *pb = nullptr;                         // the block and its input tile
        int C = 0, c0 = 0, k = 0, tr = 0;
        auto open = [&](int kk) {
            BlkDesc d;
            if (kk < 64) {
                d.a = readlane64(my.a, kk);
                d.in = readlane64(my.in, kk);
                d.C = __builtin_amdgcn_readlane(my.C, kk);
                if constexpr (HALF) d.sidx = __builtin_amdgcn_readlane(my.sidx, kk);
            } else {
                d = blks[rd.b0 + kk];
            }
            pa = reinterpret_cast<const char *>(static_cast<const double *>(L.data) + d.a);
            pb = reinterpret_cast<const char *>(xbase + d.in);
            C = d.C;
            if constexpr (HALF) tr = d.sidx;
        };
        // the row's chunks, counted first: whole rounds of the ring then hold no
        // branch around a load (the compiler's waits would become full drains)
        auto chunks_of = [&](int kk) { return kk < nb ? ((kk < 64 ? my.C : blks[rd.b0 + kk].C) + 7) >> 3 : 0; };
        int nch = 0;
        for (int kk = lane; kk < nb; kk += 64) nch += chunks_of(kk);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) nch += __shfl_xor(nch, o);
        nch = __builtin_amdgcn_readfirstlane(nch);
        if constexpr (SPLIT > 1) {
            // this wavefront's quarter: its first block k and column c0, by a
            // prefix sum over 64 blocks at a time
            const int first = nch * wv / SPLIT;
            nch = nch * (wv + 1) / SPLIT - first;
            int before = 0;
            for (int k0 = 0; k0 < nb && nch > 0; k0 += 64) {   // wave-uniform
                const int own = chunks_of(k0 + lane);
                int end = own;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const int v = __shfl_up(end, o);
                    if (lane >= o) end += v;
                }
                const uint64_t past = __ballot(before + end > first);
                if (past) {
                    const int j = __builtin_ctzll(past);
                    k = k0 + j;
                    c0 = 8 * (first - before - __builtin_amdgcn_readlane(end - own, j));
                    break;
                }
                before += __builtin_amdgcn_readlane(end, 63);
            }
        }
        open(k);
        auto load = [&](Chunk<NR> &ch) {
            ch.left = C - c0;
            ch.tr = tr;
            const int CW = (C + 1) >> 1, cg = (c0 >> 1) + g, cgc = cg < CW ? cg : CW - 1;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                int at = cgc * R + rc[t];
                if constexpr (HALF) {   // stored block: C rows, R columns
                    const int kk = c0 + 4 * t + g;
                    at = tr ? (rc[0] >> 1) * C + (kk < C ? kk : C - 1) : at;
                }
                ch.a[t] = __builtin_nontemporal_load(reinterpret_cast<const f64x2 *>(pa + uint32_t(at) * 16u));
            }
            // (tile rows up to the next multiple of 16 exist and are zero)
            const int row = c0 + (HALF && tr ? g : 2 * g), step = HALF && tr ? 4 * NR * 8 : NR * 8;
            const uint32_t ob = uint32_t(row * NR + n * NN) * 8u;
#pragma unroll
            for (int t = 0; t < 2; ++t) ch.b[t] = *reinterpret_cast<const B *>(pb + ob + uint32_t(t * step));
            if (k < nb) {   // (wave-uniform; past the last chunk it is loaded again)
                if (c0 + 8 < C) {
                    c0 += 8;
                } else if (++k < nb) {
                    c0 = 0;
                    open(k);
                }
            }
        };
        Chunk<NR> ring[D];
#pragma unroll
        for (int s = 0; s < D; ++s) load(ring[s]);
        auto products = [&](const Chunk<NR> &ch) {
            f64x2 a[2] = {ch.a[0], ch.a[1]};
            auto step = [&](int u, int t, double v) {
#pragma unroll
                for (int j = 0; j < NN; ++j)
                    acc[t][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(v, Rhs<NR>::get(ch.b[u], j), acc[t][j], 0, 0, 0);
            };
            if (HALF && ch.tr) {   // wave-uniform
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    if (4 * u + g >= ch.left) a[u] = f64x2{0.0, 0.0};   // columns past the block's width
                    step(u, 0, a[u].x);
                    step(u, 1, a[u].y);
                }
                return;
            }
            if (ch.left < 8 && 2 * g >= ch.left) {   // a block's last chunk: column pairs past its width
                a[0] = f64x2{0.0, 0.0};
                a[1] = f64x2{0.0, 0.0};
            }
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    if (t == 0 || two) step(u, t, u ? a[t].y : a[t].x);
        };
        int i = 0;
        for (; i + D <= nch; i += D) {
#pragma unroll
            for (int s = 0; s < D; ++s) {
                products(ring[s]);
                load(ring[s]);
            }
        }
#pragma unroll
        for (int s = 0; s < D - 1; ++s)
            if (i + s < nch) products(ring[s]);
    }

    if constexpr (SPLIT > 1) {
        __shared__ f64x4 part[SPLIT - 1][2 * NN][64];
        if (wv > 0) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int j = 0; j < NN; ++j) part[wv - 1][t * NN + j][lane] = acc[t][j];
        }
        __syncthreads();
        if (wv > 0) return;
#pragma unroll
        for (int w = 0; w < SPLIT - 1; ++w)
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int j = 0; j < NN; ++j) acc[t][j] += part[w][t * NN + j][lane];
    }

    // Lane (g, n) holds rows 32 mt + 16 t + g + 4 e (HALF: 32 mt + 2 (g + 4 e) + t)
    // of right-hand sides NN n + j.
    const int Rp = round16(R);
    auto out_row = [&](int t, int e) { return 32 * mt + (HALF ? 2 * (g + 4 * e) + t : 16 * t + g + 4 * e); };
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        if (!HALF && t && !two) break;   // (HALF: its padding rows are odd ones too)
        B init[4] = {};
        if (LEAF || rd.init >= 0) {   // requested for all rows before any store
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int r = out_row(t, e);
                init[e] = *reinterpret_cast<const B *>(L.init + rd.init + int64_t(r) * NR + n * NN);
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int r = out_row(t, e);
            if (r >= Rp) continue;
            B v;
            if constexpr (NR == 32) v = init[e] + f64x2{acc[t][0][e], acc[t][NN - 1][e]};
            else v = init[e] + acc[t][0][e];
            if constexpr (LEAF) {
                if (r >= R) continue;
#pragma unroll
                for (int j = 0; j < NN; ++j)
                    if (n * NN + j < L.ncols) L.Y[int64_t(n * NN + j) * L.ldy + rd.out + r] = Rhs<NR>::get(v, j);
            } else {
                if (r >= R) v = B{};   // the padding rows stay zero
                *reinterpret_cast<B *>(((rd.sel & ROW_OUT_P) ? L.out_pts : L.out_tree) + rd.out + int64_t(r) * NR + n * NN) = v;
            }
        }
    }
}

// One wavefront per work item, four per workgroup, in the dispatch order laid
// out by the host (h2_device.h), or one workgroup per item (SPLIT); one
// kernel name per phase.
#define H2_MM64_KERNEL(NAME, LEAF, HALF)                                                                             \
    template <int NR, int D, int SPLIT>                                                                        \
    __global__ __launch_bounds__(256) void NAME(Mm64Launch L, const RowDesc *__restrict__ rows,                 \
                                                const BlkDesc *__restrict__ blks) {                            \
        const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;              \
        const int64_t i = SPLIT > 1 ? int64_t(blockIdx.x) : int64_t(blockIdx.x) * 4 + wv;                      \
        const int32_t it = __builtin_amdgcn_readfirstlane(L.items[i]);                                         \
        if (it >= 0) mm64_item<NR, LEAF, D, SPLIT, HALF>(L, rows, blks, it, wv, lane);                               \
    }
H2_MM64_KERNEL(mm64_upsweep_kernel, false, false)
H2_MM64_KERNEL(mm64_stream_kernel, false, false)
H2_MM64_KERNEL(mm64_stream_half_kernel, false, true)
H2_MM64_KERNEL(mm64_downsweep_kernel, false, false)
H2_MM64_KERNEL(mm64_leafexpand_kernel, true, false)
#undef H2_MM64_KERNEL

// Right-hand sides j0 .. of the caller's column-major X into point tiles, a
// leaf (at most 64 rows) per workgroup through LDS: columns are read in runs
// of the leaf's rows, tile rows are written whole; missing rows and
// right-hand sides are zero.
template <int NR>
__global__ __launch_bounds__(256) void pack64_kernel(const double *__restrict__ X, int64_t ldx, int ncols,
                                                     const int64_t *__restrict__ leaf_begin,
                                                     const int64_t *__restrict__ leaf_end, int64_t slot,
                                                     double *__restrict__ tiles) {
    __shared__ double t[64][NR + 1];
    const int64_t leaf = blockIdx.x, b = leaf_begin[leaf];
    const int m = int(leaf_end[leaf] - b), mp = round16(m);
    const int r = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NR / 4; ++k) {
        const int j = w + 4 * k;
        t[r][j] = r < m && j < ncols ? X[(b + r) + int64_t(j) * ldx] : 0.0;
    }
    __syncthreads();
    double *o = tiles + leaf * slot;
    for (int i = threadIdx.x; i < mp * NR; i += 256) o[i] = t[i / NR][i % NR];
}

// Chunks in flight per wavefront: 4 (124 registers, 4 wavefronts per SIMD) and
// 6 or 8 (3 and 2 wavefronts) measured the same; 4 leaves the sweeps' short
// rows less to drain.
constexpr int kDepth = 4;

// Launches of at most this many items (wavefronts; a list's padding counts) run
// four wavefronts per item: too few to fill the chip, each a chain of up to
// some hundred chunks.  Above the line the extra barrier and sums cost more.
// 32 right-hand sides, whole products, one / four wavefronts per item of the
// streaming launch: 3-D, rank 64, 15,000 points (4,096 items) 567 / 459 us, 30,000
// (6,528) 1250 / 1042; 2-D, rank 49, 15,000 (2,464) 260 / 204, 30,000 (4,512)
// 380 / 397 (8 right-hand sides 311 / 301); rank 25, 60,000 (8,000) 408 / 446;
// stored by halves the same within 4 %.  Sweep launches have at most a few
// blocks per item; four wavefronts up to 8,192 / 1,024 / 512 items: 2-D, 2^18
// points 2.90 / 2.78 / 2.76 ms, 100,000 of rank 36 1342 / 1141 / 1129 us, 60,000 of
// rank 49 710 / 678 / 668; up to 256 / none: 8,000 points of rank 64 125 / 140 us.
constexpr int64_t kSplitStream = 7168, kSplitSweep = 512;

template <int NR, int SPLIT>
void launch_phase64(const Mm64Launch &L, int phase, hipStream_t st) {
    constexpr int D = kDepth;
    const dim3 grid(unsigned(SPLIT > 1 ? L.nitems : L.nitems / 4)), block(256);
    switch (phase) {
    case PHASE_UP: hipLaunchKernelGGL((mm64_upsweep_kernel<NR, D, SPLIT>), grid, block, 0, st, L, L.rows, L.blks); break;
    case PHASE_STREAM:
        if (L.half) hipLaunchKernelGGL((mm64_stream_half_kernel<NR, D, SPLIT>), grid, block, 0, st, L, L.rows, L.blks);
        else hipLaunchKernelGGL((mm64_stream_kernel<NR, D, SPLIT>), grid, block, 0, st, L, L.rows, L.blks);
        break;
    case PHASE_DOWN: hipLaunchKernelGGL((mm64_downsweep_kernel<NR, D, SPLIT>), grid, block, 0, st, L, L.rows, L.blks); break;
    default: hipLaunchKernelGGL((mm64_leafexpand_kernel<NR, D, SPLIT>), grid, block, 0, st, L, L.rows, L.blks); break;
    }
}

}  // namespace

hipError_t launch_mm64(const Mm64Launch &L, int phase, hipStream_t st) {
    if (L.nitems <= 0) return hipSuccess;
    if (L.nitems % 4 != 0 || L.ncols < 1 || L.ncols > MM_TILE) return hipErrorInvalidValue;
    const bool split = L.nitems <= (phase == PHASE_STREAM ? kSplitStream : kSplitSweep);
    if (L.ncols > 16) split ? launch_phase64<32, 4>(L, phase, st) : launch_phase64<32, 1>(L, phase, st);
    else split ? launch_phase64<16, 4>(L, phase, st) : launch_phase64<16, 1>(L, phase, st);
    return hipGetLastError();
}

hipError_t launch_pack64(const double *X, int64_t ldx, int ncols, const int64_t *leaf_begin, const int64_t *leaf_end,
                         int64_t nleaves, int64_t slot, double *tiles, hipStream_t st) {
    if (nleaves <= 0) return hipSuccess;
    if (ncols > 16)
        hipLaunchKernelGGL(pack64_kernel<32>, dim3(unsigned(nleaves)), dim3(256), 0, st, X, ldx, ncols, leaf_begin,
                           leaf_end, slot, tiles);
    else
        hipLaunchKernelGGL(pack64_kernel<16>, dim3(unsigned(nleaves)), dim3(256), 0, st, X, ldx, ncols, leaf_begin,
                           leaf_end, slot, tiles);
    return hipGetLastError();
}

}  // namespace h2
