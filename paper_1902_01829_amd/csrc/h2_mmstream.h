// The streaming launch over tiles of 16 or 32 right-hand sides, FP32 and BF16
// blocks, for all passes of at most 16 and the lists stream_by_tiles names.
// Included in h2_mm.hip's namespace.
//
// One workgroup of four wavefronts takes a unit of the pair list: a row of
// more than 32 rows, a quarter of its blocks per wavefront, or two shorter
// rows, half of a row's blocks per wavefront.  A wavefront multiplies whole
// blocks (up to 64 rows): the input tile is read, and for BF16 blocks split,
// once per block and not once per 32-row half, and the long rows of 3-D
// matrices are spread over four wavefronts.  The FP64 totals are added
// through LDS in a fixed order.
//
// Within a wavefront the row's blocks are one sequence of column chunks (one
// 16-byte item per lane and row tile), in a ring of S slots with loads in flight across block
// boundaries.  What a step costs beyond its loads and MFMAs bounds this
// kernel for blocks of rank 16 to 27, so it is kept small: block addresses
// stay in scalar registers (descriptors of 64 blocks are loaded at a time, one
// per lane, and read with lane reads), a lane's offset within a chunk is one
// multiplication, and what consuming a chunk needs to know of its block (its
// last chunk, its scale) is kept with the ring slot.  A block's products and
// their order are those of the other loops.
// 8 right-hand sides, whole products, the 32-row loops with their best launch
// shape against this one (tiles as then): 2-D 400,000 points FP32 2.13 -> 1.99
// ms, 4,096 points 63 -> 50 us, 3-D 50,021 points of rank 27 BF16 443 -> 393
// us, batch of 24 FP32 1000 -> 835 us.  Insensitive to S (2 to 10) and to two
// to four wavefronts per SIMD.  No unit is saturated (8 right-hand sides, 3-D 50,021
// points BF16 / batch of 24 FP32: L1 address units 55 / 66 % busy, matrix cores 8 /
// 28 %, vector ALU 45 / 14 %, 18.3 / 18.2 lines per load where 16 are its
// least): what is left is each wavefront's chain of dependent loads per block.

constexpr int kStreamWaves = 4;

// Rows of a wavefront: NH tiles of TW (16 or 32, the MFMA's rows and columns).
template <int KIND, int NH> struct StreamSlot {
    typename std::conditional<KIND == ELEM_F32, f32x4, u32x4>::type a[NH];
    f32x4 b[KIND == ELEM_F32 ? 1 : 2];
};
template <int TW> struct Acc;
template <> struct Acc<16> {
    typedef f32x4 type;
    static __device__ __forceinline__ type mul(float a, float b, type c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    static __device__ __forceinline__ type mul(bf16x8 a, bf16x8 b, type c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
};
template <> struct Acc<32> {
    typedef f32x16 type;
    static __device__ __forceinline__ type mul(float a, float b, type c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
    static __device__ __forceinline__ type mul(bf16x8 a, bf16x8 b, type c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
};

template <int KIND, bool BATCH, int TW, int NH, int S>
__device__ __forceinline__ void stream_blocks(const MmArgs &g, const RowDesc &rd, int first, int cnt, int lane,
                                              double (&tot)[NH][TW * TW / 64]) {
    constexpr int W = KIND == ELEM_F32 ? 4 : 8;      // columns of a 16-byte item
    constexpr int NG = 64 / TW, CH = W * NG;         // item columns and columns of a chunk
    constexpr int E = TW * TW / 64;                  // accumulator elements of a lane
    const int n = lane & (TW - 1), kq = lane / TW, R = rd.R, nh = (R + TW - 1) / TW;
    const uint32_t R16 = uint32_t(R) * 16;
    uint32_t ro[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) ro[h] = uint32_t(TW * h + n < R ? TW * h + n : R - 1) * 16;
    const char *xbase = reinterpret_cast<const char *>((rd.sel & ROW_IN_X) ? g.in_pts : g.in_tree);
    const BlkDesc *blks = g.blks + first;

    // descriptors of blocks 64 j .. 64 j + 63 (of the last block past the end), one per lane
    BlkDesc my;
    float mysc = 1.0f;
    auto load_descs = [&](int k0) {
        my = blks[k0 + lane < cnt ? k0 + lane : cnt - 1];
        if constexpr (KIND == ELEM_BF16) mysc = g.scales[my.sidx];
        asm volatile("" : "+v"(my.C), "+v"(mysc));   // waited for here, not at every later use of a load
    };
    int total = 0;   // chunks
    for (int k0 = cnt > 64 ? 64 : 0;;) {   // (the first 64 last: they stay)
        load_descs(k0);
        const int C = k0 + lane < cnt ? my.C : 0;
#pragma unroll
        for (int t = 0; t < 64; t += CH) total += __popcll(__ballot(C > t));
        if (k0 == 0) break;
        k0 = k0 + 64 < cnt ? k0 + 64 : 0;
    }
    // refill cursor: chunk c of block k
    int k = 0, c = 0, C = 0, np = 0;
    const char *ap = nullptr, *xp = nullptr;
    auto open = [&] {
        const int j = k & 63;
        const int64_t a = readlane64(my.a, j);
        if constexpr (BATCH) ap = reinterpret_cast<const char *>(a);
        else ap = static_cast<const char *>(g.data) + a * (KIND == ELEM_F32 ? 4 : 2);
        xp = xbase + readlane64(my.in, j) * 4;
        C = __builtin_amdgcn_readlane(my.C, j);
        np = (C + CH - 1) / CH;
    };
    open();
    StreamSlot<KIND, NH> ring[S];
    bool last[S];
    float sc[S];
    int rem[S];   // BF16: padded columns of the tile from the chunk's first on
    auto refill = [&](int s) {
        const uint32_t live = k < cnt ? ~0u : 0u;   // past the end: one item of the last block, unused
        const int groups = (C + W - 1) / W - NG * c;   // item columns from this chunk on
        const uint32_t ko = uint32_t(kq < groups ? kq : groups - 1) * R16;
        typedef const __attribute__((address_space(1))) char *gptr;
        typedef typename std::conditional<KIND == ELEM_F32, f32x4, u32x4>::type item;
#pragma unroll
        for (int h = 0; h < NH; ++h)
            ring[s].a[h] = __builtin_nontemporal_load(
                reinterpret_cast<const __attribute__((address_space(1))) item *>((gptr)ap + ((ko + ro[h]) & live)));
        last[s] = c + 1 == np;
        if constexpr (KIND == ELEM_F32) {
            const uint32_t xo = uint32_t(kq * TW + n) * 16;
            ring[s].b[0] = *reinterpret_cast<const __attribute__((address_space(1))) f32x4 *>((gptr)xp + xo);
        } else {
            rem[s] = round16(C) - CH * c;
            const int col = 8 * kq < rem[s] ? 8 * kq : rem[s] - 8;
            const uint32_t xo = uint32_t(col / 4 * TW + n) * 16;
            ring[s].b[0] = *reinterpret_cast<const __attribute__((address_space(1))) f32x4 *>((gptr)xp + xo);
            ring[s].b[1] = *reinterpret_cast<const __attribute__((address_space(1))) f32x4 *>((gptr)xp + xo + TW * 16);
            sc[s] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, mysc), k & 63));
        }
        if (live) {
            if (++c < np) {
                ap += NG * R16;
                xp += CH * TW * 4;
            } else if (++k < cnt) {
                if ((k & 63) == 0) load_descs(k);
                c = 0;
                open();
            } else {
                --c;   // the cursor stays on the last chunk
            }
        }
    };
    typename Acc<TW>::type acc[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int e = 0; e < E; ++e) acc[h][e] = 0.0f;
    auto consume = [&](int s) {
        if constexpr (KIND == ELEM_F32) {
            const f32x4 b = ring[s].b[0];
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                if (h >= nh) break;   // wave-uniform
                const f32x4 a = ring[s].a[h];
                acc[h] = Acc<TW>::mul(a.x, b.x, acc[h]);
                acc[h] = Acc<TW>::mul(a.y, b.y, acc[h]);
                acc[h] = Acc<TW>::mul(a.z, b.z, acc[h]);
                acc[h] = Acc<TW>::mul(a.w, b.w, acc[h]);
            }
        } else {
            bf16x8 hi, mid, lo;
            split3(ring[s].b[0], ring[s].b[1], hi, mid, lo);
            if (8 * kq >= rem[s]) {   // past the tile: zero
                const u32x4 z = {0u, 0u, 0u, 0u};
                hi = mid = lo = __builtin_bit_cast(bf16x8, z);
            }
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                if (h >= nh) break;
                const bf16x8 a = __builtin_bit_cast(bf16x8, ring[s].a[h]);
                acc[h] = Acc<TW>::mul(a, lo, acc[h]);
                acc[h] = Acc<TW>::mul(a, mid, acc[h]);
                acc[h] = Acc<TW>::mul(a, hi, acc[h]);
            }
        }
        if (last[s]) {   // the block's sum goes to the totals
            const double f = KIND == ELEM_F32 ? 1.0 : double(sc[s]);
#pragma unroll
            for (int h = 0; h < NH; ++h)
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    tot[h][e] += f * double(acc[h][e]);
                    acc[h][e] = 0.0f;
                }
        }
    };
#pragma unroll
    for (int s = 0; s < S; ++s) refill(s);
    // whole rounds with refills, then the last round (1 .. S chunks) without
    int i = 0;
    for (; i + S < total; i += S) {
#pragma unroll
        for (int s = 0; s < S; ++s) {
            consume(s);
            refill(s);
        }
    }
#pragma unroll
    for (int s = 0; s < S; ++s)
        if (i + s < total) consume(s);   // wave-uniform
}

template <int KIND, bool BATCH, int TW>
__global__ __launch_bounds__(64 * kStreamWaves) void mm_stream_tiles_kernel(MmArgs g, const RowDesc *__restrict__ rows,
                                                                      const BlkDesc *__restrict__ blks,
                                                                      const int32_t *__restrict__ items,
                                                                      const float *__restrict__ scales) {
    constexpr int E = TW * TW / 64, QT = E / 4;   // elements and groups of four rows of a lane in a tile
    constexpr int N1 = 32 / TW, N2 = 64 / TW;     // tiles of a row of at most 32, of more rows
    constexpr int S1 = KIND == ELEM_F32 ? 6 : 4, S2 = KIND == ELEM_F32 ? 4 : TW == 16 ? 2 : 3;
    __shared__ double part[kStreamWaves][N2 * E][64];   // [wavefront][tile and element][lane]
    g.rows = rows;
    g.blks = blks;
    g.items = items;
    g.scales = scales;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int32_t it0 = items[int64_t(blockIdx.x) * 2], it1 = items[int64_t(blockIdx.x) * 2 + 1];
    if (it0 < 0) return;   // padding of the list (then it1 is padding too)
    const bool wide = it1 >= 0 && (it0 >> 1) == (it1 >> 1);   // one row of more than 32 rows
    const int32_t it = wide || wv < 2 ? it0 : it1;
    RowDesc rd;
    if (it >= 0) {
        rd = rows[it >> 1];
        const int nb = rd.b1 - rd.b0;
        const int of = wide ? 4 : 2, me = wide ? wv : wv & 1;
        const int b0 = nb * me / of, cnt = nb * (me + 1) / of - b0;
        if (wide) {
            double tot[N2][E] = {};
            if (cnt > 0) stream_blocks<KIND, BATCH, TW, N2, S2>(g, rd, rd.b0 + b0, cnt, lane, tot);
#pragma unroll
            for (int e = 0; e < N2 * E; ++e) part[wv][e][lane] = tot[e / E][e % E];
        } else {
            double tot[N1][E] = {};
            if (cnt > 0) stream_blocks<KIND, BATCH, TW, N1, S1>(g, rd, rd.b0 + b0, cnt, lane, tot);
#pragma unroll
            for (int e = 0; e < N1 * E; ++e) part[wv][e][lane] = tot[e / E][e % E];
        }
    }
    __syncthreads();
    if (it < 0) return;
    // groups of four rows of the unit's row by this wavefront
    const int w0 = wide ? 0 : wv & 2, w1 = wide ? 4 : w0 + 2;
    const int n = lane & (TW - 1), kq = lane / TW, R = rd.R, Rp = round16(R);
#pragma unroll
    for (int j = 0; j < TW / 16; ++j) {
        const int id = (wide ? wv : wv & 1) * (TW / 16) + j, h = id / QT, q = id % QT;
        const int i0 = TW * h + 4 * (64 / TW) * q + 4 * kq;
        if (i0 >= Rp) continue;
        double v[4] = {};
        for (int w = w0; w < w1; ++w)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] += part[w][4 * id + e][lane];
        f32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = i0 + e < R ? float(v[e]) : 0.0f;
        float *out = ((rd.sel & ROW_OUT_P) ? g.out_pts : g.out_tree) + rd.out + tile_at<TW>(i0, n);
        *reinterpret_cast<f32x4 *>(out) = o;
    }
}
