// Internals shared by the host sources of libh2mv: the handle structures
// behind h2_handle and h2_batch, the device arena, the work lists of a
// product, and the steps each source file provides to the others.
#pragma once

#include "h2mv.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <memory>
#include <new>
#include <mutex>
#include <string>
#include <vector>

#include "h2_device.h"
#include "h2_structure.h"

namespace h2i {

using h2::BlkDesc;
using h2::RowDesc;
using h2::Structure;

// Message of the last failed call on this thread (h2_last_error).
extern thread_local std::string g_last_error;

struct Failure {
    h2_status code;
    std::string what;
};

[[noreturn]] inline void fail(h2_status code, const std::string &what) { throw Failure{code, what}; }

inline void check_hip(hipError_t e, const char *where) {
    if (e != hipSuccess) fail(H2_ERR_DEVICE, std::string(where) + ": " + hipGetErrorString(e));
}

// Device memory of arenas that are gone, for the next ones: a hipFree of a
// large block takes ~0.3 ms, and up to 10 ms where a program frees often; one
// that builds, compresses or transposes in a loop asks for the same sizes
// again (a matrix of 40,000 points transposed after others had come and gone:
// 4.6 -> 0.8 ms).  Holds at most kLimit bytes in blocks of at least kLeast;
// one that finds no room drives out those nothing asked for while kStale others
// came.  None is held while less than 1 / kShare of the device's memory is
// free, nor once the process has no matrix or batch left, nor after
// h2_release_kept.  (Built and compressed in a loop, kLimit 512 MiB / 1 GiB: 3-D,
// 14,000 points 8.6 / 8.0 ms; 2-D, 38,000 points 18.1 / 16.6, 65,536 29.1 / 29.1;
// with 256 MiB the last took 30.1 where 512 MiB took 28.2.)
// A block serves requests of exactly its size, so that what an owner counts is
// what it holds.  Blocks come here only after a wait for
// their device, so any stream may use them next.
struct DevicePool {
    static constexpr int64_t kLimit = int64_t(1) << 30, kLeast = 64 << 10, kShare = 16;
    static constexpr int64_t kStale = 256, kLook = 64;
    struct Block {
        int device;
        int64_t bytes;
        void *p;
        int64_t since = 0;   // gives when it came here
    };
    std::mutex m;
    std::vector<Block> blocks;   // oldest first
    int64_t held = 0, gives = 0, looked = 0, unlooked = 0;
    int live = 0;   // matrices and batches

    static DevicePool &get() {
        static DevicePool *pool = new DevicePool;   // never destroyed: the HIP runtime may be gone first
        return *pool;
    }
    // A block of nbytes, or null.
    void *take(int device, int64_t nbytes) {
        std::lock_guard<std::mutex> g(m);
        for (size_t i = blocks.size(); i-- > 0;)
            if (blocks[i].device == device && blocks[i].bytes == nbytes) {
                void *p = blocks[i].p;
                held -= nbytes;
                blocks.erase(blocks.begin() + long(i));
                return p;
            }
        return nullptr;
    }
    // False: not kept, the caller frees it.
    bool give(const Block &b) {
        std::vector<Block> old;   // what makes room for it
        {
            std::lock_guard<std::mutex> g(m);
            ++gives;
            if (live == 0 || b.bytes < kLeast) return false;
            try {
                size_t n = 0;
                int64_t sum = held + b.bytes;
                for (; sum > kLimit && n < blocks.size() && gives - blocks[n].since > kStale; ++n) sum -= blocks[n].bytes;
                if (sum > kLimit) return false;
                old.assign(blocks.begin(), blocks.begin() + long(n));
                blocks.push_back(b);
            } catch (const std::bad_alloc &) {
                return false;
            }
            blocks.back().since = gives;
            blocks.erase(blocks.begin(), blocks.begin() + long(old.size()));
            held += b.bytes;
            for (const Block &o : old) held -= o.bytes;
        }
        for (const Block &o : old) (void)hipFree(o.p);
        return true;
    }
    // Whether the device's free memory is to be looked up (~20 us) before up to
    // `more` bytes come: where they make more than at the last look, and at
    // every kLook-th asking (a matrix of 40,000 points transposed in a loop, a
    // look with every release / this: 833 / 815 us).
    bool look(int64_t more) {
        std::lock_guard<std::mutex> g(m);
        const int64_t then = std::min(held + more, kLimit);
        if (then <= looked && ++unlooked < kLook) return false;
        looked = then;
        unlooked = 0;
        return true;
    }
    int64_t held_on(int device) {
        std::lock_guard<std::mutex> g(m);
        int64_t sum = 0;
        for (const Block &b : blocks) sum += b.device == device ? b.bytes : 0;
        return sum;
    }
    void clear() {
        std::vector<Block> old;
        {
            std::lock_guard<std::mutex> g(m);
            old.swap(blocks);
            held = looked = 0;
        }
        for (const Block &b : old) (void)hipFree(b.p);
    }
    void enter() {
        std::lock_guard<std::mutex> g(m);
        ++live;
    }
    void leave() {
        bool last;
        {
            std::lock_guard<std::mutex> g(m);
            last = --live == 0;
        }
        if (last) clear();
    }
};

// Counts its owner among the pool's users; to be declared before (destroyed
// after) the owner's arenas.
struct PoolUser {
    PoolUser() { DevicePool::get().enter(); }
    ~PoolUser() { DevicePool::get().leave(); }
    PoolUser(const PoolUser &) = delete;
    PoolUser &operator=(const PoolUser &) = delete;
};

// Device allocations of one owner; a test-only cap (environment variable
// H2MV_DEVICE_BYTE_CAP, bytes) turns any allocation past it into H2_ERR_OOM.
struct DeviceArena {
    std::vector<DevicePool::Block> ptrs;
    int64_t bytes = 0;
    int64_t cap = -1;
    // Small set-up arrays are placed in slabs and copied a slab at a time: an
    // array of its own costs an allocation, a copy and a wait, ~40 us, and a
    // matrix has about a hundred of them (one of 40,000 points transposed:
    // 2.8 -> 1.2 ms).
    static constexpr int64_t kSlab = 1 << 20, kSlabItem = 256 << 10;
    char *slab = nullptr;
    int64_t slab_used = 0, slab_sent = 0;   // bytes placed, and of these copied
    std::vector<char> slab_host;

    DeviceArena() {
        if (const char *c = std::getenv("H2MV_DEVICE_BYTE_CAP")) cap = std::atoll(c);
    }
    DeviceArena(const DeviceArena &) = delete;
    DeviceArena &operator=(const DeviceArena &) = delete;
    ~DeviceArena() {
        release();
    }
    void swap(DeviceArena &o) {
        std::swap(ptrs, o.ptrs);
        std::swap(bytes, o.bytes);
        std::swap(cap, o.cap);
        std::swap(slab, o.slab);
        std::swap(slab_used, o.slab_used);
        std::swap(slab_sent, o.slab_sent);
        std::swap(slab_host, o.slab_host);
    }
    void *alloc(int64_t nbytes) {
        if (nbytes <= 0) nbytes = 16;
        nbytes = (nbytes + 255) / 256 * 256;
        if (cap >= 0 && bytes + nbytes > cap) fail(H2_ERR_OOM, "device byte cap exceeded");
        void *p = device_malloc(nbytes);
        bytes += nbytes;
        return p;
    }
    void *device_malloc(int64_t nbytes) {   // not counted
        int device = 0;
        check_hip(hipGetDevice(&device), "hipGetDevice");
        ptrs.reserve(ptrs.size() + 1);
        void *p = nbytes >= DevicePool::kLeast ? DevicePool::get().take(device, nbytes) : nullptr;
        if (p) {
            ptrs.push_back({device, nbytes, p});
            return p;
        }
        hipError_t e = hipMalloc(&p, size_t(nbytes));
        if (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation) {   // again without what the pool holds
            (void)hipGetLastError();
            DevicePool::get().clear();
            e = hipMalloc(&p, size_t(nbytes));
        }
        if (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation) {
            (void)hipGetLastError();
            fail(H2_ERR_OOM, "hipMalloc of " + std::to_string(nbytes) + " bytes failed");
        }
        check_hip(e, "hipMalloc");
        ptrs.push_back({device, nbytes, p});
        return p;
    }
    // Returns the memory: the smallest block to the device, and after that,
    // as hipFree waits for all work on its device, the others to the pool.
    void release() {
        if (ptrs.empty()) return;
        std::swap(*std::min_element(ptrs.begin(), ptrs.end(),
                                    [](const DevicePool::Block &x, const DevicePool::Block &y) { return x.bytes < y.bytes; }),
                  ptrs.front());
        int64_t more = 0;
        for (size_t i = 1; i < ptrs.size(); ++i) more += ptrs[i].bytes;
        bool keep = hipFree(ptrs.front().p) == hipSuccess;
        size_t free_bytes = 0, total = 0;
        if (keep && DevicePool::get().look(more) && hipMemGetInfo(&free_bytes, &total) == hipSuccess &&
            free_bytes < total / DevicePool::kShare) {
            keep = false;
            DevicePool::get().clear();
        }
        for (size_t i = 1; i < ptrs.size(); ++i) {
            const DevicePool::Block &b = ptrs[i];
            if (!keep || b.device != ptrs.front().device || !DevicePool::get().give(b)) (void)hipFree(b.p);
        }
        ptrs.clear();
    }
    // Copies v to new device memory; returns once v may be released (set-up
    // only, never inside a product).
    template <typename T>
    T *upload(const std::vector<T> &v, hipStream_t st) {
        T *d = static_cast<T *>(alloc(int64_t(v.size() * sizeof(T))));
        if (!v.empty()) {
            check_hip(hipMemcpyAsync(d, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice, st),
                      "hipMemcpyAsync");
            check_hip(hipStreamSynchronize(st), "upload");
        }
        return d;
    }
    // The same, but a small v arrives on the device with the next flush().
    // Counted as an allocation of its own.
    template <typename T>
    T *stage(const std::vector<T> &v, hipStream_t st) {
        const int64_t nbytes = std::max<int64_t>(16, int64_t(v.size() * sizeof(T))), place = (nbytes + 255) / 256 * 256;
        if (place > kSlabItem) return upload(v, st);
        if (cap >= 0 && bytes + place > cap) fail(H2_ERR_OOM, "device byte cap exceeded");
        if (!slab || slab_used + place > kSlab) {
            flush(st);
            slab = static_cast<char *>(device_malloc(kSlab));
            slab_used = slab_sent = 0;
            slab_host.resize(size_t(kSlab));
        }
        T *d = reinterpret_cast<T *>(slab + slab_used);
        if (!v.empty()) std::memcpy(slab_host.data() + slab_used, v.data(), v.size() * sizeof(T));
        slab_used += place;
        bytes += place;
        return d;
    }
    // Everything staged is on the device; no more is needed of the host's copy.
    void flush(hipStream_t st) {
        if (slab_used > slab_sent) {
            check_hip(hipMemcpyAsync(slab + slab_sent, slab_host.data() + slab_sent, size_t(slab_used - slab_sent),
                                     hipMemcpyHostToDevice, st),
                      "hipMemcpyAsync");
            check_hip(hipStreamSynchronize(st), "upload");
            slab_sent = slab_used;
        }
    }
    // Nothing more will be staged.
    void close_slab(hipStream_t st) {
        flush(st);
        slab = nullptr;
        std::vector<char>().swap(slab_host);
    }
};

enum Phase { PH_UP = 0, PH_STREAM = 1, PH_DOWN = 2, PH_LEAF = 3, PH_COUNT = 4 };

struct WorkList {
    Phase phase;
    int kind;   // element kind of its data
    const void *data;
    const h2::RowDesc *rows;
    int64_t nrows;
    const h2::BlkDesc *blks;
    const int32_t *items = nullptr;   // tile lists: wavefront items in dispatch order
    int64_t nitems = 0;
    const int32_t *pitems = nullptr;  // tile lists: pair items (two per workgroup) in dispatch order
    int64_t npitems = 0;
    // cut stream list (single vector): the rows are chunks writing FP64 partial
    // sums, which the downsweep adds up (tree_sums, near_sums)
    void *partials = nullptr;   // FP64 (FP32 for the half-storage list of a reduced-storage matrix)
    int64_t partials_bytes = 0;
    // stream list of a matrix stored by halves: the wavefronts' row groups,
    // every block's slot code and the groups' merged partial slots (see
    // h2::HalfGroup); red then adds the slots to the row sums
    const h2::ReduceDesc *red = nullptr;
    int64_t nred = 0;
    const int32_t *slot = nullptr;
    const h2::HalfGroup *groups = nullptr;
    int64_t ngroups = 0;
    const int32_t *gslot = nullptr;
    // single-vector stream list, full storage: the same rows (chunks, for a
    // cut list) with the coupling rows first and the near-field rows after,
    // each part in the list's own order -- the near field can then run as a
    // launch of its own (H2_SCHEDULE_STREAMED)
    const h2::RowDesc *srows = nullptr;
    int64_t nsrows_coupling = 0;
    std::vector<int64_t> near_cum;   // blocks of the near-field rows of srows, cumulative (size rows + 1)
};

// One launch of a tree sweep of the single-vector product (h2::SweepLaunch).
struct SweepStep {
    int level, depth, split;
    bool leaf;
};

// A single-vector stream list with fewer than two thirds as many block rows as
// the pieces it can be cut into is cut: one wavefront per row would leave the
// machine idle, at the end of the launch if not throughout (5,120 FP64
// wavefronts run at once).  Pieces hold about 8 blocks, 4,096 to 16,384 of them.
// Measured, single-vector product: 50,000 3-D points of rank 27, 6,143 rows
// of 90 blocks, uncut / 16,384 / 65,536 pieces 675 / 614 / 628 us (FP64), 298 /
// 240 / 262 (BF16); 20,011 points 4,096 / 16,384 pieces 272 / 235 us; 16,384
// 2-D points of rank 64 (16,800 blocks) 4,096 / 8,192 / 16,384 pieces 152 / 155
// / 162 us; 100,000 2-D points of rank 25 (12,287 rows) uncut / 16,384 pieces
// 360 / 372 us.
constexpr int64_t kSplitWaves = 4096, kMaxSplitWaves = 16384;

// ---------------------------------------------------------------- batches
// Many H^2 matrices of uneven size and rank per launch: the members' tile
// lists are concatenated per "level slot" -- upsweep lists aligned by their
// distance from the leaves, downsweep lists aligned at their end (the leaf
// level), one streaming slot and one leaf slot -- so every slot is one
// grid-strided launch over all members.  Tiles of all members live in one
// pool; block operands are absolute addresses into the members' storage.
struct BatchSlot {
    Phase phase;
    int kind;
    h2::RowDesc *rows;
    int64_t nrows;
    h2::BlkDesc *blks;
    int32_t *items;
    int64_t nitems;
    int32_t *pitems;
    int64_t npitems;
};

}  // namespace h2i

// The matrix behind an h2_handle: its structure, device storage and work lists.
struct h2_matrix_ {
    h2i::PoolUser pool_user;
    h2::Structure st;
    int storage = H2_FP64;
    bool structure_only = false;
    int basis_kind = h2::ELEM_F64, block_kind = h2::ELEM_F64;
    bool vec_f64 = true;
    h2i::DeviceArena mem;
    void *basis = nullptr, *blocks = nullptr;
    float *scales = nullptr;
    void *xh = nullptr, *yh = nullptr, *ynear = nullptr;
    std::vector<h2i::WorkList> lists;      // single right-hand side: the streaming list (vector offsets)
    std::vector<h2i::SweepStep> up_steps, down_steps;   // single right-hand side: the sweeps, in launch order
    int64_t *d_off_U = nullptr, *d_off_VT = nullptr, *d_off_E = nullptr, *d_off_FT = nullptr;   // off_* on the device
    h2::SumRange *d_tree_sums = nullptr, *d_near_sums = nullptr;   // cut streaming list: chunks per node / leaf
    std::vector<h2i::WorkList> mm_lists;   // tiles of MM_TILE right-hand sides (tile offsets)
    std::vector<std::vector<h2::RowDesc>> mm_host_rows;   // host copies of mm_lists (of matrices that batches take)
    std::vector<std::vector<h2::BlkDesc>> mm_host_blks;
    int64_t nscales = 0;
    int64_t tile_slot = 0;            // elements per leaf in point tiles
    int64_t *d_leaf_begin = nullptr, *d_leaf_end = nullptr;
    // tile workspace (lazy; FP32, or FP64 for FP64 matrices)
    void *t_xh = nullptr, *t_yh = nullptr, *t_x = nullptr, *t_ynear = nullptr;
    // block loop chosen at the first pass of each tile width (32, or 16 for
    // passes of at most 16 right-hand sides)
    h2::MmConfig mm_cfg[2] = {{1, 0, 0}, {1, 0, 0}};
    bool mm_tuned[2] = {false, false};
    double mm_tuned_ms[2] = {0.0, 0.0};   // timed choice's pass time (0: from the cache)
    int64_t bytes_coupling = 0, bytes_dense = 0, bytes_leaf = 0, bytes_transfer = 0;
    // layout: element offsets of U_j, V_j^T (per leaf), E_c, F_c^T (per node,
    // -1 where not stored) in basis, and of every block in blocks (coupling
    // blocks level by level in BSR order, then dense blocks)
    std::vector<int64_t> off_U, off_VT, off_E, off_FT, off_blk;
    int64_t basis_elems = 0, block_elems = 0;   // lengths of the two regions
    bool symmetric = true;                      // V = U and F = E
    // stored by halves (H2_HALF_STORAGE): only blocks with column >= row; for
    // every block of the full BSR lists (coupling levels, then dense) its
    // index in off_blk, or -(index + 1) of the stored block it mirrors
    bool half = false;
    std::vector<int64_t> blk_store;
    int batch_refs = 0;                         // batches holding addresses into this matrix
    // schedule of the single-vector product (h2_set_schedule): the near field
    // on the handle's second stream, its launch's LDS request (caps its
    // workgroups per compute unit; 0: no cap) and the share of its rows
    // launched at the start of the product (the rest follows the coupling launch)
    int schedule = H2_SCHEDULE_MERGED;
    int near_wg_per_cu = 0;
    int near_lds_bytes = 0;
    double near_early = 1.0;
    hipStream_t aux = nullptr;
    hipEvent_t ev_fork = nullptr, ev_mid = nullptr, ev_join = nullptr;
    // profiling: PH_COUNT + 1 events per recorded call
    bool prof = false;
    std::vector<hipEvent_t> pending, spare;
    double prof_ms[8] = {0};
    int64_t prof_calls = 0;

    ~h2_matrix_() {
        for (hipEvent_t e : pending) (void)hipEventDestroy(e);
        for (hipEvent_t e : spare) (void)hipEventDestroy(e);
        for (hipEvent_t e : {ev_fork, ev_mid, ev_join})
            if (e) (void)hipEventDestroy(e);
        if (aux) (void)hipStreamDestroy(aux);
    }
};

// A batch of matrices behind an h2_batch: one launch per level slot.
struct h2_batch_ {
    h2i::PoolUser pool_user;
    std::vector<h2_matrix_ *> mats;
    int nrhs = 0;
    h2i::DeviceArena mem;
    float *pool = nullptr;
    float *scales = nullptr;
    std::vector<h2i::BatchSlot> slots;
    h2::PackEntry *pack = nullptr;
    int64_t npack = 0;
    double **d_Xtab = nullptr, **d_Ytab = nullptr;
    int64_t *d_ldx = nullptr, *d_ldy = nullptr;
    hipStream_t own = nullptr;
    hipEvent_t ev_in = nullptr, ev_out = nullptr;
    // pinned host copy of the per-call tables (X, Y pointers, ldx, ldy), and
    // the event after their upload: the next call waits for it before rewriting
    int64_t *h_tables = nullptr;
    hipEvent_t ev_tables = nullptr;
    bool tables_pending = false;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    h2::MmConfig cfg{1, 0, 0};
    bool tuned = false;
    double tuned_ms = 0.0;
    std::string signature;
    int64_t cu_count = 256;
    bool counted = false;   // the members' batch_refs include this batch

    ~h2_batch_() {
        if (counted)
            for (h2_matrix_ *m : mats) --m->batch_refs;
        if (ev_tables) {
            if (tables_pending) (void)hipEventSynchronize(ev_tables);
            (void)hipEventDestroy(ev_tables);
        }
        if (h_tables) (void)hipHostFree(h_tables);
        if (exec) (void)hipGraphExecDestroy(exec);
        if (graph) (void)hipGraphDestroy(graph);
        if (ev_in) (void)hipEventDestroy(ev_in);
        if (ev_out) (void)hipEventDestroy(ev_out);
        if (own) (void)hipStreamDestroy(own);
    }
};

namespace h2i {

// h2_build.cpp
std::vector<int32_t> wave_items(const std::vector<h2::RowDesc> &rows, const std::vector<h2::BlkDesc> &blks);
std::vector<int32_t> pair_items(const std::vector<h2::RowDesc> &rows, const std::vector<h2::BlkDesc> &blks);
void convert_block(const double *src, int R, int C, bool transpose, int kind, void *dst, float *scale);
std::vector<h2::FillDesc> make_layout(h2_matrix_ &A, int64_t &ncoupling);
void build_device(h2_matrix_ &A, const h2_arrays *src, hipStream_t stream);
void build_lists(h2_matrix_ &A, const std::vector<h2::FillDesc> &fill, int64_t ncoupling, hipStream_t stream);
void validate_params(const double *points, int64_t n, const h2_params *prm);
void structure_from_arrays(const h2_arrays *a, h2::Structure &s);
void export_arrays(h2_matrix_ &A, const h2_arrays_out *o, hipStream_t st);

// h2_run.cpp
// Intermediate vectors of one single-vector product: the trees x^ and y^, the
// near field, and the partial sums of a split or half-storage stream list.
struct Workspace {
    void *xh, *yh, *ynear, *partials;
};
// Bytes of each part (rounded up to 256), in the order above; the sum is the
// whole.
void workspace_bytes(const h2_matrix_ &A, int64_t part[4]);
// Enqueues the whole single-vector product on st, in the handle's own
// workspace, or in ws (then without profiling events).
void run_product(h2_matrix_ &A, const double *x, double *y, hipStream_t st, const Workspace *ws = nullptr);
void run_tile_pass(h2_matrix_ &A, const double *X, int64_t ldx, double *Y, int64_t ldy, int nrhs, int j0,
                   const h2::MmConfig &cfg, hipStream_t st);
void run_tiles(h2_matrix_ &A, const double *X, int64_t ldx, double *Y, int64_t ldy, int nrhs, hipStream_t st);

// h2_batch.cpp
// Chooses the block loop (pipelined or not) for this matrix and the tile
// width of pass j0 by timing both on that pass, unless cached.
void tune_tiles(h2_matrix_ &A, const double *X, int64_t ldx, double *Y, int64_t ldy, int nrhs, int j0,
                hipStream_t st);

// h2_transform.cpp
void orthogonalize(h2_matrix_ &A, hipStream_t st);
h2_matrix_ *transpose_matrix(h2_matrix_ &A, hipStream_t st);
void compress(h2_matrix_ &A, double eps, hipStream_t st, int *ranks_out);

}  // namespace h2i
