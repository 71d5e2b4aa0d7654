// The product: y = A x as a fixed sequence of launches -- the upsweep, one
// streaming launch over the work list built at construction, the downsweep (the per-call marshaling of pointer
// batches of Sec. 3.2 becomes static lists), and Y = A X in tiles of
// right-hand sides on the matrix cores.
#include "h2_internal.h"

namespace h2i {

namespace {

hipEvent_t take_event(h2_matrix_ &A) {
    if (!A.spare.empty()) {
        hipEvent_t e = A.spare.back();
        A.spare.pop_back();
        return e;
    }
    hipEvent_t e;
    check_hip(hipEventCreate(&e), "hipEventCreate");
    return e;
}

// Enqueues the lists in order, with profiling events at phase boundaries
// when enabled; launch(w) enqueues one list.
template <class Launch>
void run_lists(h2_matrix_ &A, const std::vector<WorkList> &lists, hipStream_t st, Launch launch) {
    const bool prof = A.prof;
    hipEvent_t ev[PH_COUNT + 1] = {};
    if (prof)
        for (auto &e : ev) e = take_event(A);
    int next_phase = 0;   // lists are in phase order; each phase's event precedes its lists
    for (const WorkList &w : lists) {
        while (prof && next_phase <= int(w.phase))
            check_hip(hipEventRecord(ev[next_phase++], st), "hipEventRecord");
        launch(w);
    }
    if (prof) {
        while (next_phase <= PH_COUNT) check_hip(hipEventRecord(ev[next_phase++], st), "hipEventRecord");
        A.pending.insert(A.pending.end(), ev, ev + PH_COUNT + 1);
    }
}

// Bytes of the tile workspace of the many-right-hand-side product, those of
// its tree and point parts (two of each).
int64_t tile_bytes(const h2_matrix_ &A, int64_t &tree, int64_t &pts) {
    const int64_t vb = A.vec_f64 ? 8 : 4, kp = (A.st.rank + 15) / 16 * 16;
    auto r256 = [](int64_t b) { return (b + 255) / 256 * 256; };
    tree = r256(A.st.nnodes * kp * h2::MM_TILE * vb);
    pts = r256((int64_t(1) << A.st.q) * A.tile_slot * vb);
    return 2 * (tree + pts);
}

// The workspace, allocated at first use (one allocation: none of it stays
// behind when memory runs out).
void ensure_tiles(h2_matrix_ &A) {
    if (A.t_xh) return;
    int64_t tree = 0, pts = 0;
    tile_bytes(A, tree, pts);
    char *p = static_cast<char *>(A.mem.alloc(2 * tree + 2 * pts));
    A.t_xh = p;
    A.t_yh = p + tree;
    A.t_x = p + 2 * tree;
    A.t_ynear = p + 2 * tree + pts;
}

}  // namespace

void workspace_bytes(const h2_matrix_ &A, int64_t part[4]) {
    auto r256 = [](int64_t b) { return (b + 255) / 256 * 256; };
    const int64_t vb = A.vec_f64 ? 8 : 4;
    part[0] = part[1] = r256(A.st.nnodes * A.st.rank * vb);
    part[2] = r256(A.st.n * vb);
    part[3] = 0;
    for (const WorkList &w : A.lists) part[3] = std::max(part[3], r256(w.partials_bytes));
}

void run_product(h2_matrix_ &A, const double *x, double *y, hipStream_t st, const Workspace *ws) {
    const Workspace own{A.xh, A.yh, A.ynear, A.lists[0].partials};
    const Workspace &W = ws ? *ws : own;
    const WorkList &w = A.lists[0];   // the streaming list
    const bool prof = A.prof && !ws;
    hipEvent_t ev[PH_COUNT + 1] = {};
    if (prof)
        for (auto &e : ev) e = take_event(A);
    auto mark = [&](int phase) {   // the start of a phase, or the end of the last
        if (prof) check_hip(hipEventRecord(ev[phase], st), "hipEventRecord");
    };
    const bool cut = !w.slot && w.partials_bytes > 0;
    auto sweep = [&](const SweepStep &g, bool up) {
        h2::SweepLaunch L{};
        L.basis = A.basis;
        L.off_leaf = up ? A.d_off_VT : A.st.lmin <= A.st.q ? A.d_off_U : nullptr;
        L.off_tr = up ? A.d_off_FT : A.d_off_E;
        L.leaf_begin = A.d_leaf_begin;
        L.leaf_end = A.d_leaf_end;
        L.x = x;
        L.y = y;
        L.tree = up ? W.xh : W.yh;
        L.near = W.ynear;
        L.partials = cut ? static_cast<const double *>(W.partials) : nullptr;
        L.tree_sums = A.d_tree_sums;
        L.near_sums = A.d_near_sums;
        L.stride = A.st.rank;
        L.level = g.level;
        L.depth = g.depth;
        L.split = g.split;
        L.leaf = g.leaf;
        L.root_done = g.level > A.st.lmin;
        for (int p = 0; p <= g.depth; ++p) L.rank[p] = A.st.lrank[size_t(g.level + p)];
        check_hip(h2::launch_sweep(L, up, A.vec_f64, st), "sweep launch");
    };
    auto stream_rows = [&](const h2::RowDesc *rows, int64_t nrows, int lds_bytes, hipStream_t on) {
        if (nrows <= 0) return;
        h2::RowLaunch L;
        L.rows = rows;
        L.nrows = nrows;
        L.blks = w.blks;
        L.data = w.data;
        L.scales = A.scales;
        L.in0 = W.xh;
        L.in1 = x;
        L.out0 = cut ? W.partials : W.yh;
        L.out1 = cut ? W.partials : W.ynear;
        L.lds_bytes = lds_bytes;
        check_hip(h2::launch_stream(L, w.kind, A.vec_f64, cut, on), "stream launch");
    };
    // Streamed schedule: the near-field rows of the stream list run on the
    // handle's second stream, a share from the start of the product and the
    // rest after the coupling rows; the last launch (leaf phase) waits for them.
    const bool streamed = A.schedule == H2_SCHEDULE_STREAMED && w.srows;
    const h2::RowDesc *near_rows = streamed ? w.srows + w.nsrows_coupling : nullptr;
    int64_t nnear = 0, near_split = 0;
    if (streamed) {
        nnear = int64_t(w.near_cum.size()) - 1;
        const int64_t target = std::llround(A.near_early * double(w.near_cum.back()));
        near_split = std::lower_bound(w.near_cum.begin(), w.near_cum.end(), target) - w.near_cum.begin();
        near_split = std::min(near_split, nnear);
        check_hip(hipEventRecord(A.ev_fork, st), "hipEventRecord");
        check_hip(hipStreamWaitEvent(A.aux, A.ev_fork, 0), "hipStreamWaitEvent");
        stream_rows(near_rows, near_split, A.near_lds_bytes, A.aux);
    }
    mark(PH_UP);
    for (const SweepStep &g : A.up_steps) sweep(g, true);
    mark(PH_STREAM);
    if (streamed) {
        stream_rows(w.srows, w.nsrows_coupling, 0, st);
        check_hip(hipEventRecord(A.ev_mid, st), "hipEventRecord");
        check_hip(hipStreamWaitEvent(A.aux, A.ev_mid, 0), "hipStreamWaitEvent");
        stream_rows(near_rows + near_split, nnear - near_split, A.near_lds_bytes, A.aux);
        check_hip(hipEventRecord(A.ev_join, A.aux), "hipEventRecord");
    } else if (w.slot) {   // stored by halves: row sums and transposed partials, then their sums
        h2::RowLaunch L;
        L.rows = w.rows;
        L.nrows = w.nrows;
        L.blks = w.blks;
        L.data = w.data;
        L.scales = A.scales;
        L.in0 = W.xh;
        L.in1 = x;
        L.out0 = W.yh;
        L.out1 = W.ynear;
        check_hip(h2::launch_stream_half(L, w.groups, w.ngroups, w.slot, w.gslot, W.partials, w.kind, A.vec_f64, st),
                  "half-storage stream launch");
        check_hip(h2::launch_reduce_chunks(w.red, w.nred, W.partials, W.yh, W.ynear, A.vec_f64, st),
                  "partial sum launch");
    } else {
        stream_rows(w.rows, w.nrows, 0, st);
    }
    mark(PH_DOWN);
    for (const SweepStep &g : A.down_steps) {
        if (g.leaf) {
            mark(PH_LEAF);
            if (streamed) check_hip(hipStreamWaitEvent(st, A.ev_join, 0), "hipStreamWaitEvent");
        }
        sweep(g, false);
    }
    mark(PH_COUNT);
    if (prof) A.pending.insert(A.pending.end(), ev, ev + PH_COUNT + 1);
}

// One pass of up to MM_TILE right-hand sides on the matrix cores.
void run_tile_pass(h2_matrix_ &A, const double *X, int64_t ldx, double *Y, int64_t ldy, int nrhs, int j0,
                   const h2::MmConfig &cfg, hipStream_t st) {
    const int64_t nleaves = int64_t(1) << A.st.q;
    {
        check_hip(h2::launch_pack(X, ldx, j0, nrhs, A.d_leaf_begin, A.d_leaf_end, nleaves, A.tile_slot,
                                  static_cast<float *>(A.t_x),
                                  h2::mm_tile_width(cfg, std::min(h2::MM_TILE, nrhs - j0)), st),
                  "pack launch");
        run_lists(A, A.mm_lists, st, [&](const WorkList &w) {
            h2::MmLaunch L;
            L.rows = w.rows;
            L.items = w.items;
            L.nitems = w.nitems;
            L.pitems = w.pitems;
            L.npitems = w.npitems;
            L.blks = w.blks;
            L.data = w.data;
            L.scales = A.scales;
            L.in_tree = nullptr;
            L.in_pts = static_cast<float *>(A.t_x);
            L.init = nullptr;
            L.out_tree = nullptr;
            L.out_pts = nullptr;
            L.Y = Y + int64_t(j0) * ldy;
            L.ldy = ldy;
            L.ncols = std::min(h2::MM_TILE, nrhs - j0);
            switch (w.phase) {
                case PH_UP:
                    L.in_tree = static_cast<float *>(A.t_xh);
                    L.out_tree = static_cast<float *>(A.t_xh);
                    break;
                case PH_STREAM:
                    L.in_tree = static_cast<float *>(A.t_xh);
                    L.out_tree = static_cast<float *>(A.t_yh);
                    L.out_pts = static_cast<float *>(A.t_ynear);
                    break;
                case PH_DOWN:
                    L.in_tree = static_cast<float *>(A.t_yh);
                    L.init = static_cast<float *>(A.t_yh);
                    L.out_tree = static_cast<float *>(A.t_yh);
                    break;
                default:
                    L.in_tree = static_cast<float *>(A.t_yh);
                    L.init = static_cast<float *>(A.t_ynear);
                    break;
            }
            check_hip(h2::launch_mm(L, w.kind, int(w.phase), cfg, st), "mfma launch");
        });
    }
}

// Fewest right-hand sides a pass on the FP64 matrix cores is used for.  A pass
// of up to 16 costs 1.2 to 1.85 single-vector products (2-D, 2^18 points 2.23
// against 1.79 ms, 4,096 points 48 against 31 us; 3-D, 3,000 points of rank 27 60
// against 33 us); stored by halves it reads every block twice, where the
// single-vector product reads it once, and costs 2.1 to 2.6 of them from 40,000
// points up (2-D 2^18 points 2.84 against 1.16 ms), 1.5 and less below.
int least_columns64(const h2_matrix_ &A) { return A.half ? 3 : 2; }

// Y = A X for an FP64 matrix on the FP64 matrix cores, MM_TILE right-hand
// sides per pass (a pass of at most 16 takes 16-wide tiles).
void run_tiles64(h2_matrix_ &A, const double *X, int64_t ldx, double *Y, int64_t ldy, int nrhs, hipStream_t st) {
    double *xh = static_cast<double *>(A.t_xh), *yh = static_cast<double *>(A.t_yh);
    double *tx = static_cast<double *>(A.t_x), *tn = static_cast<double *>(A.t_ynear);
    for (int j0 = 0; j0 < nrhs; j0 += h2::MM_TILE) {
        const int ncols = std::min(h2::MM_TILE, nrhs - j0);
        if (ncols < least_columns64(A)) {   // the last pass
            for (int j = j0; j < nrhs; ++j) run_product(A, X + int64_t(j) * ldx, Y + int64_t(j) * ldy, st);
            break;
        }
        check_hip(h2::launch_pack64(X + int64_t(j0) * ldx, ldx, ncols, A.d_leaf_begin, A.d_leaf_end,
                                    int64_t(1) << A.st.q, A.tile_slot, tx, st),
                  "pack launch");
        run_lists(A, A.mm_lists, st, [&](const WorkList &w) {
            const bool sweep_down = w.phase == PH_DOWN || w.phase == PH_LEAF;
            h2::Mm64Launch L;
            L.rows = w.rows;
            L.items = w.items;
            L.nitems = w.nitems;
            L.blks = w.blks;
            L.data = static_cast<const double *>(w.data);
            L.in_tree = sweep_down ? yh : xh;
            L.in_pts = tx;
            L.init = w.phase == PH_LEAF ? tn : yh;
            L.out_tree = w.phase == PH_UP ? xh : yh;
            L.out_pts = tn;
            L.Y = Y + int64_t(j0) * ldy;
            L.ldy = ldy;
            L.ncols = ncols;
            L.half = A.half && w.phase == PH_STREAM;
            check_hip(h2::launch_mm64(L, int(w.phase), st), "fp64 mfma launch");
        });
    }
}

// Calls of this thread that HIP refuses while another stream of the process is
// being captured in global mode (and breaks that capture for) are let through:
// an allocation is no part of anyone's capture.
struct BesideCaptures {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    BesideCaptures() { check_hip(hipThreadExchangeStreamCaptureMode(&mode), "hipThreadExchangeStreamCaptureMode"); }
    ~BesideCaptures() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    BesideCaptures(const BesideCaptures &) = delete;
    BesideCaptures &operator=(const BesideCaptures &) = delete;
};

// Whether the FP64 tile workspace is there, allocated now if it can be: not
// while the stream is being captured, and not when memory is short (the
// product then runs column by column, in the handle's own workspace).
bool tiles64_ready(h2_matrix_ &A, hipStream_t st) {
    if (A.t_xh) return true;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    check_hip(hipStreamIsCapturing(st, &capture), "hipStreamIsCapturing");
    if (capture != hipStreamCaptureStatusNone) return false;
    const BesideCaptures beside;
    // Where the device cannot have the memory, it is not asked: a refused
    // allocation costs a wait for the device and what is kept for the next
    // handles, and this call comes back with every product.  (A sixteenth more,
    // for what the runtime rounds up.)
    int64_t tree = 0, pts = 0;
    const int64_t need = tile_bytes(A, tree, pts);
    int device = 0;
    size_t free_bytes = 0, total = 0;
    check_hip(hipGetDevice(&device), "hipGetDevice");
    check_hip(hipMemGetInfo(&free_bytes, &total), "hipMemGetInfo");
    if (int64_t(free_bytes) + DevicePool::get().held_on(device) < need + need / 16) return false;
    try {
        ensure_tiles(A);
    } catch (const Failure &f) {
        if (f.code != H2_ERR_OOM) throw;
        return false;
    }
    return true;
}

// Y = A X on the matrix cores, MM_TILE right-hand sides per pass.
void run_tiles(h2_matrix_ &A, const double *X, int64_t ldx, double *Y, int64_t ldy, int nrhs, hipStream_t st) {
    ensure_tiles(A);
    for (int j0 = 0; j0 < nrhs; j0 += h2::MM_TILE) {
        const int w = std::min(h2::MM_TILE, nrhs - j0) <= 16 ? 1 : 0;
        if (!A.mm_tuned[w]) tune_tiles(A, X, ldx, Y, ldy, nrhs, j0, st);
        run_tile_pass(A, X, ldx, Y, ldy, nrhs, j0, A.mm_cfg[w], st);
    }
}

}  // namespace h2i

using namespace h2i;

extern "C" {

h2_status h2_matvec(h2_handle A, const double *x, double *y, void *stream) {
    try {
        if (!A || !x || !y) fail(H2_ERR_INVALID_ARG, "NULL argument");
        if (A->structure_only) fail(H2_ERR_INVALID_ARG, "structure-only handle");
        run_product(*A, x, y, static_cast<hipStream_t>(stream));
        return H2_OK;
    } catch (const Failure &f) {
        g_last_error = f.what;
        return f.code;
    } catch (...) {
        g_last_error = "internal error";
        return H2_ERR_INTERNAL;
    }
}

h2_status h2_matmat(h2_handle A, const double *X, int64_t ldx, double *Y, int64_t ldy, int nrhs,
                    void *stream) {
    try {
        if (!A || !X || !Y) fail(H2_ERR_INVALID_ARG, "NULL argument");
        if (A->structure_only) fail(H2_ERR_INVALID_ARG, "structure-only handle");
        if (nrhs < 1) fail(H2_ERR_INVALID_ARG, "nrhs must be >= 1");
        if (ldx < A->st.n || ldy < A->st.n) fail(H2_ERR_INVALID_ARG, "leading dimension below n");
        const hipStream_t st = static_cast<hipStream_t>(stream);
        if (A->vec_f64 && nrhs >= least_columns64(*A) && tiles64_ready(*A, st)) {
            run_tiles64(*A, X, ldx, Y, ldy, nrhs, st);
        } else if (A->vec_f64 || A->half) {
            // too few right-hand sides, no tile workspace, or blocks stored by
            // halves in reduced storage: one single-vector product per column
            for (int j = 0; j < nrhs; ++j) run_product(*A, X + int64_t(j) * ldx, Y + int64_t(j) * ldy, st);
        } else {
            run_tiles(*A, X, ldx, Y, ldy, nrhs, st);
        }
        return H2_OK;
    } catch (const Failure &f) {
        g_last_error = f.what;
        return f.code;
    } catch (...) {
        g_last_error = "internal error";
        return H2_ERR_INTERNAL;
    }
}

h2_status h2_set_schedule(h2_handle A, int schedule, int near_wg_per_cu, double near_early) {
    try {
        if (!A) fail(H2_ERR_INVALID_ARG, "NULL handle");
        if (A->structure_only) fail(H2_ERR_INVALID_ARG, "structure-only handle");
        if (schedule != H2_SCHEDULE_MERGED && schedule != H2_SCHEDULE_STREAMED)
            fail(H2_ERR_INVALID_ARG, "unknown schedule");
        if (near_wg_per_cu < 0) fail(H2_ERR_INVALID_ARG, "near_wg_per_cu must be >= 0");
        if (!(near_early >= 0.0 && near_early <= 1.0)) fail(H2_ERR_INVALID_ARG, "near_early must be in [0, 1]");
        if (schedule == H2_SCHEDULE_MERGED) {
            A->schedule = schedule;
            return H2_OK;
        }
        if (A->half) fail(H2_ERR_UNSUPPORTED, "the streamed schedule needs full storage");
        int lds_bytes = 0;
        if (near_wg_per_cu > 0) {
            // LDS request above 1 / (cap + 1) of a compute unit's LDS: at most
            // cap of the launch's workgroups fit on one compute unit (the
            // block-row kernels' own LDS is at most 4 KiB; 1 KiB of slack per
            // workgroup for the allocation granularity)
            int dev = 0, lds_cu = 0, lds_wg = 0;
            check_hip(hipGetDevice(&dev), "hipGetDevice");
            check_hip(hipDeviceGetAttribute(&lds_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev),
                      "hipDeviceGetAttribute");
            check_hip(hipDeviceGetAttribute(&lds_wg, hipDeviceAttributeMaxSharedMemoryPerBlock, dev),
                      "hipDeviceGetAttribute");
            const int64_t own = 4096, pad = int64_t(lds_cu) / (near_wg_per_cu + 1) + 1;
            if (lds_cu <= 0 || pad + own > lds_wg || int64_t(near_wg_per_cu) * (pad + own + 1024) > lds_cu)
                fail(H2_ERR_UNSUPPORTED, "near_wg_per_cu = " + std::to_string(near_wg_per_cu) +
                                             " cannot be set through the LDS request on this device (" +
                                             std::to_string(lds_cu) + " bytes per compute unit, " +
                                             std::to_string(lds_wg) + " per workgroup)");
            lds_bytes = int(pad);
        }
        if (!A->aux) {
            hipStream_t s = nullptr;
            check_hip(hipStreamCreateWithFlags(&s, hipStreamNonBlocking), "hipStreamCreateWithFlags");
            A->aux = s;
        }
        for (hipEvent_t *e : {&A->ev_fork, &A->ev_mid, &A->ev_join})
            if (!*e) check_hip(hipEventCreateWithFlags(e, hipEventDisableTiming), "hipEventCreateWithFlags");
        A->schedule = schedule;
        A->near_wg_per_cu = near_wg_per_cu;
        A->near_lds_bytes = lds_bytes;
        A->near_early = near_early;
        return H2_OK;
    } catch (const Failure &f) {
        g_last_error = f.what;
        return f.code;
    } catch (...) {
        g_last_error = "internal error";
        return H2_ERR_INTERNAL;
    }
}

h2_status h2_profile(h2_handle A, int enable) {
    if (!A) {
        g_last_error = "NULL handle";
        return H2_ERR_INVALID_ARG;
    }
    A->prof = enable != 0;
    if (A->prof) {
        std::fill(A->prof_ms, A->prof_ms + 8, 0.0);
        A->prof_calls = 0;
    }
    return H2_OK;
}

h2_status h2_profile_read(h2_handle A, double *ms, int64_t *calls) {
    try {
        if (!A || !ms || !calls) fail(H2_ERR_INVALID_ARG, "NULL argument");
        for (size_t i = 0; i + PH_COUNT < A->pending.size(); i += PH_COUNT + 1) {
            hipEvent_t *ev = &A->pending[i];
            check_hip(hipEventSynchronize(ev[PH_COUNT]), "hipEventSynchronize");
            for (int p = 0; p < PH_COUNT; ++p) {
                float t = 0.0f;
                // end of phase p = start of the next recorded phase
                check_hip(hipEventElapsedTime(&t, ev[p], ev[p + 1]), "hipEventElapsedTime");
                A->prof_ms[p] += t;
            }
            float tot = 0.0f;
            check_hip(hipEventElapsedTime(&tot, ev[0], ev[PH_COUNT]), "hipEventElapsedTime");
            A->prof_ms[PH_COUNT] += tot;
            ++A->prof_calls;
        }
        A->spare.insert(A->spare.end(), A->pending.begin(), A->pending.end());
        A->pending.clear();
        std::copy(A->prof_ms, A->prof_ms + 8, ms);
        *calls = A->prof_calls;
        return H2_OK;
    } catch (const Failure &f) {
        g_last_error = f.what;
        return f.code;
    }
}

}  // extern "C"
