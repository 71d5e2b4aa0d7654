// A HIP runtime and device launches that only keep count, for tests of the
// library's host code without a GPU: device memory is host memory, a budget
// stands for the card's, and a capture somewhere in the process refuses
// allocations as HIP does.
#pragma once

#include "h2_internal.h"

#include <cstdio>
#include <cstdlib>
#include <map>

namespace fake {

int64_t budget = int64_t(1) << 40, used = 0;   // bytes of the card, bytes allocated
int mallocs = 0, failed_mallocs = 0, frees = 0, queries = 0;
bool other_capture = false, capture_broken = false;   // another stream is being captured, in global mode
hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;   // the thread's
int single_products = 0, tile_launches = 0;
std::map<void *, size_t> blocks;

// What HIP does with a call it counts as unsafe under a capture.
hipError_t unsafe_call() {
    if (!other_capture || mode == hipStreamCaptureModeRelaxed) return hipSuccess;
    capture_broken = true;
    return hipErrorStreamCaptureUnsupported;
}

}  // namespace fake

#define CHECK(c)                                                          \
    do {                                                                  \
        if (!(c)) {                                                       \
            std::printf("%s:%d: %s\n", __FILE__, __LINE__, #c);           \
            std::exit(1);                                                 \
        }                                                                 \
    } while (0)

extern "C" {

hipError_t hipMalloc(void **p, size_t n) {
    if (hipError_t e = fake::unsafe_call()) return e;
    ++fake::mallocs;
    if (fake::used + int64_t(n) > fake::budget) {
        ++fake::failed_mallocs;
        return hipErrorOutOfMemory;
    }
    *p = std::malloc(n);
    fake::used += int64_t(n);
    fake::blocks[*p] = n;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    if (hipError_t e = fake::unsafe_call()) return e;
    if (!p) return hipSuccess;
    CHECK(fake::blocks.count(p) == 1);
    ++fake::frees;
    fake::used -= int64_t(fake::blocks[p]);
    fake::blocks.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t *free_bytes, size_t *total) {
    ++fake::queries;
    *free_bytes = size_t(fake::budget - fake::used);
    *total = size_t(fake::budget);
    return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *m) {
    std::swap(*m, fake::mode);
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
    *s = hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *, unsigned) { return hipErrorNotSupported; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *, unsigned) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 1.0f, hipSuccess; }

}  // extern "C"

namespace h2 {

hipError_t launch_sweep(const SweepLaunch &, bool, bool, hipStream_t) { return hipSuccess; }
hipError_t launch_stream(const RowLaunch &, int, bool, bool, hipStream_t) { return ++fake::single_products, hipSuccess; }
hipError_t launch_stream_half(const RowLaunch &, const HalfGroup *, int64_t, const int32_t *, const int32_t *, void *,
                              int, bool, hipStream_t) {
    return ++fake::single_products, hipSuccess;
}
hipError_t launch_reduce_chunks(const ReduceDesc *, int64_t, const void *, void *, void *, bool, hipStream_t) {
    return hipSuccess;
}
hipError_t launch_pack(const double *, int64_t, int, int, const int64_t *, const int64_t *, int64_t, int64_t, float *,
                       int, hipStream_t) {
    return hipSuccess;
}
hipError_t launch_mm(const MmLaunch &, int, int, const MmConfig &, hipStream_t) { return ++fake::tile_launches, hipSuccess; }
hipError_t launch_pack64(const double *, int64_t, int, const int64_t *, const int64_t *, int64_t, int64_t, double *,
                         hipStream_t) {
    return hipSuccess;
}
hipError_t launch_read_probe(const void *, int64_t, int, void *, hipStream_t) { return hipSuccess; }
hipError_t launch_mm64(const Mm64Launch &, int, hipStream_t) { return ++fake::tile_launches, hipSuccess; }

}  // namespace h2

namespace fake {

// A handle of 2^q leaves of 64 points, rank 64, with one list per kind.
inline h2_matrix_ *matrix(int q, int storage) {
    h2_matrix_ *A = new h2_matrix_;
    A->st.q = q;
    A->st.n = int64_t(64) << q;
    A->st.nnodes = (int64_t(2) << q) - 1;
    A->st.rank = 64;
    A->st.lrank.assign(size_t(q) + 1, 64);
    A->tile_slot = 64 * h2::MM_TILE;
    A->storage = storage;
    A->vec_f64 = storage == H2_FP64;
    A->block_kind = storage == H2_FP64 ? h2::ELEM_F64 : h2::ELEM_F32;
    h2i::WorkList w{};
    w.phase = h2i::PH_STREAM;
    w.nrows = w.nitems = w.npitems = 64;
    A->lists.push_back(w);
    A->mm_lists.push_back(w);
    return A;
}

}  // namespace fake
