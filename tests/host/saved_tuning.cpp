// Launch shapes saved in the file that H2MV_AUTOTUNE_CACHE names (argument:
// whether this handle's shape is expected to come from it).
#include "fake_hip.h"

namespace h2i {
thread_local std::string g_last_error;
std::vector<int32_t> wave_items(const std::vector<RowDesc> &, const std::vector<BlkDesc> &) { return {}; }
std::vector<int32_t> pair_items(const std::vector<RowDesc> &, const std::vector<BlkDesc> &) { return {}; }
}  // namespace h2i

namespace h2 {
hipError_t launch_mm_batch(const MmBatchLaunch &, int, int, const MmConfig &, hipStream_t) { return hipSuccess; }
hipError_t launch_batch_pack(const PackEntry *, int64_t, double const *const *, const int64_t *, int, int, float *,
                             int64_t, hipStream_t) {
    return hipSuccess;
}
}  // namespace h2

extern "C" {
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipHostFree(void *) { return hipSuccess; }
hipError_t hipHostMalloc(void **, size_t, unsigned) { return hipErrorNotSupported; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipSuccess; }
}

int main(int, char **argv) {
    const bool saved = std::string(argv[1]) == "saved";
    std::vector<double> x(1);
    h2_matrix_ *A = fake::matrix(6, H2_FP32);
    for (int nrhs : {4, 20}) {
        CHECK(h2_matmat(A, x.data(), A->st.n, x.data(), A->st.n, nrhs, nullptr) == H2_OK);
        int pipelined = -1, tile_width = -1;
        int64_t grid = -1;
        double ms = -1.0;
        CHECK(h2_matmat_tuning(A, nrhs <= 16, &pipelined, &grid, &tile_width, &ms) == H2_OK);
        std::printf("%d right-hand sides: %d %lld %d, %g ms\n", nrhs, pipelined, static_cast<long long>(grid), tile_width, ms);
        CHECK((ms == 0.0) == saved);
        CHECK(grid == 0 && tile_width == (nrhs <= 16 ? 16 : 32));
    }
    delete A;
    return 0;
}
