// The tile workspace of FP64 handles, made by the first product of several
// columns (argument: what is checked).
#include "fake_hip.h"

namespace h2i {
thread_local std::string g_last_error;
void tune_tiles(h2_matrix_ &, const double *, int64_t, double *, int64_t, int, int, hipStream_t) {}
}  // namespace h2i

int main(int, char **argv) {
    const std::string what = argv[1];
    std::vector<double> x(1);
    h2_matrix_ *A = fake::matrix(6, H2_FP64);
    auto product = [&] { return h2_matmat(A, x.data(), A->st.n, x.data(), A->st.n, 4, nullptr); };
    if (what == "beside_a_capture") {
        // the capture of another stream goes on, and the call does what it does without one
        fake::other_capture = true;
        CHECK(product() == H2_OK);
        CHECK(!fake::capture_broken && fake::mode == hipStreamCaptureModeGlobal);
        CHECK(fake::tile_launches == 1 && fake::single_products == 0);
        fake::other_capture = false;
    }
    delete A;
    return 0;
}
