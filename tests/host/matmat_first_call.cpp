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
    } else if (what == "no_memory") {
        // too little memory, most of what is there kept for the next handle: single products,
        // without a try at the device and without giving up what is kept, call after call
        h2_matrix_ *B = fake::matrix(6, H2_FP64);
        B->mem.alloc(4096);
        B->mem.alloc(1 << 20);
        delete B;
        fake::budget = fake::used + (1 << 20);
        const int64_t used = fake::used;
        const int mallocs = fake::mallocs, frees = fake::frees;
        for (int k = 1; k <= 3; ++k) {
            CHECK(product() == H2_OK);
            CHECK(fake::single_products == 4 * k && fake::tile_launches == 0);
        }
        CHECK(fake::mallocs == mallocs && fake::frees == frees && fake::used == used);
        // memory comes back: tiles again
        fake::budget = int64_t(1) << 40;
        CHECK(product() == H2_OK && fake::single_products == 12 && fake::tile_launches == 1);
    } else if (what == "memory_kept") {
        // enough memory once what is kept for the next handle is given back
        h2_matrix_ *B = fake::matrix(6, H2_FP64);
        B->mem.alloc(4096);
        for (int k = 0; k < 8; ++k) B->mem.alloc(8 << 20);
        delete B;
        fake::budget = fake::used + (1 << 20);
        CHECK(product() == H2_OK && fake::single_products == 0 && fake::tile_launches == 1);
    }
    delete A;
    return 0;
}
