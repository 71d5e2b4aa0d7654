// Device memory that the library keeps for later calls (argument: what is
// checked).
#include "fake_hip.h"

using h2i::DeviceArena;

int main(int, char **argv) {
    const std::string what = argv[1];
    constexpr int64_t MiB = 1 << 20;
    h2_matrix_ *A = fake::matrix(2, H2_FP64), *B = fake::matrix(2, H2_FP64);
    auto dropped = [](int blocks, int64_t bytes) {   // an owner of so many blocks that comes and goes
        DeviceArena a;
        a.alloc(256);
        for (int k = 0; k < blocks; ++k) a.alloc(bytes);
    };
    if (what == "sizes") {
        // an owner holds no more than it counts
        dropped(2, 20 * MiB);
        DeviceArena a;
        for (int64_t n : {20 * MiB, 17 * MiB, 16 * MiB + 4096, 64 * int64_t(1024), int64_t(300)}) a.alloc(n);
        CHECK(fake::used - h2i::DevicePool::get().held_on(0) == a.bytes);
    } else {
        return 1;
    }
    h2_free(A);
    h2_free(B);
    return 0;
}
