// Device memory that the library keeps for later calls (argument: what is
// checked).
#include "fake_hip.h"

using h2i::DeviceArena;

int main(int, char **argv) {
    const std::string what = argv[1];
    constexpr int64_t MiB = 1 << 20, bound = 1024 * MiB;
    h2_matrix_ *A = fake::matrix(2, H2_FP64), *B = fake::matrix(2, H2_FP64);
    auto dropped = [](int blocks, int64_t bytes) {   // an owner of so many blocks that comes and goes
        DeviceArena a;
        a.alloc(256);
        for (int k = 0; k < blocks; ++k) a.alloc(bytes);
    };
    if (what == "bound") {
        for (int k = 0; k < 5; ++k) dropped(12, 96 * MiB);
        CHECK(fake::used <= bound);
        dropped(2, 2 * bound);
        CHECK(fake::used <= bound);
        // a program that moves on to other sizes finds these after a while
        auto mallocs_of = [&](int blocks, int64_t bytes) {
            const int before = fake::mallocs;
            dropped(blocks, bytes);
            return fake::mallocs - before;
        };
        for (int k = 0; k < 100; ++k) dropped(8, 32 * MiB);
        CHECK(mallocs_of(8, 32 * MiB) == 1 && fake::used <= bound);
        // more than there is room for, in turn: as much as fits is found each time
        for (int k = 0; k < 100; ++k) dropped(40, 32 * MiB);
        CHECK(mallocs_of(40, 32 * MiB) == 1 + 8 && fake::used <= bound);
    } else if (what == "given_back") {
        dropped(4, 16 * MiB);
        CHECK(fake::used > 0);
        h2_free(A);
        CHECK(fake::used > 0);
        h2_free(B);   // the last handle
        CHECK(fake::used == 0 && fake::blocks.empty());
        return 0;
    } else if (what == "release") {
        dropped(4, 16 * MiB);
        CHECK(fake::used > 0);
        h2_release_kept();
        CHECK(fake::used == 0 && fake::blocks.empty());
        dropped(4, 16 * MiB);   // kept again
        CHECK(fake::used > 0);
    } else if (what == "short_memory") {
        // less than a sixteenth of the device free: nothing is kept, and nothing stays kept
        dropped(4, 16 * MiB);
        DeviceArena other;
        fake::budget = 1600 * MiB;
        other.alloc(1510 * MiB);
        dropped(1, 2 * MiB);
        CHECK(fake::used == other.bytes);
        fake::budget = int64_t(1) << 40;
        h2_release_kept();
        dropped(1, 2 * MiB);
        const int queries = fake::queries;
        for (int k = 0; k < 128; ++k) dropped(1, 2 * MiB);   // a loop looks up now and then
        CHECK(fake::queries - queries <= 2 && fake::used == other.bytes + 2 * MiB);
    } else if (what == "sizes") {
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
