// Host-only checks of the choices that the library makes before it launches
// anything (this file includes the library source; no GPU is touched):
//   * arrays are used in place only where they are device memory of the GPU that
//     reads them.
// Prints one line per case and "ok" at the end; exits 1 after a failure.
#include "../../paper_1601_08201_amd/csrc/sgtv_api.hip"

#include <cstdio>

namespace {

int failures = 0;

#define CHECK(cond, ...)                                     \
    do {                                                     \
        if (!(cond)) {                                       \
            std::printf("FAIL %s:%d: ", __FILE__, __LINE__); \
            std::printf(__VA_ARGS__);                        \
            std::printf("\n");                               \
            ++failures;                                      \
            return;                                          \
        }                                                    \
    } while (0)

void check_memory() {
    hipPointerAttribute_t a{};
    a.type = hipMemoryTypeDevice;
    a.device = 1;
    CHECK(lies_on(a, 1), "own memory");
    CHECK(!lies_on(a, 0), "another GPU's memory");
    for (const hipMemoryType t : {hipMemoryTypeHost, hipMemoryTypeManaged, hipMemoryTypeUnregistered}) {
        a.type = t;
        CHECK(!lies_on(a, 1), "memory type %d", static_cast<int>(t));
    }
    std::printf("memory in place\n");
}

}  // namespace

int main() {
    check_memory();
    if (failures) return 1;
    std::printf("ok\n");
    return 0;
}
