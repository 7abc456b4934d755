// The dynamic-LDS limits of the tail and LU kernels (tests/test_launch_limits.py): raised on
// every device that a handle is set up on, once each. The runtime's attribute call is
// replaced by one that counts, so no GPU is needed.
#include <cstdio>
#include <cstdlib>

#include "hm_kernels.hpp"

static int raised = 0;
extern "C" hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) {
    ++raised;
    return hipSuccess;
}

int main() {
    auto on = [](int device) {
        const int before = raised;
        hm::tail_init(device);
        hm::setup_init(device);
        return raised - before;
    };
    const int first = on(0), second = on(1), again = on(0), third = on(7);
    std::printf("%d %d %d %d\n", first, second, again, third);
    return first > 1 && second == first && again == 0 && third == first ? EXIT_SUCCESS : EXIT_FAILURE;
}
