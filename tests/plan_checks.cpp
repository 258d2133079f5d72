// Host checks of bz_plan.hpp: what is decided from shapes and options alone.
#include <cstdio>
#include <cstdlib>

#include "bz_plan.hpp"

using namespace bz;

#define CHECK(x)                                                         \
    do {                                                                 \
        if (!(x)) {                                                      \
            std::printf("FAIL %s:%d: %s\n", __FILE__, __LINE__, #x);     \
            std::exit(1);                                                \
        }                                                                \
    } while (0)

// the kernel without tables is dealt to the workgroups that it was measured with
static void check_groups() {
    const int f3[] = {5, 5, 4, 4}, f7[] = {4, 3, 2, 2};
    for (int W = 1; W <= 4; W++) CHECK(prefix_groups(3, W) == f3[W - 1] && prefix_groups(7, W) == f7[W - 1]);
}

int main() {
    check_groups();
    std::printf("OK groups\n");
    return 0;
}
