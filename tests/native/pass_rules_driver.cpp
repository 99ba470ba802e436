// The compiled rules that choose a pass's form, printed for tests/test_pass_rules.py (host code
// only: built with hipcc --cuda-host-only, no kernel is launched).
#include <cstdio>

#include "../../paper_1501_04438_amd/csrc/passes.hpp"

using namespace gsk;

template <int N> static void rules() {
    const char* loop[] = {"never", "always", "beyond_cache"};
    std::printf("loop_g %d %s %s\n", N, loop[(int)gs_fused_loop_g(3, N, false)], loop[(int)gs_fused_loop_g(3, N, true)]);
    std::printf("p5_unchecked %d %d %d\n", N, (int)p5_split_len<N>(), (int)p5_unchecked<N>());
    for (double mb : {38.0, 168.0, 202.0, 236.0, 269.0, 336.0, 538.0})
        for (int e = 0; e < 2; ++e)
            std::printf("persistent_g %d %.0f %d %d %d\n", N, mb, e, (int)gs_fused_persistent_g(3, N, false, e, mb * 1e6),
                        (int)gs_fused_persistent_g(3, N, true, e, mb * 1e6));
}

int main() {
#define GS_RULES(N) rules<N>();
    GS_SIZE_LIST(GS_RULES)
#undef GS_RULES
    return 0;
}
