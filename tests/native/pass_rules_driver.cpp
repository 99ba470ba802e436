// The compiled rules that choose a pass's form, printed for tests/test_pass_rules.py (host code
// only: built with hipcc --cuda-host-only, no kernel is launched).
#include <cstdio>
#include <vector>

#include "../../paper_1501_04438_amd/csrc/passes.hpp"

using namespace gsk;

// The tiles a row of nb blocks works, each once?
template <class F> static bool each_once(F tile, int nb) {
    std::vector<char> seen(nb, 0);
    for (int b = 0; b < nb; ++b) {
        const int t = tile(b);
        if (t < 0 || t >= nb || seen[t]++) return false;
    }
    return true;
}

// The rows of tiles of the x passes with PX row pairs and of the y passes with PY pencils: whole
// rows, the rows of padding to B_3 that hold data (2/3), and rows of grids whose axes differ (any
// length), of up to 2048 points.
template <int N, int P> static void orders() {
    bool x = true, y = true, g = true;
    const int cut = N % 3 == 0 ? 2 * N / 3 : N;
    for (int m : {N, cut}) {
        const int nbx = (m + 2 * P - 1) / (2 * P), nby = (m + P - 1) / P;
        for (bool rows : {false, true}) x = x && each_once([&](int b) { return x_tile_of<N, P>(b, nbx, rows); }, nbx);
        y = y && each_once([&](int b) { return y_tile_of<N, P>(b, nby); }, nby);
    }
    for (int nb = 1; nb <= 2048 / P; ++nb) {
        g = g && each_once([&](int b) { return die_tile<line_tiles<N, P>()>(b, nb); }, nb);
        g = g && each_once([&](int b) { return die_tile<2>(b, nb); }, nb);
    }
    std::printf("orders %d %d %d %d %d\n", N, P, (int)x, (int)y, (int)g);
}

template <int N> static void rules() {
    orders<N, 1>();
    orders<N, 2>();
    orders<N, 4>();
    orders<N, 8>();
    orders<N, 16>();
    orders<N, 32>();
    // the runs of one die along a row, in the 3D x passes at the default tile and in the y passes
    std::printf("runs %d %d %d\n", N, die_run<N>(N / (2 * Geo<N>::PPX), line_tiles<N, Geo<N>::PPX>()),
                die_run<N>(N / Geo<N>::PPY, Geo<N>::PPY == 8 ? 2 : 1));
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
