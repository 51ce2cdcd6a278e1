// TEST INFRASTRUCTURE -- the in-launch selection's fold (csrc/topn_fold.hpp), one loop of 64 lanes per step of the wavefront,
// compiled under -fsanitize=address,undefined.  The column row and the importances are heap blocks of exactly the sizes the
// kernel has, so an index outside them is an ASan report; every block up to the last scored one must get its sum, and no other
// block anything.  Columns hold small integers, so sums are exact in any order.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "../../paper_2605_19893_amd/csrc/topn_fold.hpp"

static int fold(int J, int n_local, int ncv, int in_flight) {
    const int jl = ssv::fold_last_scored(J, n_local), pitch = (std::max(1, ncv) + 63) / 64 * 64;
    float* cs = new float[pitch];
    for (int c = 0; c < pitch; ++c) cs[c] = c < ncv ? (float)(1 + c * 37 % 101) : 1e9f;       // (invisible columns must not count)
    float* imp = new float[J + 1];
    std::fill(imp, imp + J + 1, -1.f);
    struct Cols { float own[4], left; };
    auto loads = [&](int j) {
        Cols r;
        const int c = ssv::fold_column(j, jl, ncv);
        for (int u = 0; u < 4; ++u) r.own[u] = cs[c + u];
        r.left = cs[ssv::fold_left_column(j, jl, ncv)];
        return r;
    };
    auto any = [&](int j, const Cols& r) {
        if (j > jl) return;
        const int c0 = 4 * j;
        float s = 0.f;
        if (c0 >= 1 && c0 - 1 < ncv) s += r.left;
        for (int u = 0; u < 4; ++u)
            if (c0 + u < ncv) s += (u == 3 ? 1.f : 2.f) * r.own[u];
        imp[j] = s;
    };
    const int groups = ssv::fold_full_groups(jl, ncv);
    Cols rest[2][64];
    for (int v = 0; v < 2; ++v)
        for (int lane = 0; lane < 64; ++lane) rest[v][lane] = loads((groups + v) * 64 + lane);
    float last63 = 0.f;
    for (int g0 = 0; g0 < groups; g0 += in_flight)
        for (int v = 0; v < in_flight; ++v) {
            const int g = std::min(g0 + v, groups - 1);
            for (int lane = 0; lane < 64; ++lane) {
                const float* x = cs + 4 * (g * 64 + lane);
                const float left = lane ? x[-1] : last63;
                imp[g * 64 + lane] = left + 2.f * x[0] + 2.f * x[1] + 2.f * x[2] + x[3];
            }
            if (g0 + v + 1 < groups) last63 = cs[4 * (g * 64 + 63) + 3];
        }
    for (int v = 0; v < 2; ++v)
        for (int lane = 0; lane < 64; ++lane) any((groups + v) * 64 + lane, rest[v][lane]);
    for (int lane = 0; lane < 64; ++lane)
        for (int j = (groups + 2) * 64 + lane; j <= jl; j += 64) any(j, loads(j));
    int bad = 0;
    for (int j = 0; j <= J; ++j) {
        float want = -1.f;
        if (j <= J - n_local) {
            want = 0.f;
            for (int u = -1; u < 4; ++u)
                if (4 * j + u >= 0 && 4 * j + u < ncv) want += (u == -1 || u == 3 ? 1.f : 2.f) * cs[4 * j + u];
        }
        bad += imp[j] != want;
    }
    if (bad) std::printf("J %d n_local %d ncv %d in flight %d: %d blocks differ\n", J, n_local, ncv, in_flight, bad);
    delete[] cs;
    delete[] imp;
    return bad;
}

int main() {
    std::vector<int> ncvs;
    for (int edge : {0, 64, 128, 256, 512, 1024, 4096, 8192})
        for (int c = std::max(0, edge - 5); c <= edge + 5; ++c) ncvs.push_back(c);
    int bad = 0, n = 0;
    for (int ncv : ncvs)
        for (int in_flight : {8, 16}) {
            for (int J = 0; J <= 33; ++J)
                for (int n_local = 0; n_local <= 32; ++n_local, ++n) bad += fold(J, n_local, ncv, in_flight);
            for (int edge : {64, 128, 512, 576, 1024, 1088, 2048})
                for (int J = edge - 3; J <= edge + 3; ++J)
                    for (int n_local : {0, 1, 2, 32}) bad += fold(J, n_local, ncv, in_flight), ++n;
        }
    std::printf("%d folds, %d blocks differ\n", n, bad);
    return bad != 0;
}
