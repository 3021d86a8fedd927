// Host check of the solve's tables (no GPU): for each N:uc:R given on the
// command line prints whether the recursion runs in steps (solve_in_steps),
// and verifies the least-squares kernel's samples by pair +-v (LsqPairs):
//  * pair j's entry of vidx is the index in W of its member on W's side (-1
//    past the last pair), every v of the half disk being some pair's;
//  * every sample of S stands in exactly one code of its w, at its place in
//    S(w), under the pair of its v, with the sign of v, and with the index of
//    w - v in W, or of its mirror and the flag for it.
// Prints one line per case ending in "bad=<count>".
#include "plan.hpp"

#include <cstdio>
#include <map>
#include <vector>

using namespace nvsm;

static long check_lsq(const HostPlan &pl) {
    const LsqPairs &lq = pl.lsq;
    const int nW = (int)pl.W.size() / 2, R = pl.R;
    if ((int)lq.vidx.size() != 64 * lq.tpl || lq.code.size() != (size_t)nW * 64 * lq.tpl) return 1;
    long bad = 0;
    std::map<std::pair<int, int>, int> at;       // W's index of (x, y)
    for (int i = 0; i < nW; ++i) at[{pl.W[2 * i], pl.W[2 * i + 1]}] = i;
    std::vector<int> seen(nW, 0);
    for (int j = 0; j < 64 * lq.tpl; ++j) {
        const int i = lq.vidx[j];
        if (i < 0) continue;
        if (i >= nW || seen[i]++) { ++bad; continue; }
        const int x = pl.W[2 * i], y = pl.W[2 * i + 1];
        bad += x * x + y * y > R * R;
    }
    for (int i = 0; i < nW; ++i) {
        const int x = pl.W[2 * i], y = pl.W[2 * i + 1];
        bad += x * x + y * y <= R * R && !seen[i];
    }
    std::vector<int32_t> wv;
    enumerate_S(pl.uc, R, &wv);
    for (int w = 0; w < nW; ++w) {
        const int n = pl.woff[w + 1] - pl.woff[w];
        std::vector<int> hit(n, 0);
        for (int l = 0; l < 64; ++l)
            for (int i = 0; i < lq.tpl; ++i) {
                const uint32_t c = lq.code[((size_t)w * 64 + l) * lq.tpl + i];
                const uint32_t place = c >> 23;
                if (place == LSQ_NONE) {
                    bad += c != LSQ_NONE << 23;
                    continue;
                }
                const int v = lq.vidx[64 * i + l];
                const uint32_t d = (c >> 4) & 0x1fffu;
                if ((int)place >= n || v < 0 || d >= (uint32_t)nW || (c & 15u)) { ++bad; continue; }
                ++hit[place];
                const int32_t *s = &wv[4 * (pl.woff[w] + place)];
                const int sv = (c >> 22) & 1 ? -1 : 1, sd = (c >> 21) & 1 ? -1 : 1;
                bad += s[0] != pl.W[2 * w] || s[1] != pl.W[2 * w + 1];
                bad += s[2] != sv * pl.W[2 * v] || s[3] != sv * pl.W[2 * v + 1];
                bad += s[0] - s[2] != sd * pl.W[2 * d] || s[1] - s[3] != sd * pl.W[2 * d + 1];
            }
        for (int k = 0; k < n; ++k) bad += hit[k] != 1;
    }
    return bad;
}

int main(int argc, char **argv) {
    for (int i = 1; i < argc; ++i) {
        int N = 0, uc = 0, R = 0;
        HostPlan pl;
        std::string err;
        if (std::sscanf(argv[i], "%d:%d:%d", &N, &uc, &R) != 3 || !build_plan(N, uc, R, 16, &pl, &err)) {
            std::printf("%s: plan failed (%s) bad=1\n", argv[i], err.c_str());
            continue;
        }
        std::printf("%s in_steps=%d pairs=%d bad=%ld\n", argv[i], (int)solve_in_steps(pl), pl.lsq.tpl,
                    pl.lsq.tpl ? check_lsq(pl) : 0L);
    }
    return 0;
}
