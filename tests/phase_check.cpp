// Host check of the phase recursion's step schedule (no GPU): for each
// N:uc:R given on the command line it verifies that
//  * every w but the seeds is finished in exactly one step, and a step's w
//    read nothing of their own or a later step;
//  * every sample of S is summed exactly once, either in its w's bulk (both
//    sides at least three steps back) or among its at most PH_FRESH fresh
//    samples, at its own place in S, with the entries of its two sides (the
//    pair's phasor conjugated exactly where the sample holds -v);
//  * the entries written by each step are those of its w and of the mirrors
//    the raster holds, and every entry lies inside the raster.
// Prints one line per case ending in "bad=<count>".
#include "plan.hpp"

#include <algorithm>
#include <cstdio>
#include <vector>

using namespace nvsm;

static long check(const HostPlan &pl) {
    const PhaseSteps &ph = pl.ph;
    long bad = 0;
    const int nW = (int)pl.W.size() / 2, uc = pl.uc, R = pl.R, pw = 2 * uc + 1;
    auto at = [&](int x, int y) { return (y + R) * pw + x + uc; };
    std::vector<int32_t> wv;
    enumerate_S(uc, R, &wv);
    if (ph.zero != (uc + R + 1) * pw || ph.entries != ph.zero + 1 || ph.entries > 0x3fff) ++bad;
    if ((int)ph.vslot.size() != 32 * ph.tpl || ph.step.size() % 128 || (int)ph.step.size() < 2 * ph.steps + 256) return bad + 1;
    // the pairs +-v, each once
    int pairs = 0;
    std::vector<int> vx(32 * ph.tpl), vy(32 * ph.tpl);
    for (int j = 0; j < 32 * ph.tpl; ++j) {
        if (ph.vslot[j] == ph.zero) continue;
        ++pairs;
        vx[j] = ph.vslot[j] % pw - uc;
        vy[j] = ph.vslot[j] / pw - R;
        if (vx[j] * vx[j] + vy[j] * vy[j] > R * R || !(vy[j] > 0 || (vy[j] == 0 && vx[j] > 0))) ++bad;
        if (j && ph.vslot[j] <= ph.vslot[j - 1]) ++bad;
    }
    int disk = 0;
    for (int y = -R; y <= R; ++y)
        for (int x = -R; x <= R; ++x) disk += x * x + y * y <= R * R && (x || y);
    if (2 * pairs != disk) ++bad;
    // the step that writes each entry
    std::vector<int> step(nW, -1);
    step[0] = step[1] = 0;
    std::vector<int> written(ph.entries, -1);
    auto rec = [&](int s, int b, int k) { return &ph.crit[(((size_t)s * PH_WIDE + b) * 8 + k) * 4]; };
    for (int w = 0; w < 2; ++w) {
        const int x = pl.W[2 * w], y = pl.W[2 * w + 1];
        if ((int)rec(0, 0, w)[0] != at(x, y) || (int)rec(0, 0, w)[1] != at(-x, -y)) return bad + 1;
        written[at(x, y)] = written[at(-x, -y)] = 0;
    }
    for (int s = 1; s < ph.steps; ++s) {
        const int w0 = (int)(ph.step[2 * s] & 0x1fff), n = (int)((ph.step[2 * s] >> 13) & 15);
        if (n > PH_WIDE) ++bad;
        if ((int)(ph.step[2 * s] >> 17) != pl.woff[w0 + n] - pl.woff[w0] || (int)ph.step[2 * s + 1] != pl.woff[w0]) ++bad;
        for (int b = 0; b < PH_WIDE; ++b) {
            const int w = b < n ? w0 + b : -1;
            int put[8];
            for (int k = 0; k < 8; ++k) {
                put[k] = (int)rec(s, b, k)[2];
                if ((int)rec(s, b, k)[3] != (k == 2 ? w : -1)) ++bad;
            }
            for (int k = 2; k < 8; ++k) bad += put[k] != -1;
            if (w < 0) {
                bad += put[0] != -1 || put[1] != -1;
                continue;
            }
            if (w >= nW || step[w] != -1) return bad + 1;
            step[w] = s;
            const int x = pl.W[2 * w], y = pl.W[2 * w + 1];
            if (put[0] != at(x, y) || put[1] != (y <= R ? at(-x, -y) : -1)) return bad + 1;
            written[at(x, y)] = s;
            if (y <= R) written[at(-x, -y)] = s;
        }
    }
    for (size_t s = 2 * ph.steps; s < ph.step.size(); ++s) bad += ph.step[s] != 0;
    bad += ph.step[0] != 0;
    for (int w = 0; w < nW; ++w) bad += step[w] < 0;
    // every sample once; an entry is read only after the step that wrote it
    std::vector<int> hit(pl.s_count, 0);
    const uint32_t none = PH_NONE | ((uint32_t)ph.zero << 4);
    if (ph.code.size() != (size_t)nW * ph.tpl * 32) return bad + 1;
    for (int w = 0; w < nW; ++w)
        for (int l = 0; l < 32; ++l) {
            for (int i = 0; i < ph.tpl; ++i) {
                const uint32_t c = ph.code[ph_code_at(w, l, i, ph.tpl)];
                if (c == none) continue;
                const int j = 32 * i + l, slot = (int)((c >> 4) & 0x3fff), s = w < 2 ? 0 : step[w];
                const int32_t t = (int32_t)(ph.step[2 * s + 1] + ((c >> 19) & 0xfff));
                if (w < 2 || t < pl.woff[w] || t >= pl.woff[w + 1] || slot >= ph.zero || (c & 0x8000000fu)) {
                    ++bad;
                    continue;
                }
                const int sx = (c >> 18) & 1 ? -vx[j] : vx[j], sy = (c >> 18) & 1 ? -vy[j] : vy[j];
                ++hit[t];
                if (wv[4 * t + 2] != sx || wv[4 * t + 3] != sy) ++bad;
                if (slot != at(pl.W[2 * w] - sx, pl.W[2 * w + 1] - sy)) ++bad;
                if (written[slot] < 0 || written[slot] > step[w] - 3) ++bad;
                if (written[ph.vslot[j]] < 0 || written[ph.vslot[j]] > step[w] - 3) ++bad;
                // past `early` + 1 the kernel keeps the pairs' phasors it last read
                if (written[ph.vslot[j]] > ph.early) ++bad;
            }
        }
    for (int s = 1; s < ph.steps; ++s)
        for (int b = 0; b < PH_WIDE; ++b)
            for (int k = 0; k < PH_FRESH; ++k) {
                const uint32_t *c = rec(s, b, k);
                const int sa = (int)(c[0] & 0xffff), sb = (int)(c[0] >> 16);
                if (c[1] == PH_NO_SAMPLE) {
                    if (sa != ph.zero || sb != ph.zero) ++bad;
                    continue;
                }
                const int w = (int)rec(s, b, 2)[3];
                const int64_t t = c[1] / 8;
                if (w < 0 || t < pl.woff[w] || t >= pl.woff[w + 1]) { ++bad; continue; }
                ++hit[t];
                const int sx = wv[4 * t + 2], sy = wv[4 * t + 3];
                if (sa != at(pl.W[2 * w] - sx, pl.W[2 * w + 1] - sy) || sb != at(sx, sy)) ++bad;
                if (written[sa] < 0 || written[sa] >= s || written[sb] < 0 || written[sb] >= s) ++bad;
            }
    for (int64_t t = 0; t < pl.s_count; ++t) bad += hit[t] != 1;
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
        std::printf("%s steps=%d tpl=%d bad=%ld\n", argv[i], pl.ph.steps, pl.ph.tpl, pl.ph.steps ? check(pl) : 0L);
    }
    return 0;
}
