// Compares the row intervals of the large rectangles' tile tests with the
// exact test of every tile, on random and adversarial ellipses: no hit lies
// outside [first, last], every tile of [sure_first, sure_last] is a hit.  The
// exact test is the oracle's (binary32 mode).  Arguments: cases, seed.
// Prints the tiles compared and the share that stays undecided.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>

#include "tile_test.hpp"

extern "C" int orc_tile_hit_api_f32(const float *state16, int tx, int ty, int W, int H);

int main(int argc, char **argv) {
    const long cases = argc > 1 ? atol(argv[1]) : 10000;
    std::mt19937_64 rng(argc > 2 ? atol(argv[2]) : 1);
    auto uni = [&](double a, double b) { return std::uniform_real_distribution<double>(a, b)(rng); };
    long tiles = 0, hits = 0, undecided = 0, bad = 0, fallback = 0;
    for (long i = 0; i < cases; ++i) {
        const int W = 1 + (int)(std::exp(uni(0.0, std::log(9000.0)))), H = 1 + (int)(std::exp(uni(0.0, std::log(6000.0))));
        // covariance of a rotated ellipse: axes from a fraction of a pixel to
        // many images, aspect up to 1e4; aligned and diagonal ones among them
        const double a = std::exp(uni(std::log(4.0), std::log(2e4))), b = std::exp(uni(std::log(0.55), std::log(a)));
        const int kind = (int)(rng() % 5);
        const double th = kind == 0 ? 0.0 : kind == 1 ? M_PI / 2 : kind == 2 ? M_PI / 4 : uni(0.0, M_PI);
        const float ca = (float)(a * a * std::cos(th) * std::cos(th) + b * b * std::sin(th) * std::sin(th));
        const float cc = (float)(a * a * std::sin(th) * std::sin(th) + b * b * std::cos(th) * std::cos(th));
        const float cb = (float)((a * a - b * b) * std::sin(th) * std::cos(th));
        const float det = ca * cc - cb * cb;
        if (!(det > 0.0f)) continue;
        const float A = cc / det, B = -cb / det, C = ca / det;
        const float k2 = (float)(rng() % 3 == 0 ? 9.0 : uni(1e-4, 9.0));
        // centres inside, at the border of, and far outside the image; some
        // exactly on sample and tile boundaries
        const double far = rng() % 4 == 0 ? 3.0 * a : 0.0;
        float u = (float)uni(-far, W + far), v = (float)uni(-far, H + far);
        if (rng() % 8 == 0) u = std::floor(u) + 0.5f;
        if (rng() % 8 == 0) v = 16.0f * std::floor(v / 16.0f) + 0.5f;
        float s[16] = {u, v, A, B, C, k2};  // the oracle's state order: u, v, A, B, C, k2, ...
        const fgs::RowTest t = fgs::row_test(u, v, A, B, C, k2);
        fallback += t.fo < 0.0f;
        const int ntx = (W + 15) / 16, nty = (H + 15) / 16;
        // some rectangles that are a part of the image's columns
        const int tx0 = rng() % 3 == 0 ? (int)(rng() % ntx) : 0, tx1 = rng() % 3 == 0 ? tx0 + (int)(rng() % (ntx - tx0)) : ntx - 1;
        const int step = nty > 40 ? 1 + (int)(rng() % (nty / 20)) : 1;
        for (int ty = (int)(rng() % step); ty < nty; ty += step) {
            float y0, y1;
            fgs::tile_row_span(v, ty, H, y0, y1);
            const fgs::RowCols r = fgs::row_columns(t, u, y0, y1, tx0, tx1, W);
            for (int tx = tx0; tx <= tx1; ++tx) {
                const bool hit = orc_tile_hit_api_f32(s, tx, ty, W, H) != 0;
                const bool poss = tx >= r.first && tx <= r.last, sure = tx >= r.sure_first && tx <= r.sure_last;
                ++tiles;
                hits += hit;
                undecided += poss && !sure && t.fo >= 0.0f;
                if (hit != fgs::tile_hit<false>(u, v, A, B, C, k2, tx, ty, W, H) ||
                    (fgs::tile_terms_finite(u, v, A, B, C) && hit != fgs::tile_hit<true>(u, v, A, B, C, k2, tx, ty, W, H)) ||
                    (hit && !poss) || (!hit && sure)) {
                    if (bad++ < 5)
                        std::printf("case %ld: u %.9g v %.9g A %.9g B %.9g C %.9g k2 %.9g W %d H %d tile %d %d hit %d "
                                    "[%d %d] sure [%d %d]\n", i, u, v, A, B, C, k2, W, H, tx, ty, hit, r.first, r.last,
                                    r.sure_first, r.sure_last);
                }
            }
        }
    }
    std::printf("tiles %ld hits %ld undecided %.5f fallback %.4f bad %ld\n", tiles, hits, (double)undecided / (double)tiles,
                (double)fallback / (double)cases, bad);
    return bad ? 1 : 0;
}
