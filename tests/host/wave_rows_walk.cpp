// Walks every tile of random layers through the row arithmetic of csrc/wave_rows.h, as the kernels of conv_wave.hip use it: every input
// row that a tap of one of the tile's pixels meets lies in the LDS row the pixel reads, once; LDS rows read for the padding hold none.
// Arguments: R (taps down), stride, largest padding, layers.  Prints the layers that are wrong.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "wave_rows.h"

using namespace cac;

// Hin rows in, Hc x Wc pixels out; tap t of output row i meets row i * is + dhmin + t.
static bool tiles_ok(int N, int Hin, int Hc, int Wc, int taps, int is, int dhmin, int pt)
{
    const int ppi = Hc * Wc;
    const WaveRows r = wave_rows(Hin, Hc, Wc, is, taps, pt);
    for (long F = 0; F < (long)N * ppi; F += pt) {
        const int n0 = (int)(F / ppi), px0 = (int)(F % ppi), i0 = px0 / Wc, first = wave_first_row(i0, is, dhmin, Hin);
        if (first > Hin) return false; // (the division by Hin is checked for Hin + IR rows)
        std::vector<int> lds(r.PH, -1); // image * Hin + row that an LDS row holds
        for (int row = 0; row < r.IR; ++row) {
            const int gi = (first + row) / Hin;
            const WaveRow at = wave_row(r, Hin, is, dhmin, i0, first, row, gi);
            if (!at.ok || n0 + gi >= N) continue;
            if (at.lr < 0 || at.lr >= r.PH || at.hin < 0 || at.hin >= Hin || lds[at.lr] >= 0) return false;
            lds[at.lr] = gi * Hin + at.hin;
        }
        for (int f = px0; f < px0 + pt; ++f) {
            const int gi = f / ppi, i = f % ppi / Wc;
            if (n0 + gi >= N) break;
            for (int t = 0; t < taps; ++t) {
                const int h = i * is + dhmin + t, at = wave_pixel_row(r, is, i0, gi, i) + t;
                if (at < 0 || at >= r.PH || lds[at] != (h >= 0 && h < Hin ? gi * Hin + h : -1)) return false;
            }
        }
    }
    return true;
}

// Every filter fragment that the waves of a tile ask for, while they multiply and ahead of that, lies in the filter: stages of KC of
// `channels`, KS waves.  (A tap's fragments are 16-channel steps of equal size; the last tap's end is the filter's.)
static bool fragments_ok(int channels, int KC, int KS)
{
    const int nkb = (channels + KC - 1) / KC;
    for (int ks = 0; ks < KS; ++ks)
        for (int s = ks; s < nkb; s += KS) {
            const int next = wave_next_stage(s, KS, nkb);
            if (next < 0 || next >= nkb || (s + KS < nkb && next != s + KS)) return false;
        }
    return true;
}

int main(int argc, char **argv)
{
    if (argc != 5) return 2;
    const int R = atoi(argv[1]), S = 9 / R, is = atoi(argv[2]), pad = atoi(argv[3]), layers = atoi(argv[4]);
    std::mt19937 rng(7);
    auto pick = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
    int done = 0, wrong = 0;
    for (int channels = 1; channels <= 1100; ++channels)
        for (int KC : {16, 32})
            for (int KS : {4, 8}) wrong += !fragments_ok(channels, KC, KS);
    if (wrong) printf("filter fragments past the last stage\n");
    while (done < layers) {
        const int N = pick(1, 9), H = pick(1, 30), W = pick(1, 30), ph = pick(0, pad), pw = pick(0, pad), pt = pick(0, 2) ? 64 : 32;
        if (H + 2 * ph < R || W + 2 * pw < S) continue;
        ++done;
        const int P = (H + 2 * ph - R) / is + 1, Q = (W + 2 * pw - S) / is + 1;
        bool ok = tiles_ok(N, H, P, Q, R, is, -ph, pt);
        if (is == 1) ok = ok && tiles_ok(N, P, H, W, R, 1, ph - (R - 1), pt); // the data gradient
        else if (R == 3) ok = ok && tiles_ok(N, P, P, Q, 2, 1, 0, pt);        // its parity classes together
        if (ok) continue;
        if (++wrong <= 5) printf("N=%d H=%d W=%d R=%d S=%d stride=%d pad=%d,%d tile=%d\n", N, H, W, R, S, is, ph, pw, pt);
    }
    printf("%d of %d layers wrong\n", wrong, done);
    return wrong != 0;
}
