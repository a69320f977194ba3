// Rows and stages of a tile of conv_wave.hip, in whole numbers: which input rows it reaches, where they lie in LDS, whose filter
// fragments a wave asks for.  (No HIP in here: planner, kernels and a host test share it.)
#pragma once
#include <numeric>

namespace cac {

// A tile's pixels run on from image to image.  In LDS an image takes VH rows, its halo rows among them, and the tile PH from the first
// tap row of its first output row on; from memory it stages up to IR rows, those of the images one after the other.
struct WaveRows {
    int VH, PH, IR;
};

// ... of tiles of pt pixels, which start at multiples of pt, on output planes of Hc x Wc; tall: input rows that an output row meets.
// Going on to the next image takes `tall` rows of LDS where the next output row of the same image takes `is`: fewer where the filter is
// flatter than the stride (1 x 9, stride 2), and the tallest tile is then one that stays in its image.
constexpr WaveRows wave_rows(int Hin, int Hc, int Wc, int is, int tall, int pt)
{
    // output rows that a tile meets, and how often it goes on to another image, at most
    const int rows = (Wc - std::gcd(pt, Wc) + pt - 1) / Wc + 1, cross = (Hc * Wc - std::gcd(pt, Hc * Wc) + pt - 1) / (Hc * Wc);
    const int gap = Hin - Hc * is > 0 ? Hin - Hc * is : 0; // input rows of an image that no output row starts at
    const int reach = (rows - 1) * is + cross * gap + tall, all = (cross + 1) * Hin;
    const int more = tall > is ? tall - is : 0;
    return WaveRows{(Hc - 1) * is + tall, (rows - 1) * is + cross * more + tall, reach < all ? reach : all};
}

// First row staged: of the image that the tile starts in, at output row i0, or, where padding alone follows in that image, the first of
// the next.
constexpr int wave_first_row(int i0, int is, int dhmin, int Hin)
{
    const int h = i0 * is + dhmin;
    return h < 0 ? 0 : h < Hin ? h : Hin;
}

// Row `row` of those that a tile stages, which lies in image gi = (first + row) / Hin from the tile's first one on: its row there and
// in LDS; ok: the tile wants it.
struct WaveRow {
    int hin, lr;
    bool ok;
};
constexpr WaveRow wave_row(const WaveRows &r, int Hin, int is, int dhmin, int i0, int first, int row, int gi)
{
    const int hin = first + row - gi * Hin, vi = hin - dhmin, lr = gi * r.VH + vi - i0 * is;
    const bool ok = (row < r.IR) & (vi >= 0) & (vi < r.VH) & (lr >= 0) & (lr < r.PH);
    return WaveRow{hin, lr, ok};
}

// LDS row of the first tap row of output row i of image gi.
constexpr int wave_pixel_row(const WaveRows &r, int is, int i0, int gi, int i) { return gi * r.VH + (i - i0) * is; }

// The stage whose filter fragments a wave asks for during stage s: its next one; after its last that one's again, never used (a scalar
// offset past the filter is not covered by the range check of the load).
constexpr int wave_next_stage(int s, int KS, int nkb) { return s + KS < nkb ? s + KS : s; }

} // namespace cac
