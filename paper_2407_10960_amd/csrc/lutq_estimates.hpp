// Estimated times of the launches that a call of up to 32 rows can take (host code; lutq_api.hip chooses by them).
//
// Why estimates: the rules of default_decomp, default_rows_decomp and sliced_rows_decomp were each measured on some twenty
// shapes, and hold there (within 4 % of the best plan found).  On drawn problems of 5..32 rows (512 to 57344 channels in
// units of 16, K 1024 to 28672, all bit widths, groups and types) they take 16 % (5..16 rows) and 42 % (17..32 rows) longer than the best of
// some fifteen launches timed (7024 x 26624 group 256, W4 fp16, M = 31: 97.4 us, row streaming in K slices 32.9); on 5603 of 1..4 rows 5.7 %.
// Fitted by least squares of the relative error to 159 000 timings of 5..32 rows on 50 000 problems (1..4 rows: 78 000; HBM-cold weights,
// MI355X); on problems not fitted to the estimates are off by 6 to 12 % (row streaming), 7 to 11 % (teams) and 6 to 7 % (panels).
// Three terms carry more than they seem to.  A workgroup that streams row blocks stages all their scale rows, whole, whatever its K
// slice: 0.07 us per KiB, 5 us with group 32 and K = 20000 (880 x 20480 group 32 W3 fp16 M = 6, eight K slices: 15.1 us, the teams 10.3).  Workgroups
// that share a row block cost by their number, and 2 to 3 us more where their parts do not end with it, each then adding two partial
// sums (W3 M = 18, 624 x 4608 in two even parts 9.3 us, 528 x 4864 in two uneven ones 12.6).
#pragma once

#include <stdint.h>

namespace lutq {

// Row streaming: rounds of workgroups; times passes; times K tiles of a wave and passes (eight side by side), the same times waves;
// K tiles of a wave, waves and row blocks; row blocks times waves (reduction); K slices; row blocks times slices; megabytes; KiB of
// scale rows that a workgroup stages, by its waves (eight: 1).
// [bits - 2][up to 16 rows, beyond]
static const double kRowsFit[3][2][10] = {
    {{2.2476, 1.9848, 0.7200, 0.1355, 0.0035, 0.0054, 2.2032, 0.0202, 0.1792, 0.0755},
     {3.3579, 0.9802, 0.5311, 0.2163, 0.0102, 0.0416, 1.7341, 0.0255, 0.2183, 0.0736}},  // 2 bits
    {{2.3153, 2.4690, 0.8867, 0.1292, 0.0159, 0.0006, 2.1116, 0.0149, 0.1416, 0.0762},
     {2.4832, 2.9228, 0.0000, 0.2351, 0.0074, 0.0000, 2.3557, 0.0201, 0.2020, 0.0711}},  // 3 bits
    {{1.6248, 2.2985, 0.8082, 0.1024, 0.0000, 0.0033, 2.1672, 0.0159, 0.1082, 0.0782},
     {2.7696, 1.1674, 0.7993, 0.1573, 0.0000, 0.0392, 1.5494, 0.0282, 0.1105, 0.0691}},  // 4 bits
};
// Teams: fixed; workgroups per compute unit; pairs of them; K tiles of a wave times R; K tiles of a wave, waves, workgroups per unit and
// R; the same without R (activations: once per K part where they are shared, by the share of the class's rows); waves per unit; partial sums across workgroups: fixed,
// per workgroup of a row block, where parts do not end with row blocks; megabytes.
// [bits - 2][1..2, 3..4, 5..8, 9..16, 17..32 rows]
static const double kTeamsFit[3][5][11] = {
    {{1.6409, 0.0654, 1.4913, 0.1391, 0.0414, 0.0000, 0.0244, 5.2359, 0.0000, 0.0000, 0.1070},
     {1.8954, 0.0712, 1.2359, 0.1263, 0.0441, 0.0046, 0.0342, 5.0205, 0.0000, 0.0000, 0.1237},
     {2.2414, 0.0000, 0.8294, 0.1685, 0.0232, 0.0544, 0.0947, 0.7999, 0.3365, 2.6171, 0.1593},
     {2.3978, 0.0000, 0.0000, 0.2071, 0.0043, 0.1416, 0.2349, 2.9510, 0.0000, 2.7246, 0.2369},
     {2.8447, 0.0000, 0.0000, 0.2055, 0.0012, 0.3221, 0.2668, 1.5912, 0.5278, 2.9114, 0.3249}},  // 2 bits
    {{2.3574, 0.0000, 0.3799, 0.1997, 0.0537, 0.0000, 0.0586, 5.1606, 0.0000, 0.0000, 0.0854},
     {2.5379, 0.0000, 0.2058, 0.1476, 0.0642, 0.0000, 0.0669, 5.2634, 0.0000, 0.0000, 0.0955},
     {2.8497, 0.0000, 0.0000, 0.2217, 0.0325, 0.0448, 0.1204, 0.5247, 0.3612, 2.9494, 0.1330},
     {2.6031, 0.0000, 0.0000, 0.1909, 0.0194, 0.1330, 0.1977, 2.8807, 0.0771, 2.1721, 0.1792},
     {2.6262, 0.0000, 0.0000, 0.2369, 0.0022, 0.3256, 0.2665, 1.5749, 0.4956, 2.7301, 0.2595}},  // 3 bits
    {{1.5489, 0.0440, 1.6252, 0.1075, 0.0267, 0.0043, 0.0024, 5.3358, 0.0000, 0.0000, 0.0724},
     {1.6439, 0.0389, 1.4969, 0.0923, 0.0286, 0.0086, 0.0057, 5.1918, 0.0000, 0.0000, 0.0730},
     {2.1586, 0.0000, 1.0265, 0.1426, 0.0164, 0.0302, 0.0304, 0.6660, 0.4631, 2.5857, 0.1160},
     {2.5023, 0.0000, 0.6140, 0.0843, 0.0222, 0.0735, 0.0429, 0.9630, 0.3768, 2.3725, 0.1145},
     {2.7457, 0.0000, 0.5554, 0.0715, 0.0193, 0.1731, 0.0653, 1.5364, 0.4893, 2.8212, 0.1587}},  // 4 bits
};

// Panels of 17..32 rows (one block of 32): rounds of workgroups; rounds times K tiles of a wavefront, 32 and 64 channels; K slices: fixed, per
// slice, per slice and 32 channels; megabytes; rounds of 64 channels.  (4000 drawn problems, 16 280 timings.  Where
// scale rows are long -- group 32 and K >= 20000 -- row streaming has no room for them in LDS: 4272 x 22272 group 32 W2 fp16 M = 23 65.7 -> 19.3 us.)
// [bits - 2][fp16, bf16]
static const double kPanelFit[3][2][8] = {
    {{3.6083, 1.4353, 2.1551, 2.0348, 0.1493, 0.0276, 0.1179, 0.5675},
     {3.5384, 1.9466, 3.3824, 2.0987, 0.1441, 0.0224, 0.1161, 0.2913}},  // 2 bits: fp16, bf16
    {{3.5524, 1.7773, 2.9189, 2.1189, 0.1416, 0.0153, 0.1005, 0.7544},
     {3.5495, 2.2876, 3.9926, 1.9464, 0.1736, 0.0000, 0.1017, 0.7374}},  // 3 bits: fp16, bf16
    {{3.8578, 0.9840, 1.6316, 2.0642, 0.1451, 0.0535, 0.0780, 0.0002},
     {4.0124, 1.1815, 1.9916, 1.8400, 0.1504, 0.0436, 0.0866, 0.3076}},  // 4 bits: fp16, bf16
};

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// kt K tiles; groups: scales per row; megabytes: packed weights and scales; side: row blocks side by side; ks: K slices (grid = shares x ks)
inline double rows_estimate_us(int bits, int64_t M, int64_t nb, int64_t kt, int64_t groups, double megabytes, int side, int grid, int nw, int ks, int cus) {
    const double* f = kRowsFit[bits - 2][M > 16];
    const int64_t shares = grid / ks;
    const double blocks = (double)ceil_div(nb, shares), passes = (double)ceil_div(ceil_div(nb, shares), side);
    const double rounds = (double)ceil_div(grid, cus), tiles = (double)ceil_div(ceil_div(kt, ks), nw);
    return rounds * (f[0] + f[1] * passes + (side == 8 ? f[2] * tiles * passes : 0.) + tiles * nw * (f[3] * passes + f[4] * blocks) + f[5] * blocks * nw +
                     f[9] * blocks * (double)groups * (16. * 2. / 1024.) * 8. / nw) +
           (ks > 1 ? f[6] + f[7] * blocks * ks : 0.) + f[8] * megabytes;
}

// r row blocks per wave, rs teams of nw / rs waves, `grid` workgroups; shared: the teams' activations go through LDS once
inline double teams_estimate_us(int bits, int64_t M, int64_t nb, int64_t kt, double megabytes, int r, int grid, int nw, int rs, bool shared, int cus) {
    static const double kMost[5] = {2., 4., 8., 16., 32.};
    const int c = M <= 2 ? 0 : M <= 4 ? 1 : M <= 8 ? 2 : M <= 16 ? 3 : 4;
    const double* f = kTeamsFit[bits - 2][c];
    const int64_t sets = nb / r / rs;
    const bool split = grid != sets;
    const double per = (double)ceil_div(grid, cus), ks = (double)(nw / rs);
    const double tiles = (double)ceil_div(split ? ceil_div(sets * kt, grid) : kt, nw / rs);
    const int64_t part = sets * kt / grid;               // K tiles of a workgroup
    const bool uneven = split && (part == 0 || sets * kt % grid != 0 || kt % part != 0);
    return f[0] + f[1] * per + f[2] * (double)ceil_div(ceil_div(grid, cus), 2) + f[3] * tiles * r + f[4] * per * tiles * nw * r +
           f[5] * per * tiles * (shared ? ks : (double)nw) * (double)M / kMost[c] + f[6] * nw * per +
           (split ? f[7] + f[8] * (double)grid / (double)sets : 0.) + (uneven ? f[9] : 0.) + f[10] * megabytes;
}

// rp: panel height / 32; a workgroup is two panels by four parts of K
inline double panel_estimate_us(int bits, bool bf16, int64_t nb, int64_t kt, double megabytes, int rp, int64_t ks, int cus) {
    const double* f = kPanelFit[bits - 2][bf16];
    const double rounds = (double)ceil_div(ceil_div(nb, 4 * rp) * ks, cus), tiles = (double)ceil_div(ceil_div(kt, ks), 4);
    return rounds * (f[0] + (rp == 1 ? f[1] * tiles : f[2] * tiles + f[7])) + (ks > 1 ? f[3] + (double)ks * (f[4] + f[5] * rp) : 0.) + f[6] * megabytes;
}

}  // namespace lutq
