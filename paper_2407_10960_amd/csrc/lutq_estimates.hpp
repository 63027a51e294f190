// Estimated times of the launches that a call of up to 32 rows can take (host code; lutq_api.hip chooses by them).
//
// Why estimates: the rules of default_decomp, default_rows_decomp and sliced_rows_decomp were each measured on some twenty
// shapes, and hold there (within 4 % of the best plan found).  On 5871 drawn problems of 5..32 rows (1024 to 57344 channels in
// units of 16, K 1024 to 28672, all bit widths, groups and types) they took 20.5 % longer than the best of about 23 plans timed,
// up to 3 times (7024 x 26624 group 256, W4 fp16, M = 31: 97.4 us, row streaming in K slices 32.9); on 5603 of 1..4 rows 5.7 %.
// Fitted by least squares of the relative error to 91 900 and 78 000 timings (HBM-cold weights, MI355X); the estimates are off by
// 7 to 16 %.  On the half of the problems of 5..32 rows that was not fitted to, the plan chosen (with the margins of lutq_api.hip) takes 14 % less
// than the rules', with 0.8 % of the problems more than 3 % slower and 0.14 % more than 10 %.
#pragma once

#include <stdint.h>

namespace lutq {

// Row streaming: rounds of workgroups; times passes; times K tiles of a wave and passes (eight side by side), the same times waves;
// K tiles of a wave, waves and row blocks; row blocks times waves (reduction); K slices; row blocks times slices; megabytes.
// [bits - 2][up to 16 rows, beyond]
static const double kRowsFit[3][2][9] = {
    {{2.1749, 1.8494, 0.7713, 0.1094, 0.0167, 0.0000, 2.3523, 0.0310, 0.1612},
     {3.0864, 0.5261, 0.5102, 0.2029, 0.0263, 0.0543, 1.5806, 0.0345, 0.1863}},  // 2 bits
    {{1.9588, 2.2526, 0.9424, 0.1253, 0.0250, 0.0000, 2.1700, 0.0280, 0.1293},
     {2.2244, 2.4819, 0.0000, 0.2276, 0.0246, 0.0009, 2.1087, 0.0490, 0.1830}},  // 3 bits
    {{2.2266, 1.8116, 0.8406, 0.0810, 0.0077, 0.0000, 2.0510, 0.0277, 0.0976},
     {3.2231, 0.0000, 0.7073, 0.1668, 0.0090, 0.0497, 1.6573, 0.0367, 0.1003}},  // 4 bits
};
// Teams: fixed; workgroups per compute unit; pairs of them; K tiles of a wave times R; K tiles of a wave, waves, workgroups per unit and
// R; the same without R (activations: once per K part where they are shared, by the share of the class's rows); waves per unit; partial sums across workgroups; megabytes.
// [bits - 2][1..2, 3..4, 5..8, 9..16, 17..32 rows]
static const double kTeamsFit[3][5][9] = {
    {{1.6409, 0.0654, 1.4913, 0.1391, 0.0414, 0.0000, 0.0244, 5.2359, 0.1070},
     {1.8954, 0.0712, 1.2359, 0.1263, 0.0441, 0.0046, 0.0342, 5.0205, 0.1237},
     {2.1169, 0.2716, 1.0189, 0.1114, 0.0462, 0.0427, 0.0148, 5.2647, 0.0894},
     {2.3578, 0.9090, 0.0000, 0.0738, 0.0440, 0.1493, 0.0412, 6.4583, 0.0916},
     {2.5721, 1.1437, 0.0318, 0.0536, 0.0611, 0.3182, 0.0422, 5.4064, 0.1625}},  // 2 bits
    {{2.3574, 0.0000, 0.3799, 0.1997, 0.0537, 0.0000, 0.0586, 5.1606, 0.0854},
     {2.5379, 0.0000, 0.2058, 0.1476, 0.0642, 0.0000, 0.0669, 5.2634, 0.0955},
     {2.8459, 0.0000, 0.3825, 0.1002, 0.0707, 0.0179, 0.0379, 5.4114, 0.1036},
     {2.5230, 0.5696, 0.0000, 0.0872, 0.0674, 0.1206, 0.0700, 6.3827, 0.1022},
     {2.1240, 0.7204, 0.5162, 0.0553, 0.1022, 0.3028, 0.0537, 5.5270, 0.0800}},  // 3 bits
    {{1.5489, 0.0440, 1.6252, 0.1075, 0.0267, 0.0043, 0.0024, 5.3358, 0.0724},
     {1.6439, 0.0389, 1.4969, 0.0923, 0.0286, 0.0086, 0.0057, 5.1918, 0.0730},
     {1.9103, 0.0000, 1.3233, 0.0651, 0.0364, 0.0237, 0.0000, 5.4417, 0.0533},
     {2.5424, 0.0000, 0.7121, 0.0038, 0.0446, 0.0690, 0.0000, 5.4326, 0.0451},
     {2.8315, 0.6381, 0.0000, 0.0000, 0.0425, 0.1783, 0.0000, 5.6294, 0.0525}},  // 4 bits
};

// Panels of 17..32 rows (one block of 32): rounds of workgroups; rounds times K tiles of a wavefront, 32 and 64 channels; K slices: fixed, per
// slice, per slice and 32 channels; megabytes; rounds of 64 channels.  (4241 drawn problems, 20 000 timings; 5 to 7 % off.  Where
// scale rows are long -- group 32 and K >= 20000 -- row streaming has no room for them in LDS: 4272 x 22272 group 32 W2 fp16 M = 23 65.7 -> 19.3 us.)
// [bits - 2][fp16, bf16]
static const double kPanelFit[3][2][8] = {
    {{3.4259, 1.5523, 2.3415, 2.1674, 0.1105, 0.0710, 0.0794, 0.5328},
     {3.2026, 2.1303, 3.5668, 2.1872, 0.1366, 0.0533, 0.0966, 0.4059}},  // 2 bits: fp16, bf16
    {{3.3496, 1.9388, 3.2046, 2.1605, 0.1118, 0.0620, 0.0755, 0.7623},
     {3.4298, 2.4676, 4.2472, 1.9216, 0.1600, 0.0329, 0.0879, 0.8455}},  // 3 bits: fp16, bf16
    {{3.5020, 1.0709, 1.7295, 2.0795, 0.1202, 0.0760, 0.0700, 0.4264},
     {3.5226, 1.3007, 2.1226, 2.0311, 0.1346, 0.0687, 0.0752, 0.5778}},  // 4 bits: fp16, bf16
};

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// kt K tiles; megabytes: packed weights and scales; side: row blocks side by side; ks: K slices (grid = shares x ks)
inline double rows_estimate_us(int bits, int64_t M, int64_t nb, int64_t kt, double megabytes, int side, int grid, int nw, int ks, int cus) {
    const double* f = kRowsFit[bits - 2][M > 16];
    const int64_t shares = grid / ks;
    const double blocks = (double)ceil_div(nb, shares), passes = (double)ceil_div(ceil_div(nb, shares), side);
    const double rounds = (double)ceil_div(grid, cus), tiles = (double)ceil_div(ceil_div(kt, ks), nw);
    return rounds * (f[0] + f[1] * passes + (side == 8 ? f[2] * tiles * passes : 0.) + tiles * nw * (f[3] * passes + f[4] * blocks) + f[5] * blocks * nw) +
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
    return f[0] + f[1] * per + f[2] * (double)ceil_div(ceil_div(grid, cus), 2) + f[3] * tiles * r + f[4] * per * tiles * nw * r +
           f[5] * per * tiles * (shared ? ks : (double)nw) * (double)M / kMost[c] + f[6] * nw * per + (split ? f[7] : 0.) + f[8] * megabytes;
}

// rp: panel height / 32; a workgroup is two panels by four parts of K
inline double panel_estimate_us(int bits, bool bf16, int64_t nb, int64_t kt, double megabytes, int rp, int64_t ks, int cus) {
    const double* f = kPanelFit[bits - 2][bf16];
    const double rounds = (double)ceil_div(ceil_div(nb, 4 * rp) * ks, cus), tiles = (double)ceil_div(ceil_div(kt, ks), 4);
    return rounds * (f[0] + (rp == 1 ? f[1] * tiles : f[2] * tiles + f[7])) + (ks > 1 ? f[3] + (double)ks * (f[4] + f[5] * rp) : 0.) + f[6] * megabytes;
}

}  // namespace lutq
