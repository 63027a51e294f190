// Estimated times of the launches that a call of up to 32 rows can take (host code; lutq_api.hip chooses by them).
//
// Why estimates: the rules of default_decomp, default_rows_decomp and sliced_rows_decomp were each measured on some twenty
// shapes, and hold there (within 4 % of the best plan found).  On 5871 drawn problems of 5..32 rows (1024 to 57344 channels in
// units of 16, K 1024 to 28672, all bit widths, groups and types) they took 20.5 % longer than the best of about 23 plans timed,
// up to 3 times (7024 x 26624 group 256, W4 fp16, M = 31: 97.4 us, row streaming in K slices 32.9); on 5603 of 1..4 rows 5.7 %.
// Fitted by least squares of the relative error to 91 900 and 78 000 timings (HBM-cold weights, MI355X); the estimates are off by
// 7 to 16 %.  On the half of the problems that was not fitted to, the plan chosen takes 2.9 % longer than the best one timed (14.7 %
// less than the rules'), with 3 % of the problems more than 3 % slower than under the rules.
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
// R; the same without R (activations; once per K part where they are shared); waves per unit; partial sums across workgroups; megabytes.
// [bits - 2][1..2, 3..4, 5..8, 9..16, 17..32 rows]
static const double kTeamsFit[3][5][9] = {
    {{1.6409, 0.0654, 1.4913, 0.1391, 0.0414, 0.0000, 0.0244, 5.2359, 0.1070},
     {1.9096, 0.0743, 1.2368, 0.1239, 0.0456, 0.0007, 0.0350, 5.0144, 0.1273},
     {2.0780, 0.2659, 1.0915, 0.1107, 0.0492, 0.0248, 0.0188, 5.2675, 0.0996},
     {2.4407, 0.8836, 0.0000, 0.0687, 0.0453, 0.1079, 0.0403, 6.4777, 0.0974},
     {2.5104, 1.1028, 0.0000, 0.0464, 0.0618, 0.2342, 0.0551, 5.4605, 0.1705}},  // 2 bits
    {{2.3574, 0.0000, 0.3799, 0.1997, 0.0537, 0.0000, 0.0586, 5.1606, 0.0854},
     {2.5379, 0.0000, 0.2058, 0.1476, 0.0642, 0.0000, 0.0669, 5.2634, 0.0955},
     {2.9110, 0.0000, 0.3815, 0.0894, 0.0766, 0.0009, 0.0424, 5.3716, 0.1165},
     {2.4949, 0.5909, 0.0000, 0.0922, 0.0689, 0.0822, 0.0750, 6.3849, 0.1122},
     {2.2451, 0.9636, 0.1101, 0.0626, 0.1058, 0.2136, 0.0596, 5.5085, 0.0807}},  // 3 bits
    {{1.5471, 0.0423, 1.6155, 0.1086, 0.0260, 0.0044, 0.0022, 5.3370, 0.0711},
     {1.6524, 0.0423, 1.4947, 0.0915, 0.0291, 0.0064, 0.0057, 5.1905, 0.0743},
     {1.9126, 0.0000, 1.3596, 0.0645, 0.0370, 0.0163, 0.0000, 5.4496, 0.0561},
     {2.4709, 0.0000, 0.7909, 0.0061, 0.0453, 0.0489, 0.0000, 5.4751, 0.0485},
     {2.8904, 0.5873, 0.0000, 0.0096, 0.0410, 0.1313, 0.0000, 5.6291, 0.0558}},  // 4 bits
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
    const double* f = kTeamsFit[bits - 2][M <= 2 ? 0 : M <= 4 ? 1 : M <= 8 ? 2 : M <= 16 ? 3 : 4];
    const int64_t sets = nb / r / rs;
    const bool split = grid != sets;
    const double per = (double)ceil_div(grid, cus), ks = (double)(nw / rs);
    const double tiles = (double)ceil_div(split ? ceil_div(sets * kt, grid) : kt, nw / rs);
    return f[0] + f[1] * per + f[2] * (double)ceil_div(ceil_div(grid, cus), 2) + f[3] * tiles * r + f[4] * per * tiles * nw * r +
           f[5] * per * tiles * (shared ? ks : (double)nw) + f[6] * nw * per + (split ? f[7] : 0.) + f[8] * megabytes;
}

}  // namespace lutq
