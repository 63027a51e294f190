// GPU quantiser: dense weights -> table indices + group scales, written directly in the packed
// layout of lutq_pack.cpp (Section 3, first equation: Q = argmin_c |W/s - T[c]|; Section 4.1 "LUT
// quantization method" / Section 4.2: one absmax scale per group, stored in the 16-bit type; Section
// 3.1: the offline reordering, here fused into the same pass).
//
// Every decision is taken in fp64 on exactly representable inputs, so the result is a function of
// the inputs alone: the scale is the group's absmax rounded once (to nearest even) to the 16-bit
// type; u = W / scale is one IEEE fp64 division; the index is the first c that minimises the fp64
// value |u - T[c]|; a group whose scale is zero takes u = 0.
//
// The index is found without a division or a scan for all but a few weights.  |u| is at most 1 + 2^-9 wherever the scale is a
// normal number (it is the rounded absmax), so the range of u is cut into 512 cells, and a table in LDS says for each cell
// which index applies below and above the one decision threshold in it (the midpoint of two table entries that are neighbours by
// value; a cell without one has a threshold that no u reaches).  A weight takes u32 = w * rcp(scale) in fp32, one table read and
// one comparison.  u32, the threshold (whose low eight mantissa bits hold the two indices: off by at most 2^-17 below 1) and
// their difference are off by less than kNear together, so a weight whose u32 is kNear or further from its cell's threshold is
// decided as the fp64 rule decides it.  The others -- about one in eight thousand with a NormalFloat table of 16 entries -- and cells
// with more than one threshold go through the fp64 rule itself, lane by lane.  With subnormal fp16 scales |u| is up to 1.5, which the
// first and the last cell take in; groups with a bf16 scale beyond 2^-100 or 2^100 go through the fp64 rule.
// That the decision away from thresholds is the nearest entry by value, and the lowest of equal entries, needs that rounding
// never reorders the distances there.  fp16 entries: distances are below 2^17 and round by less than 2^-36, and two of them that differ by
// as little are those of a weight within 2^-36 of a threshold.  bf16: with one entry of magnitude up to 1000 the smallest distance is below
// 1002, an entry beyond 2100 in magnitude is never nearest, the others' distances are below 2^12 and round by less than 2^-41, and different
// ones among them have to be 2^-40 or more apart; any other table has no thresholds and every weight goes through the fp64 rule.
//
// What bounds it: the memory traffic, with the vector unit close behind (twelve instructions a weight).  The table is built
// per workgroup, so workgroups are few (two per compute unit) and large (eight wavefronts), each walking many units.
// 8192 x 28672 bf16 to 4 bits, group 64: 129 us, 4.6 TB/s (658 us with an fp64 division and a scan of the sixteen entries per
// weight); 28672 x 4096 fp32 to 4 bits fp16 189 -> 118 us (group 256: 113), fp16 200 -> 61;
// 1024 x 4096 bf16 17.7 -> 8.9.  An instance of more than 128 registers has one workgroup a compute unit instead of two, which costs
// medium sizes most (4096 x 4096 fp32, group 128: 21.3 -> 24.8 us); none has.
// Where the cells decide less (8192 x 8192 fp32 to 4 bits, us, with the fp64 division and -- sorted fp16 tables -- a binary search -> now):
// subnormal or infinite fp16 scales 113 -> 65, an fp16 table with all but two entries within some 1e-3 of zero 115 -> 70.  The scan of the
// table alone, lane by lane, is slower than it was: bf16 scales below 2^-100, a bf16 table without an entry below 1000 or with entries closer
// than 2^-40 194 -> 260 (3 bits 122 -> 187, 2 bits 88 -> 141).  A walk of its own for these, with the table in scalar registers, takes 202 to
// 236 and 87 to 122, but its registers and code cost every fp32 call 2 to 6 %.
//
// Work unit: 16 rows x UC columns, UC = max(K tile, group), one wavefront per unit.  Lane l = 16 o + i
// holds, for every 32-column step t of the unit, the 8 weights W[16 rb + i][col0 + 32 t + 8 o + j] --
// exactly the 8 indices whose packed bits this lane owns -- so the packed tile is written with one
// 128-bit store per lane (plus one 64-bit store for the 3-bit high slice) and needs no exchange; only
// the group maximum crosses lanes (the four lanes i, 16 + i, 32 + i, 48 + i share a row).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "lutq.h"
#include "lutq_layout.hpp"

namespace lutq {

struct QuantParams {
    const void* W;            // [N, K] fp32 or 16-bit
    const uint16_t* lut;      // 2^bits entries
    uint16_t* scales;         // [N, K / group]
    uint8_t* packed;
    int N, K, KT, SG, SB;     // KT = K / TK, SG = K / group, SB = row blocks per super-block
    int upr;                  // units per row block = K / UC
    int nb;                   // row blocks
    int drb, duc;             // stride of a wavefront: all wavefronts' units, as row blocks and units of a row block
    int bf16;                 // 16-bit type of lut, scales (and of W unless fp32)
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float widen16(uint32_t h, bool bf16) {
    if (bf16) return __builtin_bit_cast(float, h << 16);
    return (float)__builtin_bit_cast(_Float16, (uint16_t)h);
}

// fp32 (finite, >= 0) -> 16-bit pattern, round to nearest even
__device__ __forceinline__ uint32_t round16(float v, bool bf16) {
    if (bf16) {
        const uint32_t b = __builtin_bit_cast(uint32_t, v);
        return (b + 0x7fffu + ((b >> 16) & 1u)) >> 16;
    }
    return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)v);
}

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

constexpr int kQuantWaves = 8;
constexpr int kCells = 512, kCellCopies = 32;          // one 4-byte entry per lane pair (l, l + 32): every lane has its own bank
constexpr float kCellScale = 254.f;                    // cell = 256 + round(u * 254): 1 .. 511 for |u| <= 1 + 2^-9
constexpr float kNear = 8.2e-6f;                       // 2^-17 (threshold) + 2^-22 (u32) + 2^-24 (difference), rounded up

// The fp64 rule: the first entry that minimises |u - T[c]|.
template <int E>
__device__ __forceinline__ uint32_t nearest_entry(double u, const double* T) {
    double best = __builtin_fabs(u - T[0]);
    uint32_t arg = 0;
#pragma unroll
    for (int c = 1; c < E; ++c) {
        const double d = __builtin_fabs(u - T[c]);
        const bool less = d < best;
        best = less ? d : best;
        arg = less ? (uint32_t)c : arg;
    }
    return arg;
}

// Entry of one cell: threshold with the index below it in bits 0..3 and the index above it in bits 4..7; a quiet NaN where the
// cell cannot be decided by one threshold below 1.
template <int E>
__device__ __forceinline__ uint32_t cell_entry(int cell, const double* T) {
    // (the margin covers how far u is from the value the cell was chosen with)
    const double centre = (double)(cell - 256) / (double)kCellScale, half = 0.5 / (double)kCellScale + 2e-5;
    // (the first and the last cell are also those of the weights beyond the cells: |u| is up to 1.5 with the smallest fp16 scales)
    const uint32_t below = nearest_entry<E>(cell == 0 ? -2.0 : centre - half, T);
    const uint32_t above = nearest_entry<E>(cell == kCells - 1 ? 2.0 : centre + half, T);
    const uint32_t code = below | (above << 4);
    if (below == above) return 0x7f000000u | code;
    const double mid = 0.5 * (T[below] + T[above]);
    const uint32_t at = nearest_entry<E>(mid, T);      // a third entry between the two would be nearest to their midpoint
    if ((at != below && at != above) || !(__builtin_fabs(mid) < 1.0)) return 0x7fc00000u | code;
    // the float nearest to the midpoint among those with these low bits (rounding in magnitude; stays below 1 + 2^-16)
    const uint32_t m = __builtin_bit_cast(uint32_t, (float)mid);
    return m + 128u < code ? code : ((m + 128u - code) & 0xffffff00u) + code;    // (a midpoint of zero: the smallest denormals)
}

// WT: how W is held: 0 fp32, 1 fp16, 2 bf16 (the latter two are also the type of the table and the scales)
template <int BITS, int GROUP, int WT>
__global__ __launch_bounds__(64 * kQuantWaves) void quantize_kernel(const QuantParams p) {
    constexpr int TK = BITS == 4 ? 128 : 256;
    constexpr int TILE_BYTES = BITS == 3 ? 1536 : 1024;
    constexpr int UC = GROUP > TK ? GROUP : TK;       // columns of one unit
    constexpr int NSTEP = UC / 32;                    // 32-column steps of one unit
    constexpr int STEPS = TK / 32;                    // steps of one tile
    constexpr int SPG = GROUP / 32;                   // steps of one group
    constexpr int NG = UC / GROUP;                    // groups of one unit (per row)
    constexpr int E = 1 << BITS;
    constexpr bool WF32 = WT == 0;
    const bool bf16 = WF32 ? p.bf16 != 0 : WT == 2;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int i = lane & 15, o = lane >> 4;

    extern __shared__ __align__(16) char smem[];      // [cells][Ts]
    double* Ts = reinterpret_cast<double*>(smem + kCells * kCellCopies * 4);
    if (threadIdx.x < E) Ts[threadIdx.x] = (double)widen16(p.lut[threadIdx.x], bf16);
    __syncthreads();
    bool close = false, small = false;                // one pair of entries per thread
    if (threadIdx.x < E * E) {
        const double a = Ts[threadIdx.x / E], b = Ts[threadIdx.x % E];
        small = __builtin_fabs(a) <= 1000.0;
        close = __builtin_fabs(a) <= 2100.0 && __builtin_fabs(b) <= 2100.0 && a != b && __builtin_fabs(a - b) < 0x1p-40;
    }
    const bool thresholds = __syncthreads_or(close) == 0 && (__syncthreads_or(small) != 0 || !bf16);
    for (int cell = threadIdx.x; cell < kCells; cell += 64 * kQuantWaves) {
        const uint32_t v = thresholds ? cell_entry<E>(cell, Ts) : 0x7fc00000u;
#pragma unroll 1
        for (int k = 0; k < kCellCopies / 4; ++k)     // (skewed, so that the lanes of one store hit different banks)
            *reinterpret_cast<u32x4*>(smem + cell * (kCellCopies * 4) + 16 * ((k + cell) & (kCellCopies / 4 - 1))) = u32x4{v, v, v, v};
    }
    __syncthreads();
    // u32 * 254 + 2^23 + 256 holds the cell in its low bits; shifted by 7 its exponent leaves 2^31, taken off with the lane's offset
    const uint32_t cell_lane = (uint32_t)(lane & (kCellCopies - 1)) * 4u - (0x4b000000u << 7);
    typedef __attribute__((address_space(3))) const uint32_t lds_cu32;
    const uint32_t cells = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)smem;

    // unit = row block x p.upr + unit of the row block; a stride of p.drb row blocks and p.duc units
    const int first = (int)blockIdx.x * kQuantWaves + wave;
    int rb = first / p.upr, uc = first % p.upr;
    for (; rb < p.nb; rb += p.drb, uc += p.duc, rb += uc >= p.upr ? 1 : 0, uc -= uc >= p.upr ? p.upr : 0) {
        const long long row = 16ll * rb + i;
        const int col0 = uc * UC;
        const long long e0 = row * p.K + col0 + 8 * o;
        u32x4 raw[NSTEP][WF32 ? 2 : 1];
        // (plain loads: a row's 128-byte lines are read by two instructions, and with non-temporal ones 138 us instead of 129)
#pragma unroll
        for (int t = 0; t < NSTEP; ++t) {
            const char* src = static_cast<const char*>(p.W) + (e0 + 32 * t) * (WF32 ? 4 : 2);
#pragma unroll
            for (int k = 0; k < (WF32 ? 2 : 1); ++k) raw[t][k] = *reinterpret_cast<const u32x4*>(src + 16 * k);
        }
        auto weight = [&](int t, int j) -> float {
            if constexpr (WF32) {
                const uint32_t v = raw[t][j / 4][j % 4];
                return __builtin_bit_cast(float, v);
            } else return widen16((j & 1) ? raw[t][0][j / 2] >> 16 : raw[t][0][j / 2] & 0xffffu, WT == 2);
        };
        // group maxima of |w| on the bit patterns (non-negative floats order like unsigned integers)
        uint32_t sbits[NG];
        float s[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            uint32_t m = 0;
            if constexpr (WF32) {
#pragma unroll
                for (int t = g * SPG; t < (g + 1) * SPG; ++t)
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const uint32_t v = raw[t][j / 4][j % 4] & 0x7fffffffu;
                        m = v > m ? v : m;
                    }
            } else {
                u16x2 m2 = u16x2{0, 0};
#pragma unroll
                for (int t = g * SPG; t < (g + 1) * SPG; ++t)
#pragma unroll
                    for (int j = 0; j < 4; ++j) m2 = __builtin_elementwise_max(m2, __builtin_bit_cast(u16x2, raw[t][0][j] & 0x7fff7fffu));
                const uint16_t h = m2.x > m2.y ? m2.x : m2.y;
                m = __builtin_bit_cast(uint32_t, widen16(h, WT == 2));
            }
            const uint32_t m1 = (uint32_t)__shfl_xor((int)m, 16);
            m = m1 > m ? m1 : m;
            const uint32_t m2 = (uint32_t)__shfl_xor((int)m, 32);
            m = m2 > m ? m2 : m;
            sbits[g] = round16(__builtin_bit_cast(float, m), bf16);
            s[g] = widen16(sbits[g], bf16);
        }
        if (o == 0) {
            uint16_t* dst = p.scales + row * p.SG + (long long)uc * NG;
#pragma unroll
            for (int g = 0; g < NG; ++g) dst[g] = (uint16_t)sbits[g];
        }
        // the 8 indices of step t of this lane, 4 bits apart; `limited`: cells outside the table, and NaN, become one inside it
        auto step_indices = [&](int t, auto limited) -> uint32_t {
            const float sg = s[t / SPG];
            // a scale that is zero or infinite makes u = 0 (of a finite weight)
            const bool ordinary = decltype(limited)::value ? sg >= (bf16 ? 0x1p-100f : 0x1p-24f) && sg <= 0x1p+100f : sg != 0.f;
            const float inv = ordinary ? __builtin_amdgcn_rcpf(sg) : 0.f;
            const float near = !decltype(limited)::value || ordinary || sg == 0.f || sg == __builtin_inff() ? kNear : __builtin_inff();
            const float to_cell = inv * kCellScale;
            uint32_t word = 0, open = 0;              // open: bit 7 - j set where weight j is not decided
            uint32_t ent[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                float cell = __builtin_fmaf(weight(t, j), to_cell, 0x1p+23f + 256.f);
                if constexpr (decltype(limited)::value) cell = __builtin_amdgcn_fmed3f(cell, 0x1p+23f, 0x1p+23f + (kCells - 1));
                ent[j] = *reinterpret_cast<lds_cu32*>((uintptr_t)((__builtin_bit_cast(uint32_t, cell) << 7) + cell_lane + cells));
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float d = weight(t, j) * inv - __builtin_bit_cast(float, ent[j]);
                const uint32_t code = d > 0.f ? ent[j] >> 4 : ent[j];
                word = __builtin_amdgcn_alignbit(code, word, 4);
                open = 2u * open + (__builtin_fabsf(d) >= near ? 0u : 1u);
            }
            while (open) {                            // (a lane at a time in effect: rare)
                const int j = __builtin_clz(open) - 24;
                open &= ~(128u >> j);
                float w;
                if constexpr (WF32) {
                    uint32_t v = raw[t][0].x;
#pragma unroll
                    for (int k = 1; k < 8; ++k) {
                        const uint32_t x = raw[t][k / 4][k % 4];
                        v = j == k ? x : v;
                    }
                    w = __builtin_bit_cast(float, v);
                } else {
                    uint32_t v = raw[t][0].x;
#pragma unroll
                    for (int k = 1; k < 4; ++k) {
                        const uint32_t x = raw[t][0][k];
                        v = (j >> 1) == k ? x : v;
                    }
                    w = widen16((j & 1) ? v >> 16 : v & 0xffffu, WT == 2);
                }
                const double u = sg == 0.f ? 0.0 : (double)w / (double)sg;
                word = (word & ~(15u << (4 * j))) | (nearest_entry<E>(u, Ts) << (4 * j));
            }
            return word;
        };
        // The cell of a weight is an LDS address, and only a group whose scale is zero or an ordinary number is sure to keep it inside
        // the table (a weight that is not finite makes its group's scale one that is not, or a zero with a sign): any other takes the
        // limits, in a copy of the code, since they cost 1 to 3 % of a call.  Where both copies would need more than 128 registers (the
        // largest fp32 unit: 134 against 126) only the one with the limits is built: 4096 x 4096 takes 22.2 us with it, 25.1 with both.
        constexpr bool always_limited = WF32 && BITS == 4 && GROUP == 256;
        uint32_t most = 0, least = 0xffffffffu;       // (of the scales' patterns; a zero counts as the largest for the least)
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            most = sbits[g] > most ? sbits[g] : most;
            least = sbits[g] - 1u < least ? sbits[g] - 1u : least;
        }
        const bool odd = most > (bf16 ? 0x7180u : 0x7bffu) || least < (bf16 ? 0x0d80u : 0x0400u) - 1u;
        uint32_t idx[NSTEP];
        if (!always_limited && __ballot(odd) == 0) {
#pragma unroll
            for (int t = 0; t < NSTEP; ++t) idx[t] = step_indices(t, std::false_type{});
        } else {
#pragma unroll
            for (int t = 0; t < NSTEP; ++t) idx[t] = step_indices(t, std::true_type{});
        }
        // packed tiles of the unit
#pragma unroll
        for (int tt = 0; tt < UC / TK; ++tt) {
            const int kt = col0 / TK + tt;
            const long long tile = ((long long)(rb / p.SB) * p.KT + kt) * p.SB + rb % p.SB;
            uint8_t* base = p.packed + tile * TILE_BYTES;
            const uint32_t* x = idx + tt * STEPS;
            if constexpr (BITS == 4) {
                *reinterpret_cast<u32x4*>(base + 16 * lane) = u32x4{x[0], x[1], x[2], x[3]};
            } else if constexpr (BITS == 2) {
                u32x4 out;
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    uint32_t v = 0;
#pragma unroll
                    for (int e = 0; e < 16; ++e) v |= ((x[2 * d + e / 8] >> (4 * (e % 8))) & 3u) << (2 * e);
                    out[d] = v;
                }
                *reinterpret_cast<u32x4*>(base + 16 * lane) = out;
            } else {
                u32x4 lo;
                u32x2 hi;
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    uint32_t v = 0;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {                 // byte q: indices 2q, 2q+1 of steps 2d, 2d+1
                        const uint32_t a0 = (x[2 * d] >> (8 * q)) & 3u, a1 = (x[2 * d] >> (8 * q + 4)) & 3u;
                        const uint32_t b0 = (x[2 * d + 1] >> (8 * q)) & 3u, b1 = (x[2 * d + 1] >> (8 * q + 4)) & 3u;
                        v |= (a0 | (a1 << 2) | (b0 << 4) | (b1 << 6)) << (8 * q);
                    }
                    lo[d] = v;
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    uint32_t v = 0;
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const uint32_t a = (x[4 * h + u] >> (8 * q + 2)) & 1u, b = (x[4 * h + u] >> (8 * q + 6)) & 1u;
                            v |= (a << (2 * u) | b << (2 * u + 1)) << (8 * q);
                        }
                    hi[h] = v;
                }
                *reinterpret_cast<u32x4*>(base + 16 * lane) = lo;
                *reinterpret_cast<u32x2*>(base + 1024 + 8 * lane) = hi;
            }
        }
    }
}

namespace {

template <int BITS, int GROUP>
hipError_t launch_q(bool wf32, const QuantParams& p, int grid, hipStream_t stream) {
    auto kernel = wf32 ? quantize_kernel<BITS, GROUP, 0> : p.bf16 ? quantize_kernel<BITS, GROUP, 2> : quantize_kernel<BITS, GROUP, 1>;
    constexpr int lds_bytes = kCells * kCellCopies * 4 + (1 << BITS) * 8;
    // more than 64 KiB of dynamic LDS has to be enabled once per kernel
    static const hipError_t attr = [] {
        for (auto k : {quantize_kernel<BITS, GROUP, 0>, quantize_kernel<BITS, GROUP, 1>, quantize_kernel<BITS, GROUP, 2>}) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, kCells * kCellCopies * 4 + (1 << BITS) * 8);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }();
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(64 * kQuantWaves), lds_bytes, stream, p);
    return hipGetLastError();
}

template <int BITS>
hipError_t launch_qb(int group, bool wf32, const QuantParams& p, int grid, hipStream_t stream) {
    switch (group) {
        case 32: return launch_q<BITS, 32>(wf32, p, grid, stream);
        case 64: return launch_q<BITS, 64>(wf32, p, grid, stream);
        case 128: return launch_q<BITS, 128>(wf32, p, grid, stream);
        case 256: return launch_q<BITS, 256>(wf32, p, grid, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace
}  // namespace lutq

extern "C" lutq_status lutq_quantize(const void* W, int w_is_f32, const void* lut, int bits, int group_size,
                                     int64_t N, int64_t K, lutq_dtype dtype, void* scales_out, void* packed_out,
                                     void* stream) {
    if (!W || !lut || !scales_out || !packed_out) return LUTQ_ERR_NULL;
    if (lutq_packed_bytes(N, K, bits, group_size) == 0) {
        if (bits < 2 || bits > 4) return LUTQ_ERR_BITS;
        if ((group_size != 32 && group_size != 64 && group_size != 128 && group_size != 256) ||
            (K > 0 && K % group_size != 0))
            return LUTQ_ERR_GROUP;
        return LUTQ_ERR_SHAPE;
    }
    if (dtype != LUTQ_F16 && dtype != LUTQ_BF16) return LUTQ_ERR_DTYPE;
    if (N > (1 << 24) || K > (1 << 24)) return LUTQ_ERR_SHAPE;
    auto aligned16 = [](const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15u) == 0; };
    if (!aligned16(W) || !aligned16(packed_out) || (reinterpret_cast<uintptr_t>(scales_out) & 1u) ||
        (reinterpret_cast<uintptr_t>(lut) & 1u))
        return LUTQ_ERR_ALIGN;
    const int tk = lutq::layout::tile_k(bits);
    const int uc = group_size > tk ? group_size : tk;
    const int64_t nb = N / 16;
    lutq::QuantParams p;
    p.W = W;
    p.lut = static_cast<const uint16_t*>(lut);
    p.scales = static_cast<uint16_t*>(scales_out);
    p.packed = static_cast<uint8_t*>(packed_out);
    p.N = (int)N; p.K = (int)K;
    p.KT = (int)(K / tk);
    p.SG = (int)(K / group_size);
    p.SB = lutq::layout::super_block(nb);
    p.upr = (int)(K / uc);
    const int64_t units = nb * (K / uc);
    p.nb = (int)nb;
    p.bf16 = dtype == LUTQ_BF16;
    // two workgroups (their tables fill the LDS) per compute unit; more would only build more tables
    const int cus = lutq::compute_units();
    if (cus < 1) return LUTQ_ERR_DEVICE;
    int64_t grid = (units + lutq::kQuantWaves - 1) / lutq::kQuantWaves;
    if (grid > 2 * (int64_t)cus) grid = 2 * (int64_t)cus;
    p.drb = (int)(grid * lutq::kQuantWaves / p.upr);
    p.duc = (int)(grid * lutq::kQuantWaves % p.upr);
    const hipStream_t s = static_cast<hipStream_t>(stream);
    const hipError_t e = bits == 2 ? lutq::launch_qb<2>(group_size, w_is_f32 != 0, p, (int)grid, s)
                       : bits == 3 ? lutq::launch_qb<3>(group_size, w_is_f32 != 0, p, (int)grid, s)
                                   : lutq::launch_qb<4>(group_size, w_is_f32 != 0, p, (int)grid, s);
    return e == hipSuccess ? LUTQ_OK : LUTQ_ERR_DEVICE;
}
