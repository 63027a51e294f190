// The fused kernel for 33 to 128 activation rows, in one pass over the weights; also for 17 to 32 where estimated to be the fastest.
//
// What is computed is that of matmul_kernel (Algorithm 1 of the paper).  From some forty rows up the matrix instructions
// take longer than the weight stream (8B gate+up at M = 128: 30 GFLOP, 12 us at 2.5 PFLOP/s, against 58.7 MB of weights),
// so this kernel is laid out like a matrix product whose A operand is dequantised on the way in:
//
//   * A wavefront owns a panel of 32 RP output channels x 32 MB activation rows (all of them, or where the matrix is small a part
//     of M per workgroup) and dequantises every weight of it exactly once; the workgroup is two panels side by side (WN) times four parts of K (WK).
//   * Matrix instruction 32x32x16.  The packed tile is in the operand order of the 16x16x32 one (lane 16 o + i = row i, K
//     octet o), so two row blocks' words are exchanged once per tile: v_permlane16_swap turns (block 0, block 1) into octets
//     {0, 2} of both blocks and octets {1, 3} of both blocks, which are A operands of two 32x32x16 instructions (K inside
//     an instruction may be permuted as long as B agrees).  One instruction per word, and every B operand read from LDS then
//     feeds twice the multiplications of a 16x16x32.
//   * Activations go through LDS, in chunks of KC columns per K part, double buffered, shared by the two panels, whose
//     wavefronts keep in step through two words in LDS (no barrier in the K loop).  A lane fetches 16 bytes of one row; its place inside the row's 2 KC bytes is permuted by the row
//     number (swz), so that global reads are whole 64- or 128-byte pieces of rows, the LDS writes are contiguous and the
//     operand reads (32 rows, one octet each) hit all banks evenly.
//   * The tables hold 16-bit pairs at every type: bf16 pairs are widened in registers, since LDS (operands, lookups) and not
//     the vector unit is what the matrix instructions wait for here.
//   * What bounds it: no unit is full.  8B gate+up, M = 128, W4 fp16, 41 us (two slices of 64 rows on the row-streaming kernel took
//     65.0; the dense fp16 product of the same shape 56).  The matrix instructions alone take 21 us of it on 224 compute units (1.66 PFLOP/s is what
//     32x32x16 reaches here), launch, table and reduction 6.  Counters: matrix units busy 45 %
//     of a compute unit's time, LDS 47 %, vector units 30 %; a wavefront issues 34 % of its time, waits at s_waitcnt 30 % and to issue
//     36 % (before the waits below were taken out 42, 42, 27; 31, 37, 32).  The waits that could be taken out (scales behind a branch, one loop for both looks at the partner's words) gave 3-8 %.  What did not:
//     operands two units ahead and two sets of table values (M = 64 27 -> 28 us), deeper activation and weight prefetch (0.96-1.0), K ranges walked from a
//     different start per workgroup, issue priority for the wavefront that is behind.
//   * K parts are added in order through LDS at the end.  Where panels are too few to fill the chip, K is also cut into KS
//     slices across workgroups: partial sums go to global slots, one arrival counter per (share, wavefront), and whichever
//     slice's wavefront arrives last adds the slots in slice order (the protocol of matmul_kernel's fix-up: nobody waits).
#pragma once

#include <type_traits>

#include "lutq_matmul_kernel.hpp"

namespace lutq {

// bf16 with 16-bit table entries
struct BF16P {};
template <> struct ScaleReg<BF16P> { float s; };
template <> __device__ __forceinline__ ScaleReg<BF16P> make_scale<BF16P>(uint32_t w, int hi) {
    ScaleReg<BF16P> r; r.s = __builtin_bit_cast(float, hi ? (w & 0xffff0000u) : (w << 16)); return r;
}
__device__ __forceinline__ uint32_t scale_pair(uint32_t pair, ScaleReg<BF16P> s) {
    ScaleReg<BF16> t; t.s = s.s;
    return scale_pair(pair, t);
}

template <typename DT> struct PanelType { typedef DT type; };
template <> struct PanelType<BF16> { typedef BF16P type; };

typedef float f32x16 __attribute__((ext_vector_type(16)));

// v_mfma_f32_32x32x16: lane 32 h + i supplies A[i][8h..8h+7] and B[8h..8h+7][i]; register 4 j + k of lane 32 h + i
// receives D[8 j + 4 h + k][i].
template <typename DT> __device__ __forceinline__ f32x16 mfma32x32x16(u32x4 a, u32x4 b, f32x16 c);
template <> __device__ __forceinline__ f32x16 mfma32x32x16<F16>(u32x4 a, u32x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
template <> __device__ __forceinline__ f32x16 mfma32x32x16<BF16>(u32x4 a, u32x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

struct PanelParams {
    const uint16_t* X;        // [M, K]
    const uint8_t* packed;
    const uint16_t* scales;   // [N, SG]
    const uint16_t* lut;
    uint16_t* Y;              // [M, N]
    uint32_t packed_bytes, scale_bytes, x_bytes;
    int M, N, K;
    int NB;                   // row blocks (N / 16)
    int SG2;                  // bytes of one row of scales
    int SBL;                  // log2 of the row blocks per super-block of the packed layout
    uint32_t tile_stride;     // packed bytes from K tile kt to kt + 1 of one row block
    uint32_t sblock_bytes;    // packed bytes of one super-block
    int G;                    // workgroups = parts of M (32 MB rows each) x shares x KS
    int shares;               // shares of the output channels, 64 RP each
    int KS;                   // K slices: workgroup b works on slice b % KS of share (b / KS) % shares of M part b / KS / shares
    int TS, KSB;              // K tiles per slice; the first KSB slices have one more
    int lut_ltpe;
    float* slots;             // KS > 1: partial sums, one slot of RP x MB x 8 KiB per workgroup
    uint32_t slot_bytes;      // ... of all workgroups
    uint32_t* counters;       // KS > 1: arrivals, eight per share and M part (one 64-byte line); zero between launches
};

constexpr int kAuxDevice = 16;   // sc1: past the compute unit's and the die's own caches, what agent-scope atomic accesses use
constexpr int kPanelPark = 2048;      // LDS bytes per wavefront for parked scales: 64 rows' eight scales, and as much that is never read
constexpr int kPanelQuarter = 1088;   // LDS bytes from one parked quarter tile to the next
constexpr int kPanelWN = 2, kPanelWK = 4, kPanelWaves = kPanelWN * kPanelWK;
// columns of K per activation chunk
__host__ __device__ constexpr int panel_kc(int mb) { return mb <= 2 ? 64 : 32; }
// chunks of activations held in registers on their way to LDS, ahead of the one being written, and K tiles of weights in flight.
// (4 bits, 33..64 rows: one and two measured faster than two and four, 8B gate+up M = 64 29.2 -> 27.6 us, 70B down 52.7 -> 50.9; 128 rows
// by 64 channels leave registers for one chunk and two tiles only; with 32 rows four tiles are 2 % faster than two.)
__host__ __device__ constexpr int panel_depth(int bits, int mb, int rp) { return (mb == 4 && rp == 2) || (bits == 4 && mb == 2) ? 1 : 2; }
__host__ __device__ constexpr int panel_stages(int bits, int mb, int rp) { return bits == 4 && rp == 1 && mb != 2 ? 4 : 2; }
// (3 bits, two bit-slices per tile: 64 channels x 128 rows do not fit the registers)
__host__ __device__ constexpr bool panel_instance_exists(int bits, int mb, int rp) { return !(bits == 3 && mb == 4 && rp == 2); }
__host__ __device__ constexpr int panel_xbuf_bytes(int mb) { return 32 * mb * panel_kc(mb) * 2; }
// [table, 256-byte entry stride][per K part: two activation buffers], of which the final reduction takes four tiles' sums; then
// [per wavefront: 64 rows' eight scales, kPanelPark][per wavefront: two progress words]
template <int BITS>
__host__ __device__ constexpr int panel_park_off(int mb) {
    const int n = lut_row_table_bytes<BITS>() + kPanelWK * 2 * panel_xbuf_bytes(mb), red = 4 * kPanelWaves * 4 * kPanelQuarter;
    return n > red ? n : red;
}
template <int BITS>
__host__ __device__ constexpr int panel_lds_bytes(int mb) { return panel_park_off<BITS>(mb) + kPanelWaves * kPanelPark + 128; }
__host__ __device__ constexpr size_t panel_slot_bytes(int mb, int rp) { return (size_t)rp * mb * 8 * 1024; }

// SCH: scales are fetched eight at a time per row (K / group a multiple of 8) and parked in LDS, else tile by tile.
template <int BITS, int GROUP, int MB, typename DT, int RP, bool SCH>
__global__ __launch_bounds__(64 * kPanelWaves) void panel_kernel(const PanelParams p) {
    using Gm = Geo<BITS>;
    using TT = typename PanelType<DT>::type;           // how table entries and scales are held
    constexpr int TK = Gm::TK, TILE_BYTES = Gm::TILE_BYTES;
    constexpr int TPS = GROUP > TK ? GROUP / TK : 1;   // tiles that share one scale
    constexpr int NS = GROUP > TK ? 1 : TK / GROUP;    // scales per tile per row
    constexpr int SPG = GROUP / 32;                    // 32-column steps per group
    constexpr int TPC = 8 * TPS / NS;                  // tiles covered by eight scales
    constexpr int LOG2C = perm_log2_copies<BITS, TT>();
    constexpr int LUT_BYTES = lut_row_table_bytes<BITS>();
    constexpr int KC = panel_kc(MB), SPC = KC / 32, CH = TK / KC;      // chunk, its steps, chunks per tile
    constexpr int D = panel_depth(BITS, MB, RP), P = panel_stages(BITS, MB, RP);
    constexpr int SL = KC / 8;                         // 16-byte slots of one row of a chunk
    constexpr int XL = MB * SL / 4;                    // activation loads per wavefront and chunk
    constexpr int XB = panel_xbuf_bytes(MB);
    // the next tile's scales are asked for a tile ahead; 128 rows by 64 channels, and 96 at 3 bits, have no registers for that
    constexpr bool CHUNK_EARLY = !(RP == 2 && (MB == 4 || (MB == 3 && BITS == 3)));
    static_assert(CH % 2 == 0 && (CH * P) % D == 0, "buffer and register rings restart with every round of P tiles");

    asm volatile("" ::"s"(p.X), "s"(p.packed), "s"(p.scales), "s"(p.lut), "s"(p.Y), "s"(p.packed_bytes), "s"(p.scale_bytes),
                 "s"(p.x_bytes), "s"(p.M), "s"(p.N), "s"(p.K), "s"(p.NB), "s"(p.SG2), "s"(p.SBL), "s"(p.tile_stride),
                 "s"(p.sblock_bytes), "s"(p.shares), "s"(p.KS), "s"(p.TS), "s"(p.KSB), "s"(p.lut_ltpe));

    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave & 1, kp = wave >> 1;
    const int l32 = lane & 31, h = lane >> 5;
    char* lut = smem;
    char* xbuf = smem + LUT_BYTES + kp * 2 * XB;

    LutSeed lut_seed = lut_fetch<BITS>(p.lut, tid, p.lut_ltpe);
    __builtin_amdgcn_sched_barrier(0);
    const LutAddr la = make_lut_addr<BITS, TT>(lut, LOG2C, lane);
    const rsrc_t rW = make_rsrc(p.packed, p.packed_bytes);
    const rsrc_t rS = make_rsrc(p.scales, p.scale_bytes);

    // workgroup = (part of M, share of the rows, K slice); a part is 32 MB activation rows
    const int gshare = (int)blockIdx.x / p.KS, slice = (int)blockIdx.x - gshare * p.KS;
    const int mpart = gshare / p.shares, share = gshare - mpart * p.shares;
    const int m0 = mpart * 32 * MB;
    const rsrc_t rX = make_rsrc(p.X + (size_t)m0 * p.K, p.x_bytes - (uint32_t)m0 * (uint32_t)p.K * 2u);
    const int rbw = (share * kPanelWN + wn) * 2 * RP;                   // first row block of the wavefront's panel
    // the slice's tiles over the four K parts
    const int st_n = p.TS + (slice < p.KSB ? 1 : 0);
    const int st_0 = slice * p.TS + (slice < p.KSB ? slice : p.KSB);
    // (with more than 64 rows in a workgroup the first two parts, whose wavefronts are the older ones on their SIMDs and run ahead, get up
    // to three sixteenths more: 8B gate+up M = 128 42.7 -> 42.2 us, 70B gate+up 154.9 -> 151.0; up to 64 rows, parts of M among them, not measured)
    const int skew = MB > 2 ? st_n / kPanelWK * 3 / 16 : 0;
    const int ka = st_0 + (st_n / kPanelWK) * kp + (kp < st_n % kPanelWK ? kp : st_n % kPanelWK) + (kp == 2 ? 2 * skew : (kp & 1) * skew);
    const int len = st_n / kPanelWK + (kp < st_n % kPanelWK ? 1 : 0) + (kp < 2 ? skew : -skew);
    // a row block beyond the last one gets a base of exactly 2 GiB: every offset formed from it stays out of range
    uint32_t wbase[2 * RP];
#pragma unroll
    for (int r = 0; r < 2 * RP; ++r) {
        const int rb = rbw + r;
        wbase[r] = rb < p.NB ? (uint32_t)(rb >> p.SBL) * p.sblock_bytes + (uint32_t)(rb & ((1 << p.SBL) - 1)) * TILE_BYTES
                             : kOutOfRange;
    }
    const uint32_t slane = ((uint32_t)rbw * 16u + (uint32_t)l32) * (uint32_t)p.SG2;    // rows beyond N lie beyond the buffer

    // activations: load i of this wavefront covers the 16-byte units (2 i + wn) 64 + lane of the chunk; unit u holds slot
    // u % SL of row u / SL, and the slot's columns are those of slot (u % SL) ^ swz(row); rows m >= M read as zero
    auto swz = [](int row) { return KC == 64 ? (row >> 1) & 7 : (row >> 2) & 3; };
    // (a step of i is 128 / SL rows, which leaves swz unchanged)
    const int xu = wn * 64 + lane;
    const uint32_t xsrc = (uint32_t)(xu / SL) * (uint32_t)p.K * 2u + 16u * (uint32_t)((xu % SL) ^ swz(xu / SL));
    const uint32_t xstep = (uint32_t)(128 / SL) * (uint32_t)p.K * 2u;
    const uint32_t xdst = (uint32_t)(wn * 64 + lane) * 16u;            // + i * 2 KiB
    // operand reads: row 32 mb + l32, slot 4 s + 2 h + q
    const uint32_t xrow = (uint32_t)l32 * (KC * 2), xslot = (uint32_t)((2 * h) ^ swz(l32));

    struct Stage {
        WFrag<BITS> w[2 * RP];
        ScaleWords<NS> s[SCH ? 1 : RP];
    };
    static_assert(RP * 512 <= kPanelPark / 2, "parked scales end where the half that is never read begins");
    char* park = smem + panel_park_off<BITS>(MB) + wave * kPanelPark;
    u32x4 chunk[RP];                                   // SCH: the next eight scales of row l32 of each half panel
    auto load_stage = [&](Stage& st, int i) {           // tile i of the wavefront's range; nothing beyond the last
        const bool in = i < len;
        const int kt = ka + i;
#pragma unroll
        for (int r = 0; r < 2 * RP; ++r)
            load_wfrag<BITS>(st.w[r], rW, in ? wbase[r] + (uint32_t)kt * p.tile_stride : kOutOfRange, lane);
        if constexpr (!SCH)
#pragma unroll
        for (int rp = 0; rp < RP; ++rp)
            load_scales<NS>(st.s[rp], rS, in ? slane + (uint32_t)rp * 32u * (uint32_t)p.SG2 + (uint32_t)(kt / TPS) * (NS * 2) : kOutOfRange);
    };
    // the eight scales that tile i is the first to use, or that the range begins with; any other tile: nothing
    auto chunk_begins = [&](int i, int kt) { return (uint32_t)kt % TPC == 0 || i == 0; };
    auto load_chunk = [&](int i) {
        const int kt = ka + i;
        const bool in = i < len && chunk_begins(i, kt);
#pragma unroll
        for (int rp = 0; rp < RP; ++rp)
            chunk[rp] = __builtin_amdgcn_raw_buffer_load_b128(rS, in ? slane + (uint32_t)rp * 32u * (uint32_t)p.SG2 + (uint32_t)(kt / TPC) * 16u : kOutOfRange, 0, kAuxNone);
    };
    // words of blocks (2 rp, 2 rp + 1) become octets {0, 2} and {1, 3} of both
    auto swap_stage = [&](Stage& st) {
        auto swap = [](uint32_t& a, uint32_t& b) {
            typedef uint32_t pair_t __attribute__((ext_vector_type(2)));
            const pair_t r = __builtin_bit_cast(pair_t, __builtin_amdgcn_permlane16_swap(a, b, false, false));
            a = r.x; b = r.y;
        };
#pragma unroll
        for (int rp = 0; rp < RP; ++rp) {
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                uint32_t a = st.w[2 * rp].w[d], b = st.w[2 * rp + 1].w[d];
                swap(a, b);
                st.w[2 * rp].w[d] = a; st.w[2 * rp + 1].w[d] = b;
            }
            if constexpr (BITS == 3) {
#pragma unroll
                for (int d = 0; d < 2; ++d) {
                    uint32_t a = st.w[2 * rp].hi[d], b = st.w[2 * rp + 1].hi[d];
                    swap(a, b);
                    st.w[2 * rp].hi[d] = a; st.w[2 * rp + 1].hi[d] = b;
                }
            }
        }
    };
    u32x4 xr[D][XL];
    auto load_x = [&](u32x4 (&x)[XL], int i, int c) {
        // (columns beyond the wavefront's range: bases of exactly 2 GiB, which no row step brings back into range)
        const uint32_t col = i < len ? (uint32_t)(ka + i) * (TK * 2) + (uint32_t)c * (KC * 2) + xsrc : kOutOfRange;
#pragma unroll
        for (int k = 0; k < XL; ++k) x[k] = __builtin_amdgcn_raw_buffer_load_b128(rX, col + (uint32_t)k * xstep, 0, kAuxNone);
    };
    auto store_x = [&](const u32x4 (&x)[XL], int parity) {
#pragma unroll
        for (int i = 0; i < XL; ++i) *reinterpret_cast<u32x4*>(xbuf + parity * XB + i * 2048 + xdst) = x[i];
    };

    f32x16 acc[RP][MB];
#pragma unroll
    for (int rp = 0; rp < RP; ++rp)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[rp][mb][i] = 0.f;

    // Activations first: they are waited for first, and loads are counted in order.
    u32x4 x0[XL];
    load_x(x0, 0, 0);
    if constexpr (SCH) load_chunk(0);
    __builtin_amdgcn_sched_barrier(0);
    Stage st[P];
    load_stage(st[0], 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int d = 0; d < D; ++d) {                      // chunk 1 + d waits in xr[(1 + d) % D]
        load_x(xr[(1 + d) % D], (1 + d) / CH, (1 + d) % CH);
        __builtin_amdgcn_sched_barrier(0);
    }
    {
        LutSeed seed = lut_seed;
        asm volatile("" : "+v"(seed.w[0]), "+v"(seed.w[1]), "+v"(seed.w[2]), "+v"(seed.w[3]));
        lut_build<BITS, TT>(lut, seed, (int)(reinterpret_cast<uintptr_t>(p.lut) >> 1) & 1, LOG2C, tid, p.lut_ltpe);
    }
    store_x(x0, 0);
    // The two wavefronts of a K part keep in step through two words each in LDS: `ready` = the last chunk whose share is
    // stored, `done` = chunks whose operands are read.  A buffer is written once the partner has read what it held, and read
    // once the partner has stored its share.  (LDS serves one wavefront's accesses in order, so a word published after
    // stores or reads is seen after them.  Both wavefronts run the same chunks and are resident together; chunk g is stored
    // after waiting for done >= g and read after waiting for ready >= g, and done = g and ready = g are published without
    // waiting for anything later: neither can wait for ever.)  The K parts run free of each other, so that one part's LDS
    // and memory phases fall into another's multiplications (a workgroup barrier per chunk: 4.4 us per K tile and wavefront at
    // M = 128 with the taller panel, this 3.6).
    uint32_t* flags = reinterpret_cast<uint32_t*>(smem + panel_park_off<BITS>(MB) + kPanelWaves * kPanelPark);
    if (tid < 2 * kPanelWaves) flags[tid] = 0;
    uint32_t* own = flags + 2 * wave;
    uint32_t* other = flags + 2 * (wave ^ 1);
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 1; q < P - 1; ++q) {                  // (before the barrier the first activations would queue behind them)
        load_stage(st[q], q);
        __builtin_amdgcn_sched_barrier(0);
    }
    auto publish = [&](int word, int v) {
        asm volatile("" ::: "memory");
        if (lane == 0) __hip_atomic_store(own + word, (uint32_t)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        asm volatile("" ::: "memory");
    };
    // the partner's words are asked for ahead of their use; only if it is late are they asked for again
    // (The first look is straight-line code: with one loop for both looks the wait in front of it was one for every LDS read under way,
    // twice per chunk.)
    uint32_t seen[2];
    auto ask = [&](int word) { seen[word] = __hip_atomic_load(other + word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
    auto wait_for = [&](int word, int v) {
        if ((int)__builtin_amdgcn_readfirstlane(seen[word]) < v) {
            do {
                ask(word);
                asm volatile("" : "+v"(seen[word]));
            } while ((int)__builtin_amdgcn_readfirstlane(seen[word]) < v);
        }
        asm volatile("" ::: "memory");
    };

    // A unit is half a 32-column step: one matrix instruction per (half panel, 32 activation rows).  While unit n is multiplied,
    // unit n + 1 is scaled and unit n + 2's table reads are issued, piece by piece between the matrix instructions: a wavefront
    // issues in order, and whatever stands in front of a matrix instruction keeps the matrix unit waiting.
    constexpr int U = 2 * SPC, UT = CH * U, NM = RP * MB;
    // units of a chunk: the next chunk is stored at the end of US (with four units early, three before it is read: 12288 x 4096 W4 M = 50
    // 16.5 -> 15.6 us; with two units the later of the two is 2 % faster); the partner's words are asked for at the start of A_DONE and A_READY
    constexpr int US = 0, A_DONE = U == 4 ? U - 1 : US, A_READY = U == 4 ? U - 2 : U - 1;
    constexpr int NPC = (BITS == 2 ? 2 : 4) * RP;       // pieces of a unit: one table read (a pair, or at 2 bits a quad) each
    u32x4 b[MB];
    u32x4 a[2][RP];                                    // operands of the unit being multiplied and of the next one
    Raw<BITS, TT> raw[RP];                             // table values of the next unit, then of the one after it
    ScaleWords<NS> sw[2][RP];                          // scales of even and odd tiles
    // operand of unit u = 2 s + q of a chunk, from the chunk's buffer
    auto read_b = [&](int parity, int mb, int u) {
        b[mb] = *reinterpret_cast<const u32x4*>(xbuf + parity * XB + xrow + ((xslot ^ (uint32_t)(4 * (u / 2) + (u & 1))) * 16u) + mb * (32 * KC * 2));
    };
    // table read `piece` of a unit (step s of the tile, half q)
    auto look = [&](const Stage& t, int s, int q, int piece) {
        const int rp = piece / (NPC / RP), e = piece % (NPC / RP);
        const uint32_t w = index_word<BITS>(t.w[2 * rp + q], s);
        if constexpr (BITS == 2) {
            const u32x2 v = (s & 1) ? (e ? lds_u64(entry_addr<true, 3>(w, la)) : lds_u64(entry_addr<true, 2>(w, la)))
                                    : (e ? lds_u64(entry_addr<true, 1>(w, la)) : lds_u64(entry_addr<true, 0>(w, la)));
            raw[rp].v[2 * e] = v.x;
            raw[rp].v[2 * e + 1] = v.y;
        } else {
            raw[rp].v[e] = lds_u32(e == 0 ? entry_addr<true, 0>(w, la) : e == 1 ? entry_addr<true, 1>(w, la)
                                   : e == 2 ? entry_addr<true, 2>(w, la) : entry_addr<true, 3>(w, la));
        }
    };
    auto scale = [&](u32x4 (&dst)[RP], const ScaleWords<NS> (&w)[RP], int s, int piece) {
        const int rp = piece / (NPC / RP), e = piece % (NPC / RP);
        const ScaleReg<TT> sc = scale_of<TT, NS>(w[rp], s / SPG);
        if constexpr (BITS == 2) {
            dst[rp][2 * e] = scale_pair(raw[rp].v[2 * e], sc);
            dst[rp][2 * e + 1] = scale_pair(raw[rp].v[2 * e + 1], sc);
        } else {
            dst[rp][e] = scale_pair(raw[rp].v[e], sc);
        }
    };
    // the scales of tile i (stage t): from the parked eight, which are replaced first where the tile is the first to use the next
    auto take_scales = [&](ScaleWords<NS> (&w)[RP], const Stage& t, int i) {
        if constexpr (SCH) {
            // No branch: where the tile is not the first to use its eight, what is stored goes to the wavefront's other KiB, and
            // the next eight are asked for at once (or with the tile's first chunk).  Behind a branch the wait for them was one for every load
            // under way, weights and activations of the tiles ahead among them, once per K tile: with that and the pairs' straight-line look, W4 fp16
            // 8B gate+up M = 128 42.8 -> 41.3 us, 70B gate+up 157 -> 148, 8B o M = 128 13.6 -> 12.5, down M = 64 21.2 -> 20.0, 12288 x 4096 M = 50 17.3 -> 16.2.
            const int kt = ka + i;
            char* const dst = park + (chunk_begins(i, kt) ? 0 : kPanelPark / 2) + 16 * l32;
            asm volatile("" ::: "memory");              // (LDS operations of one wavefront complete in order)
#pragma unroll
            for (int rp = 0; rp < RP; ++rp) *reinterpret_cast<u32x4*>(dst + rp * 512) = chunk[rp];
            asm volatile("" ::: "memory");
#pragma unroll
            for (int rp = 0; rp < RP; ++rp) lds_load_scales<NS>(w[rp], park + rp * 512 + 16 * l32 + (((uint32_t)kt % TPC) / TPS) * (NS * 2));
            if constexpr (CHUNK_EARLY) load_chunk(i + 1);
        } else {
#pragma unroll
            for (int rp = 0; rp < RP; ++rp) w[rp] = t.s[rp];
        }
    };
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) read_b(0, mb, 0);
    swap_stage(st[0]);
    take_scales(sw[0], st[0], 0);
#pragma unroll
    for (int i = 0; i < NPC; ++i) look(st[0], 0, 0, i);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NPC; ++i) {
        scale(a[0], sw[0], 0, i);
        look(st[0], 0, 1, i);
    }
    ask(1);
    __builtin_amdgcn_sched_barrier(0);

    // tile ti of a round of P (ti is a constant): stage ti; its first chunk asks for the tile P - 1 ahead, after the chunk's
    // activation loads (loads are waited for in order: the first activations behind these weights are then needed D + 1
    // chunks later)
    auto tile = [&](auto tic, int t) {
        constexpr int ti = decltype(tic)::value;
        Stage& cur = st[ti];
        Stage& nxt = st[(ti + 1) % P];
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            constexpr int R0 = ti * CH + 1;
            const int g = t * CH + c;                    // chunk of the wavefront's range
            if (c == CH - 1) {
                swap_stage(nxt);
                take_scales(sw[(ti + 1) & 1], nxt, t + 1);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int n = c * U + u, n1 = (n + 1) % UT, n2 = (n + 2) % UT;
                if (u == A_DONE) ask(1);
                if (u == A_READY) ask(0);
#pragma unroll
                for (int i = 0; i < NM; ++i) {
                    const int mb = i / RP, rp = i % RP;
                    acc[rp][mb] = mfma32x32x16<DT>(a[n & 1][rp], b[mb], acc[rp][mb]);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int e = i * NPC / NM; e < (i + 1) * NPC / NM; ++e) {
                        scale(a[(n + 1) & 1], n + 1 < UT ? sw[ti & 1] : sw[(ti + 1) & 1], n1 / 2, e);
                        look(n + 2 < UT ? cur : nxt, n2 / 2, n2 & 1, e);
                    }
                    // the operand's next unit is read as soon as its last product is issued; the next chunk's first unit
                    // once the partner has stored its share of it
                    if (rp == RP - 1) {
                        if (u + 1 < U) {
                            read_b(c & 1, mb, u + 1);
                        } else {
                            if (mb == 0) wait_for(0, g + 1);
                            read_b((c + 1) & 1, mb, 0);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (u == US) {
                    // chunk g + 1 to the other buffer, chunk g + 1 + D on its way
                    wait_for(1, g);
                    if constexpr (SCH && !CHUNK_EARLY) {
                        if (c == 0) load_chunk(t + 1);
                    }
                    store_x(xr[(R0 + c) % D], (c + 1) & 1);
                    publish(0, g + 1);
                    load_x(xr[(R0 + c) % D], t + (c + 1 + D) / CH, (c + 1 + D) % CH);
                    __builtin_amdgcn_sched_barrier(0);
                    if (c == 0) {
                        load_stage(st[(ti + P - 1) % P], t + P - 1);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                if (u == U - 2) publish(1, g + 1);          // the last unit's operands have been asked for
            }
        }
    };
    for (int t = 0; t < len; t += P) {
        tile(std::integral_constant<int, 0>{}, t);
        if (t + 1 < len) tile(std::integral_constant<int, 1 % P>{}, t + 1);
        if constexpr (P > 2) {
            if (t + 2 < len) tile(std::integral_constant<int, 2 % P>{}, t + 2);
            if (t + 3 < len) tile(std::integral_constant<int, 3 % P>{}, t + 3);
        }
    }

    // ---- add the four K parts in order through LDS, up to four tiles (32 rows x 32 columns) per wavefront and round ----
    // A lane's sums are four consecutive channels of one activation row; they are parked as quarters (8 channels x 32 rows) of
    // 1 KiB, 1088 bytes apart, and taken out as eight consecutive channels per lane, four lanes side by side: 64-byte pieces of
    // Y's rows, and sixteen lanes' reads (four rows, four quarters) cover all banks.
    constexpr int TILES = RP * MB, TR = TILES < 4 ? TILES : 4, QB = kPanelQuarter;
    const int nrow0 = share * (kPanelWN * 32 * RP);
    const rsrc_t rP = make_rsrc(p.slots, p.slot_bytes);
    const int ok = lane & 3, om = lane >> 2;            // quarter and row (of sixteen) this lane takes out
    // task = (tile, panel, half of the tile's 32 activation rows); task t is always wavefront t % 8's
    auto emit = [&](int task, f32x4 lo, f32x4 hi) {
        const int j = task >> 2, pn = (task >> 1) & 1, half = task & 1;
        const int rp = j / MB, mb = j % MB;
        const int m = m0 + 32 * mb + 16 * half + om, n = nrow0 + (pn * RP + rp) * 32 + 8 * ok;
        if (m < p.M && n < p.N) {
            const u32x2 a = pack4<DT>(lo), c = pack4<DT>(hi);
            *reinterpret_cast<u32x4*>(p.Y + (size_t)m * p.N + n) = u32x4{a.x, a.y, c.x, c.y};
        }
    };
    const uint32_t slot0 = (uint32_t)blockIdx.x * (uint32_t)panel_slot_bytes(MB, RP) + 16u * (uint32_t)lane;
#pragma unroll
    for (int j0 = 0; j0 < TILES; j0 += TR) {
        __syncthreads();
#pragma unroll
        for (int j = 0; j < TR; ++j)
            if (j0 + j < TILES) {
                const f32x16 v = acc[(j0 + j) / MB][(j0 + j) % MB];
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    *reinterpret_cast<f32x4*>(smem + (size_t)((j * kPanelWaves + wave) * 4 + k) * QB + lane * 16) =
                        f32x4{v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]};
            }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < (TR * 4 + kPanelWaves - 1) / kPanelWaves; ++i) {
            const int task = j0 * 4 + i * kPanelWaves + wave;
            const int j = (task >> 2) - j0, pn = (task >> 1) & 1, half = task & 1;
            if (j >= TR || j0 + j >= TILES) continue;
            f32x4 lo = f32x4{0.f, 0.f, 0.f, 0.f}, hi = lo;
            const char* src = smem + (size_t)((j * kPanelWaves + pn) * 4 + ok) * QB + (16 * half + om) * 16;
#pragma unroll
            for (int part = 0; part < kPanelWK; ++part) {
                lo += *reinterpret_cast<const f32x4*>(src + (size_t)part * (kPanelWN * 4 * QB));
                hi += *reinterpret_cast<const f32x4*>(src + (size_t)part * (kPanelWN * 4 * QB) + 512);
            }
            if (p.KS > 1) {
                // this slice's sums to the workgroup's own slot
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, lo), rP, slot0 + (uint32_t)task * 2048u, 0, kAuxDevice);
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, hi), rP, slot0 + (uint32_t)task * 2048u + 1024u, 0, kAuxDevice);
            } else {
                emit(task, lo, hi);
            }
        }
    }
    if (p.KS > 1) {
        // this wavefront's stores are acknowledged, then it arrives; the last of the KS slices' wavefronts of this number adds
        // their slots in slice order, its own included, and writes Y (it is the only one whose loads follow all arrivals)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0);
        uint32_t* counter = p.counters + (size_t)gshare * 16 + wave;
        uint32_t old = 0;
        if (lane == 0) old = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        old = __builtin_amdgcn_readfirstlane(old);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        if (old != (uint32_t)(p.KS - 1)) return;
        if (lane == 0) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // all of the wavefront's tasks, SB slices at a time in flight together (a slice beyond the last is not loaded -- its
        // offset is out of range -- and not added)
        constexpr int PT = (TILES * 4 + kPanelWaves - 1) / kPanelWaves, SB = PT > 2 ? 4 : 8;
        const uint32_t base = (uint32_t)(gshare * p.KS) * (uint32_t)panel_slot_bytes(MB, RP) + 16u * (uint32_t)lane;
        f32x4 lo[PT], hi[PT];
#pragma unroll
        for (int i = 0; i < PT; ++i) lo[i] = hi[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int s0 = 0; s0 < p.KS; s0 += SB) {
            u32x4 v[SB][PT][2];
#pragma unroll
            for (int s = 0; s < SB; ++s)
#pragma unroll
                for (int i = 0; i < PT; ++i)
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const int task = i * kPanelWaves + wave;
                        const bool in = s0 + s < p.KS && task < TILES * 4;
                        v[s][i][e] = __builtin_amdgcn_raw_buffer_load_b128(
                            rP, in ? base + (uint32_t)(s0 + s) * (uint32_t)panel_slot_bytes(MB, RP) + (uint32_t)task * 2048u + 1024u * e : kOutOfRange, 0, kAuxDevice);
                    }
#pragma unroll
            for (int s = 0; s < SB; ++s)
                if (s0 + s < p.KS)
#pragma unroll
                    for (int i = 0; i < PT; ++i) {
                        lo[i] += __builtin_bit_cast(f32x4, v[s][i][0]);
                        hi[i] += __builtin_bit_cast(f32x4, v[s][i][1]);
                    }
        }
#pragma unroll
        for (int i = 0; i < PT; ++i)
            if (i * kPanelWaves + wave < TILES * 4) emit(i * kPanelWaves + wave, lo[i], hi[i]);
    }
}

}  // namespace lutq
