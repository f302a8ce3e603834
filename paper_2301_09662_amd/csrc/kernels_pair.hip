// Gather gridding with both transform passes on the matrix cores, image rows
// and columns taken in pairs (j, N - j).  The FP32 form and the FP16 form of
// the hot path run this kernel; it keeps the persistent (channel, spectrum)
// schedule, the decoding and the FP32 gather of the other kernels.
//
// Pairs.  The DFT rows of bins j and N - j are conjugates, so with the real
// matrices C[j][n] = cos(2 pi j n / N), S[j][n] = sin(2 pi j n / N), j < N/2,
// four real products give both bins of a complex input v:
//   P1 = C Re v, P2 = S Im v, P3 = S Re v, P4 = C Im v
//   V[j]     = (P1 - P2) + i (P3 + P4)
//   V[N - j] = (P1 + P2) + i (P4 - P3).
// Row 0 has S = 0 and no partner; its S row holds (-1)^n instead, so that
//   V[0] = P1 + i P4,  V[N/2] = P3 + i P2.
// Against the real form [[C, -S], [S, C]] over all N rows this halves the
// matrix work, the operand reads from LDS and the registers of the DFT operand
// for two additions per output.
//
// FP32 on FP16 products (SPLIT).  Every operand x is held as hi = fp16(x) and
// lo = fp16(x - hi), 22 to 23 bits of it (2^-24.5 rms; an FP32 rounding is
// 2^-24.8), and x y is summed in FP32 as hi hi' + lo hi' + hi lo'; the dropped
// lo lo' is below 2^-23.5 rms of a product.  The depth of a product is
// the window's cells once per term, packed without padding between the terms:
// the data operand stores [hi | lo] and is read cyclically ([hi | lo | hi]), the
// DFT operand holds [hi | hi | lo].  Gridded values are scaled by a power of
// two per channel and pol, and the DFT matrix by 16; the sums are scaled back
// when they leave the registers (all exact).  A scaled value below 2^-3 has a
// subnormal lo: from there on its error is 2^-25 of the scaled unit and no
// longer follows the value.  The scale is therefore the largest that a bound of
// the window's rows allows (pair_scale), so that such values are small against
// the rest: row sums of the weights, which a crowd of antennas in one cell does
// not multiply by the window's width (2000 antennas in a cell, 60 outriggers in
// 61 x 63 cells, samples of 0 and +-1: 0.6e-6 from 64-bit images, 5.8e-6 with the
// largest cell's sum times the width), and, where the antennas' weights differ
// by kPairSpread or more, the samples they meet in the call (range_kernel): a
// silent antenna with a gain of 1e6 among 256 put the images off by 2e-4.  In the
// FP16 form (no SPLIT) operands are rounded to FP16 once.
//
// A workgroup holds one spectrum at a time: gather -> row pass (the window's
// rows times the DFT, i pairs) -> column pass (the DFT times the columns, j
// pairs) -> products of Eq. 5 into registers.  Wave w owns the j tile w % JT
// (16 pairs = 32 image rows) and ITW tiles of 16 columns.
//
// What bounds it: issue slots.  A product occupies the matrix cores 16 cycles
// and takes about 8 cycles of VALU issue with it (two kinds of waves on one
// SIMD: 0.52 ms of products and 0.54 ms of FMAs take 0.78 ms together), so
// products and VALU instructions add up; at the station shape (N = 64, 18 x 18
// cells) that sum is 85 % of the cycles.  Hence the pairs, one-instruction
// conversions, a gather program read with uniform loops and no address
// arithmetic, and spectra loaded without branches so that nothing waits for
// them before they are decoded.  Eight waves of at most 128 registers (N = 64)
// keep two workgroups on a CU.  Whole calls, against the kernels this one
// replaced (vector-ALU transforms in FP32; one DFT row per image row in FP16):
// station FP32 1099 -> 568 us, FP16 530 -> 430 us; 2048 antennas, N = 128, FP32
// 2414 -> 1690 us; station on a 256 grid, FP32 2239 -> 1285 us.  With 2048
// antennas the gather's LDS reads and scattered writes bound it instead (1.06 of
// 1.97 ms when each phase was left out in turn).  FP32 errors
// against 64-bit images are below those of the vector-ALU transforms on arrays of
// evenly weighted antennas (station 1.7e-7 against 1.8e-7, 77 antennas at N = 48
// 0.6e-7 against 1.0e-7, 256 grid 2.0e-7 against 2.2e-7); for the others see
// above.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "epic_device.hpp"
#include "epic_gather.hpp"
#include "epic_internal.hpp"
#include "epic_mfma.hpp"
#include "epic_sched.hpp"

namespace epic {

namespace {

// FP16, N = 192, both pols, windows beyond 32 cells (products of two steps): six
// column parts of two column tiles each, gathered six times instead of four but
// with shared products (62 antennas, 16 channels x 200 spectra, 38 x 38 cells:
// 148 us; half-split, below, 248; unpaired rows 168.  1002 antennas, 62 x 62
// cells: 294, 332 and 330).
constexpr bool pair_six(int N, bool split, int P, int WD) { return N == 192 && !split && P == 2 && WD > 32; }

constexpr int pair_ks(int N, bool split, int P, int WD) {
    return N <= 64 ? 1 : (N <= 128 ? 2 : (pair_six(N, split, P, WD) ? 6 : (N == 192 && !split ? 4 : 8)));
}
// Column tiles per wave.  FP16 single-pol grids of 48 and 96 have three column
// tiles and few registers: all three in one wave make workgroups of two or three
// waves, several to a CU, whose barriers overlap (station, 4 channels x 1000
// spectra: N = 96 50.1 -> 35.8 us, N = 48 30.2 -> 23.9; unpaired rows 40.2, 23.4).
constexpr int pair_itw(int N, bool split, int P, int WD) {
    if (pair_six(N, split, P, WD)) return 1;
    if (!split && P == 1 && (N == 48 || N == 96)) return 3;
    return N == 128 || (N == 192 && !split) || (N == 256 && split) ? 2 : 1;
}

// The narrower windows there: twelve waves of at most 168 registers.  With the
// column tiles split (two tiles and one, 64 accumulators) 40 to 90 registers
// spill; with each wave computing one output of every pair (chained, twice the
// products, 48 accumulators) none do: 215 against 139 us for 4 channels x 1000
// spectra of the station (unpaired rows took 155).
constexpr bool pair_half(int N, bool split, int P, int WD) {
    return N == 192 && !split && P == 2 && !pair_six(N, split, P, WD);
}

template <int N_, int WD_, bool SPLIT_, int P_ = 2>
struct PairShape {
    static constexpr int N = N_;
    static constexpr int WD = WD_;                  // window rows / columns held per part (multiple of 4)
    static constexpr bool SPLIT = SPLIT_;
    static constexpr int NH = N / 2;                // pairs
    static constexpr int JT = (NH + 15) / 16;       // tiles of 16 row pairs
    static constexpr int KS = pair_ks(N, SPLIT, P_, WD);    // workgroups sharing a spectrum's columns
    static constexpr int NK = N / KS;               // columns per workgroup: NK / 2 pairs
    static constexpr int NKH = NK / 2;
    static constexpr int NIT = (NKH + 15) / 16;     // column-pair tiles of the row pass
    static constexpr int NCT = (NK + 15) / 16;      // column tiles of the column pass
    static constexpr int NKP = 16 * NCT;            // columns held in LDS
    // half-split: two waves share a row-pair tile by outputs, rows j and rows
    // N - j, and take every column tile (see pair_half)
    static constexpr bool HS = pair_half(N, SPLIT, P_, WD);
    static constexpr int ITW = HS ? NCT : pair_itw(N, SPLIT, P_, WD);   // column tiles per wave
    static constexpr int CG = HS ? 2 : (NCT + ITW - 1) / ITW;   // column groups (half-split: the halves)
    static constexpr int WAVES = JT * CG;
    static constexpr int TH = 64 * WAVES;
    static constexpr int RW = WAVES / NIT * NIT;    // waves of the row pass
    // rows of the DFT operand's planes: every pair tile of either pass
    static constexpr int TR = 16 * JT > (KS - 1) * NKH + 16 * NIT ? 16 * JT : (KS - 1) * NKH + 16 * NIT;
    static constexpr int SD = SPLIT ? 2 * WD : WD;  // stored halfs of a real or imaginary part
    static constexpr int DEPTH = SPLIT ? 3 * WD : WD;
    static constexpr int ST = (DEPTH + 31) / 32;    // MFMA steps of a product
    // LDS pitch of a row of either operand, [Re | Im]: an odd number of 16-byte
    // groups, so that 16 lanes reading 16 rows touch every bank group once
    static constexpr int PITCH = ((2 * SD / 8) | 1) * 8;
    // unsplit workgroups: a wave's row-pass operand is its column-pass operand
    static constexpr bool SHARE = KS == 1;
    // chained products: each output is summed over both parts by the matrix
    // cores (twice the products, no additions); else the four products are
    // shared by a pair and added.  Chained pays for single-step products whose
    // operands fit the registers (station FP16 143 against 148 us at 250
    // spectra); with two steps it loses (station FP32 797 against 708 us).
    static constexpr bool CHAIN = (SHARE && ST == 1) || HS;
    static constexpr int PL = CHAIN ? 4 : 2;        // planes of the DFT operand
    static_assert((SPLIT ? WD % 4 : WD % 8) == 0 && WAVES <= 16, "");
    static_assert(!SHARE || (NIT == JT && WAVES % NIT == 0), "row-pass tile = column-pass tile");
};

// Register budget (waves per SIMD).
template <class Sh>
constexpr int pair_waves() {
    return Sh::WAVES == 9 || Sh::WAVES == 12 ? 3 : (Sh::ITW == 1 || Sh::ITW == 3 ? 4 : 2);
}

struct PairArgs {
    const uint8_t* samples;   // [T][C][A][P]
    const ChanInfo* chans;    // of the sliced gather program
    const CellDesc* desc;     // x: operand offset r * PITCH + w | groups << 16; y: first group of the slice
    const uint2* grp_ant;     // 4 x u16 per group
    const float4* grp_w;
    const _Float16* dft;      // [planes][TR][32 ST]
    const float* row_bound;   // [C][kRowBounds][P] bounds of |Re G| + |Im G| summed over a window row (SPLIT)
    float* slots;             // [S][C][NPP][N][N]
    int64_t T;
    int C, A;
    int M1max;                // rows of the row-pass operand (multiple of 16)
    int nibble_order, fresh;
    int grid_wg, wg_per_xcd;
    uint32_t off_w, off_ant, off_desc, off_A1, off_B2;   // the samples are at 0
};

// One real value into its operand position: rounded to FP16, or hi and lo
// (neg1 = -1: with a variable factor the residual is one mixed-precision FMA
// whose result is rounded to FP16 directly).
template <bool SPLIT, int WD>
__device__ __forceinline__ void put_part(_Float16* dst, float v, float neg1) {
    const _Float16 hi = (_Float16)v;
    dst[0] = hi;
    if constexpr (SPLIT) dst[WD] = (_Float16)fmaf((float)hi, neg1, v);
}
template <bool SPLIT, int WD>
__device__ __forceinline__ void put_part4(_Float16* dst, const floatx4 v, float neg1) {
    typedef float float2v __attribute__((ext_vector_type(2)));
    const h2v a = __builtin_convertvector((float2v{v[0], v[1]}), h2v), b = __builtin_convertvector((float2v{v[2], v[3]}), h2v);
    *reinterpret_cast<half4*>(dst) = half4{a[0], a[1], b[0], b[1]};
    if constexpr (SPLIT) {
        half4 lo;
        lo[0] = (_Float16)fmaf((float)a[0], neg1, v[0]);
        lo[1] = (_Float16)fmaf((float)a[1], neg1, v[1]);
        lo[2] = (_Float16)fmaf((float)b[0], neg1, v[2]);
        lo[3] = (_Float16)fmaf((float)b[1], neg1, v[3]);
        *reinterpret_cast<half4*>(dst + WD) = lo;
    }
}

// Scale of the gridded values of one pol: the largest power of two for which,
// with row a bound of |Re G| + |Im G| summed over a window row, neither a
// gridded component nor the row pass's sum of such a row times the scaled DFT
// operand can leave half of FP16's range.
__device__ __forceinline__ float pair_scale(int row_bits) {   // uniform: scalar registers
    if (row_bits <= 0) return 1.0f;
    int e = 15 - kDftScaleLog2 - (((row_bits >> 23) & 255) - 126);   // 16 row < 2^(15 - e); inf: smallest scale
    e = e > 100 ? 100 : (e < -100 ? -100 : e);
    return __int_as_float((e + 127) << 23);
}

// Decoded sample(s) of an antenna at an LDS address, FP16 (re, im per pol).
template <int P>
struct RawSample;
template <>
struct RawSample<1> {
    h2v h;
    __device__ __forceinline__ void load(uint32_t addr) { h = *(const __attribute__((address_space(3))) h2v*)(addr); }
    __device__ __forceinline__ float2 get() const { return make_float2((float)h[0], (float)h[1]); }
};
template <>
struct RawSample<2> {
    h4v h;
    __device__ __forceinline__ void load(uint32_t addr) { h = *(const __attribute__((address_space(3))) h4v*)(addr); }
    __device__ __forceinline__ float4 get() const {
        return make_float4((float)h[0], (float)h[1], (float)h[2], (float)h[3]);
    }
};
__device__ __forceinline__ uint32_t lds_address(const unsigned char* p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) unsigned char*)p;
}

// Gather gridding over the sliced program: 64 cells (sorted by their groups)
// form a slice whose lanes loop equally long, group j of the slice's lanes
// stored side by side, so its reads are contiguous over the lanes.  In LDS the
// antenna indices are held as the LDS addresses of their samples.  A program
// too large for LDS is streamed from L2; from LDS up to three groups are taken
// together, all their index and weight reads before all their sample reads
// before the sums, so that a slice waits for LDS twice (station FP32 601 -> 572
// us a call, FP16 438 -> 430).  Streaming gains nothing from more in flight (2048
// antennas: 1707 us two groups at a time, 1812 with three): the bank conflicts of
// its sample reads bound it.
template <class Sh, int P, int WM, bool PROG>
__device__ __forceinline__ void pair_gather(const unsigned char* smem, const PairArgs& a, const uint2* g_ant,
                                            const float4* g_w, int wave, int lane, CellDesc d, int n_cell, int prow,
                                            float sx, float sy, float neg1, _Float16* s_A1) {
    constexpr int GF4 = group_f4<P, WM>();
    const CellDesc* s_desc = reinterpret_cast<const CellDesc*>(smem + a.off_desc);
    auto put = [&](const CellDesc& cd, int k, float2 gx, float2 gy) {
        if (k >= n_cell) return;
        if constexpr (Sh::SPLIT) {
            gx.x *= sx; gx.y *= sx; gy.x *= sy; gy.y *= sy;
        }
        _Float16* dst = s_A1 + (cd.x & 0xFFFFu);
        put_part<Sh::SPLIT, Sh::WD>(dst, gx.x, neg1);
        put_part<Sh::SPLIT, Sh::WD>(dst + Sh::SD, gx.y, neg1);
        if constexpr (P == 2) {
            put_part<Sh::SPLIT, Sh::WD>(dst + prow, gy.x, neg1);
            put_part<Sh::SPLIT, Sh::WD>(dst + prow + Sh::SD, gy.y, neg1);
        }
    };
    // slices wave, wave + WAVES, ...; the first one's descriptor d is at hand
    const uint32_t s0 = lds_address(smem);
    for (int k0 = 64 * wave; k0 < n_cell; k0 += Sh::TH) {
        const int k = k0 + lane;
        if (k0 != 64 * wave) d = s_desc[k];
        const int ng = __builtin_amdgcn_readfirstlane((int)(d.x >> 16));
        const int g0 = __builtin_amdgcn_readfirstlane((int)d.y);
        float2 gx = make_float2(0.f, 0.f), gy = make_float2(0.f, 0.f);
        auto groups = [&](auto nb, int j0) {   // nb groups from j0 on
            constexpr int NB = decltype(nb)::value;
            uint32_t at[NB][4];
            float4 w[NB][GF4];
            RawSample<P> x[NB][4];
#pragma unroll
            for (int u = 0; u < NB; ++u) {
                const int j = j0 + u;
                const uint4 o = (reinterpret_cast<const uint4*>(smem + a.off_ant) + g0 + lane)[64 * j];
                at[u][0] = o.x; at[u][1] = o.y; at[u][2] = o.z; at[u][3] = o.w;
#pragma unroll
                for (int q = 0; q < GF4; ++q)   // a slice's 64 lanes side by side per weight word
                    w[u][q] = (reinterpret_cast<const float4*>(smem + a.off_w) + g0 * GF4 + lane)[64 * (j * GF4 + q)];
            }
#pragma unroll
            for (int u = 0; u < NB; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) x[u][q].load(at[u][q]);
#pragma unroll
            for (int u = 0; u < NB; ++u)
                gather_fma<P, WM>(gx, gy, w[u], x[u][0].get(), x[u][1].get(), x[u][2].get(), x[u][3].get());
        };
        if constexpr (PROG) {
            constexpr int NBM = GF4 == 1 ? (Sh::N >= 192 ? 2 : 3) : (GF4 == 2 ? 2 : 1);
            int j = 0;
            for (; j + NBM <= ng; j += NBM) groups(std::integral_constant<int, NBM>{}, j);
            if (NBM > 2 && ng - j >= 2) {
                groups(std::integral_constant<int, 2>{}, j);
                j += 2;
            }
            if (NBM > 1 && ng - j >= 1) groups(std::integral_constant<int, 1>{}, j);
        } else {
            constexpr uint32_t B = 4 * P;   // bytes per antenna
            const uint2* ant = g_ant + g0;
            const float4* w = g_w + (int64_t)g0 * GF4;
#pragma unroll 2
            for (int j = 0; j < ng; ++j) {
                const uint2 o = ant[64 * j + lane];
                float4 ww[GF4];
#pragma unroll
                for (int q = 0; q < GF4; ++q) ww[q] = w[(64 * j + lane) * GF4 + q];
                RawSample<P> x[4];
                x[0].load(s0 + (o.x & 0xFFFFu) * B);
                x[1].load(s0 + (o.x >> 16) * B);
                x[2].load(s0 + (o.y & 0xFFFFu) * B);
                x[3].load(s0 + (o.y >> 16) * B);
                gather_fma<P, WM>(gx, gy, ww, x[0].get(), x[1].get(), x[2].get(), x[3].get());
            }
        }
        put(d, k, gx, gy);
    }
}

template <int N_, int WD_, int P, int WM, bool SPLIT, bool PROG>
__global__ void __launch_bounds__((PairShape<N_, WD_, SPLIT, P>::TH))
__attribute__((amdgpu_waves_per_eu(pair_waves<PairShape<N_, WD_, SPLIT, P>>()))) pair_kernel(PairArgs a) {
    using Sh = PairShape<N_, WD_, SPLIT, P>;
    constexpr int N = Sh::N, WD = Sh::WD, SD = Sh::SD, PITCH = Sh::PITCH, ST = Sh::ST, NK = Sh::NK, NKH = Sh::NKH, NKP = Sh::NKP;
    constexpr int JT = Sh::JT, NIT = Sh::NIT, ITW = Sh::ITW, TH = Sh::TH, KS = Sh::KS, RW = Sh::RW;
    constexpr int NPP = (P == 2) ? 4 : 1;
    constexpr int GF4 = group_f4<P, WM>();
    // half-split: the row-pass operand and the passes' addresses are loaded and
    // computed for each spectrum instead of being kept in registers
    constexpr bool LOW = Sh::HS;
    constexpr int HH = Sh::HS ? 1 : 2;   // outputs of a pair that a wave computes
    // persistent, XCD-aware: consecutive runs (mostly the same channel) share an XCD's L2
    const int b = blockIdx.x;
    const int g = (b & 7) * a.wg_per_xcd + (b >> 3);
    if (g >= a.grid_wg) return;
    const int64_t T = a.T;
    const PartSplit ps = part_split(g, a.grid_wg, KS);
    const int kpart = ps.kpart;
    const int64_t total = (int64_t)a.C * T;   // this column part's (channel, spectrum) sequence
    const int64_t L = (total + ps.Gp - 1) / ps.Gp;
    int64_t k0, k1;
    owned_range(ps.gp, L, 0, 1, total, &k0, &k1);
    if (k0 >= k1) return;

    extern __shared__ __align__(16) unsigned char smem[];
    const int AP = a.A * P;
    _Float16* s_A1 = reinterpret_cast<_Float16*>(smem + a.off_A1);
    _Float16* s_B2 = reinterpret_cast<_Float16*>(smem + a.off_B2);
    float neg1 = -1.0f;
    asm volatile("" : "+s"(neg1));   // see put_part

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, l4 = lane >> 4;
    const int jt = wave % JT, cg = wave / JT;          // column pass: row-pair tile, column group
    const int cgt = Sh::HS ? 0 : cg * ITW;             // first column tile
    const int itile = wave % NIT, mt0 = wave / NIT;    // row pass: column-pair tile, first row tile

    // DFT operands (the same lane layout serves as either MFMA operand)
    // CHAIN: C, C with (-1)^n in row 0, S, -S; else C, S with (-1)^n in row 0
    half8 fd[LOW ? 3 : Sh::PL][ST], rd[Sh::SHARE || LOW ? 1 : Sh::PL][Sh::SHARE || LOW ? 1 : ST];
    {
        constexpr int plane = Sh::TR * 32 * ST;
        const _Float16* row = a.dft + (16 * jt + l16) * 32 * ST + 8 * l4;
#pragma unroll
        for (int q = 0; q < (LOW ? 3 : Sh::PL); ++q) {
            // half-split, output h = cg: C or C', the factor of Im v in the real
            // part (-S or S) and of Re v in the imaginary part (S or -S)
            const int pl = LOW ? (q == 0 ? cg : (q == 1 ? 3 - cg : 2 + cg)) : q;
#pragma unroll
            for (int ks = 0; ks < ST; ++ks) fd[q][ks] = *reinterpret_cast<const half8*>(row + pl * plane + 32 * ks);
        }
    }
    // row-pass operand of a split workgroup (LOW: from L2 for each spectrum)
    auto load_rd = [&](auto& dst) {
        constexpr int plane = Sh::TR * 32 * ST;
        const int ol = LOW ? opaque(lane) : lane;
        const _Float16* rrow = a.dft + (kpart * NKH + 16 * itile + (ol & 15)) * 32 * ST + 8 * (ol >> 4);
#pragma unroll
        for (int q = 0; q < Sh::PL; ++q)
#pragma unroll
            for (int ks = 0; ks < ST; ++ks) dst[q][ks] = *reinterpret_cast<const half8*>(rrow + q * plane + 32 * ks);
    };
    if constexpr (!Sh::SHARE && !LOW) load_rd(rd);
    // operand position of the lane's eight depth elements per step, cyclic in
    // the stored parts (beyond the depth the DFT operand is zero)
    auto pos_at = [&](int ks, int lq) {
        int q = 32 * ks + 8 * lq;
        if (q >= SD) q -= SD;
        if (q >= SD) q -= SD;
        if (q >= SD) q -= SD;
        return q;
    };
    int pos[ST];
#pragma unroll
    for (int ks = 0; ks < ST; ++ks) pos[ks] = pos_at(ks, l4);
    auto pos_of = [&](int ks, int lq) { return LOW ? pos_at(ks, lq) : pos[ks]; };

    // Decoding runs on the workgroup's last waves, a 32-bit word (four samples)
    // per lane: the first waves carry the longest gather chains and the row
    // pass.  A row that starts at no word boundary is read as the words that
    // hold it, shifted together.  Lanes past the row's end read its last words
    // again and a word's samples past the end are never used, so the loads have
    // no branch and stay in flight until the next spectrum's decoding.
    constexpr int kPre = 2;   // words per lane loaded a spectrum ahead (more are loaded directly)
    const int nwords = (AP + 3) >> 2;
    const int dw0 = 64 * (Sh::WAVES - 1 - wave);   // the wave's first word
    const bool dwave = dw0 < nwords;
    uint32_t pre[kPre], pre_hi[kPre];
    const int64_t row_stride = (int64_t)a.C * AP;   // bytes from one spectrum to the next
    auto word = [&](const uint8_t* row, int w) {   // (second << 32 | first) words holding samples 4 w ..
        const int m = (int)(reinterpret_cast<uintptr_t>(row) & 3);
        const uint32_t* q = reinterpret_cast<const uint32_t*>(row - m);
        const int last = (m + AP - 1) >> 2;
        return make_uint2(q[w], q[w + 1 < last ? w + 1 : last]);
    };
    auto prefetch = [&](const uint8_t* row) {
        const int ln = opaque(tid) & 63;
#pragma unroll
        for (int k = 0; k < kPre; ++k) {
            const int w = dw0 + k * TH + ln;
            const uint2 x = word(row, w < nwords ? w : nwords - 1);
            pre[k] = x.x;
            pre_hi[k] = x.y;
        }
    };
    // decode the row into the sample buffer: the prefetched words first, any
    // further words straight from memory
    auto decode = [&](const uint8_t* row) {
        uint4* dst = reinterpret_cast<uint4*>(smem);
        const int m = (int)(reinterpret_cast<uintptr_t>(row) & 3);
        const int ln = opaque(tid) & 63;
#pragma unroll
        for (int k = 0; k < kPre; ++k) {
            const int w = dw0 + k * TH + ln;
            if (w < nwords) dst[w] = unpack44_h4(__builtin_amdgcn_alignbyte(pre_hi[k], pre[k], m), a.nibble_order);
        }
        for (int w = dw0 + kPre * TH + ln; w < nwords; w += TH) {
            const uint2 x = word(row, w);
            dst[w] = unpack44_h4(__builtin_amdgcn_alignbyte(x.y, x.x, m), a.nibble_order);
        }
    };

    int c = (int)(k0 / T);
    int64_t t = k0 - (int64_t)c * T;
    const uint8_t* row = a.samples + (t * a.C + c) * AP;   // the spectrum to decode next
    if (dwave) prefetch(row);
    for (int64_t f = k0; f < k1;) {
        // one channel segment: spectra t .. t+n-1 of channel c
        const int64_t n = (k1 - f < T - t) ? k1 - f : T - t;
        const int slot = slot_of(ps.gp, c, t, T, 0, 1, L);
        const ChanInfo ci = a.chans[c];
        const int n_cell = ci.n_cell;
        const int R4 = (ci.R + 3) & ~3;
        const int M1 = P * R4;
        const CellDesc* g_desc = a.desc + ci.cell_off;
        const uint2* g_ant = a.grp_ant + 64 * (int64_t)ci.grp_off;
        const float4* g_w = a.grp_w + 64 * (int64_t)ci.grp_off * GF4;
        // with products of three steps and more, or a row-pass operand of its own,
        // registers are too few to keep what a lane number gives in this segment's
        // loads over the whole kernel (N = 192, 44 x 44 cells, both pols: 720 us
        // with, 509 without; N = 96, 8 x 8 cells, 1000 antennas 177 and 152; station,
        // two steps: 564 with, 575 without)
        const int ls = ST > 2 || !Sh::SHARE ? opaque(lane) : lane;
        // the rows' bounds, a lane each, are loaded here and reduced after the
        // copies below
        float most = 0.f;
        if constexpr (SPLIT) most = a.row_bound[(int64_t)c * kRowBounds * P + (ls & (kRowBounds * P - 1))];
        CellDesc d0 = make_uint2(0u, 0u);   // of the wave's first slice
        if (64 * wave < n_cell) d0 = g_desc[64 * wave + ls];
        __syncthreads();   // the previous segment is done with every LDS buffer
        const int ptid = opaque(tid);
        if constexpr (PROG) {
            uint4* s_ant = reinterpret_cast<uint4*>(smem + a.off_ant);
            float4* s_w = reinterpret_cast<float4*>(smem + a.off_w);
            constexpr uint32_t B = 4 * P;   // bytes per antenna
            const uint32_t s0 = lds_address(smem);
            for (int k = ptid; k < ci.n_grp; k += TH) {
                const uint2 o = g_ant[k];
                s_ant[k] = make_uint4(s0 + (o.x & 0xFFFFu) * B, s0 + (o.x >> 16) * B, s0 + (o.y & 0xFFFFu) * B,
                                      s0 + (o.y >> 16) * B);
#pragma unroll
                for (int q = 0; q < GF4; ++q)   // a slice's 64 lanes side by side per weight word
                    s_w[((k >> 6) * GF4 + q) * 64 + (k & 63)] = g_w[(int64_t)k * GF4 + q];
            }
        }
        {
            CellDesc* s_desc = reinterpret_cast<CellDesc*>(smem + a.off_desc);
            for (int k = ptid; k < ((n_cell + 63) & ~63); k += TH) s_desc[k] = g_desc[k];
        }
        // zero both operand buffers: cells outside the window, rows beyond R
        // and the padding up to whole MFMA steps are never written again
        {
            uint4* z1 = reinterpret_cast<uint4*>(s_A1);
            for (int k = ptid; k < a.M1max * PITCH / 8; k += TH) z1[k] = make_uint4(0, 0, 0, 0);
            uint4* z2 = reinterpret_cast<uint4*>(s_B2);
            for (int k = ptid; k < P * NKP * PITCH / 8; k += TH) z2[k] = make_uint4(0, 0, 0, 0);
        }
        float acc[ITW][4][HH][NPP];   // column tile, row 4 l4 + e of the pair tile, j or N - j, product
#pragma unroll
        for (int it = 0; it < ITW; ++it)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int h = 0; h < HH; ++h)
#pragma unroll
                    for (int k = 0; k < NPP; ++k) acc[it][e][h][k] = 0.f;

        // decode the segment's first spectrum (each next one is decoded while
        // the current one is transformed)
        // the row after `row` in the workgroup's run (its last row again at the end)
        auto next_row = [&](int64_t tn, int64_t left) {
            if (left <= 0) return row;
            return tn < T ? row + row_stride : a.samples + (int64_t)(c + 1) * AP;
        };
        {
            const uint8_t* nx = next_row(t + 1, k1 - f - 1);
            if (dwave) {
                decode(row);
                prefetch(nx);
            }
            row = nx;
        }
        float sx = 1.f, sy = 1.f;   // scale of the gridded values per pol
        if constexpr (SPLIT) {
#pragma unroll
            for (int x = P; x < kRowBounds * P; x *= 2) most = fmaxf(most, __shfl_xor(most, x));
            sx = pair_scale(__builtin_amdgcn_readlane(__float_as_int(most), 0));
            sy = pair_scale(__builtin_amdgcn_readlane(__float_as_int(most), P - 1));
        }
        asm volatile("" : "+v"(d0.x), "+v"(d0.y));   // arrived before the loop
        __syncthreads();

        for (int64_t i = 0; i < n; ++i) {
            // Wave priorities: the latency-bound gathering and row pass ahead
            // of the column pass of a CU's other workgroups.
            __builtin_amdgcn_s_setprio(2);
            // 2. gather gridding (FP32), stored as the row-pass operand: row
            //    p R4 + r, columns [Re G(r, 0..) | Im G(r, 0..)]
            pair_gather<Sh, P, WM, PROG>(smem, a, g_ant, g_w, wave, opaque(lane), d0, n_cell, R4 * PITCH, sx, sy, neg1,
                                         s_A1);
            half8 rl[LOW ? Sh::PL : 1][LOW ? ST : 1];
            if constexpr (LOW) load_rd(rl);   // arrives across the barrier
            __syncthreads();

            __builtin_amdgcn_s_setprio(1);
            // 1'. decode the next spectrum of this segment (every gather read of
            //     the current one is done; the next barrier orders it before
            //     the next gather)
            if (i + 1 < n) {
                const uint8_t* nx = next_row(t + i + 2, k1 - f - i - 2);
                if (dwave) {
                    decode(row);
                    prefetch(nx);
                }
                row = nx;
            }
            // 3a. row pass: rows 16 mt.. of the window times the column pairs of
            //     itile -> column-pass operand, column li: pair li of this part,
            //     NKH + li: its partner; [Re Y(0..) | Im Y(0..)]
            const int p16 = LOW ? opaque(l16) : l16, p4 = LOW ? opaque(l4) : l4;
            for (int mt = wave < RW ? mt0 : 64; 16 * mt < M1; mt += RW / NIT) {
                const _Float16* src = s_A1 + (16 * mt + p16) * PITCH;
                half8 ar[ST], ai[ST];
#pragma unroll
                for (int ks = 0; ks < ST; ++ks) {
                    ar[ks] = *reinterpret_cast<const half8*>(src + pos_of(ks, p4));
                    ai[ks] = *reinterpret_cast<const half8*>(src + SD + pos_of(ks, p4));
                }
                const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
                floatx4 yr = zero, yi = zero, zr = zero, zi = zero;   // pair li and its partner
                if constexpr (Sh::CHAIN) {
                    auto op = [&](int q, int ks) {
                        if constexpr (LOW) return rl[q][ks];
                        else return fd[q][ks];
                    };
#pragma unroll
                    for (int ks = 0; ks < ST; ++ks) {
                        yr = mfma16(ar[ks], op(0, ks), yr);
                        zr = mfma16(ar[ks], op(1, ks), zr);
                        yi = mfma16(ar[ks], op(2, ks), yi);
                        zi = mfma16(ar[ks], op(3, ks), zi);
                    }
#pragma unroll
                    for (int ks = 0; ks < ST; ++ks) {
                        yr = mfma16(ai[ks], op(3, ks), yr);
                        zr = mfma16(ai[ks], op(2, ks), zr);
                        yi = mfma16(ai[ks], op(0, ks), yi);
                        zi = mfma16(ai[ks], op(1, ks), zi);
                    }
                } else {
                    floatx4 p1 = zero, p2 = zero, p3 = zero, p4 = zero;
#pragma unroll
                    for (int ks = 0; ks < ST; ++ks) {
                        half8 oc, os;
                        if constexpr (Sh::SHARE) { oc = fd[0][ks]; os = fd[1][ks]; }
                        else { oc = rd[0][ks]; os = rd[1][ks]; }
                        p1 = mfma16(ar[ks], oc, p1);
                        p3 = mfma16(ar[ks], os, p3);
                        p2 = mfma16(ai[ks], os, p2);
                        p4 = mfma16(ai[ks], oc, p4);
                    }
                    yr = p1 - p2; yi = p3 + p4; zr = p1 + p2; zi = p4 - p3;
                    if (kpart == 0 && itile == 0 && p16 == 0) {   // pair 0: bins 0 and N/2
                        yr = p1; yi = p4; zr = p3; zi = p2;
                    }
                }
                const int m0 = 16 * mt + 4 * p4;
                const int li = 16 * itile + p16;
                if (m0 < M1 && (NKH % 16 == 0 || li < NKH)) {
                    const int p = (P == 2 && m0 >= R4) ? 1 : 0;
                    _Float16* dst = s_B2 + (p * NKP + li) * PITCH + (m0 - p * R4);
                    put_part4<SPLIT, WD>(dst, yr, neg1);
                    put_part4<SPLIT, WD>(dst + SD, yi, neg1);
                    put_part4<SPLIT, WD>(dst + NKH * PITCH, zr, neg1);
                    put_part4<SPLIT, WD>(dst + NKH * PITCH + SD, zi, neg1);
                }
            }
            __syncthreads();

            __builtin_amdgcn_s_setprio(0);
            // 3b + 4. column pass, both pols, products of Eq. 5 into registers
            const int c16 = LOW ? opaque(l16) : l16, c4 = LOW ? opaque(l4) : l4;
#pragma unroll
            for (int it = 0; it < ITW; ++it) {
                if (Sh::NCT % ITW != 0 && cgt + it >= Sh::NCT) break;
                if (ITW > 1) __builtin_amdgcn_sched_barrier(0);   // one tile's temporaries at a time
                floatx4 er[P][HH], ei[P][HH];
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    const _Float16* src = s_B2 + (p * NKP + 16 * (cgt + it) + c16) * PITCH;
                    const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
                    if constexpr (Sh::HS) {
                        floatx4 yr = zero, yi = zero;
#pragma unroll
                        for (int ks = 0; ks < ST; ++ks) {
                            const half8 br = *reinterpret_cast<const half8*>(src + pos_of(ks, c4));
                            const half8 bi = *reinterpret_cast<const half8*>(src + SD + pos_of(ks, c4));
                            yr = mfma16(fd[0][ks], br, yr);
                            yi = mfma16(fd[2][ks], br, yi);
                            yr = mfma16(fd[1][ks], bi, yr);
                            yi = mfma16(fd[0][ks], bi, yi);
                        }
                        er[p][0] = yr; ei[p][0] = yi;
                    } else if constexpr (Sh::CHAIN) {
                        floatx4 yr = zero, yi = zero, zr = zero, zi = zero;
                        half8 bi[ST];
#pragma unroll
                        for (int ks = 0; ks < ST; ++ks) {
                            const half8 br = *reinterpret_cast<const half8*>(src + pos_of(ks, c4));
                            bi[ks] = *reinterpret_cast<const half8*>(src + SD + pos_of(ks, c4));
                            yr = mfma16(fd[0][ks], br, yr);
                            zr = mfma16(fd[1][ks], br, zr);
                            yi = mfma16(fd[2][ks], br, yi);
                            zi = mfma16(fd[3][ks], br, zi);
                        }
#pragma unroll
                        for (int ks = 0; ks < ST; ++ks) {
                            yr = mfma16(fd[3][ks], bi[ks], yr);
                            zr = mfma16(fd[2][ks], bi[ks], zr);
                            yi = mfma16(fd[0][ks], bi[ks], yi);
                            zi = mfma16(fd[1][ks], bi[ks], zi);
                        }
                        er[p][0] = yr; ei[p][0] = yi; er[p][1] = zr; ei[p][1] = zi;
                    } else {
                        floatx4 p1 = zero, p2 = zero, p3 = zero, p4 = zero;
#pragma unroll
                        for (int ks = 0; ks < ST; ++ks) {
                            const half8 br = *reinterpret_cast<const half8*>(src + pos_of(ks, c4));
                            const half8 bi = *reinterpret_cast<const half8*>(src + SD + pos_of(ks, c4));
                            p1 = mfma16(fd[0][ks], br, p1);
                            p3 = mfma16(fd[1][ks], br, p3);
                            p2 = mfma16(fd[1][ks], bi, p2);
                            p4 = mfma16(fd[0][ks], bi, p4);
                        }
                        er[p][0] = p1 - p2;
                        ei[p][0] = p3 + p4;
                        er[p][1] = p1 + p2;
                        ei[p][1] = p4 - p3;
                        if (jt == 0 && c4 == 0) {   // pair 0 (element 0): bins 0 and N/2
                            er[p][0][0] = p1[0];
                            ei[p][0][0] = p4[0];
                            er[p][1][0] = p3[0];
                            ei[p][1][0] = p2[0];
                        }
                    }
                }
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int h = 0; h < HH; ++h) {
                        const float xr = er[0][h][e], xi = ei[0][h][e];
                        float (&s)[NPP] = acc[it][e][h];
                        s[0] = fmaf(xr, xr, fmaf(xi, xi, s[0]));
                        if constexpr (P == 2) {
                            const float yr = er[1][h][e], yi = ei[1][h][e];
                            s[1] = fmaf(yr, yr, fmaf(yi, yi, s[1]));
                            s[2] = fmaf(xr, yr, fmaf(xi, yi, s[2]));
                            s[3] = fmaf(xi, yr, fmaf(-xr, yi, s[3]));
                        }
                    }
            }
        }

        // add the segment's sums into its slot; bin -> pixel (+N/2 mod N)
        {
            float ux = 1.f, uy = 1.f;   // inverse scales of the two fields
            if constexpr (SPLIT) {
                ux = 1.0f / (sx * (kDftScale * kDftScale));
                uy = 1.0f / (sy * (kDftScale * kDftScale));
            }
            float* base = a.slots + ((int64_t)slot * a.C + c) * NPP * N * N;
            const int fl = opaque(lane), f16 = fl & 15, f4 = fl >> 4;
#pragma unroll
            for (int it = 0; it < ITW; ++it) {
                const int li = 16 * (cgt + it) + f16;
                if (!Sh::HS && Sh::CG * ITW * 16 != NK && li >= NK) continue;
                const int q = li < NKH ? li : li - NKH;
                const int i = kpart * NKH + q;
                const int kx = li < NKH ? i : (i == 0 ? N / 2 : N - i);
                const int ii = kx + N / 2 < N ? kx + N / 2 : kx - N / 2;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int j = 16 * jt + 4 * f4 + e;
                    if (Sh::NH % 16 != 0 && j >= Sh::NH) continue;
#pragma unroll
                    for (int h = 0; h < HH; ++h) {
                        const int ky = (Sh::HS ? cg : h) == 0 ? j : (j == 0 ? N / 2 : N - j);
                        const int jj = ky + N / 2 < N ? ky + N / 2 : ky - N / 2;
                        float* px = base + (int64_t)jj * N + ii;
#pragma unroll
                        for (int k = 0; k < NPP; ++k) {
                            float v = acc[it][e][h][k];
                            if constexpr (SPLIT) v = (v * ((k == 1) ? uy : ux)) * ((k == 0) ? ux : uy);
                            slot_put(px + (int64_t)k * N * N, v, a.fresh != 0);
                        }
                    }
                }
            }
        }
        f += n;
        ++c;
        t = 0;
    }
}

// Planes of the DFT operand [TR][32 ST]: element (j, k) holds cos / sin
// (2 pi j n / N), n the window position of depth k, evaluated in FP64; split:
// times 16, hi for the first two terms and lo for the third.  Two planes: C, and
// S whose row 0 holds (-1)^n; four (chained products): C, C whose row 0 holds
// (-1)^n, S, -S.  Rows beyond N/2 and depth beyond the terms are 0.
__global__ void pair_table_kernel(_Float16* __restrict__ m, int N, int WD, int split, int planes, int rows,
                                  int depth32) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= planes * rows * depth32) return;
    const int plane = idx / (rows * depth32);
    const int j = (idx / depth32) % rows, k = idx % depth32;
    const int n = k % WD, term = k / WD;
    double v = 0.0;
    if (term < (split ? 3 : 1) && j < N / 2) {
        double s, c;
        sincospi(2.0 * (double)((int64_t)j * n % N) / (double)N, &s, &c);
        if (plane == 0) v = c;
        else if (plane == 1) v = j == 0 ? ((n & 1) ? -1.0 : 1.0) : (planes == 4 ? c : s);
        else v = plane == 2 ? s : -s;
        if (split) {
            v *= (double)kDftScale;
            const double hi = (double)(_Float16)v;
            v = term == 2 ? v - hi : hi;
        }
    }
    m[idx] = (_Float16)v;
}

// ---- launch shapes -----------------------------------------------------------
// Host view of PairShape.
struct PairDims {
    int WD, SD, ST, PITCH, KS, NKP, TR, TH, PL;
};

PairDims pair_dims(int N, int WD, bool split, int P) {
    PairDims d{};
    d.WD = WD;
    d.SD = split ? 2 * WD : WD;
    d.ST = ((split ? 3 * WD : WD) + 31) / 32;
    d.PITCH = ((2 * d.SD / 8) | 1) * 8;
    const bool hs = pair_half(N, split, P, WD);
    d.PL = (pair_ks(N, split, P, WD) == 1 && d.ST == 1) || hs ? 4 : 2;
    d.KS = pair_ks(N, split, P, WD);
    const int NK = N / d.KS, NCT = (NK + 15) / 16, NIT = (NK / 2 + 15) / 16, JT = (N / 2 + 15) / 16;
    const int ITW = pair_itw(N, split, P, WD);
    d.NKP = 16 * NCT;
    d.TR = std::max(16 * JT, (d.KS - 1) * (NK / 2) + 16 * NIT);
    d.TH = 64 * JT * (hs ? 2 : (NCT + ITW - 1) / ITW);
    return d;
}

// Window sizes compiled per form: FP32, the largest of each count of MFMA steps;
// FP16, 16 to 32 (one step) and 48, 64 (two), which differ in LDS.
int pair_wd(int need, bool split) {
    if (split) {
        for (int w : {8, 20, 32, 40, 52, 64})
            if (need <= w) return w;
    } else {
        for (int w : {16, 24, 32, 48, 64})
            if (need <= w) return w;
    }
    return 0;
}

struct PairLayout {
    uint32_t off_w, off_ant, off_desc, off_A1, off_B2;
    int M1max;
    size_t total;
};

PairLayout pair_layout(const SubDev& d, bool prog) {
    const PairDims s = pair_dims(d.N, d.pair_wd, d.precision == EPIC_FP32, d.P);
    PairLayout L{};
    size_t b = 0;
    auto take = [&](size_t n) {
        b = (b + 15) & ~(size_t)15;
        const size_t o = b;
        b += n;
        return (uint32_t)o;
    };
    const int gf4 = group_f4_of(d.P, d.wmode);
    L.M1max = (d.P * d.R4max + 15) / 16 * 16;
    (void)take((size_t)((d.A * d.P + 3) & ~3) * 4);   // the decoded samples, at 0
    L.off_w = prog ? take((size_t)d.pair_gmax * gf4 * 16) : 0;
    L.off_ant = prog ? take((size_t)d.pair_gmax * 16) : 0;
    L.off_desc = take((size_t)((d.CellMax + 63) & ~63) * 8);
    L.off_A1 = take((size_t)L.M1max * s.PITCH * 2);
    L.off_B2 = take((size_t)d.P * s.NKP * s.PITCH * 2);
    L.total = (b + 15) & ~(size_t)15;
    return L;
}

using KernelFn = void (*)(PairArgs);

// FP32, N = 192, both pols, windows beyond 52 cells: more than 90 of twelve waves'
// registers spill (62 antennas, 16 channels x 200 spectra: 834 us, the vector
// kernel 735), so there are no such instances.
constexpr bool pair_spills(int N, bool split, int P, int WD) { return split && N == 192 && P == 2 && WD > 52; }

template <int N, int WD, bool SPLIT, bool PROG>
KernelFn pair_pick2(int P, int wm) {
    if (P == 2) {
        if constexpr (pair_spills(N, SPLIT, 2, WD)) {
            return nullptr;
        } else {
            if (wm == kWComplex) return pair_kernel<N, WD, 2, kWComplex, SPLIT, PROG>;
            return wm == kWShared ? pair_kernel<N, WD, 2, kWShared, SPLIT, PROG> : pair_kernel<N, WD, 2, kWReal, SPLIT, PROG>;
        }
    }
    return wm == kWComplex ? pair_kernel<N, WD, 1, kWComplex, SPLIT, PROG> : pair_kernel<N, WD, 1, kWReal, SPLIT, PROG>;
}

template <int N, int WD, bool SPLIT>
void* pair_pick(int P, int wm, bool prog) {
    return reinterpret_cast<void*>(prog ? pair_pick2<N, WD, SPLIT, true>(P, wm) : pair_pick2<N, WD, SPLIT, false>(P, wm));
}

constexpr size_t kLdsLimit = 160 * 1024;

}  // namespace

// The instances are spread over several translation units of this file, each
// compiled with EPIC_PAIR_UNIT = 0, 1, ...; unit 0 also holds the host side.
// A grid holds windows up to its own side, in the smallest compiled size that
// fits them: 32 at N = 32, FP32 52 and FP16 48 at N = 48.
#define EPIC_PAIR_CASE(NN, WD, SPLIT) \
    case NN * 64 + (WD == 64 ? 63 : WD): return pair_pick<NN, WD, SPLIT>(P, wm, prog);
#define EPIC_PAIR_SPLIT32(NN) EPIC_PAIR_CASE(NN, 8, true) EPIC_PAIR_CASE(NN, 20, true) EPIC_PAIR_CASE(NN, 32, true)
#define EPIC_PAIR_SPLIT52(NN) EPIC_PAIR_SPLIT32(NN) EPIC_PAIR_CASE(NN, 40, true) EPIC_PAIR_CASE(NN, 52, true)
#define EPIC_PAIR_SPLIT64(NN) EPIC_PAIR_SPLIT52(NN) EPIC_PAIR_CASE(NN, 64, true)
#define EPIC_PAIR_HALF32(NN) EPIC_PAIR_CASE(NN, 16, false) EPIC_PAIR_CASE(NN, 24, false) EPIC_PAIR_CASE(NN, 32, false)
#define EPIC_PAIR_HALF48(NN) EPIC_PAIR_HALF32(NN) EPIC_PAIR_CASE(NN, 48, false)
#define EPIC_PAIR_HALF64(NN) EPIC_PAIR_HALF48(NN) EPIC_PAIR_CASE(NN, 64, false)

#define EPIC_PAIR_SELECT(NAME, CASES)                       \
    void* NAME(int key, int P, int wm, bool prog) {         \
        switch (key) { CASES }                              \
        return nullptr;                                     \
    }

#if EPIC_PAIR_UNIT == 0
EPIC_PAIR_SELECT(pair_select_split_32, EPIC_PAIR_SPLIT32(32) EPIC_PAIR_SPLIT52(48))
#elif EPIC_PAIR_UNIT == 1
EPIC_PAIR_SELECT(pair_select_split_64, EPIC_PAIR_SPLIT64(64))
#elif EPIC_PAIR_UNIT == 2
EPIC_PAIR_SELECT(pair_select_split_96, EPIC_PAIR_SPLIT64(96))
#elif EPIC_PAIR_UNIT == 3
EPIC_PAIR_SELECT(pair_select_split_128, EPIC_PAIR_SPLIT64(128))
#elif EPIC_PAIR_UNIT == 4
EPIC_PAIR_SELECT(pair_select_split_192, EPIC_PAIR_SPLIT64(192))
#elif EPIC_PAIR_UNIT == 5
EPIC_PAIR_SELECT(pair_select_split_256, EPIC_PAIR_SPLIT64(256))
#elif EPIC_PAIR_UNIT == 6
EPIC_PAIR_SELECT(pair_select_half_small, EPIC_PAIR_HALF32(32) EPIC_PAIR_HALF48(48) EPIC_PAIR_HALF64(64))
#elif EPIC_PAIR_UNIT == 7
EPIC_PAIR_SELECT(pair_select_half_large, EPIC_PAIR_HALF64(96) EPIC_PAIR_HALF64(128) EPIC_PAIR_HALF64(192) EPIC_PAIR_HALF64(256))
#endif

#if EPIC_PAIR_UNIT == 0
#define EPIC_PAIR_DECL(NAME) void* NAME(int key, int P, int wm, bool prog);
EPIC_PAIR_DECL(pair_select_split_64) EPIC_PAIR_DECL(pair_select_split_96) EPIC_PAIR_DECL(pair_select_split_128)
EPIC_PAIR_DECL(pair_select_split_192) EPIC_PAIR_DECL(pair_select_split_256) EPIC_PAIR_DECL(pair_select_half_small)
EPIC_PAIR_DECL(pair_select_half_large)

namespace {
const void* pair_select(const SubDev& d) {
    const int key = d.N * 64 + (d.pair_wd == 64 ? 63 : d.pair_wd);
    const bool prog = d.prog_lds != 0;
    if (d.precision != EPIC_FP32)
        return d.N <= 64 ? pair_select_half_small(key, d.P, d.wmode, prog) : pair_select_half_large(key, d.P, d.wmode, prog);
    switch (d.N) {
        case 32: case 48: return pair_select_split_32(key, d.P, d.wmode, prog);
        case 64: return pair_select_split_64(key, d.P, d.wmode, prog);
        case 96: return pair_select_split_96(key, d.P, d.wmode, prog);
        case 128: return pair_select_split_128(key, d.P, d.wmode, prog);
        case 192: return pair_select_split_192(key, d.P, d.wmode, prog);
        default: return pair_select_split_256(key, d.P, d.wmode, prog);
    }
}
}  // namespace

// Launch shape: grids of 32..128 (multiples of 16, not 80 / 112), 192 and 256
// with windows of at most 64 cells whose operands fit LDS; the gather program in
// LDS unless that costs a resident workgroup, else streamed from L2.
hipError_t pair_configure(SubDev& d, int device, int num_cu, int force_prog) {
    const bool grid_ok = d.N == 32 || d.N == 48 || d.N == 64 || d.N == 96 || d.N == 128 || d.N == 192 || d.N == 256;
    if (!grid_ok) return hipErrorNotSupported;
    const bool split = d.precision == EPIC_FP32;
    d.pair_wd = pair_wd(std::max(d.R4max, d.W4max), split);
    if (d.pair_wd == 0) return hipErrorNotSupported;
    if (pair_spills(d.N, split, d.P, d.pair_wd)) return hipErrorNotSupported;
    const PairDims s = pair_dims(d.N, d.pair_wd, split, d.P);
    const PairLayout with = pair_layout(d, true), without = pair_layout(d, false);
    // workgroups per CU with the program in LDS or streamed (device < 0: by LDS only)
    int occ[2] = {0, 0};   // streamed, in LDS
    for (int pl = 0; pl < 2; ++pl) {
        const PairLayout& L = pl ? with : without;
        if (L.total > kLdsLimit) continue;
        SubDev t = d;
        t.prog_lds = pl;
        const int by_lds = (int)(kLdsLimit / L.total);
        occ[pl] = by_lds > 2 ? 2 : by_lds;
        if (device < 0) continue;
        const void* fn = pair_select(t);
        if (!fn) return hipErrorNotSupported;
        hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsLimit);
        if (e != hipSuccess) return e;
        int blocks = 0;
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, fn, s.TH, L.total);
        if (e != hipSuccess) return e;
        // Workgroups of six or nine waves are counted as if their waves filled the
        // SIMDs' slots evenly; what runs side by side is what fits with the odd
        // waves on the same SIMDs.  The rest would wait for a second round of the
        // persistent launch (N = 48, single pol, 18 x 18 cells, 16 channels x 301
        // spectra: 39.8 us for the three counted, 29.8 for two; N = 96, 8 x 8 cells,
        // 1000 antennas: 355 us for two, 164 for one).
        const int waves = s.TH / 64;
        if (waves > 4 && waves % 4 != 0) {
            hipFuncAttributes at{};
            if ((e = hipFuncGetAttributes(&at, fn)) != hipSuccess) return e;
            const int slots = std::min(8, 512 / ((std::max(at.numRegs, 1) + 7) / 8 * 8));   // waves per SIMD
            blocks = std::min(blocks, slots / ((waves + 3) / 4));
        }
        occ[pl] = blocks > 0 ? blocks : 1;
    }
    // the program in LDS unless that costs a resident workgroup
    const bool prog = force_prog < 0 ? occ[1] > 0 && occ[1] >= occ[0] : force_prog != 0;
    if (occ[prog ? 1 : 0] == 0) return hipErrorNotSupported;
    d.pair = 1;
    d.prog_lds = prog ? 1 : 0;
    d.KS = s.KS;
    d.threads = s.TH;
    d.lds_bytes = (prog ? with : without).total;
    d.grid_wg = num_cu * occ[prog ? 1 : 0] / d.KS * d.KS;
    return hipSuccess;
}

int pair_pitch(const SubDev& d) { return pair_dims(d.N, d.pair_wd, d.precision == EPIC_FP32, d.P).PITCH; }

int64_t pair_table_halfs(const SubDev& d) {
    const PairDims s = pair_dims(d.N, d.pair_wd, d.precision == EPIC_FP32, d.P);
    return (int64_t)s.PL * s.TR * 32 * s.ST;
}

hipError_t launch_pair_table(const SubDev& d, hipStream_t st) {
    const PairDims s = pair_dims(d.N, d.pair_wd, d.precision == EPIC_FP32, d.P);
    const int n = s.PL * s.TR * 32 * s.ST;
    pair_table_kernel<<<dim3((n + 255) / 256), dim3(256), 0, st>>>(reinterpret_cast<_Float16*>(d.pair_dft), d.N, s.WD,
                                                                   d.precision == EPIC_FP32, s.PL, s.TR, 32 * s.ST);
    return hipGetLastError();
}

hipError_t launch_pair(const SubDev& d, const uint8_t* samples, int64_t n_time, hipStream_t st) {
    const PairLayout L = pair_layout(d, d.prog_lds != 0);
    PairArgs a{};
    a.samples = samples;
    a.chans = d.pair_chans;
    a.desc = d.pair_desc;
    a.grp_ant = reinterpret_cast<const uint2*>(d.pair_ant);
    a.grp_w = reinterpret_cast<const float4*>(d.pair_w);
    a.dft = reinterpret_cast<const _Float16*>(d.pair_dft);
    a.row_bound = d.use_range ? d.range : d.row_bound;
    a.slots = d.slots;
    a.T = n_time;
    a.C = d.C; a.A = d.A;
    a.M1max = L.M1max;
    a.nibble_order = d.nibble_order; a.fresh = d.fresh;
    a.grid_wg = d.grid_wg;
    a.wg_per_xcd = (d.grid_wg + 7) / 8;
    a.off_w = L.off_w; a.off_ant = L.off_ant; a.off_desc = L.off_desc;
    a.off_A1 = L.off_A1; a.off_B2 = L.off_B2;
    const void* fn = pair_select(d);
    if (!fn) return hipErrorNotSupported;
    hipLaunchKernelGGL(reinterpret_cast<KernelFn>(const_cast<void*>(fn)), dim3(8 * a.wg_per_xcd), dim3(d.threads),
                       L.total, st, a);
    return hipGetLastError();
}
#endif

}  // namespace epic
