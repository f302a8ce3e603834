// Gridding on the matrix cores (EPIC_GRID_BLOCK_GEMM / EPIC_GRID_DENSE_GEMM).
//
// Gridding (Eq. 4: the antenna fields W_a * E_a summed over antennas) of a
// channel is the product G = Wc E of the channel's kernel matrix Wc [cells x
// antennas] with the spectra's fields E [antennas x (spectrum, pol, re/im)].
// With real weights one real product gives both the real and the imaginary
// part of every pol.  The product runs on 16 x 16 x 32 MFMA tiles:
//   rows     16 aperture cells of the channel's window: four quads of four
//            neighbouring cells of a row, in bands of four rows, so that a
//            tile of a filled window is a square of 4 x 4 cells;
//   depth    32 antennas out of the tile's own list, the antennas with a
//            non-zero weight in it (block-sparse form), in raster order of
//            their positions, or of all antennas (dense form);
//   columns  TB spectra x P pols x (re, im) of the current step.
// The weights of the (tile, 32 antennas) blocks are a stream that every step
// reads once, and that stream bounds the form for large arrays: it is as short
// as the footprints let it be, since a square tile meets fewer footprints than
// a strip of 16 cells does, and a list per tile holds no antenna that only its
// neighbour tile needs.  The fields lie in LDS by antenna, a row of TB spectra
// each, and the transposing LDS reads (ds_read_b64_tr) take the rows of any 32
// antennas as the operand of a block.  Measured, 2048 antennas, 256 channels,
// 128 x 128, FP8: strips of cells over shared blocks of 32 antennas 698 blocks
// per channel and 7.60 ms; squares with lists of their own 229 blocks and
// 2.25 ms; with the next step's first entries, samples and row operand on their
// way across the barriers 1.98 ms; with one descriptor load per block and the
// FP8 parts 0 and 1 in one load 1.86 ms.  Of that the gridding product takes
// 0.85 ms (13.8 GB of weights and descriptors per call; 46 % of the requests
// miss the XCD's L2), the readout 0.07 ms and the transforms the rest.
// The weights are split into parts in the
// operand type whose products are summed in FP32: FP16 high + low (~2^-22
// relative), or FP8 e4m3 with a power-of-two scale, high + middle + low, each
// part holding the previous one's rounding error times 16 (<= 2^-12 relative;
// two e4m3 parts leave up to 2^-8, which measurably exceeds the 1e-3 image bar
// for arrays of a few antennas).  The 4-bit samples are exact in either type.
// The gridded cells go
// to the FP16 row-pass operand, and the two transform passes, the products of
// Eq. 5 and the time sums run as in the gather-gridding kernel.
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

// Operand of one 16 x 32 (A) or 32 x 16 (B) block per lane: 8 elements.
template <int OP>
struct Operand;
template <>
struct Operand<kBgFp16> {
    using type = half8;               // 16 bytes
    static constexpr int bytes = 2;
};
template <>
struct Operand<kBgFp8> {
    using type = long;                // 8 bytes of e4m3
    static constexpr int bytes = 1;
};

template <int OP>
__device__ __forceinline__ floatx4 mfma_op(typename Operand<OP>::type a, typename Operand<OP>::type b, floatx4 c) {
    if constexpr (OP == kBgFp16)
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a, b, c, 0, 0, 0);
}

typedef _Float16 half2 __attribute__((ext_vector_type(2)));

// The (re, im) pair of one sample in the field operand: 4-bit integers, exact
// in both types.
template <int OP>
__device__ __forceinline__ uint32_t field_pair(float2 v) {
    if constexpr (OP == kBgFp16) {
        const half2 h = {(_Float16)v.x, (_Float16)v.y};
        return __builtin_bit_cast(uint32_t, h);
    } else {
        return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(v.x, v.y, 0, false) & 0xFFFFu;
    }
}

// Fields of 32 antennas as the 32 x 16 operand, read transposed from rows in
// LDS.  Lanes 16 l4 .. of a read give the addresses of 8 bytes each: of the
// rows of antennas 8 l4 + i, i = (l % 16) / 2, columns 8 (l % 2) .. (FP8), or
// of i = (l % 16) / 4, columns 4 (l % 4) .. (FP16, two reads: i and i + 4).
// Lane l receives column l % 16 of its antennas 8 l4 ...  (Layout verified on
// the device.)
typedef long long2v __attribute__((ext_vector_type(2)));
typedef int int2v __attribute__((ext_vector_type(2)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef short short8v __attribute__((ext_vector_type(8)));

__device__ __forceinline__ long field_block(const unsigned char* row) {
    const int2v r = __builtin_amdgcn_ds_read_tr8_b64_v2i32((__attribute__((address_space(3))) int2v*)row);
    return __builtin_bit_cast(long, r);
}

__device__ __forceinline__ half8 field_block(const unsigned char* row0, const unsigned char* row1) {
    const short4v x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)row0);
    const short4v y = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)row1);
    const short8v r = {x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
    return __builtin_bit_cast(half8, r);
}

// One block entry in flight: its weights, this lane's antennas and the quad of
// cells that the lane's products belong to.
template <int OP, int NTERM>
struct BgEntry {
    typename Operand<OP>::type w[NTERM];
    uint32_t ant, quad;   // FP8: the quad is the high half of ant; FP16: that is the antenna four rows on
};

struct BgArgs {
    const uint8_t* samples;   // [T][C][A][P]
    const ChanInfo* chans;
    const int32_t* waves;     // [C][N / 16 + 1] first block entry of each wave's share
    const uint16_t* desc;     // [entry][64] antennas and cells as the lanes read them
    const unsigned char* w;   // [entry] operand elements (bg_weights_kernel)
    const float* scale;       // [2]: weight scale, its inverse
    const _Float16* dft;      // [2N][K2] real-form DFT matrix
    float* slots;             // [S][C][NPP][N][N]
    int fresh;                // 1: the slots hold zeros, store instead of add
    int64_t T;
    int C, A, nibble_order, TB, V;
    int erow_log2;            // bytes per antenna of the field operand
    uint32_t off_E, off_A1, off_B2;
    int A1rows;               // rows of the A1 region (zeroed per segment)
    int grid_wg, wg_per_xcd;
};

// Register budget: two waves per SIMD for the grids up to 64 with at most two
// MFMA steps (their ~220 live registers fit without spilling: measured at the
// station shape, 1.19 ms with three waves and ~60 spilled registers against
// 0.80 ms with two); the compiler's choice otherwise.
template <int N_, int KK_>
constexpr int bg_waves_per_eu() { return (N_ <= 64 && KK_ <= 2) ? 2 : 1; }

// Block entries of a wave that load together, and (spectrum, antenna) pairs of a
// thread whose samples load ahead (kRawMin of them where a step has no more).
constexpr int kBgFly = 2;
constexpr int kRaw = 8, kRawMin = 2;

template <int N_, int KK_, int P, int OP>
__global__ void __launch_bounds__(mfma_threads<N_>())
__attribute__((amdgpu_waves_per_eu(bg_waves_per_eu<N_, KK_>()))) bg_kernel(BgArgs a) {
    using Sh = MShape<N_, KK_>;
    using Op = typename Operand<OP>::type;
    using Raw = std::conditional_t<P == 2, uint16_t, uint8_t>;
    constexpr int TH = mfma_threads<N_>(), NW = TH / 64;
    constexpr int KS = Sh::KS, KPAD = Sh::KPAD, A1P = Sh::A1P, B2P = Sh::B2P, NK = Sh::NK, IT = Sh::IT;
    constexpr int NPP = (P == 2) ? 4 : 1;
    constexpr int EB = Operand<OP>::bytes;
    constexpr int NTERM = (OP == kBgFp16) ? 2 : 3;
    const int b = blockIdx.x;
    const int g = (b & 7) * a.wg_per_xcd + (b >> 3);
    if (g >= a.grid_wg) return;
    const PartSplit ps = part_split(g, a.grid_wg, KS);
    const int64_t T = a.T;
    const int64_t total = (int64_t)(a.V / KS) * T;   // this column part's (channel, spectrum) sequence
    const int64_t L = (total + ps.Gp - 1) / ps.Gp;
    int64_t k0, k1;
    owned_range(ps.gp, L, 0, 1, total, &k0, &k1);
    if (k0 >= k1) return;

    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* s_E = smem + a.off_E;                                      // [A][columns]
    _Float16* s_A1 = reinterpret_cast<_Float16*>(smem + a.off_A1);
    _Float16* s_B2 = reinterpret_cast<_Float16*>(smem + a.off_B2);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, l4 = lane >> 4;
    const int mw = wave;   // every wave owns 16 image rows
    const int kpart = ps.kpart;

    half8 a2[2][Sh::KK];
    load_col_fragments<Sh>(a2, a.dft, mw, l16, l4);
    float inv_scale = 1.0f;
    if constexpr (OP == kBgFp8) inv_scale = a.scale[1];

    // decode spectra t .. t+nb-1 of channel c into the field operand: column
    // u 2P + 2p + ri of the antenna's row.  Columns from 2 P nb on hold whatever
    // was there: their products are never stored.  The samples of the first kRaw
    // (spectrum, antenna) pairs of a thread are loaded ahead of the transforms
    // and written when the field operand is free; more pairs follow directly.
    const int AP = a.A * P;
    const int el = a.erow_log2;
    const float inv_A = 1.0f / (float)a.A;
    auto pair_of = [&](int k, int& u, int& an) {   // exact: k < 2^17, (k + 1/2) / A is no integer
        u = (int)(((float)k + 0.5f) * inv_A);
        an = k - u * a.A;
    };
    auto load_raw = [&](int cc, int64_t t, int u, int an) {
        const uint8_t* src = a.samples + ((t + u) * a.C + cc) * (int64_t)AP + an * P;
        Raw r;
        __builtin_memcpy(&r, src, sizeof(Raw));   // any byte alignment
        return r;
    };
    auto put_raw = [&](Raw r, int u, int an) {
        uint32_t h[P];
#pragma unroll
        for (int p = 0; p < P; ++p) h[p] = field_pair<OP>(unpack44((uint8_t)(r >> (8 * p)), a.nibble_order));
        unsigned char* q = s_E + u * 2 * P * EB + (an << el);
        if constexpr (EB * P == 4) *reinterpret_cast<uint2*>(q) = make_uint2(h[0], h[P - 1]);
        else if constexpr (EB == 2) *reinterpret_cast<uint32_t*>(q) = h[0];
        else if constexpr (P == 2) *reinterpret_cast<uint32_t*>(q) = h[0] | (h[P - 1] << 16);
        else *reinterpret_cast<uint16_t*>(q) = (uint16_t)h[0];
    };
    Raw raw[kRaw];
    auto load_step = [&](int cc, int64_t t, int nb) {
        const int k0 = opaque(tid);
        auto load = [&](int j) {
            int u, an;
            pair_of(std::min(k0 + j * TH, nb * a.A - 1), u, an);
            raw[j] = load_raw(cc, t, u, an);
        };
#pragma unroll
        for (int j = 0; j < kRawMin; ++j) load(j);
        if (nb * a.A > kRawMin * TH) {
#pragma unroll
            for (int j = kRawMin; j < kRaw; ++j) load(j);
        }
    };
    auto put_step = [&](int cc, int64_t t, int nb) {
        const int k0 = opaque(tid);
        int u, an;
        auto put = [&](int j) {
            const int k = k0 + j * TH;
            pair_of(k, u, an);
            if (k < nb * a.A) put_raw(raw[j], u, an);
        };
#pragma unroll
        for (int j = 0; j < kRawMin; ++j) put(j);
        if (nb * a.A <= kRawMin * TH) return;
#pragma unroll
        for (int j = kRawMin; j < kRaw; ++j) put(j);
        for (int k = k0 + kRaw * TH; k < nb * a.A; k += TH) {
            pair_of(k, u, an);
            put_raw(load_raw(cc, t, u, an), u, an);
        }
    };
    // this lane's part of the antenna list and of an antenna's row (see field_block)
    const int lsub = (OP == kBgFp16) ? 4 * l4 + (l16 >> 2) : 8 * l4 + (l16 >> 1);
    const unsigned char* s_El = s_E + ((OP == kBgFp16) ? 8 * (l16 & 3) : 8 * (l16 & 1)) % (1 << el);
    using Entry = BgEntry<OP, NTERM>;
    auto fetch = [&](int ent, Entry& r) {
        const unsigned char* src = a.w + (size_t)ent * NTERM * 512 * EB;
        if constexpr (OP == kBgFp16) {
#pragma unroll
            for (int h = 0; h < NTERM; ++h) r.w[h] = *reinterpret_cast<const Op*>(src + lane * 16 + h * 1024);
            const uint2 q = *reinterpret_cast<const uint2*>(a.desc + (size_t)ent * 64 + 4 * lsub);
            r.ant = q.x;
            r.quad = q.y;
        } else {
            const long2v w01 = *reinterpret_cast<const long2v*>(src + lane * 16);
            r.w[0] = w01[0];
            r.w[1] = w01[1];
            r.w[2] = *reinterpret_cast<const Op*>(src + 1024 + lane * 8);
            r.ant = *reinterpret_cast<const uint32_t*>(a.desc + (size_t)ent * 64 + 2 * lsub);
        }
    };

    int s_ch = (int)(k0 / T);
    int64_t t = k0 - (int64_t)s_ch * T;
    int v = s_ch * KS + kpart;
    for (int64_t f = k0; f < k1;) {
        const int64_t n = (k1 - f < T - t) ? k1 - f : T - t;
        const int c = v / KS;
        const int slot = slot_of(ps.gp, s_ch, t, T, 0, 1, L);
        const ChanInfo ci = a.chans[c];
        const int ent0 = a.waves[c * (NW + 1) + wave], ent1 = a.waves[c * (NW + 1) + wave + 1];
        const int R4 = (ci.R + 3) & ~3;
        const int M1 = P * R4;
        __syncthreads();   // the previous segment is done with every LDS buffer
        {
            uint4* z1 = reinterpret_cast<uint4*>(s_A1);
            for (int k = tid; k < a.A1rows * A1P / 8; k += TH) z1[k] = make_uint4(0, 0, 0, 0);
            uint4* z2 = reinterpret_cast<uint4*>(s_B2);
            for (int k = tid; k < P * NK * B2P / 8; k += TH) z2[k] = make_uint4(0, 0, 0, 0);
        }
        float acc[IT][4][NPP];
#pragma unroll
        for (int it = 0; it < IT; ++it)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int k = 0; k < NPP; ++k) acc[it][e][k] = 0.f;

        load_step(c, t, (int)std::min<int64_t>(a.TB, n));
        Entry x[kBgFly], y[kBgFly];
        if (ent0 < ent1) {
#pragma unroll
            for (int q = 0; q < kBgFly; ++q) fetch(std::min(ent0 + q, ent1 - 1), x[q]);
        }
        put_step(c, t, (int)std::min<int64_t>(a.TB, n));
        __syncthreads();

        for (int64_t u0 = 0; u0 < n; u0 += a.TB) {
            const int nb = (int)std::min<int64_t>(a.TB, n - u0);
            __builtin_amdgcn_s_setprio(2);
            // 2. gridding product: G rows (cells) x columns (u, p, re/im), over
            //    the wave's share of the channel's block entries, kBgFly of them
            //    loading while the kBgFly before them are multiplied
            if (ent0 < ent1) {
                const int ucol = l16 / (2 * P);
                _Float16* dst = s_A1 + (ucol * M1 + ((P == 2) ? ((l16 >> 1) & 1) * R4 : 0)) * A1P + (l16 & 1) * KPAD;
                floatx4 d[NTERM];
#pragma unroll
                for (int h = 0; h < NTERM; ++h) d[h] = floatx4{0.f, 0.f, 0.f, 0.f};
                bool first = true;   // FP8: the first entry of a tile adds to nothing
                auto multiply = [&](const Entry& r) {
                    const bool last = (__builtin_amdgcn_readfirstlane(r.ant) & kBgLast) != 0;
                    const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
                    const unsigned char* row = s_El + ((r.ant & (kBgLast - 1)) << el);
                    if constexpr (OP == kBgFp16) {
                        const Op eb = field_block(row, s_El + ((r.ant >> 16) << el));
                        d[0] = mfma_op<OP>(r.w[0], eb, d[0]);
                        d[0] = mfma_op<OP>(r.w[1], eb, d[0]);
                    } else {
                        const Op eb = field_block(row);
                        if (first) {
#pragma unroll
                            for (int h = 0; h < NTERM; ++h) d[h] = mfma_op<OP>(r.w[h], eb, zero);
                        } else {
#pragma unroll
                            for (int h = 0; h < NTERM; ++h) d[h] = mfma_op<OP>(r.w[h], eb, d[h]);
                        }
                    }
                    first = last;
                    if (!last) return;
                    // D lane l: cells 4 (l / 16) + e of the tile (a quad), column l % 16
                    half4 g;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if constexpr (OP == kBgFp8)
                            g[e] = (_Float16)fmaf(fmaf(fmaf(d[2][e], 0.0625f, d[1][e]), 0.0625f, d[0][e]), inv_scale, 0.f);
                        else
                            g[e] = (_Float16)d[0][e];
                    }
                    if constexpr (OP == kBgFp16) d[0] = zero;
                    const uint32_t quad = (OP == kBgFp16) ? r.quad : r.ant >> 16;
                    if (ucol < nb && quad != 0xFFFFu)
                        *reinterpret_cast<half4*>(dst + (int)(quad >> 8) * A1P + (int)(quad & 0xFFu)) = g;
                };
                for (int q0 = ent0; q0 < ent1; q0 += 2 * kBgFly) {
#pragma unroll
                    for (int q = 0; q < kBgFly; ++q) fetch(std::min(q0 + kBgFly + q, ent1 - 1), y[q]);
#pragma unroll
                    for (int q = 0; q < kBgFly; ++q)
                        if (q0 + q < ent1) multiply(x[q]);
                    // past the end: the first entries again, for the next step
                    const int qn = (q0 + 2 * kBgFly < ent1) ? q0 + 2 * kBgFly : ent0;
#pragma unroll
                    for (int q = 0; q < kBgFly; ++q) fetch(std::min(qn + q, ent1 - 1), x[q]);
#pragma unroll
                    for (int q = 0; q < kBgFly; ++q)
                        if (q0 + kBgFly + q < ent1) multiply(y[q]);
                }
            }
            // row-pass operand of this wave (L2-resident; loaded per step so that
            // its registers are free during the gridding product) and the next
            // step's samples, on their way across the barrier
            half8 b1[Sh::NT1][Sh::KK];
            load_row_fragments<Sh>(b1, a.dft, kpart, mw, opaque(l16), opaque(l4));
            const int64_t tn = t + u0 + a.TB;
            const int nbn = (int)std::min<int64_t>(a.TB, n - u0 - a.TB);   // <= 0: the last step
            if (nbn > 0) load_step(c, tn, nbn);
            __syncthreads();
            for (int u = 0; u < nb; ++u) {
                __builtin_amdgcn_s_setprio(1);
                row_pass<Sh, P>(s_A1 + u * M1 * A1P, s_B2, b1, M1, R4, mw, opaque(l16), opaque(l4));
                // 1'. the next step's fields, ahead of the step's last barrier
                if (u + 1 == nb && nbn > 0) put_step(c, tn, nbn);
                __syncthreads();
                __builtin_amdgcn_s_setprio(0);
                col_pass<Sh, P>(s_B2, a2, acc, opaque(l16), opaque(l4));
                // the next row pass overwrites B2; the next gridding product
                // touches neither B2 nor anything the column pass reads
                if (u + 1 < nb) __syncthreads();
            }
        }
        flush_slot<Sh, P>(a.slots, slot, a.C, c, kpart, acc, mw, l16, l4, a.fresh != 0);
        f += n;
        ++s_ch;
        v += KS;
        t = 0;
    }
}

// FP8 weight scale: the largest |w| of the sub-array's entries (a grid-stride
// maximum per workgroup, combined with an integer maximum on the float bits,
// which order like the values for |w| >= 0), then scale = 2^e with
// 224 <= s max|w| < 448 and its inverse.
__global__ void bg_absmax_kernel(const float* __restrict__ grp_w, int64_t n, unsigned int* __restrict__ bits) {
    __shared__ float red[256];
    float m = 0.f;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x)
        m = fmaxf(m, fabsf(grp_w[k]));
    red[threadIdx.x] = m;
    __syncthreads();
    for (int w = blockDim.x / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) atomicMax(bits, __float_as_uint(red[0]));
}

__global__ void bg_scale_kernel(float* __restrict__ scale) {
    if (threadIdx.x != 0) return;
    const float mx0 = __uint_as_float(reinterpret_cast<unsigned int*>(scale)[0]);
    const float mx = mx0 > 0.f ? mx0 : 1.f;
    const int e = (int)floorf(log2f(224.f / mx));
    scale[0] = ldexpf(1.f, e);
    scale[1] = ldexpf(1.f, -e);
}

// Split every gather entry's weight w into the operand parts of its block
// element (element el[k], lane el / 8, position el % 8, of each part of entry
// ent[k]; FP16 parts follow each other, FP8 parts 0 and 1 are side by side in
// 16 bytes per lane, which load at once, and part 2 follows): FP16 hi = fp16(w),
// lo = fp16(w - hi); FP8 r0 = s w, part t = e4m3(r_t), r_{t+1} = 16 (r_t - part t),
// t = 0, 1, 2.  Padding entries (ent < 0) are skipped; elements no entry maps to
// stay zero.
template <int OP>
__global__ void bg_weights_kernel(const float* __restrict__ grp_w, const int32_t* __restrict__ ent,
                                  const uint16_t* __restrict__ el, int64_t n, const float* __restrict__ scale,
                                  unsigned char* __restrict__ w8) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const int32_t q = ent[k];
    if (q < 0) return;
    const float w = grp_w[k];
    if constexpr (OP == kBgFp16) {
        _Float16* wh = reinterpret_cast<_Float16*>(w8) + (int64_t)q * 2 * 512 + el[k];
        const _Float16 h = (_Float16)w;
        wh[0] = h;
        wh[512] = (_Float16)(w - (float)h);
    } else {
        unsigned char* wb = w8 + (int64_t)q * 3 * 512;
        const int lane8 = el[k] >> 3, pos = el[k] & 7;
        float r = w * scale[0];
        for (int t = 0; t < 3; ++t) {
            const int b = __builtin_amdgcn_cvt_pk_fp8_f32(r, 0.0f, 0, false);
            wb[t < 2 ? lane8 * 16 + t * 8 + pos : 1024 + el[k]] = (unsigned char)(b & 0xFF);
            r = (r - __builtin_amdgcn_cvt_f32_fp8(b, 0)) * 16.0f;
        }
    }
}

// ---- launch shapes -----------------------------------------------------------
struct BgLayout {
    uint32_t off_E, off_A1, off_B2;
    int A1rows, erow_log2;
    size_t total;
};

size_t take16(size_t& b, size_t n) {
    b = (b + 15) & ~(size_t)15;
    const size_t o = b;
    b += n;
    return o;
}

BgLayout bg_layout(const SubDev& d, int TB) {
    BgLayout L{};
    size_t b = 0;
    const int eb = d.precision == EPIC_FP8 ? 1 : 2;
    const int K2 = 32 * d.KK;
    const int NK = d.N / mfma_ks(d.N);
    L.A1rows = TB * d.P * d.R4max + 16;
    // an antenna's row of the field operand: its columns, at least the 8 bytes of one read
    for (L.erow_log2 = 3; (1 << L.erow_log2) < TB * 2 * d.P * eb; ++L.erow_log2) {}
    L.off_E = (uint32_t)take16(b, (size_t)d.A << L.erow_log2);
    L.off_A1 = (uint32_t)take16(b, (size_t)L.A1rows * (K2 + kPadH) * 2);
    L.off_B2 = (uint32_t)take16(b, (size_t)d.P * NK * (K2 + kPadH) * 2);
    L.total = (b + 15) & ~(size_t)15;
    return L;
}

using BgFn = void (*)(BgArgs);

template <int N, int KK>
BgFn bg_pick2(int P, int op) {
    if (P == 2) return op == kBgFp8 ? bg_kernel<N, KK, 2, kBgFp8> : bg_kernel<N, KK, 2, kBgFp16>;
    return op == kBgFp8 ? bg_kernel<N, KK, 1, kBgFp8> : bg_kernel<N, KK, 1, kBgFp16>;
}

BgFn bg_select(int N, int KK, int P, int op) {
    switch (N * 8 + KK) {
#define EPIC_BG(NN, KKK) case NN * 8 + KKK: return bg_pick2<NN, KKK>(P, op);
        EPIC_BG(32, 1) EPIC_BG(32, 2)
        EPIC_BG(48, 1) EPIC_BG(48, 2) EPIC_BG(48, 3)
        EPIC_BG(64, 1) EPIC_BG(64, 2) EPIC_BG(64, 3) EPIC_BG(64, 4)
        EPIC_BG(96, 1) EPIC_BG(96, 2) EPIC_BG(96, 3) EPIC_BG(96, 4)
        EPIC_BG(128, 1) EPIC_BG(128, 2) EPIC_BG(128, 3) EPIC_BG(128, 4)
#undef EPIC_BG
    }
    return nullptr;
}

constexpr size_t kLdsLimit = 160 * 1024;

int op_of(const SubDev& d) { return d.precision == EPIC_FP8 ? kBgFp8 : kBgFp16; }

}  // namespace

// Launch shape of the GEMM-gridding form: the same grids and column split as
// the gather form; TB spectra per gridding step, the most of 16 / (2 P),
// 8 / (2 P), ... whose LDS lets the shape's target workgroups share a CU
// (two for N <= 64 with at most two MFMA steps, as the registers allow, else
// one).
hipError_t bg_configure(SubDev& d, int device, int num_cu, int force_tb) {
    const int need = std::max(d.Rmax, d.Wmax);
    d.KK = (need + 15) / 16;
    if (d.N < 32 || d.N > 128 || d.N % 16 != 0 || d.N == 80 || d.N == 112) return hipErrorNotSupported;
    if (d.KK < 1 || 16 * d.KK > d.N || d.KK > 4) return hipErrorNotSupported;
    if (!(d.wmode == kWShared || (d.P == 1 && d.wmode == kWReal))) return hipErrorNotSupported;
    d.KS = mfma_ks(d.N);
    d.threads = 64 * (d.N / 16);
    const int target = (d.N <= 64 && d.KK <= 2) ? 2 : 1;   // workgroups per CU the registers allow
    const int tbmax = 16 / (2 * d.P);
    int tb = 0;
    for (int cand = tbmax; cand >= 1 && tb == 0; cand /= 2)
        if (bg_layout(d, cand).total <= kLdsLimit / target) tb = cand;
    for (int cand = tbmax; cand >= 1 && tb == 0; cand /= 2)
        if (bg_layout(d, cand).total <= kLdsLimit) tb = cand;
    if (tb == 0) return hipErrorNotSupported;
    if (force_tb > 0) {   // a candidate of the autotuner: any step size whose LDS fits
        if (force_tb > tbmax || bg_layout(d, force_tb).total > kLdsLimit) return hipErrorNotSupported;
        tb = force_tb;
    }
    d.bg_tb = tb;
    const BgLayout L = bg_layout(d, tb);
    d.lds_bytes = L.total;
    d.prog_lds = 0;
    int occ = 1;
    if (device >= 0) {
        BgFn fn = bg_select(d.N, d.KK, d.P, op_of(d));
        if (!fn) return hipErrorNotSupported;
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsLimit);
        if (e != hipSuccess) return e;
        int blocks = 0;
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, reinterpret_cast<const void*>(fn), d.threads,
                                                         L.total);
        if (e != hipSuccess) return e;
        occ = blocks > 0 ? blocks : 1;
    }
    d.grid_wg = ((num_cu * occ + 7) / 8) * 8;
    return hipSuccess;
}

hipError_t launch_bg_weights(const SubDev& d, hipStream_t st) {
    const int64_t n = d.bg_nentries;   // gather entries
    if (d.precision == EPIC_FP8) {
        unsigned int* bits = reinterpret_cast<unsigned int*>(d.bg_scale);
        hipError_t e = launch_zero(d.bg_scale, 1, st);   // the maximum's bits start at +0
        if (e != hipSuccess) return e;
        const int64_t nb = std::min<int64_t>(1024, (n + 255) / 256);
        bg_absmax_kernel<<<dim3((unsigned)std::max<int64_t>(1, nb)), dim3(256), 0, st>>>(d.grp_w, n, bits);
        bg_scale_kernel<<<dim3(1), dim3(64), 0, st>>>(d.bg_scale);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const int bs = 256;
    const dim3 grid((unsigned)((n + bs - 1) / bs));
    if (d.precision == EPIC_FP8)
        bg_weights_kernel<kBgFp8><<<grid, dim3(bs), 0, st>>>(d.grp_w, d.bg_dst_ent, d.bg_dst_el, n, d.bg_scale, d.bg_w);
    else
        bg_weights_kernel<kBgFp16><<<grid, dim3(bs), 0, st>>>(d.grp_w, d.bg_dst_ent, d.bg_dst_el, n, d.bg_scale, d.bg_w);
    return hipGetLastError();
}

hipError_t launch_bgemm(const SubDev& d, const uint8_t* samples, int64_t n_time, hipStream_t st) {
    const BgLayout L = bg_layout(d, d.bg_tb);
    BgArgs a{};
    a.samples = samples;
    a.chans = d.chans;
    a.waves = d.bg_waves;
    a.desc = d.bg_desc;
    a.w = d.bg_w;
    a.scale = d.bg_scale;
    a.dft = reinterpret_cast<const _Float16*>(d.dft16);
    a.slots = d.slots;
    a.fresh = d.fresh;
    a.T = n_time;
    a.C = d.C; a.A = d.A; a.nibble_order = d.nibble_order; a.TB = d.bg_tb; a.erow_log2 = L.erow_log2;
    a.V = d.C * d.KS;
    a.off_E = L.off_E; a.off_A1 = L.off_A1; a.off_B2 = L.off_B2;
    a.A1rows = L.A1rows;
    a.grid_wg = d.grid_wg;
    a.wg_per_xcd = (d.grid_wg + 7) / 8;
    BgFn fn = bg_select(d.N, d.KK, d.P, op_of(d));
    if (!fn) return hipErrorNotSupported;
    hipLaunchKernelGGL(fn, dim3(8 * a.wg_per_xcd), dim3(d.threads), L.total, st, a);
    return hipGetLastError();
}

}  // namespace epic
