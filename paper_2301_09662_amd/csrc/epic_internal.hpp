// Internal declarations shared by the host plan (plan.cpp) and the HIP kernel
// translation units.  Not part of the public ABI (include/epic.h).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "../../include/epic.h"

namespace epic {

constexpr int kMaxSub = 16;
constexpr int kMaxGridN = 256;

// Aperture window of one (sub-array, channel): the bounding box of every
// antenna's kernel footprint.  Cells outside it are identically zero, so the
// transform only reads the window.  Because a cyclic shift of the aperture
// multiplies both polarisations' sky fields by the same unit phase, the
// products of Eq. 5 do not depend on where the window sits in the grid; the
// kernels place it at the origin.
//
// Gridding runs as a "gather program": the non-empty window cells, sorted by
// their number of contributions (so neighbouring lanes loop equally long),
// each with a list of (antenna, tap) contributions padded with zero-weight
// entries to whole groups of kGroup.
constexpr int kGroup = 4;

struct ChanInfo {
    int32_t x0, y0;      // absolute cell of window element (0, 0)
    int32_t R, W;        // window rows (y extent) and columns (x extent)
    int32_t n_cell;      // non-empty cells
    int32_t cell_off;    // offset of this channel's cell descriptors
    int32_t n_grp;       // groups of kGroup entries
    int32_t grp_off;     // offset of this channel's first group
};

// Cell descriptor: x = LDS float2 offset of the cell within one pol's window
// (row * pitch + col) | (groups << 16); y = first group (channel-relative).
using CellDesc = uint2;

// A gather program's tables, as the set-up kernels see them.
struct GatherProgram {
    const ChanInfo* chans;
    const CellDesc* desc;
    const uint16_t* ant;
    const uint8_t* tap;
    float* w;
};

// of the split FP16 DFT operand (kernels_pair.hip)
constexpr int kDftScaleLog2 = 4;
constexpr float kDftScale = 1 << kDftScaleLog2;
constexpr int kRowBounds = 16;   // bounds per channel and pol: of four window rows each

// Operand types of the GEMM-gridding form (gridding on the matrix cores).
constexpr int kBgFp16 = 0, kBgFp8 = 1;

// Flag in the antenna list of a GEMM-gridding block entry: the last entry of
// its tile (antenna numbers stay below it: their fields would not fit LDS).
constexpr uint32_t kBgLast = 0x8000u;

// Device resources of one sub-array.
struct SubDev {
    // shape
    int A, P, C, N, K, NPP, nibble_order;
    int S;               // partial accumulator slots per channel
    int KS;              // column split of the image across workgroups
    int Rmax, Wmax;      // largest window over channels
    int WP;              // LDS row pitch (float2) of the gridded window
    int Gmax, CellMax;   // largest group / non-empty cell count over channels
    int wmode;           // gather weights: 0 complex, 1 real per pol, 2 real shared by both pols
    int grid_wg;         // resident workgroups of one launch (persistent)
    // tables
    ChanInfo* chans;          // [C]
    CellDesc* cells_desc;     // [sum n_cell]
    uint16_t* grp_ant;        // [sum n_grp * kGroup] antenna per entry (0 for padding)
    uint8_t* grp_tap;         // [sum n_grp * kGroup] tap dy*K+dx, 255 for padding
    float* grp_w;             // [sum n_grp * kGroup][WF] entry weights, WF = 2P, P or 1 by wmode
    int32_t* cells;           // [C][A][2] nearest cell
    double* gfrac;            // [C][A][2] fractional cell coordinate
    float* taps;              // [C][A][P][K][K][2] FP32 taps (before gains)
    float* gains;             // [C][A][P][2] complex gains in effect (or nullptr = unit)
    float* gains_buf = nullptr;   // device storage of the gains once any were set
    float2* twiddle;          // [N] exp(+2 pi i r / N)
    float* slots;             // [S][C][NPP][N][N] partial accumulators
    int32_t* vaa = nullptr;   // [C][A][4 or 1] zero-lag antenna correlations (autocorrelation removal)
    float* lag = nullptr;     // [C][(2K-1)^2][3 or 1][2] lag sums of the autocorrelation image
    float* lag_total = nullptr;   // the same, as of the read-out under way
    // launch shape
    int threads;
    size_t lds_bytes;
    int prog_lds;        // gather program copied to LDS (else read through L2)
    int smp_bufs = 2;    // FP32: decoded sample buffers (2: decode overlaps gridding)
    // matrix-core (reduced precision) form
    int precision;       // epic_precision of this sub-array's kernel
    int KK;              // 32-deep MFMA steps per transform product
    void* dft16;         // [2N][32 KK] FP16 real-form DFT matrix
    // gather form with paired transforms on the matrix cores (kernels_pair.hip)
    int pair = 0;                     // 1: the gather form runs that kernel
    int pair_wd = 0;                  // compiled window size
    // its gather program, in slices of 64 cells whose groups lie side by side
    int pair_gmax = 0;                // largest group count over channels
    ChanInfo* pair_chans = nullptr;   // grp_off in units of 64 groups
    CellDesc* pair_desc = nullptr;    // x: operand offset | groups of the slice << 16, y: first group of the slice
    uint16_t* pair_ant = nullptr;
    uint8_t* pair_tap = nullptr;
    float* pair_w = nullptr;
    void* pair_dft = nullptr;         // FP16 DFT operand
    // scales of its FP32 form
    float* row_bound = nullptr;       // [C][kRowBounds][P] bounds of |Re G| + |Im G| summed over a window row
    float* peak = nullptr;            // [C][A][P] largest |weight| of an antenna
    int32_t* row_top = nullptr;       // [C] most entries of a window row
    float* range = nullptr;           // [2][C][kRowBounds][P] the same by a call's samples too (accumulate, noalloc)
    int use_range = 0;                // per call: the samples are looked through for that bound
    // gridding on the matrix cores (EPIC_GRID_DENSE_GEMM / EPIC_GRID_BLOCK_GEMM)
    int gridder = EPIC_GRID_GATHER;   // gridding form this sub-array's kernel runs
    int R4max = 0;                    // largest window row count, rounded up to 4
    int W4max = 0;                    // largest window column count, rounded up to 4
    int bg_tb = 1;                    // spectra per gridding step
    int64_t bg_nentries = 0;          // gather entries (length of bg_dst_ent, bg_dst_el)
    int32_t* bg_waves = nullptr;      // [C][N / 16 + 1] first block entry of each wave's share
    uint16_t* bg_desc = nullptr;      // [entries][64] per lane group: antennas (kBgLast flags) and the
                                      // (r << 8 | w) of the quad's first cell, 0xFFFF padding
    int32_t* bg_dst_ent = nullptr;    // [gather entries] block entry that holds the weight, -1 padding
    uint16_t* bg_dst_el = nullptr;    // [gather entries] its element there
    unsigned char* bg_w = nullptr;    // [entries][terms * 512] split weights
    int bg_nterm = 2;                 // terms of the split (FP16: 2, FP8: 3)
    float* bg_scale = nullptr;        // [2] FP8 weight scale and its inverse
    // direct imaging (EPIC_GRID_DIRECT_GEMM): per-channel kernel-image matrix
    void* dir_m = nullptr;            // [C][N^2 / 8][A / 16][2 terms][64 lanes][8] FP16
    int dir_chunks = 1;               // time chunks (partial accumulator slots) of a launch
    int fresh = 0;                    // per call: the slots hold zeros (stores replace adds)
};

// One sub-array as seen by the batched (several sub-arrays in one launch)
// matrix-core kernel; a device copy of the table is passed to the kernel.
struct BatchSub {
    const ChanInfo* chans;
    const CellDesc* cells_desc;
    const uint16_t* grp_ant;
    const float* grp_w;
    const uint16_t* dft;      // FP16 real-form DFT matrix [2N][32 KK]
    float* slots;             // [S][C][NPP][N][N]
    int C, A, V;              // channels, antennas, virtual channels (C * KS)
    int N, KK, KS, NK, IT, WAVES, NT1, WP, M1max;
    int nibble_order, S, weight, prog_lds;
};

// Launch state of a batched plan.
struct BatchDev {
    BatchSub* table;          // device [n_sub]
    int grid_wg, threads, kkmax, P, wmode, prog_lds, smp_stride;
    size_t lds_bytes;
    uint32_t off[6];
    int fresh = 0;            // per call: the slots hold zeros (stores replace adds)
};

// Slots of a channel that a read-out sums.  By default all S.  After a single
// call of T spectra on fresh slots (split in runs of L of the channel-major
// sequence) the channel's owners are consecutive workgroups and only their
// pieces were stored; the other slots hold nothing and are not read.
struct SlotUse {
    int64_t T = -1, L = 0;
    __host__ __device__ int count(int64_t c, int S) const {
        if (T < 0) return S;
        if (T == 0) return 0;
        return L <= 1 ? (int)T : (int)((c * T + T - 1) / L - c * T / L) + 1;
    }
};

// ---- launchers (defined in the .hip translation units) -----------------

// One-off FP64 set-up on the device.
hipError_t launch_gaussian_taps(const SubDev& d, double sigma, hipStream_t st);
hipError_t launch_twiddles(const SubDev& d, hipStream_t st);
// the weights of the gather programs the plan holds
hipError_t launch_weights(const SubDev& d, hipStream_t st);

// The bounds that a call's samples give (d.range), for channels whose antennas'
// weights differ by kPairSpread or more; the weights' bounds for the others.
// Below that spread the weights' bounds do by themselves: 255 of 256 antennas
// silent and 15 times the live one's weight, samples of +-1, leave 0.7e-6 on 18 x
// 18 cells (1.4e-7 by the samples).  Ordinary gains do not pay for the look.
constexpr float kPairSpread = 16.0f;
hipError_t launch_range(const SubDev& d, const uint8_t* samples, int64_t n_time, hipStream_t st);

// The FP32 hot path for one sub-array: n_time spectra of uint8 [T][C][A][P].
// fp32_configure picks the launch shape; with device < 0 it makes no HIP call.
hipError_t fp32_configure(SubDev& d, int device, int num_cu);
hipError_t launch_fp32(const SubDev& d, const uint8_t* samples, int64_t n_time, hipStream_t st,
                       float* efield = nullptr);

// FP16 DFT matrix in real form, of the batched and GEMM-gridding kernels.
hipError_t launch_dft_matrix(const SubDev& d, hipStream_t st);

// The gather form with paired transforms on the matrix cores: FP32 (split FP16
// operands) and FP16 (same contract as launch_fp32).
// force_prog: -1 library choice, 0 / 1 gather program streamed from L2 / in LDS
hipError_t pair_configure(SubDev& d, int device, int num_cu, int force_prog = -1);
int pair_pitch(const SubDev& d);
int64_t pair_table_halfs(const SubDev& d);
hipError_t launch_pair_table(const SubDev& d, hipStream_t st);
hipError_t launch_pair(const SubDev& d, const uint8_t* samples, int64_t n_time, hipStream_t st);

// Gridding on the matrix cores (kernels_bgemm.hip): launch shape, the split
// operand weights (after launch_weights), and the hot path.
// force_tb: 0 library choice, else that many spectra per gridding step
hipError_t bg_configure(SubDev& d, int device, int num_cu, int force_tb = 0);
hipError_t launch_bg_weights(const SubDev& d, hipStream_t st);
hipError_t launch_bgemm(const SubDev& d, const uint8_t* samples, int64_t n_time, hipStream_t st);

// Direct imaging on the matrix cores (kernels_direct.hip): launch shape,
// the kernel-image matrix (FP64, split FP16 hi + lo), and the hot path.
hipError_t direct_configure(SubDev& d, int num_cu, int64_t max_time);
int64_t direct_matrix_halfs(const SubDev& d);
hipError_t launch_direct_matrix(const SubDev& d, hipStream_t st);
hipError_t launch_direct(const SubDev& d, const uint8_t* samples, int64_t n_time, hipStream_t st);

// Several FP16 sub-arrays in one persistent launch.
hipError_t batch_configure(SubDev* subs, int n_sub, BatchDev& bd, int device, int num_cu);
BatchSub batch_entry(const SubDev& d, int weight);
hipError_t launch_batch(const BatchDev& bd, const uint8_t* const* samples, int n_sub, int64_t n_time,
                        hipStream_t st);

// Ordered reduction of the slots into [C][NPP][N][N] (or Stokes), optional reset.
hipError_t launch_autocorr(const SubDev& d, const uint8_t* samples, int64_t n_time, hipStream_t st);
hipError_t launch_autocorr_fold(const SubDev& d, hipStream_t st);
hipError_t launch_zero(float* x, int64_t n, hipStream_t st);
int64_t vaa_count(const SubDev& d);
hipError_t launch_readout(const SubDev& d, float* out, int stokes, int reset, hipStream_t st, SlotUse use = {});

// Debug decode of n bytes into float (re, im) pairs.
hipError_t launch_unpack_debug(const uint8_t* in, int64_t n, int order, float* out, hipStream_t st);

}  // namespace epic
