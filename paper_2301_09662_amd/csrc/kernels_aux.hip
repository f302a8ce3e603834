// One-off FP64 set-up kernels (kernel taps, transform tables, gather-entry
// weights), the zero-lag correlations and ordered read-out of the partial
// accumulators, and the debug decoder.  FP64 appears only in the set-up
// kernels, never on the per-spectrum or per-integration path.
#include "epic_internal.hpp"
#include "epic_device.hpp"
#include "epic_gather.hpp"

namespace epic {

namespace {

// Default gridding kernel: a K x K Gaussian of the distance between each tap's
// cell centre and the antenna's fractional position g, normalised to unit sum
// (nearest-cell kernels of Sec. 3.1; the shape is this library's choice).
// One thread per (channel, antenna); the same kernel is used for every pol.
__global__ void gaussian_taps_kernel(const int32_t* __restrict__ cells, const double* __restrict__ g,
                                     float* __restrict__ taps, int C, int A, int P, int K, double sigma) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)C * A) return;
    const int h = K / 2;
    const double cx = (double)cells[2 * idx], cy = (double)cells[2 * idx + 1];
    const double gx = g[2 * idx], gy = g[2 * idx + 1];
    const double inv = 1.0 / (2.0 * sigma * sigma);
    double w[49];
    double sum = 0.0;
    for (int dy = -h; dy <= h; ++dy)
        for (int dx = -h; dx <= h; ++dx) {
            const double ex = cx + dx - gx, ey = cy + dy - gy;
            const double v = exp(-(ex * ex + ey * ey) * inv);
            w[(dy + h) * K + (dx + h)] = v;
            sum += v;
        }
    float* out = taps + idx * (int64_t)P * K * K * 2;
    for (int p = 0; p < P; ++p)
        for (int k = 0; k < K * K; ++k) {
            out[(p * K * K + k) * 2 + 0] = (float)(w[k] / sum);
            out[(p * K * K + k) * 2 + 1] = 0.0f;
        }
}

// exp(+2 pi i r / N), r = 0..N-1, evaluated in FP64 and rounded once.
__global__ void twiddle_kernel(float2* __restrict__ tw, int N) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= N) return;
    double s, c;
    sincospi(2.0 * (double)r / (double)N, &s, &c);
    tw[r] = make_float2((float)c, (float)s);
}

// Weight of one gather entry for pol p: the entry's tap times the antenna's
// gain, complex product in FP64 (rounded once by the caller).  Padding entries
// (tap 255) weigh 0.
__device__ __forceinline__ void entry_weight(const float* __restrict__ taps, const float* __restrict__ gains, int64_t c,
                                             int A, int P, int K, int a, int tap, int p, double* wr, double* wi) {
    double r = 0.0, i = 0.0;
    if (tap != 255) {
        const int64_t cap = (c * A + a) * P + p;
        const int64_t ti = (cap * K * K + tap) * 2;
        r = taps[ti];
        i = taps[ti + 1];
        if (gains) {
            const double gr = gains[2 * cap], gi = gains[2 * cap + 1];
            const double t = gr * r - gi * i;
            i = gr * i + gi * r;
            r = t;
        }
    }
    *wr = r;
    *wi = i;
}

__device__ __forceinline__ void put_weight(float* __restrict__ w, int64_t e, int wm, int P, int p, double wr, double wi) {
    if (wm == kWComplex) {
        w[(e * P + p) * 2] = (float)wr;
        w[(e * P + p) * 2 + 1] = (float)wi;
    } else {
        w[e * (wm == kWReal ? P : 1) + p] = (float)wr;
    }
}

// |w_re| + |w_im| of an antenna's tap: the most it makes of a component of size 1.
__device__ __forceinline__ float weight_size(const float* __restrict__ taps, const float* __restrict__ gains,
                                             int64_t cap, int kk, int tap) {
    const float2 t = reinterpret_cast<const float2*>(taps)[cap * kk + tap];
    float2 g = make_float2(1.f, 0.f);
    if (gains) g = reinterpret_cast<const float2*>(gains)[cap];
    return fabsf(g.x * t.x - g.y * t.y) + fabsf(g.x * t.y + g.y * t.x);
}

// Weights of the gather programs (the plain one and the sliced one, either may
// be absent) in one launch: blockIdx.y is the channel, blockIdx.x counts the
// blocks of the plain program (an entry per thread), then of the sliced one (a
// slice per block: lanes take its cells, the four waves its groups in turn),
// then, for the scales of the FP32 form, of the window's rows (a wave sums the
// weights of a row's entries, a block takes the largest of four rows: a sample's
// two components are at most eight, so 16 times the sum bounds the row's
// |Re G| + |Im G|) and of the antennas (eight lanes take the largest of an
// antenna's and pol's).  Layout per entry by weight mode:
// complex -> 2P floats (re, im per pol); real -> P floats (re per pol); shared
// -> 1 float (the X weight, equal to Y).
template <int P, int wm>
__global__ void __launch_bounds__(256) weights_kernel(GatherProgram plain, int nb_plain, GatherProgram sliced,
                                                      int nb_sliced, const float* __restrict__ taps,
                                                      const float* __restrict__ gains,
                                                      const int32_t* __restrict__ cells, int A, int K,
                                                      float* __restrict__ row_bound, float* __restrict__ peak) {
    const int c = blockIdx.y, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    constexpr int np = wm == kWShared ? 1 : P;
    int b = blockIdx.x;
    if (b < nb_plain) {
        const ChanInfo ci = plain.chans[c];
        const int e = b * 256 + threadIdx.x;
        if (e >= ci.n_grp * kGroup) return;
        const int64_t ge = (int64_t)ci.grp_off * kGroup + e;
        const int a = plain.ant[ge], tap = plain.tap[ge];
        for (int p = 0; p < np; ++p) {
            double wr, wi;
            entry_weight(taps, gains, c, A, P, K, a, tap, p, &wr, &wi);
            put_weight(plain.w, ge, wm, P, p, wr, wi);
        }
        return;
    }
    b -= nb_plain;
    const ChanInfo ci = sliced.chans[c];
    if (b < nb_sliced) {
        if (64 * b >= ci.n_cell) return;
        const CellDesc d = sliced.desc[ci.cell_off + 64 * b + lane];
        for (int j = wv; j < (int)(d.x >> 16); j += 4) {
            // a group's indices, then all its taps and gains: two round trips
            const int64_t ge = (64 * (int64_t)ci.grp_off + d.y + 64 * j + lane) * kGroup;
            const ushort4 an = *reinterpret_cast<const ushort4*>(sliced.ant + ge);
            const uchar4 tp = *reinterpret_cast<const uchar4*>(sliced.tap + ge);
            const int aa[4] = {an.x, an.y, an.z, an.w}, tt[4] = {tp.x, tp.y, tp.z, tp.w};
            double wr[np][kGroup], wi[np][kGroup];
#pragma unroll
            for (int q = 0; q < kGroup; ++q)
#pragma unroll
                for (int p = 0; p < np; ++p)   // padding: any tap's loads, so that no branch parts them
                    entry_weight(taps, gains, c, A, P, K, aa[q], tt[q] == 255 ? 0 : tt[q], p, &wr[p][q], &wi[p][q]);
#pragma unroll
            for (int q = 0; q < kGroup; ++q)
#pragma unroll
                for (int p = 0; p < np; ++p) {
                    const bool on = tt[q] != 255;
                    put_weight(sliced.w, ge + q, wm, P, p, on ? wr[p][q] : 0.0, on ? wi[p][q] : 0.0);
                }
        }
        return;
    }
    b -= nb_sliced;
    if (b < kRowBounds) {
        __shared__ float red[4][2];
        const int row = 4 * b + wv;
        float s[2] = {0.f, 0.f};
        for (int k = lane; row < ci.R && k < A * K; k += 64) {   // an antenna's taps in neighbouring lanes
            const int a = k / K, dx = k - a * K;
            const int64_t ca = (int64_t)c * A + a;
            const int dy = ci.y0 + row - (cells[ca * 2 + 1] - K / 2);
            if (dy < 0 || dy >= K) continue;
#pragma unroll
            for (int p = 0; p < P; ++p) s[p] += weight_size(taps, gains, ca * P + p, K * K, dy * K + dx);
        }
        for (int m = 32; m > 0; m >>= 1)
            for (int p = 0; p < P; ++p) s[p] += __shfl_xor(s[p], m);
        if (lane == 0)
            for (int p = 0; p < P; ++p) red[wv][p] = s[p];
        __syncthreads();
        const int p = threadIdx.x;
        if (p < P)
            row_bound[((int64_t)c * kRowBounds + b) * P + p] =
                16.0f * fmaxf(fmaxf(red[0][p], red[1][p]), fmaxf(red[2][p], red[3][p]));
        return;
    }
    const int k = (b - kRowBounds) * 32 + threadIdx.x / 8;
    if (k >= A * P) return;
    const int64_t cap = (int64_t)c * A * P + k;
    float w = 0.f;
    for (int tap = threadIdx.x & 7; tap < K * K; tap += 8) w = fmaxf(w, weight_size(taps, gains, cap, K * K, tap));
    for (int m = 4; m > 0; m >>= 1) w = fmaxf(w, __shfl_xor(w, m));
    if ((threadIdx.x & 7) == 0) peak[cap] = w;
}

// ---- the range of the gridded values (FP32 form) --------------------------
// A call's bounds of the window's rows, [C][kRowBounds][P] like the weights' own
// (row_bound): those, where the antennas of a pol (the ones that weigh anything)
// differ by less than kPairSpread; else bound b of a channel is what its b-th
// share of the spectra can make of a row.  Block (share, channel).  A row gathers
// at most 2 row_top[c] components, none above the largest product of an antenna's
// weight and a bound of its samples: a thread takes a word of the samples' row
// (four samples; a byte where rows are no aligned words) and ORs the magnitudes of
// its nibbles over the spectra, at least the largest of them and less than twice
// that.  Bound by reading the samples, eight words in flight (station, 132
// channels x 1000 spectra: 64 us a call at a byte and a maximum per sample, 19 us
// by words; where the weights are even, 4 us).
template <int P, typename Word>
__global__ void __launch_bounds__(256) range_kernel(const Word* __restrict__ samples, int64_t T, int C, int W,
                                                    const float* __restrict__ peak, const int32_t* __restrict__ row_top,
                                                    const float* __restrict__ row_bound, float* __restrict__ range) {
    constexpr int NS = sizeof(Word);   // samples per word
    __shared__ float red[4][2][2];
    const int c = blockIdx.y, share = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const float* pk = peak + (int64_t)c * W * NS;
    const float* rb = row_bound + (int64_t)c * kRowBounds * P;
    float* out = range + ((int64_t)c * kRowBounds + share) * P;
    {   // largest and smallest weight of the thread's pol (the block's size is even)
        float hi = 0.f, lo = __builtin_huge_valf();
#pragma unroll 8
        for (int k = tid; k < W * NS; k += 256) {
            const float w = pk[k];
            hi = fmaxf(hi, w);
            if (w > 0.f) lo = fminf(lo, w);
        }
        for (int x = 32; x >= P; x >>= 1) {
            hi = fmaxf(hi, __shfl_xor(hi, x));
            lo = fminf(lo, __shfl_xor(lo, x));
        }
        if (lane < P) {
            red[wv][lane][0] = hi;
            red[wv][lane][1] = lo;
        }
    }
    __syncthreads();
    bool far = false;
    for (int p = 0; p < P; ++p) {
        const float hi = fmaxf(fmaxf(red[0][p][0], red[1][p][0]), fmaxf(red[2][p][0], red[3][p][0]));
        const float lo = fminf(fminf(red[0][p][1], red[1][p][1]), fminf(red[2][p][1], red[3][p][1]));
        far = far || (hi > 0.f && !(hi < kPairSpread * lo));
    }
    if (!far) {
        if (tid < P) out[tid] = rb[share * P + tid];
        return;
    }
    const int64_t t0 = T * share / kRowBounds, n = T * (share + 1) / kRowBounds - t0, CW = (int64_t)C * W;
    // short rows: several thread groups take every so-manieth spectrum
    const int groups = W < 256 ? 256 / W : 1, group = W < 256 ? tid / W : 0;
    float m[2] = {0.f, 0.f};
    for (int k = tid - group * W; group < groups && k < W; k += 256) {
        const Word* src = samples + (t0 * C + c) * W + k;
        uint32_t most = 0;
        for (int64_t u = group; u < n; u += 8 * groups) {
            uint32_t x[8];   // past the end: the last spectrum again
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = src[(u + j * groups < n ? u + j * groups : n - 1) * CW];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const uint32_t neg = (x[j] >> 3) & 0x11111111u;
                most |= (x[j] ^ (neg * 15u)) + neg;   // nibble magnitudes, 0 to 8
            }
        }
        most |= most >> 4;
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            const int s = k * NS + q, p = P == 2 ? (NS > 1 ? q & 1 : s & 1) : 0;
            const uint32_t size = (most >> (8 * q)) & 15u;
            m[p] = fmaxf(m[p], size ? (float)size * pk[s] : 0.f);
        }
    }
    __syncthreads();   // red has been read
#pragma unroll
    for (int p = 0; p < P; ++p) {
        for (int x = 32; x > 0; x >>= 1) m[p] = fmaxf(m[p], __shfl_xor(m[p], x));
        if (lane == 0) red[wv][p][0] = m[p];
    }
    __syncthreads();
    if (tid >= P) return;
    const float r = fmaxf(fmaxf(red[0][tid][0], red[1][tid][0]), fmaxf(red[2][tid][0], red[3][tid][0]));
    float rows = 0.f;   // what the weights alone allow
    for (int k = 0; k < kRowBounds; ++k) rows = fmaxf(rows, rb[k * P + tid]);
    out[tid] = fminf(rows, 2.0f * (float)row_top[c] * r);
}

// ---- autocorrelations (the a = b terms of Eq. 3) ---------------------------
// Zero-lag correlations of every antenna over the spectra of a call:
// vaa[c][a] += (XX*, YY*, Re XY*, Im XY*) (single pol: XX* only).  Every term
// is an integer of magnitude at most 128 (products of 4-bit numbers), so the
// int32 sums are exact and independent of the order of the atomics up to
// 2^24 - 1 spectra; the host folds them into the lag sums before a call would
// pass that count.
constexpr int kAutoChunk = 64;   // spectra per thread (byte form) or per block (word form)

__device__ __forceinline__ int2 unpack44_int(uint32_t byte, int order) {
    const int hi = ((int)(byte << 24)) >> 28;
    const int lo = ((int)(byte << 28)) >> 28;
    return order == 0 ? make_int2(hi, lo) : make_int2(lo, hi);
}

// Rows whose length or address is no multiple of four bytes: one thread per
// (channel, antenna), a byte at a time.
__global__ void autocorr_bytes_kernel(const uint8_t* __restrict__ samples, int64_t T, int C, int A, int P,
                                      int nibble_order, int32_t* __restrict__ vaa) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;   // c * A + a
    if (idx >= (int64_t)C * A) return;
    const int64_t c = idx / A, a = idx - c * A;
    const int64_t t0 = (int64_t)blockIdx.y * kAutoChunk;
    const int64_t t1 = (t0 + kAutoChunk < T) ? t0 + kAutoChunk : T;
    const int64_t AP = (int64_t)A * P;
    int xx = 0, yy = 0, xyr = 0, xyi = 0;
    for (int64_t t = t0; t < t1; ++t) {
        const uint8_t* row = samples + (t * C + c) * AP + a * P;
        const int2 x = unpack44_int(row[0], nibble_order);
        xx += x.x * x.x + x.y * x.y;
        if (P == 2) {
            const int2 y = unpack44_int(row[1], nibble_order);
            yy += y.x * y.x + y.y * y.y;
            xyr += x.x * y.x + x.y * y.y;
            xyi += x.y * y.x - x.x * y.y;
        }
    }
    const int npa = (P == 2) ? 4 : 1;
    int32_t* dst = vaa + idx * npa;
    atomicAdd(dst, xx);
    if (P == 2) {
        atomicAdd(dst + 1, yy);
        atomicAdd(dst + 2, xyr);
        atomicAdd(dst + 3, xyi);
    }
}

// One thread per (channel, 4-byte word of the row): two dual-pol or four
// single-pol antennas.  Four spectra's words are transposed bytewise, so a word
// holds one antenna and pol at four spectra, and the signed 4-bit dot product
// of eight nibbles sums their products: three (XX*, YY*, Re XY*) plus two
// (Im XY*, on the nibble-swapped Y) per antenna and four spectra.  Bound by
// latency, so a block's four thread rows take 16 spectra each, all loads issued
// ahead, and are added in LDS before the atomics.  66 channels x 256 antennas x
// 250 spectra: 26.7 us a byte at a time, now 4.9 us.
template <int P>
__global__ void __launch_bounds__(256) autocorr_words_kernel(const uint32_t* __restrict__ samples, int64_t T, int C,
                                                             int W, int nibble_order, int32_t* __restrict__ vaa) {
    constexpr int NS = 8;   // sums per word: 2 antennas x 4 products, or 4 antennas x 1
    constexpr int kRow = kAutoChunk / 4;
    __shared__ int red[4][64][NS + 1];
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int64_t idx = (int64_t)blockIdx.x * 64 + tx;   // c * W + word
    const int64_t CW = (int64_t)C * W;
    const bool on = idx < CW;
    const int64_t t0 = (int64_t)blockIdx.y * kAutoChunk + ty * kRow;
    uint32_t w[kRow];
#pragma unroll
    for (int k = 0; k < kRow; ++k) w[k] = (on && t0 + k < T) ? samples[(t0 + k) * CW + idx] : 0u;
    int sum[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) sum[k] = 0;
#pragma unroll
    for (int k = 0; k < kRow; k += 4) {
        // bytes b of four spectra -> word b
        const uint32_t a01 = __builtin_amdgcn_perm(w[k + 1], w[k], 0x05010400u);       // w0.b0 w1.b0 w0.b1 w1.b1
        const uint32_t a23 = __builtin_amdgcn_perm(w[k + 1], w[k], 0x07030602u);       // w0.b2 w1.b2 w0.b3 w1.b3
        const uint32_t b01 = __builtin_amdgcn_perm(w[k + 3], w[k + 2], 0x05010400u);
        const uint32_t b23 = __builtin_amdgcn_perm(w[k + 3], w[k + 2], 0x07030602u);
        const uint32_t v[4] = {__builtin_amdgcn_perm(b01, a01, 0x05040100u), __builtin_amdgcn_perm(b01, a01, 0x07060302u),
                               __builtin_amdgcn_perm(b23, a23, 0x05040100u), __builtin_amdgcn_perm(b23, a23, 0x07060302u)};
        if constexpr (P == 2) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const uint32_t x = v[2 * q], y = v[2 * q + 1];
                const uint32_t ys = ((y >> 4) & 0x0F0F0F0Fu) | ((y & 0x0F0F0F0Fu) << 4);
                sum[4 * q + 0] = __builtin_amdgcn_sdot8((int)x, (int)x, sum[4 * q + 0], false);
                sum[4 * q + 1] = __builtin_amdgcn_sdot8((int)y, (int)y, sum[4 * q + 1], false);
                sum[4 * q + 2] = __builtin_amdgcn_sdot8((int)x, (int)y, sum[4 * q + 2], false);
                // low nibbles of x times high of y, minus the other way round
                const int lh = __builtin_amdgcn_sdot8((int)(x & 0x0F0F0F0Fu), (int)ys, 0, false);
                const int hl = __builtin_amdgcn_sdot8((int)(x & 0xF0F0F0F0u), (int)ys, 0, false);
                sum[4 * q + 3] += lh - hl;   // Im XY* when the imaginary part is the low nibble
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) sum[q] = __builtin_amdgcn_sdot8((int)v[q], (int)v[q], sum[q], false);
        }
    }
    constexpr int N = P == 2 ? 8 : 4;
#pragma unroll
    for (int k = 0; k < N; ++k) red[ty][tx][k] = sum[k];
    __syncthreads();
    // 64 words x N sums, four per thread row: consecutive threads on consecutive sums
    for (int k = threadIdx.x; k < 64 * N; k += 256) {
        const int word = k / N, q = k - word * N;
        const int64_t wi = (int64_t)blockIdx.x * 64 + word;
        if (wi >= CW) continue;
        int v = red[0][word][q] + red[1][word][q] + red[2][word][q] + red[3][word][q];
        if (P == 2 && (q & 3) == 3 && nibble_order != 0) v = -v;
        atomicAdd(vaa + wi * N + q, v);
    }
}

__device__ __forceinline__ float2 times(float2 v, float s) { return make_float2(v.x * s, v.y * s); }
// Divides g by the power of two of its larger component and returns that.
__device__ __forceinline__ float take_power(float2& g) {
    int e = (__float_as_int(fmaxf(fabsf(g.x), fabsf(g.y))) >> 23) - 127;   // zero and subnormal: -127
    e = e < -126 ? 0 : (e > 126 ? 126 : e);
    g = times(g, __int_as_float((127 - e) << 23));
    return __int_as_float((127 + e) << 23);
}

// Lag sums of one channel: R^{pq}(d) = sum_a V^{pq}_aa sum_u w^p_a(u + d) conj(w^q_a(u))
// for every tap offset d in [-(K-1), K-1]^2 (the correlation of the antenna's
// kernel with itself, weighted by its zero-lag correlation).  An antenna's
// kernel image times its conjugate depends on these lags only, not on where
// the antenna sits, so sum_d R(d) exp(+2 pi i d.k / N) is the image of the
// a = b terms.  Products: 0 XX* (w^X, w^X), 1 YY* (w^Y, w^Y), 2 XY* (w^X, w^Y).
// Block (dy of the lag, channel); threads stride over antennas and take every
// dx; FP32 sums in a fixed order, added into the lag accumulator (which thus
// holds the a = b terms of several stretches of an integration with different
// gains).  A read-out passes `total`: the sums so far go there, and the
// accumulator restarts from them, or from zero with `reset`.
// lag layout: [C][L][npl][2] with L = (2K-1)^2, npl = 3 (dual pol) or 1.
// Bound by the latency of the tap loads: K is compiled in, so a tap row's loads
// issue together and serve every dx, and the gains multiply the lag's sum once
// per antenna instead of every tap (w' = g w: the sum is |g|^2 or g_x g_y*
// times the taps' own).  66 channels x 256 antennas, K = 3: 34.5 us with a block
// per lag, now 12.1 us.
template <int K, int P>
__global__ void __launch_bounds__(256) autocorr_lag_kernel(const int32_t* __restrict__ vaa,
                                                           const float* __restrict__ taps,
                                                           const float* __restrict__ gains, float* __restrict__ lag,
                                                           float* __restrict__ total, int reset, int A) {
    constexpr int L1 = 2 * K - 1, L = L1 * L1;
    constexpr int npl = (P == 2) ? 3 : 1, npa = (P == 2) ? 4 : 1;
    const int ddy = (int)blockIdx.x - (K - 1), c = blockIdx.y;
    float acc[L1][npl][2];
#pragma unroll
    for (int x = 0; x < L1; ++x)
#pragma unroll
        for (int q = 0; q < npl; ++q) acc[x][q][0] = acc[x][q][1] = 0.f;
    const int uy0 = ddy < 0 ? -ddy : 0, uy1 = ddy < 0 ? K : K - ddy;   // rows with uy and uy + ddy in the kernel
    for (int a = threadIdx.x; a < A; a += 256) {
        const int64_t ca = (int64_t)c * A + a;
        const int32_t* v = vaa + ca * npa;
        const float2* t = reinterpret_cast<const float2*>(taps) + ca * P * K * K;
        // a gain's power of two goes to the taps, exactly: their products stay in
        // range wherever the weights' do
        float2 gx = make_float2(1.f, 0.f), gy = gx;
        float tx = 1.f, ty = 1.f;
        if (gains) {
            gx = reinterpret_cast<const float2*>(gains)[ca * P];
            tx = take_power(gx);
            if (P == 2) {
                gy = reinterpret_cast<const float2*>(gains)[ca * P + 1];
                ty = take_power(gy);
            }
        }
        float s[L1][npl][2];
#pragma unroll
        for (int x = 0; x < L1; ++x)
#pragma unroll
            for (int q = 0; q < npl; ++q) s[x][q][0] = s[x][q][1] = 0.f;
#pragma unroll 1
        for (int uy = uy0; uy < uy1; ++uy) {
            float2 xa[K], xb[K], ya[K], yb[K];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                xa[k] = times(t[(uy + ddy) * K + k], tx);
                xb[k] = times(t[uy * K + k], tx);
                if constexpr (P == 2) {
                    ya[k] = times(t[K * K + (uy + ddy) * K + k], ty);
                    yb[k] = times(t[K * K + uy * K + k], ty);
                }
            }
#pragma unroll
            for (int x = 0; x < L1; ++x)
#pragma unroll
                for (int ux = 0; ux < K; ++ux) {
                    const int vx = ux + x - (K - 1);
                    if (vx < 0 || vx >= K) continue;
                    s[x][0][0] += xa[vx].x * xb[ux].x + xa[vx].y * xb[ux].y;
                    s[x][0][1] += xa[vx].y * xb[ux].x - xa[vx].x * xb[ux].y;
                    if constexpr (P == 2) {
                        s[x][1][0] += ya[vx].x * yb[ux].x + ya[vx].y * yb[ux].y;
                        s[x][1][1] += ya[vx].y * yb[ux].x - ya[vx].x * yb[ux].y;
                        s[x][2][0] += xa[vx].x * yb[ux].x + xa[vx].y * yb[ux].y;
                        s[x][2][1] += xa[vx].y * yb[ux].x - xa[vx].x * yb[ux].y;
                    }
                }
        }
        const float vx = (float)v[0] * (gx.x * gx.x + gx.y * gx.y);
        float vy = 0.f, wr = 0.f, wi = 0.f;
        if constexpr (P == 2) {
            vy = (float)v[1] * (gy.x * gy.x + gy.y * gy.y);
            const float gr = gx.x * gy.x + gx.y * gy.y, gi = gx.y * gy.x - gx.x * gy.y;   // g_x g_y*
            const float vr = (float)v[2], vi = (float)v[3];
            wr = vr * gr - vi * gi;
            wi = vr * gi + vi * gr;
        }
#pragma unroll
        for (int x = 0; x < L1; ++x) {
            acc[x][0][0] = fmaf(vx, s[x][0][0], acc[x][0][0]);
            acc[x][0][1] = fmaf(vx, s[x][0][1], acc[x][0][1]);
            if constexpr (P == 2) {
                acc[x][1][0] = fmaf(vy, s[x][1][0], acc[x][1][0]);
                acc[x][1][1] = fmaf(vy, s[x][1][1], acc[x][1][1]);
                acc[x][2][0] += wr * s[x][2][0] - wi * s[x][2][1];
                acc[x][2][1] += wr * s[x][2][1] + wi * s[x][2][0];
            }
        }
    }
    // block reduction (fixed order: deterministic): lanes, then waves
    constexpr int n = L1 * npl * 2;
    __shared__ float red[4][n];
#pragma unroll
    for (int x = 0; x < L1; ++x)
#pragma unroll
        for (int q = 0; q < npl; ++q)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float r = acc[x][q][h];
                for (int m = 32; m > 0; m >>= 1) r += __shfl_xor(r, m);
                if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][(x * npl + q) * 2 + h] = r;
            }
    __syncthreads();
    if ((int)threadIdx.x < n) {
        const int k = threadIdx.x;
        const int64_t o = ((int64_t)c * L + (int64_t)blockIdx.x * L1) * npl * 2 + k;
        const float r = lag[o] + ((red[0][k] + red[1][k]) + (red[2][k] + red[3][k]));
        if (total) total[o] = r;
        lag[o] = reset ? 0.f : r;
    }
}

// out[c][k][j][i] = sum_s slots[s][c][k][j][i] in an order fixed by the shape,
// so the result is identical from run to run; minus the autocorrelation image
// when lag != nullptr; Stokes form on request (linear feeds, XY* = (U + i V) / 2:
// I = XX+YY, Q = XX-YY, U = 2 Re XY*, V = 2 Im XY*); optional reset of the
// slots, and the zero-lag sums cleared (their lag sums are in `lag` by now).
// The autocorrelation image at pixel (i, j) reads frequency bin
// k = (i + N/2, j + N/2) mod N, where exp(+2 pi i d.k / N) =
// (-1)^(dx+dy) exp(+2 pi i (dx i + dy j) / N) = exp(+2 pi i r / N) with N/2
// added to r for odd dx + dy, the phase from the plan's table tw[r] (FP64 at
// plan time, rounded once to FP32).
//
// Bound by memory: every live slot is read once.  A thread sums four
// neighbouring pixels of every product (16-byte loads, four slots in flight).
// Few channels on a small grid have many slots (the launch splits a channel
// over all workgroups), so a block also splits the slots into SP interleaved
// groups, added through LDS.  One thread per pixel with one slot at a time
// was a chain of 64 dependent round trips on 16 blocks at 4 channels, N = 32:
// 28.6 us, now 4.4; station (7 slots, 60 MB read and cleared) 29 us, now 19
// (7 TB/s over the cache and HBM).
template <int NPP>
__global__ void __launch_bounds__(256) readout_kernel(float* __restrict__ slots, float* __restrict__ out, int S,
                                                      SlotUse use, int C, int N, int SP, int stokes, int reset,
                                                      int out_aligned, const float* __restrict__ lag, int K,
                                                      const float2* __restrict__ tw, int32_t* __restrict__ vaa,
                                                      int64_t n_vaa) {
    __shared__ float4 red[256][NPP];
    __shared__ float2 s_tw[kMaxGridN];
    const int NN = N * N;
    const int TX = 256 / SP;
    const int tx = threadIdx.x & (TX - 1), ty = threadIdx.x / TX;
    const int64_t quad = (int64_t)blockIdx.x * TX + tx;   // four pixels of one row
    const bool on = quad < (int64_t)C * (NN / 4);
    const int64_t c = on ? quad / (NN / 4) : 0;
    const int pix = on ? (int)(quad - c * (NN / 4)) * 4 : 0;
    if (lag) {
        for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n_vaa; k += (int64_t)gridDim.x * 256) vaa[k] = 0;
        for (int k = threadIdx.x; k < N; k += 256) s_tw[k] = tw[k];
        __syncthreads();
    }
    float4 v[NPP];
#pragma unroll
    for (int k = 0; k < NPP; ++k) v[k] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (on) {
        const int n = use.count(c, S);
        const int64_t per_slot = (int64_t)C * NPP * NN;
        float* p0 = slots + c * NPP * NN + pix;
        auto add = [&](const float4 (&x)[NPP]) {
#pragma unroll
            for (int k = 0; k < NPP; ++k) {
                v[k].x += x[k].x; v[k].y += x[k].y; v[k].z += x[k].z; v[k].w += x[k].w;
            }
        };
        constexpr int kFly = 4;   // slots in flight
        int s = ty;
        for (; s + (kFly - 1) * SP < n; s += kFly * SP) {
            float4 x[kFly][NPP];
#pragma unroll
            for (int u = 0; u < kFly; ++u)
#pragma unroll
                for (int k = 0; k < NPP; ++k)
                    x[u][k] = *reinterpret_cast<const float4*>(p0 + (s + u * SP) * per_slot + (int64_t)k * NN);
#pragma unroll
            for (int u = 0; u < kFly; ++u) add(x[u]);
        }
        for (; s < n; s += SP) {
            float4 x[NPP];
#pragma unroll
            for (int k = 0; k < NPP; ++k) x[k] = *reinterpret_cast<const float4*>(p0 + s * per_slot + (int64_t)k * NN);
            add(x);
        }
        if (reset)
            for (int z = ty; z < n; z += SP)
#pragma unroll
                for (int k = 0; k < NPP; ++k)
                    *reinterpret_cast<float4*>(p0 + z * per_slot + (int64_t)k * NN) = make_float4(0.f, 0.f, 0.f, 0.f);
        // the a = b terms, the lags shared out over the slot groups.  XX* and YY*
        // lag sums are Hermitian (R(-d) = R(d)*), so lags d and -d are taken
        // together with one phase.
        if (lag) {
            const int i0 = pix % N, j = pix / N;
            const int L1 = 2 * K - 1, L = L1 * L1, npl = (NPP == 4) ? 3 : 1;
            const float* lc = lag + c * L * npl * 2;
            const float inv_n = 1.0f / (float)N;
            float a[NPP][4];
#pragma unroll
            for (int k = 0; k < NPP; ++k)
#pragma unroll
                for (int m = 0; m < 4; ++m) a[k][m] = 0.f;
            for (int l = L / 2 + ty; l < L; l += SP) {   // d = 0 at l = L/2, then d > 0; -d is lag L - 1 - l
                const int dy = l / L1 - (K - 1), dx = l - (dy + K - 1) * L1 - (K - 1);
                const float* lp = lc + l * npl * 2;
                const float* lm = lc + (L - 1 - l) * npl * 2;
                const bool zero = l == L / 2;
                float pr[4], pi[4];
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    // offset by 32 N: positive, below 2^14 (|dx|, |dy| <= 6, i, j < N)
                    const int t = dx * (i0 + m) + dy * j + (((dx + dy) & 1) ? N / 2 : 0) + 32 * N;
                    int r = t - (int)((float)t * inv_n) * N;
                    if (r < 0) r += N;
                    if (r >= N) r -= N;
                    pr[m] = s_tw[r].x;
                    pi[m] = s_tw[r].y;
                }
                const float two = zero ? 1.f : 2.f;
                const float xr = two * lp[0], xi = two * lp[1];
#pragma unroll
                for (int m = 0; m < 4; ++m) a[0][m] = fmaf(xr, pr[m], fmaf(-xi, pi[m], a[0][m]));
                if constexpr (NPP == 4) {
                    const float yr = two * lp[2], yi = two * lp[3];
                    // XY*: R(d) e + R(-d) e*
                    const float mr = zero ? 0.f : lm[4], mi = zero ? 0.f : lm[5];
                    const float sr = lp[4] + mr, dr = lp[4] - mr, si = lp[5] + mi, di = lp[5] - mi;
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        a[1][m] = fmaf(yr, pr[m], fmaf(-yi, pi[m], a[1][m]));
                        a[2][m] = fmaf(sr, pr[m], fmaf(-di, pi[m], a[2][m]));
                        a[3][m] = fmaf(si, pr[m], fmaf(dr, pi[m], a[3][m]));
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < NPP; ++k) {
                v[k].x -= a[k][0]; v[k].y -= a[k][1]; v[k].z -= a[k][2]; v[k].w -= a[k][3];
            }
        }
    }
    if (SP > 1) {
#pragma unroll
        for (int k = 0; k < NPP; ++k) red[threadIdx.x][k] = v[k];
        for (int w = SP / 2; w > 0; w >>= 1) {
            __syncthreads();
            if (ty < w)
#pragma unroll
                for (int k = 0; k < NPP; ++k) {
                    const float4 o = red[threadIdx.x + w * TX][k];
                    v[k].x += o.x; v[k].y += o.y; v[k].z += o.z; v[k].w += o.w;
                    red[threadIdx.x][k] = v[k];
                }
        }
    }
    if (!on || ty != 0) return;
    if constexpr (NPP == 4)
        if (stokes) {
            const float4 x = v[0], y = v[1];
            v[0] = make_float4(x.x + y.x, x.y + y.y, x.z + y.z, x.w + y.w);
            v[1] = make_float4(x.x - y.x, x.y - y.y, x.z - y.z, x.w - y.w);
            v[2] = make_float4(2.f * v[2].x, 2.f * v[2].y, 2.f * v[2].z, 2.f * v[2].w);
            v[3] = make_float4(2.f * v[3].x, 2.f * v[3].y, 2.f * v[3].z, 2.f * v[3].w);
        }
#pragma unroll
    for (int k = 0; k < NPP; ++k) {
        float* o = out + (c * NPP + k) * NN + pix;
        if (out_aligned) {
            *reinterpret_cast<float4*>(o) = v[k];
        } else {   // a caller's buffer need only be aligned to its floats
            o[0] = v[k].x; o[1] = v[k].y; o[2] = v[k].z; o[3] = v[k].w;
        }
    }
}

__global__ void zero_kernel(float* __restrict__ x, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = 0.0f;
}

__global__ void unpack_debug_kernel(const uint8_t* __restrict__ in, int64_t n, int order, float2* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    out[i] = unpack44(in[i], order);
}

}  // namespace

hipError_t launch_gaussian_taps(const SubDev& d, double sigma, hipStream_t st) {
    const int64_t n = (int64_t)d.C * d.A;
    const int bs = 128;
    gaussian_taps_kernel<<<dim3((unsigned)((n + bs - 1) / bs)), dim3(bs), 0, st>>>(d.cells, d.gfrac, d.taps, d.C, d.A,
                                                                                   d.P, d.K, sigma);
    return hipGetLastError();
}

hipError_t launch_twiddles(const SubDev& d, hipStream_t st) {
    twiddle_kernel<<<dim3((d.N + 63) / 64), dim3(64), 0, st>>>(d.twiddle, d.N);
    return hipGetLastError();
}

hipError_t launch_weights(const SubDev& d, hipStream_t st) {
    const GatherProgram g0{d.chans, d.cells_desc, d.grp_ant, d.grp_tap, d.grp_w};
    const GatherProgram g1{d.pair_chans, d.pair_desc, d.pair_ant, d.pair_tap, d.pair_w};
    const int nb0 = d.grp_w ? (d.Gmax * kGroup + 255) / 256 : 0, nb1 = d.pair_w ? (d.CellMax + 63) / 64 : 0;
    const int nb2 = d.row_bound ? kRowBounds + (d.A * d.P + 31) / 32 : 0;
    const dim3 grid(nb0 + nb1 + nb2, d.C), block(256);
#define EPIC_WEIGHTS(PP, WM) \
    weights_kernel<PP, WM><<<grid, block, 0, st>>>(g0, nb0, g1, nb1, d.taps, d.gains, d.cells, d.A, d.K, d.row_bound, \
                                                   d.peak)
    if (d.P == 2) {
        if (d.wmode == kWComplex) EPIC_WEIGHTS(2, kWComplex);
        else if (d.wmode == kWReal) EPIC_WEIGHTS(2, kWReal);
        else EPIC_WEIGHTS(2, kWShared);
    } else {
        if (d.wmode == kWComplex) EPIC_WEIGHTS(1, kWComplex);
        else EPIC_WEIGHTS(1, kWReal);
    }
#undef EPIC_WEIGHTS
    return hipGetLastError();
}

hipError_t launch_range(const SubDev& d, const uint8_t* samples, int64_t n_time, hipStream_t st) {
    const int AP = d.A * d.P;
    const dim3 grid(kRowBounds, d.C), block(256);
    if ((AP & 3) == 0 && (reinterpret_cast<uintptr_t>(samples) & 3) == 0) {
        const auto fn = d.P == 2 ? range_kernel<2, uint32_t> : range_kernel<1, uint32_t>;
        fn<<<grid, block, 0, st>>>(reinterpret_cast<const uint32_t*>(samples), n_time, d.C, AP / 4, d.peak, d.row_top,
                                   d.row_bound, d.range);
    } else {
        const auto fn = d.P == 2 ? range_kernel<2, uint8_t> : range_kernel<1, uint8_t>;
        fn<<<grid, block, 0, st>>>(samples, n_time, d.C, AP, d.peak, d.row_top, d.row_bound, d.range);
    }
    return hipGetLastError();
}

hipError_t launch_autocorr(const SubDev& d, const uint8_t* samples, int64_t n_time, hipStream_t st) {
    const int64_t chunks = (n_time + kAutoChunk - 1) / kAutoChunk;
    if (chunks > 65535) return hipErrorInvalidValue;
    const int AP = d.A * d.P;
    // whole aligned words of every row: the word form (a byte form costs 26.7
    // against 4.9 us at 66 channels x 256 dual-pol antennas x 250 spectra)
    if ((AP & 3) == 0 && (reinterpret_cast<uintptr_t>(samples) & 3) == 0) {
        const int W = AP / 4;
        const dim3 grid((unsigned)(((int64_t)d.C * W + 63) / 64), (unsigned)chunks);
        const uint32_t* w = reinterpret_cast<const uint32_t*>(samples);
        if (d.P == 2)
            autocorr_words_kernel<2><<<grid, dim3(256), 0, st>>>(w, n_time, d.C, W, d.nibble_order, d.vaa);
        else
            autocorr_words_kernel<1><<<grid, dim3(256), 0, st>>>(w, n_time, d.C, W, d.nibble_order, d.vaa);
        return hipGetLastError();
    }
    const int64_t n = (int64_t)d.C * d.A;
    const int bs = 256;
    autocorr_bytes_kernel<<<dim3((unsigned)((n + bs - 1) / bs), (unsigned)chunks), dim3(bs), 0, st>>>(
        samples, n_time, d.C, d.A, d.P, d.nibble_order, d.vaa);
    return hipGetLastError();
}

hipError_t launch_zero(float* x, int64_t n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    zero_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st>>>(x, n);
    return hipGetLastError();
}

int64_t vaa_count(const SubDev& d) { return (int64_t)d.C * d.A * (d.P == 2 ? 4 : 1); }

namespace {

hipError_t launch_lag(const SubDev& d, float* total, int reset, hipStream_t st) {
    const dim3 grid(2 * d.K - 1, d.C);
    switch (d.K * 2 + d.P) {
#define EPIC_LAG(KK, PP)                                                                                      \
    case KK * 2 + PP:                                                                                         \
        autocorr_lag_kernel<KK, PP><<<grid, dim3(256), 0, st>>>(d.vaa, d.taps, d.gains, d.lag, total, reset, d.A); \
        break;
        EPIC_LAG(1, 1) EPIC_LAG(1, 2) EPIC_LAG(3, 1) EPIC_LAG(3, 2) EPIC_LAG(5, 1) EPIC_LAG(5, 2) EPIC_LAG(7, 1)
        EPIC_LAG(7, 2)
#undef EPIC_LAG
    }
    return hipGetLastError();
}

}  // namespace

// Move the zero-lag correlations gathered so far into the lag accumulator
// (with the gains in effect while they were gathered) and clear them.
hipError_t launch_autocorr_fold(const SubDev& d, hipStream_t st) {
    if (!d.vaa) return hipSuccess;
    hipError_t e = launch_lag(d, nullptr, 0, st);
    if (e != hipSuccess) return e;
    return launch_zero(reinterpret_cast<float*>(d.vaa), vaa_count(d), st);   // all-zero bits: 0 as int32 too
}

hipError_t launch_readout(const SubDev& d, float* out, int stokes, int reset, hipStream_t st, SlotUse use) {
    hipError_t e = hipSuccess;
    const float* lag = nullptr;
    if (d.vaa) {   // this read-out's lag sums; the kernel below clears the zero-lag sums
        if ((e = launch_lag(d, d.lag_total, reset, st)) != hipSuccess) return e;
        lag = d.lag_total;
    }
    const int64_t n_vaa = d.vaa ? vaa_count(d) : 0;
    // slot groups per block: enough threads for the loads in flight to cover
    // the memory latency (2^17), whatever the number of slots is, so that the
    // order of the sum depends on the shape only
    const int64_t quads = (int64_t)d.C * d.N * d.N / 4;
    int SP = 1;
    while (SP < 32 && quads * SP < (1 << 17)) SP *= 2;
    const int TX = 256 / SP;
    const dim3 grid((unsigned)((quads + TX - 1) / TX));
    const int al = (reinterpret_cast<uintptr_t>(out) & 15) == 0;
    if (d.NPP == 4)
        readout_kernel<4><<<grid, dim3(256), 0, st>>>(d.slots, out, d.S, use, d.C, d.N, SP, stokes, reset, al, lag, d.K,
                                                      d.twiddle, d.vaa, n_vaa);
    else
        readout_kernel<1><<<grid, dim3(256), 0, st>>>(d.slots, out, d.S, use, d.C, d.N, SP, stokes, reset, al, lag, d.K,
                                                      d.twiddle, d.vaa, n_vaa);
    return hipGetLastError();
}

hipError_t launch_unpack_debug(const uint8_t* in, int64_t n, int order, float* out, hipStream_t st) {
    const int bs = 256;
    unpack_debug_kernel<<<dim3((unsigned)((n + bs - 1) / bs)), dim3(bs), 0, st>>>(in, n, order,
                                                                                 reinterpret_cast<float2*>(out));
    return hipGetLastError();
}

}  // namespace epic
