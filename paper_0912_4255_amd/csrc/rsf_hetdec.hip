// Time-domain front end (paper Sec. III.A.1, eqs. eq14-eq16): heterodyne a
// real high-rate series, low-pass filter it at the new Nyquist frequency and
// keep every D-th sample.  The heterodyne factor of raw sample
// m = j D + c - i splits into exp(-2 pi i f_h j D dt) exp(-2 pi i f_h (c - i) dt),
// so the filter runs with complex taps g[i] = h[i] exp(-2 pi i f_h (c - i) dt)
// on the real series and each output takes one FP64 phase factor.
//
// Two forms: filters of L >= 4 D + 1 taps with L + 7 D <= 5120 whose window
// fits LDS run as a product on the FP32 matrix cores (rsf_hetdec_mfma_k, below;
// mm_shape has the rule); the others a
// direct sum (rsf_hetdec_k): one workgroup per 64 outputs, the raw samples its outputs
// touch and the taps in LDS, each wave computing four outputs at a time with
// its lanes striding over the taps (consecutive lanes read consecutive
// samples and taps), then summing across the wave.
#include <algorithm>

#include "rsf_device.h"
#include "rsf_launch.h"

namespace rsf {

namespace {
constexpr int kHdThreads = 256;
constexpr int kHdOut = 64;     // outputs per workgroup
constexpr int kHdIlp = 4;      // outputs per wave pass
}  // namespace

__global__ __launch_bounds__(kHdThreads) void rsf_hetdec_k(HetdecArgs a) {
    extern __shared__ float sm[];
    float2* g = reinterpret_cast<float2*>(sm);      // L taps
    float* xs = sm + 2 * a.L;                         // raw window
    const int64_t j0 = (int64_t)blockIdx.x * kHdOut;
    const int nj = (int)min((int64_t)kHdOut, a.n_out - j0);
    const int64_t m0 = j0 * a.D + a.c - (a.L - 1);    // first raw sample touched
    const int span = (nj - 1) * a.D + a.L;
    for (int i = threadIdx.x; i < a.L; i += kHdThreads) g[i] = a.g[i];
    for (int i = threadIdx.x; i < span; i += kHdThreads) {
        const int64_t m = m0 + i;
        xs[i] = (m >= 0 && m < a.n_raw) ? a.x[m] : 0.f;
    }
    __syncthreads();
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int jb = wave * kHdIlp; jb < nj; jb += 4 * kHdIlp) {
        float re[kHdIlp], im[kHdIlp];
#pragma unroll
        for (int q = 0; q < kHdIlp; ++q) re[q] = im[q] = 0.f;
        // output jb + q reads window index (jb + q) D + (L - 1) - i for tap i
        const int base = jb * a.D + (a.L - 1);
        for (int i = lane; i < a.L; i += 64) {
            const float2 t = g[i];
#pragma unroll
            for (int q = 0; q < kHdIlp; ++q) {
                if (jb + q < nj) {
                    const float v = xs[base + q * a.D - i];
                    re[q] += t.x * v;
                    im[q] += t.y * v;
                }
            }
        }
#pragma unroll
        for (int q = 0; q < kHdIlp; ++q) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                re[q] += __shfl_xor(re[q], off);
                im[q] += __shfl_xor(im[q], off);
            }
        }
        if (lane < kHdIlp && jb + lane < nj) {
            float r = re[0], m = im[0];
#pragma unroll
            for (int q = 1; q < kHdIlp; ++q)
                if (lane == q) {
                    r = re[q];
                    m = im[q];
                }
            const int64_t j = j0 + jb + lane;
            const double cyc = a.cyc_per_out * (double)j;
            float s, c;
            sincospif(-2.0f * (float)(cyc - rint(cyc)), &s, &c);
            a.out[j] = make_float2(r * c - m * s, r * s + m * c);
        }
    }
}

// Matrix-core form.  Output j = 8 J + n (n < 8) reads
// x[8 D J + n D + c - i] g[i], so with row J's window starting at its sample
// 8 D J + c - (L - 1), output (J, n) is the product of that window with the
// taps shifted by n D:
//   y_{8J+n} = sum_kk X[8 D J + kk] G[kk][n],  G[kk][n] = g[(L - 1) + n D - kk]
// (zero outside the filter), kk < Kd = L + 7 D.  The 16 columns (8 outputs, real
// and imaginary parts) and 16 rows J are one FP32 MFMA 16x16x4 tile; the
// columns' zero taps cost 7 / (2 K) more products than the direct sum.  The
// length Kd is split over WK waves, each holding its slice of G in registers
// for the whole launch; the 16 / WK row tiles of a block are the other way the
// waves divide.  Whatever WK, an output is the same sum of 16 partial sums in the
// same order: a wave keeps 16 / WK of them apart and adds them as the sum of the
// waves' partial tiles through LDS goes on, so the bits depend on the filter alone
// and the error against 64 bits is the direct sum's (0.94 to 1.05 times it for D =
// 10 to 128 and K = 8 to 20; one partial sum per wave gave up to 1.23 times it at
// WK = 4 and 8).  Keeping them apart costs up to 4 % (D = 32, K = 8, 3,000,000
// outputs: 149 -> 155 us).
//
// Persistent workgroups walk consecutive blocks (the overlap of neighbouring
// windows stays in their caches).  One barrier per block: after it, the next
// block's window comes by DMA into the other buffer, the last block's partial
// tiles are added and written, and this block's products run.  The buffers are
// LDS arrays of their own, so no LDS read of one waits for the DMA into the
// other.  Rows start 8 D samples apart, on the same banks when D is even; then
// four floats between the window's chunks of 8 D samples move the rows' 16-byte
// reads to different banks (an odd D has at most two rows on a bank).  Windows
// of which two do not fit LDS run with one buffer and no prefetch.
//
// The columns' zero taps would spread a sample that is not finite over its
// row: outputs whose sum is not finite are formed again from the samples that
// their own filter reaches, after the workgroup's last block (not_finite, below).
// Ten days at 256 Hz, D = 64, K = 16 (431 us when all samples are finite): 502 us with an
// hour of NaN, 1.27 ms with a NaN in every 1009 samples, 2.8 ms with an hour of
// infinities; with every such output summed where it is finished, by one thread,
// 17.2, 26.4 and 17.1 ms.
//
// What bounds it: the FP32 matrix rate (4 flops per tap and output, 153.8
// TFLOP/s measured by a large product).  Ten days at 256 Hz, D = 64, K = 16:
// 277 us for the products alone (82 % of that rate with the zero taps), 201 us
// for the samples alone (5 TB/s), about 400 us for both together; the product
// form for D = 64 alone that this replaces (rows of 64 samples, one output tap
// phase per column, a diagonal sum through LDS) took 404 us.  One day at 1 kHz,
// D = 100, K = 16: 175 us against 1530 us for the direct sum.  Vector
// instructions hold up FP32 products: with the samples staged through registers
// (237 vector instructions per wave and block, 17 of them products) the D = 64
// case took 546 us.  A third window buffer changed nothing.
namespace {
constexpr int kMmThreads = 1024;  // 16 waves, 4 per SIMD
constexpr int kMmWaves = kMmThreads / 64;
// floats of one of NB window buffers (the partial tiles have the other 32 KiB of LDS)
constexpr int mm_buf(int NB) { return 32768 / NB; }
typedef float mm_v4f __attribute__((ext_vector_type(4)));

// The split of one plan: WK waves along the taps, NG groups of 16 taps each.
struct MmShape {
    int WK = 0, NG = 0, NB = 0;  // NB window buffers
};

// NG is compiled for these values: up to 8 for 4 waves along the taps, 12 for 8 waves and
// 16 for 16, beyond which the taps do not fit the registers beside the partial
// sums (D = 50, K = 16, 400,000 outputs: 59.7 us with 16 groups on 8 waves, 49.7
// with 8 on 16; D = 25, K = 16: 45.8 with 16 groups on 4 waves, 34.4 with 8 on 8);
// 18 and 20 with one buffer only, so filters of Kd <= 5120
constexpr int kMmGroups[] = {1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16, 18, 20};
constexpr int mm_groups_max(int WK, int NB) { return NB == 1 ? 20 : WK == 4 ? 8 : WK == 8 ? 12 : 16; }

int mm_pad(int D) { return (D & 1) ? 0 : 4; }

MmShape mm_shape_of(int L, int D, int WK) {
    MmShape m;
    const int Kd = L + 7 * D, WM = kMmWaves / WK;
    const int need = (Kd + 16 * WK - 1) / (16 * WK);
    for (int NG : kMmGroups) {
        if (NG < need) continue;
        // the last row reads KR taps from its start; its window has Kd of them in whole chunks of 8 D
        const int KR = 16 * NG * WK;
        const int64_t stride = 8 * D + mm_pad(D), rows = 16 * WM - 1;
        const int64_t floats = std::max((rows + (Kd + 8 * D - 1) / (8 * D)) * stride,
                                        rows * stride + KR + (int64_t)(KR / (8 * D)) * mm_pad(D) + 16);
        const int NB = floats <= mm_buf(2) ? 2 : floats <= mm_buf(1) ? 1 : 0;
        if (NB == 1 && NG == 7) continue;  // the one-buffer kernels start at 8
        if (!NB || NG > mm_groups_max(WK, NB) || (NB == 1 && (WK != kMmWaves || NG < 8))) return m;
        m.NB = NB;
        m.WK = WK;
        m.NG = NG;
        return m;
    }
    return m;
}

// The form a plan of L taps takes for n_out outputs (WK = 0: the direct sum).
// Filters under 4 D + 1 taps would meet more zero taps than their own.
MmShape mm_shape(int L, int D, int64_t n_out, int n_cu) {
    MmShape best;
    if (D < 2 || L < 4 * D + 1) return best;
    for (int WK : {4, 8, 16}) {
        const MmShape m = mm_shape_of(L, D, WK);
        if (!m.WK || (best.WK && m.NB < 2)) continue;
        if (best.WK) {
            // fewer row tiles per block only where larger blocks leave compute units
            // idle; the same bits (D = 10, K = 8: 40,000 outputs 7.9 us on 16 waves
            // and 9.6 on 4, 4,000,000 outputs 171 and 131 us)
            const int64_t per_block = 128 * (kMmWaves / best.WK);
            if ((n_out + per_block - 1) / per_block >= 2 * (int64_t)n_cu) break;
        }
        best = m;
    }
    return best;
}
}  // namespace

// Outputs that are not finite, taken from the samples that their own filter
// reaches: the wave's 32 outputs from j0, output j0 + lane / 2 in two lanes (its
// real and imaginary parts).  An output that reaches a NaN is NaN; whether it does
// is looked up at its centre sample, which answers for the inside of a stretch of
// NaN, then in one pass over all that the 32 outputs reach.  The others (they reach
// infinities, overflow, or only share a row with such a sample) are summed again,
// four at a time, the lanes striding over the taps.
__device__ __forceinline__ void not_finite(const HetdecArgs& a, int64_t j0) {
    const int lane = threadIdx.x & 63, o = lane >> 1;
    const bool im = lane & 1;
    const int64_t j = j0 + o;
    float* out = reinterpret_cast<float*>(a.out);
    const float now = j < a.n_out ? out[2 * j + im] : 0.f, other = __shfl_xor(now, 1);
    const bool bad = !(fabsf(now) <= 3.402823466e38f && fabsf(other) <= 3.402823466e38f);
    if (!__any(bad)) return;
    const int64_t m0 = j0 * a.D - a.c;  // the first sample that output j0 reaches
    auto sample = [&](int64_t m) { return m >= 0 && m < a.n_raw ? a.x[m] : 0.f; };
    bool nan = bad && isnan(sample(j * a.D));
    if (__any(bad && !nan)) {
        const int reach = 31 * a.D + a.L;
        for (int p = 0; p < reach; p += 512) {
            float v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = sample(m0 + p + 64 * q + lane);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const uint64_t at = __ballot(isnan(v[q]));
                // this output reaches samples o D .. o D + L - 1 from m0
                const int lo = max(o * a.D - (p + 64 * q), 0), hi = min(o * a.D + a.L - 1 - (p + 64 * q), 63);
                if (hi >= lo) nan = nan || (bad && ((at >> lo) << (63 - hi + lo)) != 0);
            }
        }
    }
    float s = __int_as_float(0x7fc00000), t = s;  // real and imaginary sums
    uint64_t todo = __ballot(bad && !nan);
    while (todo) {
        const int k = (__ffsll((long long)todo) - 1) >> 1;  // outputs k .. k + 3
        float re[4] = {0.f, 0.f, 0.f, 0.f}, imag[4] = {0.f, 0.f, 0.f, 0.f};
        for (int i0 = 0; i0 < a.L; i0 += 128) {
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int i = i0 + 64 * r + lane;
                const float2 g = i < a.L ? a.g[i] : make_float2(0.f, 0.f);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float v = i < a.L ? sample((j0 + k + q) * a.D + a.c - i) : 0.f;
                    re[q] += g.x * v;
                    imag[q] += g.y * v;
                }
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                re[q] += __shfl_xor(re[q], off);
                imag[q] += __shfl_xor(imag[q], off);
            }
            if (o == k + q && !nan) {
                s = re[q];
                t = imag[q];
            }
        }
        todo &= ~__ballot(o >= k && o < k + 4);
    }
    if (bad) {
        const double cyc = a.cyc_per_out * (double)j;
        float sn, cs;
        sincospif(-2.0f * (float)(cyc - rint(cyc)), &sn, &cs);
        out[2 * j + im] = im ? s * sn + t * cs : s * cs - t * sn;
    }
}

template <int WK, int NG, int NB>
__global__ __launch_bounds__(kMmThreads) void rsf_hetdec_mfma_k(HetdecArgs a, int pad, unsigned inv_chunk, bool wide,
                                                                 int64_t n_blk) {
    constexpr int WM = kMmWaves / WK;
    constexpr int NO = 128 * WM;  // outputs per block
    __shared__ __align__(16) float buf0[mm_buf(NB)];
    __shared__ __align__(16) float buf1[NB > 1 ? mm_buf(NB) : 4];
    __shared__ __align__(16) float red[2][kMmWaves][256];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kw = wave % WK, mt = wave / WK;
    const int D = a.D, L = a.L, chunk = 8 * D, stride = chunk + pad;
    const int J = lane & 15, q = lane >> 4;
    // This wave's group g of 16 taps is kk = 16 (kw + WK g): the partial sums take
    // groups in turn, so none holds the filter's main lobe alone, and the four taps
    // of a lane have an accumulator each: chains as short as the direct sum's.
    // With contiguous slices and two accumulators the error at D = 100, K = 16 was
    // 2.2e-7 at 158 us, against 1.5e-7.
    // B operand: lane holds G[16 (kw + WK g) + 4 q + t][lane % 16]; taps
    // outside the filter are outside the buffer and read zero
    float bop[NG][4];
    {
        const __amdgpu_buffer_rsrc_t taps =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<float2*>(a.g), 0, 8 * L, 0x00027000);
        const int at = 8 * ((L - 1) + (J >> 1) * D - (16 * kw + 4 * q)) + 4 * (J & 1);
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                bop[g][t] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(taps, at - 8 * (16 * WK * g + t), 0, 0));
    }

    // consecutive blocks per workgroup
    const int64_t per = n_blk / gridDim.x, rest = n_blk - per * gridDim.x;
    const int64_t b0 = per * blockIdx.x + min((int64_t)blockIdx.x, rest);
    const int n_it = (int)(per + ((int64_t)blockIdx.x < rest ? 1 : 0));

    // The window of block b: chunks of 8 D samples (all that the rows' Kd taps
    // reach), a piece of 64 lanes per wave instruction, 16 bytes a lane where
    // every window starts on 16 bytes; samples outside the series are zero.
    // The addresses are a scalar base and the lane's offset, and the waves that
    // issue go first (priority): vector instructions wait behind the products of
    // the waves that are done with it.
    const int n_chunks = 16 * WM - 1 + (L + 7 * D + chunk - 1) / chunk;
    // what the last rows' zero taps read past the window is zero, once
    for (int i = n_chunks * stride + tid; i < mm_buf(NB); i += kMmThreads) {
        buf0[i] = 0.f;
        if (NB > 1) buf1[i] = 0.f;
    }
    const int piece = wide ? 256 : 64, pieces = (chunk + piece - 1) / piece;
    auto stage = [&](int64_t b, float* w) {
        const int64_t m0 = b * NO * (int64_t)D + a.c - (L - 1);  // raw sample of the window's first
        __builtin_amdgcn_s_setprio(3);
        if (m0 >= 0 && m0 + (int64_t)n_chunks * chunk <= a.n_raw) {
            const float* x0 = a.x + m0;
            int c = wave / pieces, p = wave - c * pieces;
            while (c < n_chunks) {
                const float* from = x0 + c * chunk + p * piece;
                float* to = w + c * stride + p * piece;
                if (wide) {
                    if (4 * lane < chunk - p * piece)
                        __builtin_amdgcn_global_load_lds((const void*)(from + 4 * lane),
                                                         (__attribute__((address_space(3))) void*)to, 16, 0, 0);
                } else {
                    if (lane < chunk - p * piece)
                        __builtin_amdgcn_global_load_lds((const void*)(from + lane),
                                                         (__attribute__((address_space(3))) void*)to, 4, 0, 0);
                }
                p += kMmWaves;
                while (p >= pieces) {
                    p -= pieces;
                    ++c;
                }
            }
        } else {
            for (int i = tid; i < n_chunks * chunk; i += kMmThreads) {
                const int64_t m = m0 + i;
                const int c = i / chunk;
                w[i + c * pad] = (m >= 0 && m < a.n_raw) ? a.x[m] : 0.f;
            }
        }
        __builtin_amdgcn_s_setprio(0);
    };

    int first = n_it, last = -1;  // the blocks with a sum that is not finite, of this wave
    // adds the WK partial tiles of block b and writes its outputs: thread
    // e of a tile has element (row 4 (l / 16) + v, column l % 16), l = e / 4, v = e % 4
    auto finish = [&](int64_t b, const float (*part)[256]) {
        if (tid < 256 * WM) {  // whole waves
            const int tile = tid >> 8, e = tid & 255, l = e >> 2, v = e & 3;
            float t[WK];
#pragma unroll
            for (int w = 0; w < WK; ++w) t[w] = part[tile * WK + w][e];
#pragma unroll
            for (int h = WK / 2; h > 0; h /= 2)
#pragma unroll
                for (int w = 0; w < h; ++w) t[w] += t[w + h];
            float s = t[0];
            float o = __shfl_xor(s, 4);  // the other part of the same output
            const bool im = l & 1;
            const int64_t j = b * NO + 128 * tile + 8 * (4 * (l >> 4) + v) + ((l & 15) >> 1);
            if (__any(!(fabsf(s) <= 3.402823466e38f))) {
                first = min(first, (int)(b - b0));
                last = (int)(b - b0);
            }
            if (j >= a.n_out) return;
            const double cyc = a.cyc_per_out * (double)j;
            float sn, cs;
            sincospif(-2.0f * (float)(cyc - rint(cyc)), &sn, &cs);
            reinterpret_cast<float*>(a.out)[2 * j + (im ? 1 : 0)] = im ? o * sn + s * cs : s * cs - o * sn;
        }
    };

    // this block's products into its wave's partial tile.  Partial sum v < 16 has
    // groups v, v + 16, ..: 16 / WK of them are this wave's, added here in the order
    // of finish's tree
    auto multiply = [&](const float* w, float (*part)[256]) {
        const float* row = w + (16 * mt + J) * stride + 4 * q;
        constexpr int U = kMmWaves / WK;
        // with padding 8 D is a multiple of 16, so a group of 16 taps lies in one chunk
        auto partial = [&](int u) {
            mm_v4f acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = acc0, acc2 = acc0, acc3 = acc0;
#pragma unroll
            for (int g = u; g < NG; g += U) {
                const unsigned kk = 16 * (kw + WK * g);
                const float4 x = *reinterpret_cast<const float4*>(row + kk + pad * (int)(((uint64_t)kk * inv_chunk) >> 32));
                acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x, bop[g][0], acc0, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(x.y, bop[g][1], acc1, 0, 0, 0);
                acc2 = __builtin_amdgcn_mfma_f32_16x16x4f32(x.z, bop[g][2], acc2, 0, 0, 0);
                acc3 = __builtin_amdgcn_mfma_f32_16x16x4f32(x.w, bop[g][3], acc3, 0, 0, 0);
            }
            return (acc0 + acc1) + (acc2 + acc3);
        };
        mm_v4f sum = partial(0);
        if constexpr (U == 2 && NG > 1) sum += partial(1);
        if constexpr (U == 4) {
            if constexpr (NG > 2) sum += partial(2);
            if constexpr (NG > 1) {
                mm_v4f odd = partial(1);
                if constexpr (NG > 3) odd += partial(3);
                sum += odd;
            }
        }
        // D layout: lane holds rows 4 (lane / 16) + v, column lane % 16
        *reinterpret_cast<float4*>(part[mt * WK + kw] + 4 * lane) = make_float4(sum[0], sum[1], sum[2], sum[3]);
    };

    if constexpr (NB > 1) {
        auto step = [&](int it, const float* w, float* next, float (*part)[256], const float (*last)[256]) {
            __builtin_amdgcn_s_waitcnt(0);  // this wave's DMA for the block has landed
            __syncthreads();
            if (it + 1 < n_it) stage(b0 + it + 1, next);
            if (it > 0) finish(b0 + it - 1, last);
            multiply(w, part);
        };
        if (n_it > 0) stage(b0, buf0);
        for (int it = 0; it < n_it; it += 2) {
            step(it, buf0, buf1, red[0], red[1]);
            if (it + 1 < n_it) step(it + 1, buf1, buf0, red[1], red[0]);
        }
    } else {
        for (int it = 0; it < n_it; ++it) {
            __syncthreads();
            stage(b0 + it, buf0);
            if (it > 0) finish(b0 + it - 1, red[(it - 1) & 1]);
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            multiply(buf0, red[it & 1]);
        }
    }
    __syncthreads();
    if (n_it > 0) finish(b0 + n_it - 1, red[(n_it - 1) & 1]);

    // outputs that are not finite, by all waves, when the taps' registers are free
    int* range = reinterpret_cast<int*>(red[n_it & 1]);  // the partial tiles that no wave reads any more
    if (lane == 0) {
        range[2 * wave] = first;
        range[2 * wave + 1] = last;
    }
    __syncthreads();  // and the outputs are written
#pragma unroll
    for (int w = 0; w < 4 * WM; ++w) {  // the waves that finish
        first = min(first, range[2 * w]);
        last = max(last, range[2 * w + 1]);
    }
    for (int64_t j = (b0 + first) * NO + 32 * wave; j < (b0 + last + 1) * NO; j += 32 * kMmWaves) not_finite(a, j);
}

namespace {
typedef void (*MmFn)(HetdecArgs, int, unsigned, bool, int64_t);

template <int WK, int NG>
MmFn mm_fn2() {
    if constexpr (NG <= mm_groups_max(WK, 2))
        return rsf_hetdec_mfma_k<WK, NG, 2>;
    else
        return nullptr;
}

template <int WK>
MmFn mm_fn(int NG) {
    switch (NG) {
        case 1: return mm_fn2<WK, 1>();
        case 2: return mm_fn2<WK, 2>();
        case 3: return mm_fn2<WK, 3>();
        case 4: return mm_fn2<WK, 4>();
        case 5: return mm_fn2<WK, 5>();
        case 6: return mm_fn2<WK, 6>();
        case 7: return mm_fn2<WK, 7>();
        case 8: return mm_fn2<WK, 8>();
        case 10: return mm_fn2<WK, 10>();
        case 12: return mm_fn2<WK, 12>();
        case 14: return mm_fn2<WK, 14>();
        case 16: return mm_fn2<WK, 16>();
        default: return nullptr;
    }
}

MmFn mm_kernel(const MmShape& m) {
    if (m.NB == 1) {
        switch (m.NG) {
            case 8: return rsf_hetdec_mfma_k<16, 8, 1>;
            case 10: return rsf_hetdec_mfma_k<16, 10, 1>;
            case 12: return rsf_hetdec_mfma_k<16, 12, 1>;
            case 14: return rsf_hetdec_mfma_k<16, 14, 1>;
            case 16: return rsf_hetdec_mfma_k<16, 16, 1>;
            case 18: return rsf_hetdec_mfma_k<16, 18, 1>;
            case 20: return rsf_hetdec_mfma_k<16, 20, 1>;
            default: return nullptr;
        }
    }
    return m.WK == 4 ? mm_fn<4>(m.NG) : m.WK == 8 ? mm_fn<8>(m.NG) : m.WK == 16 ? mm_fn<16>(m.NG) : nullptr;
}
}  // namespace

// The direct sum's LDS: what a plan's taps and decimation may need at most.
size_t hetdec_lds(int L, int D) {
    return (size_t)2 * L * sizeof(float) + (size_t)((kHdOut - 1) * D + L) * sizeof(float);
}

hipError_t launch_hetdec(const HetdecArgs& a, int n_cu, hipStream_t s) {
    const MmShape m = mm_shape(a.L, a.D, a.n_out, n_cu);
    if (MmFn fn = mm_kernel(m)) {
        const int64_t no = 128 * (kMmWaves / m.WK);
        const int64_t n_blk = (a.n_out + no - 1) / no;
        const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>(n_blk, n_cu));
        // a window starts at sample 128 k D - K D of the series, a row 8 D samples after another
        const bool wide = reinterpret_cast<uintptr_t>(a.x) % 16 == 0 && a.c % 4 == 0;
        // kk / (8 D) for kk < 2^16 by the reciprocal rounded up
        const unsigned inv = (unsigned)(((1ull << 32) + 8ull * a.D - 1) / (8ull * a.D));
        hipLaunchKernelGGL(fn, dim3(grid), dim3(kMmThreads), 0, s, a, mm_pad(a.D), inv, wide, n_blk);
        return hipGetLastError();
    }
    const unsigned grid = (unsigned)((a.n_out + kHdOut - 1) / kHdOut);
    hipLaunchKernelGGL(rsf_hetdec_k, dim3(grid), dim3(kHdThreads), hetdec_lds(a.L, a.D), s, a);
    return hipGetLastError();
}

// Grants the direct sum's LDS, which only grows (the matrix-core form's is static).
hipError_t hetdec_set_lds_limit(size_t bytes) {
    static size_t granted = 0;
    if (bytes <= granted) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute((const void*)rsf_hetdec_k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) granted = bytes;
    return e;
}

}  // namespace rsf
