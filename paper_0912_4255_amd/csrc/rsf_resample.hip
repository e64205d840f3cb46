// Barycentric resampling (paper Sec. III.A.2, steps 1-5) for gfx950.
//
// One workgroup (8 waves) resamples a 16 x 128 tile of the SSB grid
// k = LB * n_a + n_b (16 runs of 128 consecutive samples).  Two kernels:
// rsf_resample_run_k interpolates the timing chain along each run and carries
// every ordinary call; rsf_resample_k evaluates it per sample (long sampling
// intervals, fast or refused orbits; orbits in half tiles), per run of 64 samples:
//   1. every lane inverts eq. eq21 for its k in FP64 (one fixed-point step
//      and one Newton step, residual below 1e-12 s);
//   2. the wave loads the detector-grid window its 64 outputs need into LDS,
//      applying the heterodyne correction z = x_h exp(-2 pi i f_h t_m) on the
//      way (eqs. absorb/Fa3; t_m at the detector samples from a third-order
//      expansion about the first lane's inversion, the phase f_h t_m reduced
//      mod 1 in FP64);
//   3. every lane interpolates z at T^k with the W-tap kernel in FP32;
//   4. a(T^k), b(T^k) come from the detector tensor in FP64, and the masked
//      antenna sums A', B', C' (eqs. eq9/eq10) accumulate in FP64.
// The FFT layout (row n_b, what the first FFT pass reads contiguously) goes
// through a tile in LDS; the natural order (API outputs) is written directly.
#include <climits>

#include "rsf_chain.h"
#include "rsf_launch.h"

namespace rsf {

namespace {
constexpr int kTileB = 128;   // n_b: two groups of 64 lanes
constexpr int kTileA = 16;
constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kWinMax = 64 + kMaxTaps + 8;

__device__ __forceinline__ uint32_t pack_half2(float re, float im) {
    const __half2 h = __floats2half2_rn(re, im);
    return *reinterpret_cast<const uint32_t*>(&h);
}
}  // namespace

namespace {
// The series' runs: 128 samples.
struct SeriesRun {
    static constexpr double mid = 63.5, half = 82.0, p = 78.0, q = 48.25;
};
constexpr int kRunLen = 128;
static_assert(kRunLen == kTileB, "a run is a tile row");
// window of a run: 64 samples and their compression (104 - W slots each half,
// as the general kernel stages), and the taps
constexpr int kRunWin = 208;

// Interpolation weight at distance x, sx = sin(pi x): Lanczos-W, or the
// Dirichlet kernel of n samples (pin = pi / n).
__device__ __forceinline__ float tap_weight(const InterpDev& ip, float x, float sx, float pin) {
    if (x == 0.f) return 1.f;
    const float rx = __builtin_amdgcn_rcpf(kPiF * x);  // 1 / (pi x)
    if (ip.kernel == 0) {
        // sin(2 pi x / W) straight from x: x is exact (frac + integer) and
        // an angle-addition form would cancel when x -> 0 off the centre tap
        const float s2 = sinpif(2.f * x / (float)ip.taps);
        return sx * s2 * (0.5f * (float)ip.taps) * rx * rx;
    }
    // sin(pi x) / (n tan(pi x / n)) = sinc(x) g(y), y = pi x / n, with
    // g = y / tan(y) (n even) or y / sin(y) (n odd), a series when small
    const float y = x * pin;
    float g;
    if (fabsf(y) < 0.01f) {
        const float y2 = y * y;
        g = ip.n_odd ? 1.f + y2 * (1.f / 6.f + y2 * (7.f / 360.f)) : 1.f - y2 * (1.f / 3.f + y2 * (1.f / 45.f));
    } else {
        g = ip.n_odd ? y / sinf(y) : y / tanf(y);
    }
    return sx * rx * g;
}

// One resampled sample: to the tile (FFT layout), or straight to the API
// outputs (natural order: the lanes hold consecutive k; whole waves call this).
__device__ __forceinline__ void put_sample(const ResampleArgs& A, int sky, int64_t k, bool valid, float2 zt, double tm,
                                           double av, double bv, bool mk, float4& main, float& tile_tm) {
    if (A.layout == 1) {
        const float4 m = A.f16 ? make_float4(__uint_as_float(pack_half2(zt.x, zt.y)), (float)av, (float)bv, (float)tm)
                               : make_float4(zt.x, zt.y, (float)av, (float)bv);
        main = valid ? m : make_float4(0.f, 0.f, 0.f, 0.f);
        tile_tm = valid ? (float)tm : 0.f;
        return;
    }
    const int64_t at = (int64_t)sky * A.n + k;
    if (valid) {
        if (A.out_z) A.out_z[at] = A.f16 ? make_float2(0.f, 0.f) : zt;
        if (A.out_zh) A.out_zh[at] = pack_half2(zt.x, zt.y);
        if (A.out_a) A.out_a[at] = (float)av;
        if (A.out_b) A.out_b[at] = (float)bv;
        if (A.out_tm) A.out_tm[at] = tm;
        if (A.out_u) A.out_u[at] = ((double)k * A.dt - tm) / A.dt;
    }
    const uint64_t bal = __ballot(valid && mk);
    if (A.out_mask && (threadIdx.x & 63) == 0) {  // k: the first of 64, a multiple of 32
        uint32_t* out = A.out_mask + (int64_t)sky * A.n_words;
        const int64_t word = k / 32;
        if (word < A.n_words) out[word] = (uint32_t)bal;
        if (word + 1 < A.n_words) out[word + 1] = (uint32_t)(bal >> 32);
    }
}

// The tile to the FFT layout: element (n_b, n_a) at n_b P + n_a, 16 n_a at a time.
template <int COLS>
__device__ __forceinline__ void write_tile(const ResampleArgs& A, int sky, int b0, int64_t a0,
                                           const float4 (&main)[kTileA][COLS + 1], const float (&tm)[kTileA][COLS + 1]) {
    if (A.layout != 1) return;
    const int64_t sky_off = (int64_t)sky * A.rs_sky_stride;
    constexpr int threads = 4 * COLS;
#pragma unroll
    for (int q = 0; q < kTileA * COLS / threads; ++q) {
        const int e = threadIdx.x + q * threads;
        const int nb = e / kTileA, na = e % kTileA;
        if (b0 + nb < A.LB && a0 + na < A.P) {
            const int64_t idx = sky_off + (int64_t)(b0 + nb) * A.P + a0 + na;
            A.rs_main[idx] = main[na][nb];
            if (!A.f16) A.rs_tm[idx] = tm[na][nb];
        }
    }
}

// antenna-sum partials of the workgroup, fixed reduction order, to (or, ADD, into)
// the sums of tile `tile` of a row of tiles
template <bool ADD, int WAVES>
__device__ __forceinline__ void antenna_partials(const ResampleArgs& A, int sky, int tile, int row_tiles, double sA,
                                                 double sB, double sC, double (&red)[WAVES][3]) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        sA += __shfl_xor(sA, off);
        sB += __shfl_xor(sB, off);
        sC += __shfl_xor(sC, off);
    }
    if ((threadIdx.x & 63) == 0) {
        double* r = red[threadIdx.x >> 6];
        r[0] = sA;
        r[1] = sB;
        r[2] = sC;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) t += red[w][threadIdx.x];
        double* p = A.partials + ((int64_t)sky * A.n_blocks + blockIdx.y * row_tiles + tile) * 3 + threadIdx.x;
        if (ADD)
            atomicAdd(p, t);
        else
            *p = t;
    }
}
}  // namespace

// BIN: the source is in a circular binary orbit; the grid is regular in
// emission time (target t_b + R(t_s + t_b) of the inversion) and the delay
// used by the correction and stored for the spindown phase is the total
// d = t_m - R(tau_e), tau_e from tau_e + R(tau_e) = tau + t_m(tau).
// COLS: 128, or 64 with orbits: half tiles in workgroups of 4 waves, of which a CU
// holds three where it holds one of 8 (161 registers), adding their antenna sums
// into the tile's, which rsf_resample_run_k<true> or the launch clears: two numbers
// added to 0, the same in either order.  Four rows of 864,001 samples with an orbit of
// one hour: 270 us, 302 us in whole tiles; one of 86,400: 40 and 48 us.
template <bool BIN, int COLS>
__global__ __launch_bounds__(4 * COLS) void rsf_resample_k(ResampleArgs A) {
    constexpr int kWaves = COLS / 16, kHalves = COLS / 64;
    __shared__ float2 win[kWaves][kWinMax];
    __shared__ float4 tile_main[kTileA][COLS + 1];
    __shared__ float tile_tm[kTileA][COLS + 1];
    __shared__ double red[kWaves][3];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int b0 = blockIdx.x * COLS;
    const int64_t a0 = (int64_t)blockIdx.y * kTileA;
    const int sky = blockIdx.z;
    const double* srow = A.sky + (int64_t)A.sky_stride * sky;
    const double alpha = srow[0], delta = srow[1];
    BinaryOrbit bo{};
    bool orbit_ok = true;
    if constexpr (BIN) {
        const BinaryOrbit given{srow[2], srow[3], srow[4]};
        orbit_ok = orbit_admitted(given);
        bo = orbit_or_none(given);
        if (A.run && orbit_ok && orbit_slow(bo, SeriesRun::half * A.dt, A.run_delay)) return;
    }
    const double3 n0 = sky_unit(alpha, delta);
    const SkyFrame fr = sky_frame(alpha, delta);
    const int W = A.ip.taps;
    const int hw = W / 2;
    const float pin = kPiF / (float)A.ip.n;  // pi / n of the Dirichlet kernel
    // Dirichlet kernel of a long series: |y| = pi |x| / n < pi (hw + 1) / n
    // keeps y / tan(y) (or y / sin(y)) within 1 + 3e-8, so in FP32 every
    // weight is sin(pi x) / (pi x) = (-1)^m sin(pi frac) / (pi x), m = hw - i
    const bool flat = A.ip.kernel == 1 && pin * (float)(hw + 1) < 2.9e-4f;
    double sA = 0.0, sB = 0.0, sC = 0.0;
    bool window_overflow = false;
    for (int unit = wave; unit < kHalves * kTileA; unit += kWaves) {
        const int ia = unit >> (kHalves - 1), ib = (unit & (kHalves - 1)) * 64 + lane;
        const int64_t n_a = a0 + ia;
        const int n_b = b0 + ib;
        const int64_t k = (int64_t)A.LB * n_a + n_b;
        const bool valid = (n_b < A.LB) && (n_a < A.P) && (k < A.n);

        int j = 0;
        float frac = 0.f;
        double tm = 0.0, av = 0.0, bv = 0.0;
        bool mk = false;
        Inversion inv{};
        if (valid) {
            const double tb = (double)k * A.dt;
            double target = tb;
            if constexpr (BIN) target = tb + binary_delay(bo, A.t_start + tb);
            inv = invert_ssb(A.t_start, target, n0, A.eph, A.det);
            const double T = inv.T;
            tm = tb - T;
            beam_ab(inv.ang, A.det, fr, &av, &bv);
            const double u = T / A.dt;
            const double fl = floor(u);
            j = (int)fl;
            frac = (float)(u - fl);
            const int64_t jn = (int64_t)floor(u + 0.5);
            mk = (jn >= 0) && (jn < A.n) && !in_gap(A.gaps, A.n_gaps, jn);
        }
        // expansion point of t_m for this run's window: the first valid lane
        // (lane 0 whenever any lane is valid: it has the run's smallest k)
        const uint64_t vmask = __ballot(valid);
        const int src = vmask ? __ffsll((long long)vmask) - 1 : 0;
        const RoemerD rref = readlane_rd(inv.r1, src);
        const double t_ref = readlane_d(inv.T1, src);

        // window of detector samples needed by this run
        int jmin = valid ? j : INT_MAX;
        int jmax = valid ? j : INT_MIN;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            jmin = min(jmin, __shfl_xor(jmin, off));
            jmax = max(jmax, __shfl_xor(jmax, off));
        }
        const bool any = jmin != INT_MAX;
        const int w0 = any ? jmin - hw + 1 : 0;
        const int wlen = any ? (jmax - jmin + W) : 0;
        const bool ok = wlen <= kWinMax;
        if (any && ok) {
            for (int p = lane; p < wlen; p += 64) {
                const int64_t jj = (int64_t)w0 + p;
                float2 z = make_float2(0.f, 0.f);
                if (jj >= 0 && jj < A.n) {
                    const float2 xv = A.x[jj];
                    double tmj = tm_expand(rref, (double)jj * A.dt - t_ref);
                    if constexpr (BIN)
                        tmj -= binary_delay(bo, emission_time(bo, A.t_start + (double)jj * A.dt + tmj));
                    const double cyc = A.f_het * tmj;
                    const float ph = (float)(cyc - rint(cyc));
                    const float s = __builtin_amdgcn_sinf(ph), c = __builtin_amdgcn_cosf(ph);  // revolutions
                    z = make_float2(xv.x * c + xv.y * s, xv.y * c - xv.x * s);  // x * (c - i s)
                }
                win[wave][p] = z;
            }
        }
        if (any && !ok) window_overflow = true;
        // the window is this wave's own: its LDS operations complete in order,
        // so a wave-level barrier (no workgroup synchronisation) suffices
        __builtin_amdgcn_wave_barrier();

        float2 zt = make_float2(0.f, 0.f);
        if (valid) {
            if (ok && flat) {
                const int base = j - hw + 1 - w0;
                if (frac == 0.f || frac == 1.f) {
                    // x = 0 at one tap (the centre, or the next one when the
                    // fraction rounded up to 1 in FP32), sin(pi x) = 0 at the others
                    zt = win[wave][base + hw - 1 + (frac == 1.f ? 1 : 0)];
                } else {
                    // sum of (-1)^m z / x, then the common factor sin(pi frac) / pi
                    float ax = 0.f, ay = 0.f;
                    for (int i = 1; i <= W; ++i) {
                        const float x = frac + (float)(hw - i);
                        float r = __builtin_amdgcn_rcpf(x);
                        if ((hw - i) & 1) r = -r;
                        const float2 zz = win[wave][base + i - 1];
                        ax += r * zz.x;
                        ay += r * zz.y;
                    }
                    const float sc = sinpif(frac) * (1.0f / kPiF);
                    zt = make_float2(ax * sc, ay * sc);
                }
            } else if (ok) {
                const float sf = sinpif(frac);
                const int base = j - hw + 1 - w0;
                for (int i = 1; i <= W; ++i) {
                    const float w = tap_weight(A.ip, frac + (float)(hw - i), ((hw - i) & 1) ? -sf : sf, pin);
                    const float2 zz = win[wave][base + i - 1];
                    zt.x += w * zz.x;
                    zt.y += w * zz.y;
                }
            } else {
                zt = make_float2(__int_as_float(0x7fc00000), __int_as_float(0x7fc00000));
            }
            if (!orbit_ok) zt = make_float2(__int_as_float(0x7fc00000), __int_as_float(0x7fc00000));
            if (mk) {
                sA += av * av;
                sB += bv * bv;
                sC += av * bv;
            }
        }
        put_sample(A, sky, k, valid, zt, tm, av, bv, mk, tile_main[ia][ib], tile_tm[ia][ib]);
        __builtin_amdgcn_wave_barrier();  // the next run rewrites this wave's window
    }
    __syncthreads();  // the tile rows of all waves are complete

    if (window_overflow && lane == 0) atomicOr(A.flags, 2u);
    if (!orbit_ok && threadIdx.x == 0) atomicOr(A.flags, 4u);
    write_tile<COLS>(A, sky, b0, a0, tile_main, tile_tm);
    if constexpr (COLS == kTileB)
        antenna_partials<false>(A, sky, blockIdx.x, gridDim.x, sA, sB, sC, red);
    else
        antenna_partials<true>(A, sky, blockIdx.x / 2, (gridDim.x + 1) / 2, sA, sB, sC, red);
}

// The interpolated chain: the tile's 16 runs of 128 samples, two per wave.  The
// 80 nodes are evaluated first, one per thread, and turned into quartics of
// V = d / dt, a and b and of the window's delay; a run's detector samples are
// heterodyne-corrected into its wave's window once for 128 outputs; the gaps are
// looked up per run.  What bounds it: vector issue (the window's phases and the
// taps), then latency.  3,456,000 samples, 16 taps: 69 us against 109 for runs of
// 64 with quadratics from three nodes per wave and run, a division and a search
// of the gap list per sample; 5,184,000 samples 94 against 145 us; 8 binary rows
// of 864,001 samples 133 against 452 us (every sample's chain, and the emission
// time's fixed point per window sample).
template <bool BIN>
__global__ __launch_bounds__(kThreads, 4) void rsf_resample_run_k(ResampleArgs A) {
    struct Run {
        double poly[3][5], het[5], vn[5], u_c;
        int gap, pad;
    };
    __shared__ Run runs[kTileA];
    __shared__ float2 win[kWaves][kRunWin];
    __shared__ float4 tile_main[kTileA][kTileB + 1];
    __shared__ float tile_tm[kTileA][kTileB + 1];
    __shared__ double red[kWaves][3];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b0 = blockIdx.x * kTileB;
    const int64_t a0 = (int64_t)blockIdx.y * kTileA;
    const int sky = blockIdx.z;
    const double* srow = A.sky + (int64_t)A.sky_stride * sky;
    BinaryOrbit bo{};
    if constexpr (BIN) {
        bo = BinaryOrbit{srow[2], srow[3], srow[4]};
        if (!orbit_admitted(bo) || !orbit_slow(bo, SeriesRun::half * A.dt, A.run_delay)) {  // rsf_resample_k's
            if (tid < 3) A.partials[((int64_t)sky * A.n_blocks + blockIdx.y * gridDim.x + blockIdx.x) * 3 + tid] = 0.0;
            return;
        }
    }
    const int W = A.ip.taps, hw = W / 2;
    const float pin = kPiF / (float)A.ip.n;  // pi / n of the Dirichlet kernel
    // Dirichlet kernel of a long series: |y| = pi |x| / n < pi (hw + 1) / n
    // keeps y / tan(y) (or y / sin(y)) within 1 + 3e-8, so in FP32 every
    // weight is sin(pi x) / (pi x) = (-1)^m sin(pi frac) / (pi x), m = hw - i
    const bool flat = A.ip.kernel == 1 && pin * (float)(hw + 1) < 2.9e-4f;

    if (tid < 5 * kTileA) {
        const int rr = tid / 5, i = tid - 5 * rr;
        const double alpha = srow[0], delta = srow[1];
        const double tb = ((double)((int64_t)A.LB * (a0 + rr) + b0) + (SeriesRun::mid + node_at<SeriesRun>(i))) * A.dt;
        double target = tb;
        if constexpr (BIN) target = tb + binary_delay(bo, A.t_start + tb);
        const Inversion inv = invert_ssb(A.t_start, target, sky_unit(alpha, delta), A.eph, A.det);
        double av, bv;
        beam_ab(inv.ang, A.det, sky_frame(alpha, delta), &av, &bv);
        const double V = (tb - inv.T) / A.dt;
        Run& v = runs[rr];
        v.vn[i] = V;
        v.poly[0][i] = V;
        v.poly[1][i] = av;
        v.poly[2][i] = bv;
    }
    __syncthreads();
    if (tid < 4 * kTileA) {
        const int rr = tid >> 2, qi = tid & 3;
        Run& v = runs[rr];
        const double k0 = (double)((int64_t)A.LB * (a0 + rr) + b0);
        if (qi < 3) {
            to_quartic<SeriesRun>(v.poly[qi]);
        } else {
            window_delay<SeriesRun>(v.vn, A.f_het * A.dt, v.het);
            v.u_c = k0 + SeriesRun::mid - v.vn[2];
        }
    } else if (tid < 5 * kTileA) {  // the second wave, beside the first
        Run& v = runs[tid - 4 * kTileA];
        // the run's detector samples, from the nodes just outside its ends
        const double c = (double)((int64_t)A.LB * (a0 + tid - 4 * kTileA) + b0) + SeriesRun::mid;
        v.gap = gap_state(A.gaps, A.n_gaps, (int64_t)floor(c - SeriesRun::p - v.vn[0]) - 1,
                          (int64_t)floor(c + SeriesRun::p - v.vn[4]) + 2);
    }
    __syncthreads();

    double sA = 0.0, sB = 0.0, sC = 0.0;
    bool overflow = false;
    for (int ia = wave; ia < kTileA; ia += kWaves) {
        const Run& v = runs[ia];
        const int64_t n_a = a0 + ia;
        const int64_t k0 = (int64_t)A.LB * n_a + b0;
        // samples of the run: inside the row, the rows stored and the series
        const int count = n_a < A.P ? (int)max((int64_t)0, min((int64_t)min(kRunLen, A.LB - b0), A.n - k0)) : 0;
        int64_t w0 = 0;
        int wlen = 0;
        bool ok = true;
        if (count > 0) {
            const int64_t j0 = (int64_t)floor((double)k0 - quartic(v.poly[0], -SeriesRun::mid));
            const int64_t j1 = (int64_t)floor((double)(k0 + count - 1) -
                                              quartic(v.poly[0], (double)(count - 1) - SeriesRun::mid));
            w0 = j0 - hw + 1;
            const int64_t need = j1 - j0 + W;
            ok = j1 >= j0 && need <= 2 * (104 - W) + W;
            wlen = ok ? (int)need : 0;
            const double xc = (double)w0 - v.u_c;
            for (int p0 = 0; p0 < wlen; p0 += 192) {
                float2 xv[3];
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const int p = p0 + 64 * q + lane;
                    const int64_t jj = w0 + p;
                    xv[q] = (p < wlen && jj >= 0 && jj < A.n) ? A.x[jj] : make_float2(0.f, 0.f);
                }
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const int p = p0 + 64 * q + lane;
                    if (p0 + 64 * q < wlen) {
                        const double cyc = quartic(v.het, xc + (double)p);
                        const float ph = (float)(cyc - rint(cyc));
                        const float s = __builtin_amdgcn_sinf(ph), c = __builtin_amdgcn_cosf(ph);  // revolutions
                        if (p < wlen)  // x * (c - i s)
                            win[wave][p] = make_float2(xv[q].x * c + xv[q].y * s, xv[q].y * c - xv[q].x * s);
                    }
                }
            }
            if (!ok) overflow = true;
        }
        // the window is this wave's own: its LDS operations complete in order,
        // so a wave-level barrier (no workgroup synchronisation) suffices
        __builtin_amdgcn_wave_barrier();
        for (int h = 0; h < 2; ++h) {
            const int l = 64 * h + lane;
            const int64_t k = k0 + l;
            const bool valid = l < count;
            float2 zt = make_float2(0.f, 0.f);
            double tm = 0.0, av = 0.0, bv = 0.0;
            bool mk = false;
            if (valid) {
                const double s = (double)l - SeriesRun::mid;
                const double V = quartic(v.poly[0], s);
                tm = V * A.dt;
                av = quartic(v.poly[1], s);
                bv = quartic(v.poly[2], s);
                const double u = (double)k - V, fl = floor(u);
                const float frac = (float)(u - fl);
                const int base = (int)((int64_t)fl - hw + 1 - w0);
                const double fn = floor(u + 0.5);
                // a position that is not a number (a sky that is not) is looked up as
                // sample 0, as the general kernel does, and so reaches A', B', C'
                mk = v.gap != 1 && !(fn < 0.0) && !(fn >= (double)A.n);
                if (v.gap == 2) mk = mk && !in_gap(A.gaps, A.n_gaps, (int64_t)fn);
                if (mk) {
                    sA += av * av;
                    sB += bv * bv;
                    sC += av * bv;
                }
                const float2* wz = win[wave] + base;
                const float sf = sinpif(frac);
                if (!ok || base < 0 || base + W > wlen) {
                    overflow = true;
                    zt = make_float2(__int_as_float(0x7fc00000), __int_as_float(0x7fc00000));
                } else if (flat) {
                    // sum of (-1)^m z / x over the taps beside the two next to u,
                    // times sin(pi frac) / pi; taps hw - m and hw + 1 + m in pairs
                    const float x1 = frac - 1.f;
                    float w0_, w1_, unused;
                    sinc_d(frac, sf, 0.f, w0_, unused);
                    sinc_d(x1, -sf, 0.f, w1_, unused);
                    float ax = 0.f, ay = 0.f;
                    auto pair = [&](int m, float sg) {
                        const float2 zl = wz[hw - 1 - m], zr = wz[hw + m];
                        const float rl = sg * __builtin_amdgcn_rcpf(frac + (float)m);
                        const float rr = -sg * __builtin_amdgcn_rcpf(x1 - (float)m);
                        ax += rl * zl.x + rr * zr.x;
                        ay += rl * zl.y + rr * zr.y;
                    };
                    int m = 1;
                    for (; m + 1 < hw; m += 2) {
                        pair(m, -1.f);
                        pair(m + 1, 1.f);
                    }
                    if (m < hw) pair(m, -1.f);
                    const float sp = sf * (1.0f / kPiF);
                    const float2 za = wz[hw - 1], zb = wz[hw];
                    zt = make_float2(sp * ax + (w0_ * za.x + w1_ * zb.x), sp * ay + (w0_ * za.y + w1_ * zb.y));
                    // u on a sample: that one alone, also beside one that is not finite
                    if (__builtin_expect(__any(sf == 0.f), 0) && sf == 0.f) zt = frac < 0.5f ? za : zb;
                } else {
                    for (int i = 1; i <= W; ++i) {
                        const float w = tap_weight(A.ip, frac + (float)(hw - i), ((hw - i) & 1) ? -sf : sf, pin);
                        const float2 zz = wz[i - 1];
                        zt.x += w * zz.x;
                        zt.y += w * zz.y;
                    }
                }
            }
            put_sample(A, sky, k, valid, zt, tm, av, bv, mk, tile_main[ia][l], tile_tm[ia][l]);
        }
        __builtin_amdgcn_wave_barrier();  // the next run rewrites this wave's window
    }
    __syncthreads();  // the tile rows of all waves are complete
    if (__any(overflow) && lane == 0) atomicOr(A.flags, 2u);
    write_tile<kTileB>(A, sky, b0, a0, tile_main, tile_tm);
    antenna_partials<false>(A, sky, blockIdx.x, gridDim.x, sA, sB, sC, red);
}

// One workgroup per sky: sums the block partials of every detector in a
// fixed order and forms the F-statistic coefficients 2B'/D', 2A'/D', -4C'/D'
// (eq. eq6 with noise-weighted sums) in FP64.
__global__ __launch_bounds__(256) void rsf_antenna_reduce_k(ReduceArgs R) {
    __shared__ double red[256][3];
    const int sky = blockIdx.x;
    double wsum[3] = {0.0, 0.0, 0.0};
    for (int X = 0; X < R.n_det; ++X) {
        double s[3] = {0.0, 0.0, 0.0};
        const double* p = R.partials + ((int64_t)X * R.n_sky + sky) * (int64_t)R.n_blocks * 3;
        for (int i = threadIdx.x; i < R.n_blocks; i += 256) {
            s[0] += p[3 * i + 0];
            s[1] += p[3 * i + 1];
            s[2] += p[3 * i + 2];
        }
        red[threadIdx.x][0] = s[0];
        red[threadIdx.x][1] = s[1];
        red[threadIdx.x][2] = s[2];
        __syncthreads();
        for (int h = 128; h > 0; h >>= 1) {
            if (threadIdx.x < h) {
                red[threadIdx.x][0] += red[threadIdx.x + h][0];
                red[threadIdx.x][1] += red[threadIdx.x + h][1];
                red[threadIdx.x][2] += red[threadIdx.x + h][2];
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            if (R.abc_det[X]) {
                double* o = R.abc_det[X] + (int64_t)sky * 3;
                o[0] = red[0][0];
                o[1] = red[0][1];
                o[2] = red[0][2];
            }
            wsum[0] += R.w[X] * red[0][0];
            wsum[1] += R.w[X] * red[0][1];
            wsum[2] += R.w[X] * red[0][2];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double A = wsum[0], B = wsum[1], C = wsum[2];
        const double D = A * B - C * C;
        if (R.abc_w) {
            R.abc_w[3 * sky + 0] = A;
            R.abc_w[3 * sky + 1] = B;
            R.abc_w[3 * sky + 2] = C;
        }
        float* cf = R.coef + 4 * sky;
        if (D > 0.0 && A > 0.0 && B > 0.0) {
            cf[0] = (float)(2.0 * B / D);
            cf[1] = (float)(2.0 * A / D);
            cf[2] = (float)(-4.0 * C / D);
            cf[3] = 0.f;
        } else {
            const float nan = __int_as_float(0x7fc00000);
            cf[0] = cf[1] = cf[2] = nan;
            cf[3] = 1.f;
            atomicOr(R.flags, 1u);
        }
    }
}

// Into an FFT what is resampled goes in FP32: sampling intervals up to 2.3 s, with t_m to
// kDelayErr and A', B', C' to 1e-11.  The API outputs t_m, u, A', B', C' are FP64, so there
// the remainders stay below the exact chain's own error (the inversion's residual of up
// to 1e-12 s): 3e-13 s and 1e-13, sampling intervals up to 0.95 s.  At the other rule's limits
// t_m was off by 9.2e-12 s (a_p = 10 s, P_b = 4 h, dt = 0.5 s) against 6.3e-13 s for the
// exact chain, A', B', C' by 5.7e-13 (dt = 2 s) against 6e-15.  Four binary rows of 864,001 samples:
// 82 us interpolated, 227 us where the orbit is faster than that.
double resample_run_delay(bool api) { return api ? 3e-13 : kDelayErr; }
bool resample_interpolates(double dt, const EphDev& e, bool api) {
    return chain_interpolates(e, SeriesRun::half * dt, resample_run_delay(api), api ? 1e-13 : 1e-11);
}

hipError_t launch_resample(const ResampleArgs& a, int n_sky, hipStream_t s) {
    const dim3 grid((unsigned)((a.LB + kTileB - 1) / kTileB), (unsigned)((a.P + kTileA - 1) / kTileA), (unsigned)n_sky);
    if (a.run) {
        if (a.binary)
            hipLaunchKernelGGL(rsf_resample_run_k<true>, grid, dim3(kThreads), 0, s, a);
        else
            hipLaunchKernelGGL(rsf_resample_run_k<false>, grid, dim3(kThreads), 0, s, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess || !a.binary) return e;
    }
    if (!a.binary) {
        hipLaunchKernelGGL((rsf_resample_k<false, kTileB>), grid, dim3(kThreads), 0, s, a);
        return hipGetLastError();
    }
    // a binary plan's sky rows choose their kernel on the device, by their orbit;
    // the half tiles' antenna sums are added into cleared ones
    const dim3 halves((unsigned)((a.LB + 63) / 64), grid.y, grid.z);
    if (!a.run) {
        const hipError_t e = launch_fill_u32((unsigned int*)a.partials, 6 * a.n_blocks * n_sky, 0u, s);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((rsf_resample_k<true, 64>), halves, dim3(256), 0, s, a);
    return hipGetLastError();
}

int resample_blocks(int LB, int64_t P) {
    return ((LB + kTileB - 1) / kTileB) * (int)((P + kTileA - 1) / kTileA);
}

hipError_t launch_antenna_reduce(const ReduceArgs& r, hipStream_t s) {
    hipLaunchKernelGGL(rsf_antenna_reduce_k, dim3((unsigned)r.n_sky), dim3(256), 0, s, r);
    return hipGetLastError();
}

}  // namespace rsf
