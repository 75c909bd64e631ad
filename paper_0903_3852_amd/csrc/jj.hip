// jj.hip -- ensemble integration of the driven, damped, noisy Brownian
// particle of Eq. 1 over many independent paths and parameter points,
// stochastic Heun (Alg. 2) or Euler-Maruyama.  Per point, either potential:
//   SDE_POTENTIAL_SIN     m phi'' + gamma phi' = -sin phi + a cos wt + f + noise
//                         (Josephson-junction form, phi in radians)
//   SDE_POTENTIAL_SIN2PI  m x'' + gamma x' = -2 pi cos(2 pi x) + a cos wt + f
//                         + noise: the paper's V(x) = sin(2 pi x), x in periods
// The state is the coordinate in units of its period (theta + winding), so
// the two differ only in the trigonometric function of the force and in
// per-point constants.
//
// Design (gfx950):
//  * One persistent launch.  Every wavefront pops work items (point, path
//    chunk of 64*PPT paths) from a device-scope counter until the queue is
//    empty; items are queued longest-first so uneven batches finish together.
//    Paths are independent (Sec. 4.1), so which wave runs an item does not
//    change any result.
//  * Per-path state stays in VGPRs for the whole item (Alg. 1 keeps x, v in
//    registers for m steps and touches global memory only at the ends); the
//    point's parameters are wave-uniform and live in SGPRs.
//  * The phase is kept in revolutions, theta in [0, 1), plus an integer
//    winding count, so the hardware v_sin_f32 (which takes revolutions) needs
//    no range reduction and FP32 never adds a tiny increment to a large phase
//    (the precision issue of Sec. 5).  The drive phase is the step index mod
//    S read from a cos table, the integer form of keeping time modulo the
//    drive period (Sec. 5).
//  * One Philox4x32-10 block per path gives the Gaussians of four
//    consecutive steps; Box-Muller uses the hardware log2/sqrt/sin/cos.
//  * The time average of v is summed in FP32 over M steps and folded into an
//    FP64 accumulator every M absolute steps (Sec. 4.1 samples every M).
//  * Per-chunk FP64 sums of vbar and vbar^2 are written without atomics and
//    combined per point in a fixed order by a second kernel, so results are
//    bitwise reproducible.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdlib>
#include <map>
#include <mutex>
#include <type_traits>

#include "device_common.h"
#include "sde_internal.h"

namespace sde {

// Per-point constants in the arithmetic type R of the integration (float:
// the FP32 path; double: the FP64 path).
template <typename R>
struct JJPointT {
    R dt, hdt, dtp, hdtp;          // dt, dt/2, dt/L, dt/(2L) with L the coordinate's period
                                   // (2 pi for phi, 1 for x): theta' = v / L
    R gim, kv, a_im, f_im;         // gamma/m, (force amplitude)/m, a/m, f/m with force
                                   // amplitude 1 (sin phi) or 2 pi (2 pi cos 2 pi x);
                                   // overdamped: 1/gamma for 1/m
    R c2, sig_v;                   // c2 = -2 ln2 sigma^2 with sigma the noise increment per
                                   // Gaussian: on v (inertial) or on theta in periods
                                   // (overdamped); sig_v = L / dt turns the latter into
                                   // a velocity
    uint32_t S, lut_off, n_paths, inertial;
    uint64_t path_first, n_steps, n_transient;
    double inv_W;
    uint32_t chunk_first, n_chunks;
};
using JJPointDev = JJPointT<float>;
static_assert(sizeof(JJPointT<float>) % 8 == 0 && sizeof(JJPointT<double>) % 8 == 0, "layout");

struct JJItem {
    uint32_t point, chunk;
};

struct JJArgs {
    const void* pts;      // JJPointT<R>[]
    const JJItem* items;
    const void* lut;      // R[]
    const void* tables;   // F64Tables (FP64 only)
    uint32_t* queue;
    int* flag;
    void* theta;          // R[]
    int32_t* winding;
    void* v;              // R[]
    double* acc;
    double* partials;
    int32_t* rec;         // optional windings every rec_every steps: [row][rec_pitch]
    uint64_t rec_pitch;   // paths of the call
    uint64_t step0;
    uint32_t key0, key1;
    uint32_t n_items, M;
    uint32_t rec_every;   // a multiple of 4 (records fall on block ends)
    int32_t init_from_state;
};

// One step n -> n + 1 of the PPT paths held by this lane.  e0, e1 are the
// uniform drive terms (a cos(w t) + f)/m at t_n and t_{n+1} (the second
// drift evaluation of Alg. 2 is taken at t + dt), ns the noise increments.
// The potential's shape at theta (in periods): sin(2 pi theta) for the
// -sin phi force, cos(2 pi theta) for -V'(x) = -2 pi cos(2 pi x).  FP32: the
// hardware v_sin/v_cos, which take revolutions; FP64: the table functions.

// ---- FP64 functions of the path integrator ----
// The arguments are special enough that table lookups beat general library
// functions: the uniforms are 24-bit fractions, phases are in revolutions.
// A workgroup keeps in LDS sin and cos of i/256 revolution (in two parts) and,
// for the logarithm of a mantissa near 1 + i/256, a 24-bit reciprocal v with
// -log2 v (in two parts, the first short enough to add an exponent exactly).
// The remainders are exact and small, so 3 polynomial terms (log: 6) reach
// FP64, and each result is rounded once: errors stay near half an ulp
// (sines and cosines keep it at their zeros, which are table points).
// Coefficients: Chebyshev fits, relative errors below 2.2e-17 of the small
// correction they give.  262144 paths x 400 Heun steps: 582 us with the
// library's sinpi, log2, sqrt and sincospi, 313 us with these.
struct F64Tables {
    double2 sc[256];     // sin, cos of 2 pi i / 256
    double2 sc_lo[256];  // what their rounding left
    struct Log {
        double hi;       // -log2 v (of 2 v from kLogFold on), a multiple of 2^-40
        float lo, v;     // its rest; v = 256 / (256 + i)
    } lg[257];
};
// Mantissas from 1 + kLogFold / 256 (about sqrt 2) on count to the next power
// of two, so that the logarithm of a uniform just below 1 has no cancellation.
constexpr uint32_t kLogFold = 106;

template <typename R>
struct JJTables {};  // FP32 has hardware functions
template <>
struct JJTables<double> : F64Tables {};
static_assert(sizeof(F64Tables) % 16 == 0, "copied in 16-byte pieces");

__device__ __forceinline__ void fill_tables(JJTables<float>&, const void*) {}
__device__ __forceinline__ void fill_tables(JJTables<double>& T, const void* src)
{
    for (uint32_t i = threadIdx.x; i < sizeof(F64Tables) / 16; i += blockDim.x)
        reinterpret_cast<double2*>(&T)[i] = static_cast<const double2*>(src)[i];
    __syncthreads();
}

// The tables, from long double functions.
static const F64Tables& host_tables()
{
    static const F64Tables tables = [] {
        F64Tables t{};
        const long double pi = 3.14159265358979323846264338327950288L;
        for (int i = 0; i < 256; ++i) {
            long double sn = std::sin(2 * pi * i / 256), cs = std::cos(2 * pi * i / 256);
            if (i % 64 == 0) {  // exact at the quarters
                sn = i == 64 ? 1 : i == 192 ? -1 : 0;
                cs = i == 0 ? 1 : i == 128 ? -1 : 0;
            }
            t.sc[i] = make_double2((double)sn, (double)cs);
            t.sc_lo[i] = make_double2((double)(sn - t.sc[i].x), (double)(cs - t.sc[i].y));
        }
        for (int i = 0; i <= 256; ++i) {
            const float v = (float)(256.0L / (256 + i));
            const long double l = -std::log2((long double)v * (i < (int)kLogFold ? 1 : 2));
            t.lg[i].v = v;
            t.lg[i].hi = (double)(std::nearbyint(l * 0x1p40L) * 0x1p-40L);
            t.lg[i].lo = (float)(l - t.lg[i].hi);
        }
        return t;
    }();
    return tables;
}

// sin and cos of 2 pi (entry i + r) revolutions, |r| <= 1/512 exact: the
// entry's pair rotated by the small angle.
template <bool SIN, bool COS>
__device__ __forceinline__ void rotate_entry(const F64Tables& T, uint32_t i, double r, double& sn, double& cs)
{
    const double2 e = T.sc[i];
    const double z = r * r;
    const double sd = fma(fma(0x1.466b53685f962p+6, z, -0x1.4abbce6246526p+5), z, 0x1.921fb54442d18p+2) * r;
    const double cm = fma(fma(-0x1.55d36d85e5ebfp+6, z, 0x1.03c1f081ad337p+6), z, -0x1.3bd3cc9be45dep+4) * z;
    if (SIN) sn = e.x + fma(e.x, cm, fma(e.y, sd, T.sc_lo[i].x));
    if (COS) cs = e.y + fma(e.y, cm, fma(-e.x, sd, T.sc_lo[i].y));
}

// The force's shape at theta.
template <bool COSF>
__device__ __forceinline__ float jj_shape(float theta, const JJTables<float>&)
{
    return COSF ? cos_rev(theta) : sin_rev(theta);
}
template <bool COSF>
__device__ __forceinline__ double jj_shape(double theta, const JJTables<double>& T)
{
#pragma clang fp contract(off)
    // whole revolutions out (exactly, whatever their number: a predictor of a
    // path that diverges may be anywhere), then 256 of the rest to the nearest
    // integer, in the low bits of t
    constexpr double kMagic = 0x1.8p52;
    const double f = theta - __builtin_rint(theta);
    const double t = fma(256.0, f, kMagic);
    const double r = fma(-0x1p-8, t - kMagic, f);
    double sn, cs;
    rotate_entry<!COSF, COSF>(T, (uint32_t)__double_as_longlong(t) & 255u, r, sn, cs);
    return COSF ? cs : sn;
}

__device__ __forceinline__ float fm(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fm(double a, double b, double c) { return fma(a, b, c); }

// sigma * (the four Gaussians of Philox block c), c2 = -2 ln2 sigma^2.  Each
// is rounded to R before a step adds it, whether or not the compiler sees
// both in one basic block (no contraction of the radius' product into the
// step's additions): a path's numbers do not depend on which loop runs it.
__device__ __forceinline__ void jj_gauss4(U4 c, uint32_t k0, uint32_t k1, float c2, const JJTables<float>&, float g[4])
{
#pragma clang fp contract(off)
    const U4 x = philox4x32_10(c, k0, k1);
    const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const float u1 = (float)((w[2 * p] >> 8) + 1u) * 0x1p-24f;
        const float u2 = (float)(w[2 * p + 1] >> 8) * 0x1p-24f;
        const float rho = __builtin_amdgcn_sqrtf(c2 * __builtin_amdgcn_logf(u1));
        g[2 * p] = rho * __builtin_amdgcn_cosf(u2);
        g[2 * p + 1] = rho * __builtin_amdgcn_sinf(u2);
    }
}
__device__ __forceinline__ void jj_gauss4(U4 c, uint32_t k0, uint32_t k1, double c2, const JJTables<double>& T,
                                          double g[4])
{
#pragma clang fp contract(off)
    const U4 x = philox4x32_10(c, k0, k1);
    const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        // u1 = k 2^-24, k = 2^E m exact in FP32; the mantissa m to the nearest
        // 1/256 selects v: log2 u1 = (E - 24) - log2 v + log2(m v)
        const uint32_t b = __float_as_uint((float)((w[2 * p] >> 8) + 1u));
        constexpr uint32_t kFold = 0x800000u - ((kLogFold << 15) - (1u << 14));
        const F64Tables::Log lg = T.lg[((b & 0x7fffffu) + 0x4000u) >> 15];
        const double r = fma((double)__uint_as_float((b & 0x7fffffu) | 0x3f800000u), (double)lg.v, -1.0);
        double q = fma(-0x1.ec71295a0d4acp-3, r, 0x1.277714d2a5458p-2);
        q = fma(q, r, -0x1.71547652b197bp-2);
        q = fma(q, r, 0x1.ec709dc398b67p-2);
        q = fma(q, r, -0x1.71547652b82fep-1);
        q = fma(q, r, 0x1.71547652b82fep+0);
        const double l = ((double)((int)((b + kFold) >> 23) - 151) + lg.hi) + fma(r, q, (double)lg.lo);
        // rho sigma = sqrt(c2 l): hardware estimate, one Goldschmidt step, one
        // correction (zero for u1 = 1 or no noise)
        const double x2 = c2 * l;
        const double y = __builtin_amdgcn_rsq(fmax(x2, 0x1p-1000));
        double rho = x2 * y, h = 0.5 * y;
        const double d = fma(-h, rho, 0.5);
        rho = fma(rho, d, rho);
        h = fma(h, d, h);
        rho = fma(fma(-rho, rho, x2), h, rho);
        // u2 to the nearest 1/256 revolution (the top byte, rounded) and the
        // signed rest of its 24 bits
        const uint32_t v = w[2 * p + 1];
        double sn, cs;
        rotate_entry<true, true>(T, (v + 0x800000u) >> 24, (double)((int32_t)(v << 8) >> 16) * 0x1p-24, sn, cs);
        g[2 * p] = rho * cs;
        g[2 * p + 1] = rho * sn;
    }
}

template <typename R, int PPT, int SCHEME, bool INERTIAL, bool COSF, bool ACC>
__device__ __forceinline__ void jj_step(const JJPointT<R>& P, const JJTables<R>& T, R e0, R e1,
                                        const R (&ns)[PPT], R (&th)[PPT], R (&vv)[PPT], R (&af)[PPT])
{
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        if (INERTIAL) {
            // X = (coordinate, v), F = (v, (force - gamma v + a cos wt + f)/m), noise on v
            const R F1 = fm(-P.kv, jj_shape<COSF>(th[k], T), fm(-P.gim, vv[k], e0));
            if (SCHEME == SDE_HEUN) {
                const R vt = fm(P.dt, F1, vv[k]) + ns[k];
                const R tt = fm(P.dtp, vv[k], th[k]);
                const R F2 = fm(-P.kv, jj_shape<COSF>(tt, T), fm(-P.gim, vt, e1));
                th[k] = fm(P.hdtp, vv[k] + vt, th[k]);
                vv[k] = fm(P.hdt, F1 + F2, vv[k]) + ns[k];
            } else {
                th[k] = fm(P.dtp, vv[k], th[k]);
                vv[k] = fm(P.dt, F1, vv[k]) + ns[k];
            }
        } else {
            // overdamped: coordinate' = (force + a cos wt + f)/gamma + noise on
            // the coordinate; v reports the step's mean velocity (change / dt)
            const R F1 = fm(-P.kv, jj_shape<COSF>(th[k], T), e0);
            if (SCHEME == SDE_HEUN) {
                const R tt = fm(P.dtp, F1, th[k]) + ns[k];
                const R F2 = fm(-P.kv, jj_shape<COSF>(tt, T), e1);
                th[k] = fm(P.hdtp, F1 + F2, th[k]) + ns[k];
                vv[k] = fm(R(0.5), F1 + F2, P.sig_v * ns[k]);
            } else {
                th[k] = fm(P.dtp, F1, th[k]) + ns[k];
                vv[k] = fm(P.sig_v, ns[k], F1);
            }
        }
        if (ACC) af[k] += vv[k];
    }
}

// Where an item's noise and drive come from: blocks in ascending order, each
// taken once, avail() of them (at least one after ensure()) without another
// ensure().  take() gives the four Gaussians of block b of each path and, for
// a whole block that begins at drive phase kk, the drive terms e of its steps.
//
// Drawn by the wave itself, right where it is used.  The drive terms of a
// point come from a table in LDS that the wave fills once per item (TAB), or
// are formed from the cos table at every block.  The table leaves the loop
// without scalar loads to wait for and without the 5 multiply-adds and 5
// moves that wave-uniform FP32 arithmetic takes on the vector unit (1500
// points x 1000 paths x 2000 steps at 1, 2, 4 paths per lane: 3402, 3143,
// 2928 -> 3148, 2949, 2846 us, and 2829, 2716, 2728 with the present block
// loop; FP64: no change, so its kernels go without).
constexpr uint32_t kDriveTable = 1024;  // entries per wave: periods of up to kDriveTable - 8 steps

template <typename R, int PPT, bool TAB>
struct OwnNoise {
    uint32_t key0, key1, q;
    const uint32_t (&pid)[PPT];
    const JJTables<R>& T;
    R c2, a_im, f_im;
    const R* lut;  // cos(2 pi k / S), or with TAB the drive terms
    static constexpr uint32_t kUnroll = 1;

    __device__ __forceinline__ void ensure() {}
    __device__ __forceinline__ uint32_t avail() const { return 1u << 28; }
    template <int N>
    __device__ __forceinline__ void take(uint32_t b, uint32_t kk, R (&g)[N][PPT][4], R (&e)[N][5])
    {
        static_assert(N == 1, "one block at a time");
#pragma unroll
        for (int k = 0; k < PPT; ++k) 
            jj_gauss4(U4{b, pid[k], q, (uint32_t)SDE_TAG_NOISE}, key0, key1, c2, T, g[0][k]);
#pragma unroll
        for (int j = 0; j < 5; ++j) e[0][j] = TAB ? lut[kk + j] : fm(a_im, load_uniform(lut + kk + j), f_im);
    }
};

// Drawn ahead by other waves of the workgroup into a double-buffered LDS ring
// (kBlocks blocks per buffer, one barrier per buffer): see jj_split_kernel.
template <typename R>
struct JJRing {
    static constexpr uint32_t kBlocks = 64 / sizeof(R);  // 16 KB per buffer
    R g[2 * kBlocks][kWave][4];
    R e[2 * kBlocks][8];  // the drive terms, the same for every lane
};

template <typename R, bool INERTIAL>
struct RingNoise {
    // Blocks taken per loop iteration: a wave alone on its SIMD issues an
    // instruction every ~6 cycles whatever it is, so the loop's scalar work
    // and register copies count like the steps.  Two in FP64 with inertia: the
    // values of four leave no registers to start a force before the one ahead
    // of it is done (1000 paths x 3000 steps, Heun 497 -> 389 us, Euler-Maruyama
    // 275 -> 223).  Without inertia a force waits for the one ahead of it anyway
    // (446 : 451 and 259 : 262 with four : two).
    static constexpr uint32_t kUnroll = sizeof(R) == 8 && INERTIAL ? 2 : 4;
    static constexpr uint32_t kBlocks = JJRing<R>::kBlocks;
    const JJRing<R>& ring;
    uint32_t left = 0, at = 0;  // blocks left in the current buffer; its next slot

    __device__ __forceinline__ void ensure()
    {
        if (left) return;
        __syncthreads();  // the other buffer is full, and its writers go on to the one just used up
        at = at == 2 * kBlocks ? 0u : at;
        left = kBlocks;
    }
    __device__ __forceinline__ uint32_t avail() const { return left; }
    template <int N>
    __device__ __forceinline__ void take(uint32_t, uint32_t, R (&g)[N][1][4], R (&e)[N][5])
    {
#pragma unroll
        for (int i = 0; i < N; ++i) {
#pragma unroll
            for (int j = 0; j < 4; ++j) e[i][j] = ring.e[at + i][j];
#pragma unroll
            for (int j = 0; j < 4; ++j) g[i][0][j] = ring.g[at + i][threadIdx.x & (kWave - 1)][j];
        }
#pragma unroll
        for (int i = 0; i < N; ++i) e[i][4] = i + 1 < N ? e[i + 1][0] : ring.e[at + i][4];
        left -= N;
        at += N;
    }
};

template <typename R, int PPT, int SCHEME, bool INERTIAL, bool COSF, typename Noise>
__device__ __forceinline__ void jj_item(const JJArgs& A, const JJPointT<R>& P, const JJTables<R>& T, uint32_t q,
                                        uint32_t chunk, const uint32_t (&pid)[PPT], Noise& src)
{
    const uint32_t lane = threadIdx.x & (kWave - 1);
    R* theta = static_cast<R*>(A.theta);
    R* vel = static_cast<R*>(A.v);

    R th[PPT], vv[PPT], af[PPT];
    int32_t wd[PPT];
    double ad[PPT];
    bool live[PPT];
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        live[k] = pid[k] < P.n_paths;
        const uint64_t gi = P.path_first + pid[k];
        if (A.init_from_state) {
            th[k] = live[k] ? theta[gi] : R(0);
            vv[k] = live[k] ? vel[gi] : R(0);
            wd[k] = live[k] ? A.winding[gi] : 0;
            ad[k] = live[k] ? A.acc[gi] : 0.0;
        } else {
            const U4 x = philox4x32_10(U4{0u, pid[k], q, (uint32_t)SDE_TAG_INIT}, A.key0, A.key1);
            th[k] = (R)(x.x >> 8) * R(0x1p-24);
            vv[k] = R(-2) + R(4) * ((R)(x.y >> 8) * R(0x1p-24));
            wd[k] = 0;
            ad[k] = 0.0;
        }
        af[k] = R(0);
    }

    const R* lut = static_cast<const R*>(A.lut) + P.lut_off;  // cos(2 pi k / S) for k < S + 8
    const uint64_t n_end = A.step0 + P.n_steps;
    uint64_t n = A.step0;
    uint32_t kk = (uint32_t)(n % P.S);               // drive phase index of step n
    const uint32_t kk4 = P.S < 4 ? 4 % P.S : 4u;     // what a block moves it by
    // steps until the next multiple of M, kept from the window's start on (no
    // sum is open before it, so folds there would add nothing)
    uint32_t to_fold = 0;
    bool opened = false;
    auto open_window = [&]() {
        if (opened) return;
        opened = true;
        to_fold = A.M - (uint32_t)(n % A.M);
    };
    // recording: rc = n mod rec_every; row r holds the state after the
    // (r + 1)-th multiple of rec_every past step0
    const bool recording = sizeof(R) == 4 && A.rec;  // FP32 only
    uint32_t rc = recording ? (uint32_t)(n % A.rec_every) : 0u;
    uint64_t row = 0;

    auto fold = [&]() {
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            ad[k] += (double)af[k];
            af[k] = R(0);
        }
        to_fold = A.M;
    };
    // keep theta in [0, 1): move whole revolutions into the winding count
    auto wrap = [&]() {
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            const R fl = floor(th[k]);
            th[k] -= fl;
            wd[k] += (int32_t)fl;
        }
    };
    auto record = [&]() {
        rc = 0;
        int32_t* out = A.rec + row * A.rec_pitch + P.path_first;
#pragma unroll
        for (int k = 0; k < PPT; ++k)
            if (live[k]) out[pid[k]] = wd[k];
        ++row;
    };
    // `count` whole 4-step blocks, U at a time, outside the window, in it, or
    // (kTick) in it with folds wherever they fall.  A tick has no branch; it is
    // for the launch whose step chain has the SIMD to itself (in the other one
    // it would pay by the instruction).
    enum { kPlain, kWindow, kTick };
    auto run_some = [&](auto mode, auto unroll, uint32_t iterations, uint32_t blk) {
        constexpr int kMode = decltype(mode)::value;
        constexpr uint32_t U = decltype(unroll)::value;
        for (uint32_t i = 0; i < iterations; ++i, blk += U) {
            R g[U][PPT][4], e[U][5];
            src.take(blk, kk, g, e);
            if constexpr (Noise::kUnroll == 1) {
                kk += kk4;
                kk -= kk >= P.S ? P.S : 0u;
            }
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    R ns[PPT];
#pragma unroll
                    for (int k = 0; k < PPT; ++k) ns[k] = g[u][k][j];
                    jj_step<R, PPT, SCHEME, INERTIAL, COSF, kMode != kPlain>(P, T, e[u][j], e[u][j + 1], ns, th, vv, af);
                    if constexpr (kMode == kTick) {
                        const bool due = --to_fold == 0;
                        to_fold = due ? A.M : to_fold;
#pragma unroll
                        for (int k = 0; k < PPT; ++k) {
                            ad[k] += (double)(due ? af[k] : R(0));
                            af[k] = due ? R(0) : af[k];
                        }
                    }
                }
                wrap();
            }
        }
    };
    auto run_blocks = [&](auto mode, uint32_t count, uint32_t blk) {
        constexpr uint32_t U = Noise::kUnroll;
        run_some(mode, std::integral_constant<uint32_t, U>{}, count / U, blk);
        if constexpr (U > 1) run_some(mode, std::integral_constant<uint32_t, 1>{}, count % U, blk + count / U * U);
    };

    while (n < n_end) {
        const uint32_t j0 = (uint32_t)n & 3u;
        const uint64_t left = n_end - n;
        if (j0 == 0 && left >= 4) {
            // The whole blocks up to the next event: the end of the call, the
            // start of the window, the block that a fold falls into (or ends
            // at).  Their loop is one basic block: the compiler overlaps the
            // noise, the four steps and the drive's loads, which branches for
            // the window and the fold between the steps had kept apart (one
            // point of 4096 paths, one wave per SIMD: 1335 -> 885 us for 10^4
            // steps; 4096 x 1024 paths x 5000 steps, ALU-bound: 18.4 -> 17.7 ms;
            // a ragged batch 4.41 -> 3.72 ms).
            constexpr bool kTicks = Noise::kUnroll > 1;
            const bool window = n >= P.n_transient;
            uint64_t blocks = left >> 2;
            bool tick = false;
            if (window) {
                open_window();
                // folds in every other block or more are no events: a loop of
                // one or two blocks costs more than the ticks (1000 paths, 2000
                // steps, sample_every 1: 409 us with events, 120 so)
                tick = kTicks && (A.M < 8 || to_fold < 4);
                if (!kTicks || A.M >= 8) blocks = min(blocks, (uint64_t)max(to_fold >> 2, tick ? 1u : 0u));
            } else
                blocks = min(blocks, (P.n_transient - n) >> 2);
            const uint32_t count = (uint32_t)min(blocks, (uint64_t)1 << 28);
            if (count) {
                // as the noise and the records come
                uint32_t todo = count, blk = (uint32_t)(n >> 2);
                do {
                    src.ensure();
                    uint32_t some = min(todo, src.avail());
                    if (recording) some = min(some, (A.rec_every - rc) >> 2);
                    if (kTicks && tick)
                        run_blocks(std::integral_constant<int, kTicks ? kTick : kPlain>{}, some, blk);
                    else if (window)
                        run_blocks(std::integral_constant<int, kWindow>{}, some, blk);
                    else
                        run_blocks(std::integral_constant<int, kPlain>{}, some, blk);
                    blk += some;
                    if (recording) {
                        rc += 4 * some;
                        if (rc == A.rec_every) record();
                    }
                    todo -= some;
                } while ((kTicks || sizeof(R) == 4) && todo);  // FP64 drawing its own: at once
                n += 4 * (uint64_t)count;
                if (kTicks) {  // the ring holds the drive: its phase only matters to steps taken one by one
                    kk += 4 * count;
                    if (kk >= P.S) kk %= P.S;
                }
                if (window && !tick) {
                    to_fold -= 4 * count;
                    if (to_fold == 0) fold();
                }
                continue;
            }
        }
        src.ensure();
        const uint32_t jn = left >= (uint64_t)(4u - j0) ? 4u : j0 + (uint32_t)left;
        R g[1][PPT][4], e[1][5];
        src.take((uint32_t)(n >> 2), kk, g, e);
        auto step = [&](R ea, R eb, const R (&ns)[PPT]) {
            if (n >= P.n_transient) {
                open_window();
                jj_step<R, PPT, SCHEME, INERTIAL, COSF, true>(P, T, ea, eb, ns, th, vv, af);
                if (--to_fold == 0) fold();
            } else {
                jj_step<R, PPT, SCHEME, INERTIAL, COSF, false>(P, T, ea, eb, ns, th, vv, af);
            }
            ++n;
        };
        if (j0 == 0 && jn == 4) {
            // a whole block that the window begins in, or with a fold between
            // its steps; its drive terms come with the noise
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                R ns[PPT];
#pragma unroll
                for (int k = 0; k < PPT; ++k) ns[k] = g[0][k][j];
                step(e[0][j], e[0][j + 1], ns);
            }
            kk += kk4;
            kk -= kk >= P.S ? P.S : 0u;
        } else {  // a first or last partial block of the call
            for (uint32_t j = j0; j < jn; ++j) {
                R ns[PPT];
#pragma unroll
                for (int k = 0; k < PPT; ++k)
                    ns[k] = j == 0 ? g[0][k][0] : j == 1 ? g[0][k][1] : j == 2 ? g[0][k][2] : g[0][k][3];
                step(fm(P.a_im, load_uniform(lut + kk), P.f_im), fm(P.a_im, load_uniform(lut + kk + 1), P.f_im), ns);
                kk = (kk + 1 == P.S) ? 0u : kk + 1;
            }
        }
        wrap();
        // a block never crosses a multiple of 4, hence of rec_every
        if (recording) {
            rc += jn - j0;
            if (rc == A.rec_every) record();
        }
    }

    double s1 = 0.0, s2 = 0.0;
    bool bad = false;
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        ad[k] += (double)af[k];
        if (live[k]) {
            const uint64_t gi = P.path_first + pid[k];
            if (theta) theta[gi] = th[k];
            if (A.winding) A.winding[gi] = wd[k];
            if (vel) vel[gi] = vv[k];
            if (A.acc) A.acc[gi] = ad[k];
            const double vb = ad[k] * P.inv_W;
            s1 += vb;
            s2 += vb * vb;
            bad |= !(isfinite(th[k]) && isfinite(vv[k]));
        }
    }
    s1 = wave_sum(s1);
    s2 = wave_sum(s2);
    if (lane == 0) {
        A.partials[2 * (P.chunk_first + chunk)] = s1;
        A.partials[2 * (P.chunk_first + chunk) + 1] = s2;
    }
    if (__ballot(bad) != 0 && lane == 0) atomicOr(A.flag, 1);
}

// Most waves per SIMD that the compiler is to leave registers for.  FP64 steps
// are chains of table lookups; two or three waves whose lookups are ahead of
// their use do better than five that wait for each one, which is what the
// compiler makes by itself or not, as the code around the loop happens to
// be.  2^18 paths x 400 steps at 2 paths per lane, as it came out : 2 waves : 3,
// us: Heun 313 : 309 : 344, overdamped 340 : 301 : 301, Euler-Maruyama 260 :
// 236 : 235; at 1 path per lane 341 : 314 : 320, 331 : 367 : 315, 261 : 287 : 250.
template <typename R, int PPT>
constexpr int kMostWaves = sizeof(R) == 4 ? 8 : PPT == 2 ? 2 : 3;

template <typename R, int PPT, int SCHEME, bool INERTIAL, bool COSF, bool TAB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, kMostWaves<R, PPT>))) void
jj_persistent_kernel(JJArgs A)
{
    __shared__ __attribute__((aligned(16))) R drive[4][TAB ? kDriveTable : 1];
    R* mine = drive[threadIdx.x / kWave];  // this wave's own: no barrier
    __shared__ JJTables<R> T;
    fill_tables(T, A.tables);
    const uint32_t lane = threadIdx.x & (kWave - 1);
    for (;;) {
        uint32_t item = 0;
        if (lane == 0) item = atomicAdd(A.queue, 1u);
        item = uniform_u32(__shfl(item, 0, kWave));
        if (item >= A.n_items) break;
        const JJItem it = load_uniform(A.items + item);
        const JJPointT<R> P = load_uniform(static_cast<const JJPointT<R>*>(A.pts) + it.point);
        uint32_t pid[PPT];
#pragma unroll
        for (int k = 0; k < PPT; ++k) pid[k] = it.chunk * (kWave * PPT) + k * kWave + lane;
        const R* lut = static_cast<const R*>(A.lut) + P.lut_off;
        if constexpr (TAB) {
            for (uint32_t t = lane; t < P.S + 8; t += kWave) mine[t] = fm(P.a_im, lut[t], P.f_im);
            // the wave's own LDS writes are complete before its reads
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        OwnNoise<R, PPT, TAB> src{A.key0, A.key1, it.point, pid, T, P.c2, P.a_im, P.f_im, TAB ? mine : lut};
        jj_item<R, PPT, SCHEME, INERTIAL, COSF>(A, P, T, it.point, it.chunk, pid, src);
    }
}

// The same integration for calls with too few paths to fill the chip, where
// a wave is alone on its SIMD and waits out the latency of every dependent
// instruction.  The noise does not depend on the path, so it leaves the
// chain: one workgroup per item of 64 paths, wave 0 runs the steps, the other
// waves (on SIMDs that would idle) draw the Gaussians of the blocks ahead
// into LDS.  With kB the blocks of a ring buffer, block b of the call goes
// through slot b mod 2 kB; the waves meet at one barrier per buffer: past
// barrier c, buffer c mod 2 is full and its predecessor used up.  Every wave
// of a workgroup passes exactly ceil(blocks / kB) barriers.
constexpr int kSplitDrawers = 3;
constexpr int kSplitThreads = (1 + kSplitDrawers) * kWave;

template <typename R, int SCHEME, bool INERTIAL, bool COSF>
__global__ __launch_bounds__(kSplitThreads) void jj_split_kernel(JJArgs A)
{
    __shared__ __attribute__((aligned(16))) JJRing<R> ring;
    __shared__ JJTables<R> T;
    fill_tables(T, A.tables);
    constexpr uint32_t kB = JJRing<R>::kBlocks;
    const JJItem it = load_uniform(A.items + blockIdx.x);
    const JJPointT<R> P = load_uniform(static_cast<const JJPointT<R>*>(A.pts) + it.point);
    const uint32_t lane = threadIdx.x & (kWave - 1), wave = uniform_u32(threadIdx.x / kWave);
    const uint32_t pid[1] = {it.chunk * kWave + lane};
    if (wave == 0) {
        RingNoise<R, INERTIAL> src{ring};
        jj_item<R, 1, SCHEME, INERTIAL, COSF>(A, P, T, it.point, it.chunk, pid, src);
        return;
    }
    if (P.n_steps == 0) return;
    const uint64_t b0 = A.step0 >> 2, blocks = ((A.step0 + P.n_steps - 1) >> 2) - b0 + 1;
    const R* lut = static_cast<const R*>(A.lut) + P.lut_off;
    uint32_t phase = (uint32_t)((4 * b0) % P.S);  // drive phase of the buffer's first block
    for (uint64_t c = 0; c < blocks; c += kB) {
        const uint32_t cnt = (uint32_t)min(blocks - c, (uint64_t)kB);
        const uint32_t base = (c / kB) & 1u ? kB : 0u;
        for (uint32_t i = wave - 1; i < cnt; i += kSplitDrawers) {
            R g[4];
            jj_gauss4(U4{(uint32_t)(b0 + c) + i, pid[0], it.point, (uint32_t)SDE_TAG_NOISE}, A.key0, A.key1, P.c2, T, g);
#pragma unroll
            for (int j = 0; j < 4; ++j) ring.g[base + i][lane][j] = g[j];
            if (lane < 5) ring.e[base + i][lane] = fm(P.a_im, lut[(phase + 4 * i) % P.S + lane], P.f_im);
        }
        phase = (phase + 4 * kB) % P.S;
        __syncthreads();
    }
}

// Stage 2: per point, its chunk partials -- one wavefront a point, lane l
// adding chunks l, l + 64, ..., then the fixed butterfly.  (One thread a point
// walked its chunks one load latency at a time: 195 us for the 2048 chunks of
// a single point of 2^18 paths, a quarter of that call; 17 us for a ragged
// batch.)
constexpr uint32_t kPointSumWaves = 4;  // points per workgroup

template <typename R>
__global__ __launch_bounds__(kPointSumWaves* kWave) void jj_point_sums_kernel(const JJPointT<R>* pts, uint32_t n_pts,
                                                                              const double* partials, double* out)
{
    const uint32_t q = blockIdx.x * kPointSumWaves + threadIdx.x / kWave;
    if (q >= n_pts) return;
    const uint32_t first = pts[q].chunk_first, nc = pts[q].n_chunks, lane = threadIdx.x & (kWave - 1);
    const double2* p = reinterpret_cast<const double2*>(partials) + first;
    double s1 = 0.0, s2 = 0.0;
#pragma unroll 4
    for (uint32_t c = lane; c < nc; c += kWave) {
        const double2 x = p[c];
        s1 += x.x;
        s2 += x.y;
    }
    s1 = wave_sum(s1);
    s2 = wave_sum(s2);
    if (lane == 0) {
        out[2 * (uint64_t)q] = s1;
        out[2 * (uint64_t)q + 1] = s2;
    }
}

// Test hooks: raw Philox words and the integrators' Gaussians.
__global__ void philox_dump_kernel(uint32_t k0, uint32_t k1, uint32_t tag, uint32_t a, uint32_t b,
                                   uint64_t c0, uint64_t n, uint32_t* out)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const U4 x = philox4x32_10(U4{(uint32_t)(c0 + i), a, b, tag}, k0, k1);
    out[4 * i] = x.x;
    out[4 * i + 1] = x.y;
    out[4 * i + 2] = x.z;
    out[4 * i + 3] = x.w;
}

__global__ void gauss_dump_kernel(uint32_t k0, uint32_t k1, uint32_t tag, uint32_t a, uint32_t b,
                                  uint64_t n0, uint64_t n, float* out)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint64_t s = n0 + i;
    float g[4];
    gauss4(U4{(uint32_t)(s >> 2), a, b, tag}, k0, k1, g);
    const uint32_t j = (uint32_t)s & 3u;
    out[i] = j == 0 ? g[0] : j == 1 ? g[1] : j == 2 ? g[2] : g[3];
}

// ------------------------------------------------------------------ host --

using JJKernel = void (*)(JJArgs);

// Paths per lane: 1, 2 or 4 in FP32; FP64 holds twice the registers per
// path and stops at 2.
template <typename R, bool INERTIAL, bool COSF, bool TAB>
static JJKernel pick_kernel_t(int ppt, int scheme)
{
    constexpr bool f32 = sizeof(R) == 4;
    if (scheme == SDE_HEUN) {
        if (ppt == 1) return jj_persistent_kernel<R, 1, SDE_HEUN, INERTIAL, COSF, TAB>;
        if (f32 && ppt == 4) return jj_persistent_kernel<R, f32 ? 4 : 2, SDE_HEUN, INERTIAL, COSF, TAB>;
        return jj_persistent_kernel<R, 2, SDE_HEUN, INERTIAL, COSF, TAB>;
    }
    if (ppt == 1) return jj_persistent_kernel<R, 1, SDE_EULER, INERTIAL, COSF, TAB>;
    if (f32 && ppt == 4) return jj_persistent_kernel<R, f32 ? 4 : 2, SDE_EULER, INERTIAL, COSF, TAB>;
    return jj_persistent_kernel<R, 2, SDE_EULER, INERTIAL, COSF, TAB>;
}

template <typename R>
static JJKernel pick_split(int kind, int scheme)
{
    const bool heun = scheme == SDE_HEUN;
    switch (kind) {
    case 0: return heun ? jj_split_kernel<R, SDE_HEUN, true, false> : jj_split_kernel<R, SDE_EULER, true, false>;
    case 1: return heun ? jj_split_kernel<R, SDE_HEUN, false, false> : jj_split_kernel<R, SDE_EULER, false, false>;
    case 2: return heun ? jj_split_kernel<R, SDE_HEUN, true, true> : jj_split_kernel<R, SDE_EULER, true, true>;
    default: return heun ? jj_split_kernel<R, SDE_HEUN, false, true> : jj_split_kernel<R, SDE_EULER, false, true>;
    }
}

// Point kinds, one persistent launch each: bit 0 = overdamped, bit 1 = the
// sin(2 pi x) potential.
constexpr int kJJKinds = 4;

template <typename R, bool TAB>
static JJKernel pick_kind(int kind, int ppt, int scheme)
{
    switch (kind) {
    case 0: return pick_kernel_t<R, true, false, TAB>(ppt, scheme);
    case 1: return pick_kernel_t<R, false, false, TAB>(ppt, scheme);
    case 2: return pick_kernel_t<R, true, true, TAB>(ppt, scheme);
    default: return pick_kernel_t<R, false, true, TAB>(ppt, scheme);
    }
}

// `tab`: every point's drive fits the table in LDS (FP32 only).
template <typename R>
static JJKernel pick_kernel(int kind, int ppt, int scheme, bool tab)
{
    if constexpr (sizeof(R) == 4)
        if (tab) return pick_kind<R, true>(kind, ppt, scheme);
    return pick_kind<R, false>(kind, ppt, scheme);
}

static bool finite_point(const sde_jj_point& p)
{
    return std::isfinite(p.m) && std::isfinite(p.gamma) && std::isfinite(p.a) && std::isfinite(p.omega) &&
           std::isfinite(p.f) && std::isfinite(p.D);
}

// Work items of one paths-per-lane choice: chunk layout per point and the
// queue of each point kind (longest first within a kind).
template <typename R>
struct JJPlan {
    std::vector<JJPointT<R>> pts;
    std::vector<JJItem> items;
    uint32_t kind_begin[kJJKinds + 1] = {};  // items of kind k: [kind_begin[k], kind_begin[k + 1])
    uint32_t n_chunks = 0;
};

template <typename R>
static void plan_items(std::vector<JJPointT<R>>& P, const std::vector<int>& kinds, int ppt, JJPlan<R>& out)
{
    const uint32_t chunk_paths = (uint32_t)(kWave * ppt);
    std::vector<JJItem> it[kJJKinds];
    uint32_t chunk_first = 0;
    for (uint32_t q = 0; q < (uint32_t)P.size(); ++q) {
        JJPointT<R>& d = P[q];
        d.n_chunks = (d.n_paths + chunk_paths - 1) / chunk_paths;
        d.chunk_first = chunk_first;
        for (uint32_t c = 0; c < d.n_chunks; ++c) it[kinds[q]].push_back(JJItem{q, c});
        chunk_first += d.n_chunks;
    }
    auto longest_first = [&](const JJItem& x, const JJItem& y) { return P[x.point].n_steps > P[y.point].n_steps; };
    out.pts = P;
    out.items.clear();
    for (int k = 0; k < kJJKinds; ++k) {
        std::stable_sort(it[k].begin(), it[k].end(), longest_first);
        out.kind_begin[k] = (uint32_t)out.items.size();
        out.items.insert(out.items.end(), it[k].begin(), it[k].end());
    }
    out.kind_begin[kJJKinds] = (uint32_t)out.items.size();
    out.n_chunks = chunk_first;
}

// How the items run: 1, 2 or 4 paths per lane of the persistent kernel, or
// kSplitChoice for jj_split_kernel (1 path per lane).  These are the values
// the tune cache holds.
constexpr int kSplitChoice = 17;

// Most items (of 64 paths) per CU the split kernel is tried for, FP32 and
// FP64.  With more, every SIMD has waves enough to switch between, and the
// waves that draw ahead only take issue slots.  One point, best persistent
// against split, us: 10^4 FP32 steps of 4096 paths 802 : 439, 32768 (2 per
// CU) 808 : 569, 65536 (4) 823 : 824, 98304 (6) 1336 : 1143; 2000 FP64 steps of
// 4096 paths 445 : 269, 32768 (2) 451 : 320, 49152 (3) 455 : 370.  Past the
// lines, of earlier versions of both: 131072 FP32 paths (8) 1329 : 1566, 65536
// FP64 paths (4) 643 : 755.
constexpr uint32_t kSplitItemsPerCU32 = 6, kSplitItemsPerCU64 = 3;

struct JJLaunch {
    JJArgs A;
    uint32_t* queues;  // kJJKinds work-queue words, zeroed by each launch sequence
    int ppt;
    bool split;  // jj_split_kernel (ppt = 1)
    bool tab;    // the persistent kernel's drive terms from LDS
    int scheme;
    uint32_t kind_begin[kJJKinds + 1];
    uint32_t n_items, n_pts;
    uint32_t grid[kJJKinds];
    double* point_sums;
};

template <typename R>
static int jj_grids(sde_ctx* ctx, JJLaunch& L)
{
    for (int kind = 0; kind < kJJKinds; ++kind) {
        const uint32_t count = L.kind_begin[kind + 1] - L.kind_begin[kind];
        L.grid[kind] = 0;
        if (!count) continue;
        if (L.split) {  // one workgroup per item
            L.grid[kind] = count;
            continue;
        }
        JJKernel kern = pick_kernel<R>(kind, L.ppt, L.scheme, L.tab);
        int per_cu = 0;
        SDE_HIP(ctx, hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(kern), 256, 0));
        if (per_cu < 1) per_cu = 1;
        const uint64_t want = ((uint64_t)count + 3) / 4;  // 4 waves per block, one item each at least
        L.grid[kind] = (uint32_t)std::min<uint64_t>(want, (uint64_t)per_cu * ctx->n_cu);
    }
    return SDE_OK;
}

__global__ void jj_zero_queues_kernel(uint32_t* q)
{
    if (threadIdx.x < (uint32_t)kJJKinds) q[threadIdx.x] = 0u;
}

// The launch sequence of one call: reset the queues, the persistent kernel
// of each point kind present, the per-point sums.
template <typename R>
static int jj_record(sde_ctx* ctx, const JJLaunch& L, hipStream_t s)
{
    hipLaunchKernelGGL(jj_zero_queues_kernel, dim3(1), dim3(64), 0, s, L.queues);
    SDE_HIP(ctx, hipGetLastError());
    const JJItem* all = L.A.items;
    for (int kind = 0; kind < kJJKinds; ++kind) {
        if (!L.grid[kind]) continue;
        JJArgs A = L.A;
        A.items = all + L.kind_begin[kind];
        A.n_items = L.kind_begin[kind + 1] - L.kind_begin[kind];
        A.queue = L.queues + kind;
        JJKernel kern = L.split ? pick_split<R>(kind, L.scheme) : pick_kernel<R>(kind, L.ppt, L.scheme, L.tab);
        hipLaunchKernelGGL(kern, dim3(L.grid[kind]), dim3(L.split ? kSplitThreads : 256), 0, s, A);
        SDE_HIP(ctx, hipGetLastError());
    }
    if (L.point_sums) {
        hipLaunchKernelGGL(jj_point_sums_kernel<R>, dim3((L.n_pts + kPointSumWaves - 1) / kPointSumWaves),
                           dim3(kPointSumWaves * kWave), 0, s, static_cast<const JJPointT<R>*>(L.A.pts), L.n_pts,
                           static_cast<const double*>(L.A.partials), L.point_sums);
        SDE_HIP(ctx, hipGetLastError());
    }
    return SDE_OK;
}

// The graph cache key of one call: every value the recorded launches bake
// in -- each field of the kernel arguments (the per-kind item range and queue
// word are derived from kind_begin and the queue words), the kernel choice,
// the grids and the point-sum launch.  A field left out would let a later call replay a graph recorded
// with a stale value.
static std::string jj_graph_key(const char* prec, const JJLaunch& L)
{
    const JJArgs& A = L.A;
    char buf[640];
    snprintf(buf, sizeof buf,
             "jj|%s|pts%p|it%p|lut%p|tab%p|q%p|fl%p|th%p|wd%p|v%p|acc%p|pa%p|rec%p/%llu/%u|n0%llu|k%u.%u|ni%u|M%u|ini%d|"
             "ppt%d/%d/%d|sch%d|np%u|ps%p",
             prec, A.pts, (const void*)A.items, A.lut, A.tables, (void*)L.queues, (void*)A.flag, A.theta, (void*)A.winding, A.v,
             (void*)A.acc, (void*)A.partials, (void*)A.rec, (unsigned long long)A.rec_pitch, A.rec_every,
             (unsigned long long)A.step0, A.key0, A.key1, L.n_items, A.M, A.init_from_state, L.ppt, (int)L.split, (int)L.tab, L.scheme,
             L.n_pts, (void*)L.point_sums);
    std::string k = buf;
    for (int kind = 0; kind < kJJKinds; ++kind)
        k += "|" + std::to_string(L.kind_begin[kind + 1]) + "/" + std::to_string(L.grid[kind]);
    return k;
}

template <typename R>
static int jj_upload_plan(sde_ctx* ctx, const JJPlan<R>& plan, hipStream_t stream, JJLaunch& L)
{
    int st;
    if ((st = upload(ctx, kSlotJJPoints, 0, plan.pts.data(), plan.pts.size() * sizeof(JJPointT<R>), stream)))
        return st;
    if ((st = upload(ctx, kSlotJJItems, 1, plan.items.data(), plan.items.size() * sizeof(JJItem), stream))) return st;
    void* partials = nullptr;
    if ((st = ensure_ws(ctx, kSlotJJPartials, (size_t)std::max(plan.n_chunks, 1u) * 2 * sizeof(double), &partials)))
        return st;
    if ((st = ensure_counters(ctx, kJJKinds))) return st;
    L.queues = ctx->counters;
    L.A.pts = ctx->ws[kSlotJJPoints].ptr;
    L.A.items = static_cast<const JJItem*>(ctx->ws[kSlotJJItems].ptr);
    L.A.partials = static_cast<double*>(partials);
    std::copy(plan.kind_begin, plan.kind_begin + kJJKinds + 1, L.kind_begin);
    L.n_items = (uint32_t)plan.items.size();
    L.n_pts = (uint32_t)plan.pts.size();
    return jj_grids<R>(ctx, L);
}

static int ilog2u64(uint64_t x)
{
    int r = 0;
    while (x > 1) {
        x >>= 1;
        ++r;
    }
    return r;
}

static void set_choice(JJLaunch& L, int choice)
{
    L.split = choice == kSplitChoice;
    L.ppt = L.split ? 1 : choice;
}

// Whether a call is small enough for the split kernel.
template <typename R>
static bool split_fits(const sde_ctx* ctx, const std::vector<JJPointT<R>>& P)
{
    uint64_t items = 0;
    for (const auto& d : P) items += (d.n_paths + kWave - 1) / kWave;
    return items <= (uint64_t)(sizeof(R) == 4 ? kSplitItemsPerCU32 : kSplitItemsPerCU64) * ctx->n_cu;
}

// Times the candidate choices on a short slice of the call
// (same points, at most 2048 steps, no per-path outputs) and returns the
// fastest.  Nothing the caller passed is written.
template <typename R>
static int jj_tune(sde_ctx* ctx, const std::vector<JJPointT<R>>& P0, const std::vector<int>& kinds,
                   const JJLaunch& base, hipStream_t stream, int* best_choice)
{
    std::vector<JJPointT<R>> P = P0;
    uint64_t work = 0;
    for (auto& d : P) {
        d.n_steps = std::min<uint64_t>(d.n_steps, 2048);
        work += (uint64_t)d.n_paths * d.n_steps;
    }
    if (work == 0) {
        *best_choice = 2;
        return SDE_OK;
    }
    hipEvent_t e0, e1;
    SDE_HIP(ctx, hipEventCreate(&e0));
    SDE_HIP(ctx, hipEventCreate(&e1));
    double best = 1e300;
    int st = SDE_OK;
    std::vector<int> cands = sizeof(R) == 4 ? std::vector<int>{1, 2, 4} : std::vector<int>{1, 2};
    if (split_fits(ctx, P)) cands.push_back(kSplitChoice);
    for (int choice : cands) {
        JJLaunch L = base;
        set_choice(L, choice);
        JJPlan<R> plan;
        plan_items(P, kinds, L.ppt, plan);
        L.point_sums = nullptr;
        L.A.theta = nullptr;
        L.A.winding = nullptr;
        L.A.v = nullptr;
        L.A.acc = nullptr;
        L.A.rec = nullptr;
        L.A.init_from_state = 0;
        L.A.flag = ctx->tune_flag;  // a trial run's NaN is not the caller's
        if ((st = jj_upload_plan(ctx, plan, stream, L))) break;
        float ms = 0.f;
        for (int rep = 0; rep < 3; ++rep) {  // the first launch loads the code object; the faster of the others
            if ((st = hipEventRecord(e0, stream) == hipSuccess ? SDE_OK : SDE_ERR_DEVICE)) break;
            if ((st = jj_record<R>(ctx, L, stream))) break;
            if ((st = hipEventRecord(e1, stream) == hipSuccess ? SDE_OK : SDE_ERR_DEVICE)) break;
            if (hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(&ms, e0, e1) != hipSuccess) {
                st = SDE_ERR_DEVICE;
                break;
            }
            if (rep > 0 && ms < best) {
                best = ms;
                *best_choice = choice;
            }
        }
        if (st) break;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (st == SDE_ERR_DEVICE) return fail(ctx, st, "autotuner: HIP event or launch failed");
    return st;
}

// What one call computes, from its arguments: per-point constants, point
// kinds, the drive tables, and the shape class of the call.
template <typename R>
struct JJSetup {
    std::vector<JJPointT<R>> P;
    std::vector<int> kinds;
    std::vector<R> lut;
    uint64_t path_first = 0, max_steps = 0;
    unsigned kinds_present = 0;
    uint32_t M = 100, max_period = 0;
};

// Whether every point's drive terms fit the persistent kernel's LDS table.
template <typename R>
static bool drive_fits(const JJSetup<R>& S)
{
    return S.max_period <= kDriveTable - 8;
}

// Validates a call's arguments (nothing is launched on an error) and builds
// its per-point constants and drive tables.
template <typename R>
static int jj_setup(sde_ctx* ctx, const sde_jj_point* pts, uint32_t n_pts, const sde_run* run, R* theta,
                    int32_t* winding, R* v, double* acc, double* point_sums, JJSetup<R>& out)
{
    ctx->last = sde_stats{};
    if (!pts || !run || n_pts == 0) return fail(ctx, SDE_ERR_INVALID, "null points/run or n_pts = 0");
    if (run->scheme != SDE_HEUN && run->scheme != SDE_EULER)
        return fail(ctx, SDE_ERR_INVALID, "unknown scheme %d", run->scheme);
    if (run->init != SDE_INIT_PHILOX && run->init != SDE_INIT_FROM_STATE)
        return fail(ctx, SDE_ERR_INVALID, "unknown init %d", run->init);
    if (run->init == SDE_INIT_FROM_STATE && (!theta || !winding || !v || !acc))
        return fail(ctx, SDE_ERR_INVALID, "SDE_INIT_FROM_STATE needs theta, winding, v and acc");
    if (!aligned(theta, sizeof(R)) || !aligned(winding, 4) || !aligned(v, sizeof(R)) || !aligned(acc, 8) ||
        !aligned(point_sums, 8))
        return fail(ctx, SDE_ERR_INVALID, "misaligned device pointer");
    out.M = run->sample_every ? run->sample_every : 100u;

    std::vector<JJPointT<R>>& P = out.P;
    std::vector<int>& kinds = out.kinds;
    std::vector<R>& lut = out.lut;
    P.assign(n_pts, JJPointT<R>{});
    kinds.assign(n_pts, 0);
    lut.clear();
    std::map<uint32_t, uint32_t> lut_of;  // S -> offset
    uint64_t path_first = 0, max_steps = 0;
    unsigned kinds_present = 0;
    for (uint32_t q = 0; q < n_pts; ++q) {
        const sde_jj_point& p = pts[q];
        if (!finite_point(p)) return fail(ctx, SDE_ERR_INVALID, "point %u: non-finite parameter", q);
        if (p.n_paths == 0 || p.steps_per_period == 0)
            return fail(ctx, SDE_ERR_INVALID, "point %u: n_paths and steps_per_period must be > 0", q);
        if (p.n_paths > (1u << 31)) return fail(ctx, SDE_ERR_INVALID, "point %u: more than 2^31 paths", q);
        if (!(p.omega > 0) || p.m < 0 || p.gamma < 0 || p.D < 0 || (p.m == 0 && !(p.gamma > 0)))
            return fail(ctx, SDE_ERR_INVALID, "point %u: need omega > 0, m >= 0, D >= 0, gamma >= 0 "
                        "(gamma > 0 when m = 0)", q);
        if (p.potential != SDE_POTENTIAL_SIN && p.potential != SDE_POTENTIAL_SIN2PI)
            return fail(ctx, SDE_ERR_INVALID, "point %u: unknown potential %d", q, p.potential);
        if (p.reserved != 0) return fail(ctx, SDE_ERR_INVALID, "point %u: reserved must be 0", q);
        const bool sin2pi = p.potential == SDE_POTENTIAL_SIN2PI;
        const double L = sin2pi ? 1.0 : 2.0 * M_PI;   // period of the coordinate
        const double amp = sin2pi ? 2.0 * M_PI : 1.0;  // amplitude of the potential force
        const double dt = 2.0 * M_PI / (p.omega * (double)p.steps_per_period);
        JJPointT<R>& d = P[q];
        d.dt = (R)dt;
        d.hdt = (R)(0.5 * dt);
        d.dtp = (R)(dt / L);
        d.hdtp = (R)(0.5 * dt / L);
        d.inertial = p.m > 0 ? 1u : 0u;
        if (d.inertial) {
            d.kv = (R)(amp / p.m);
            d.gim = (R)(p.gamma / p.m);
            d.a_im = (R)(p.a / p.m);
            d.f_im = (R)(p.f / p.m);
            const double sig = std::sqrt(2.0 * p.gamma * p.D * dt) / p.m;
            d.c2 = (R)(-2.0 * M_LN2 * sig * sig);
            d.sig_v = (R)0;
        } else {
            const double s = std::sqrt(2.0 * p.D * dt / p.gamma);
            d.kv = (R)(amp / p.gamma);
            d.gim = (R)0;
            d.a_im = (R)(p.a / p.gamma);
            d.f_im = (R)(p.f / p.gamma);
            const double sig = s / L;
            d.c2 = (R)(-2.0 * M_LN2 * sig * sig);
            d.sig_v = (R)(L / dt);
        }
        kinds[q] = (d.inertial ? 0 : 1) + (sin2pi ? 2 : 0);
        kinds_present |= 1u << kinds[q];
        d.S = p.steps_per_period;
        auto it = lut_of.find(d.S);
        if (it == lut_of.end()) {
            const uint32_t off = (uint32_t)lut.size();
            for (uint32_t k = 0; k < d.S + 8; ++k)
                lut.push_back((R)std::cos(2.0 * M_PI * (double)(k % d.S) / (double)d.S));
            it = lut_of.emplace(d.S, off).first;
        }
        d.lut_off = it->second;
        d.n_paths = p.n_paths;
        d.path_first = path_first;
        d.n_steps = p.n_steps;
        d.n_transient = p.n_transient;
        const uint64_t end = run->step0 + p.n_steps;
        const uint64_t W = end > p.n_transient ? end - p.n_transient : 0;
        d.inv_W = W ? 1.0 / (double)W : 0.0;
        path_first += p.n_paths;
        max_steps = std::max<uint64_t>(max_steps, p.n_steps);
        out.max_period = std::max(out.max_period, p.steps_per_period);
    }
    if (path_first / kWave > 0xffffffffull) return fail(ctx, SDE_ERR_INVALID, "too many paths in one call");
    out.path_first = path_first;
    out.max_steps = max_steps;
    out.kinds_present = kinds_present;
    return SDE_OK;
}

// The kernel arguments that come from the run options and the caller's
// buffers (the workspace pointers are filled in by the caller).
template <typename R>
static void jj_fill_args(sde_ctx* ctx, const sde_run* run, const JJSetup<R>& S, R* theta, int32_t* winding, R* v,
                         double* acc, double* point_sums, JJLaunch& L)
{
    L.scheme = run->scheme;
    L.tab = drive_fits(S);
    L.point_sums = point_sums;
    L.A.flag = ctx->flag;
    L.A.theta = theta;
    L.A.winding = winding;
    L.A.v = v;
    L.A.acc = acc;
    L.A.step0 = run->step0;
    L.A.tables = nullptr;
    L.A.rec = nullptr;
    L.A.rec_pitch = S.path_first;
    L.A.rec_every = 0u;
    L.A.key0 = (uint32_t)(run->seed & 0xffffffffu);
    L.A.key1 = (uint32_t)(run->seed >> 32);
    L.A.M = S.M;
    L.A.init_from_state = run->init == SDE_INIT_FROM_STATE;
}

// The choice of a call that is neither forced nor tuned.
template <typename R>
static int default_choice(const sde_ctx* ctx, const JJSetup<R>& S)
{
    return split_fits(ctx, S.P) ? kSplitChoice : 2;
}

// Tune-cache key of a call's shape class (paths per lane).  Calls that have
// other candidates or kernels are classes of their own: those small enough for
// the split kernel (the limit lies inside a power of two of paths), and FP32
// periods past the drive table.
template <typename R>
static std::string jj_tune_key(sde_ctx* ctx, const sde_run* run, const JJSetup<R>& S)
{
    char key[192];
    snprintf(key, sizeof key, "jj|%s|%s|scheme%d|kinds%x|paths2^%d|steps2^%d%s%s", ctx->arch.c_str(),
             sizeof(R) == 4 ? "f32" : "f64", run->scheme, S.kinds_present, ilog2u64(S.path_first),
             ilog2u64(std::max<uint64_t>(S.max_steps, 1)), split_fits(ctx, S.P) ? "|few" : "",
             sizeof(R) == 4 && !drive_fits(S) ? "|long-drive" : "");
    return key;
}

// The choice cached for a call's class, if it can run it.
template <typename R>
static bool cached_choice(sde_ctx* ctx, const sde_run* run, const JJSetup<R>& S, int* choice)
{
    int c;
    if (!tune_lookup(ctx, jj_tune_key<R>(ctx, run, S), &c) || (c == kSplitChoice && !split_fits(ctx, S.P))) return false;
    *choice = c;
    return true;
}

template <typename R>
static int jj_integrate_t(sde_ctx* ctx, const sde_jj_point* pts, uint32_t n_pts, const sde_run* run, R* theta,
                          int32_t* winding, R* v, double* acc, double* point_sums, int32_t* rec,
                          uint32_t rec_every, uint64_t rec_rows, hipStream_t stream)
{
    JJSetup<R> S;
    int st = jj_setup<R>(ctx, pts, n_pts, run, theta, winding, v, acc, point_sums, S);
    if (st) return st;
    if (rec) {
        if (rec_every == 0 || rec_every % 4 != 0)
            return fail(ctx, SDE_ERR_INVALID, "record_every must be a positive multiple of 4");
        if (!aligned(rec, 4)) return fail(ctx, SDE_ERR_INVALID, "misaligned record buffer");
        for (uint32_t q = 0; q < n_pts; ++q) {
            const uint64_t rows = (run->step0 + pts[q].n_steps) / rec_every - run->step0 / rec_every;
            if (rows > rec_rows)
                return fail(ctx, SDE_ERR_INVALID, "point %u needs %llu record rows, the buffer has %llu", q,
                            (unsigned long long)rows, (unsigned long long)rec_rows);
        }
    }

    if ((st = upload(ctx, kSlotJJLut, 2, S.lut.data(), S.lut.size() * sizeof(R), stream))) return st;
    JJLaunch L;
    jj_fill_args<R>(ctx, run, S, theta, winding, v, acc, point_sums, L);
    L.A.lut = ctx->ws[kSlotJJLut].ptr;
    if (sizeof(R) == 8) {
        if ((st = upload(ctx, kSlotJJTables, 3, &host_tables(), sizeof(F64Tables), stream))) return st;
        L.A.tables = ctx->ws[kSlotJJTables].ptr;
    }
    L.A.rec = rec;
    L.A.rec_every = rec ? rec_every : 0u;
    const char* prec = sizeof(R) == 4 ? "f32" : "f64";

    // the launch choice: paths per lane as forced, cached, or tuned on this
    // call's shape class
    int choice = ctx->jj_ppt;
    if (sizeof(R) == 8 && choice == 4) choice = 2;
    if (!choice) {
        if (!cached_choice(ctx, run, S, &choice)) {
            choice = default_choice(ctx, S);
            if (ctx->autotune) {
                const auto t0 = std::chrono::steady_clock::now();
                if ((st = jj_tune<R>(ctx, S.P, S.kinds, L, stream, &choice))) return st;
                ctx->last.tuned = 1;
                ctx->last.tune_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
                tune_store(ctx, jj_tune_key<R>(ctx, run, S), choice);
            }
        }
    }
    set_choice(L, choice);
    JJPlan<R> plan;
    plan_items(S.P, S.kinds, L.ppt, plan);
    if ((st = jj_upload_plan(ctx, plan, stream, L))) return st;
    ctx->last.jj_paths_per_lane = L.ppt;
    ctx->last.work_items = plan.items.size();

    if ((st = run_recorded(ctx, jj_graph_key(prec, L), stream, [&](hipStream_t s) { return jj_record<R>(ctx, L, s); })))
        return st;
    if (run->sync) return sync_and_check(ctx, stream);
    return SDE_OK;
}

int jj_integrate_impl(sde_ctx* ctx, const sde_jj_point* pts, uint32_t n_pts, const sde_run* run,
                      float* theta, int32_t* winding, float* v, double* acc, double* point_sums,
                      hipStream_t stream)
{
    return jj_integrate_t<float>(ctx, pts, n_pts, run, theta, winding, v, acc, point_sums, nullptr, 0, 0, stream);
}

int jj_integrate_recorded_impl(sde_ctx* ctx, const sde_jj_point* pts, uint32_t n_pts, const sde_run* run,
                               float* theta, int32_t* winding, float* v, double* acc, double* point_sums,
                               uint32_t record_every, uint64_t n_rows, int32_t* rec_winding, hipStream_t stream)
{
    if (!rec_winding) return fail(ctx, SDE_ERR_INVALID, "null record buffer");
    return jj_integrate_t<float>(ctx, pts, n_pts, run, theta, winding, v, acc, point_sums, rec_winding,
                                 record_every, n_rows, stream);
}

int jj_integrate_f64_impl(sde_ctx* ctx, const sde_jj_point* pts, uint32_t n_pts, const sde_run* run,
                          double* theta, int32_t* winding, double* v, double* acc, double* point_sums,
                          hipStream_t stream)
{
    return jj_integrate_t<double>(ctx, pts, n_pts, run, theta, winding, v, acc, point_sums, nullptr, 0, 0, stream);
}

// ---------------------------------------------- the no-allocation variant --
// Device scratch of sde_jj_integrate_noalloc: the queue words, point table,
// work items, drive tables and per-chunk partial sums of one call, in
// 256-byte aligned sections.  Each GPU the library runs on holds its own copy
// until the process ends; every such call on that GPU uses it.
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

// Device address of `scratch` per device (host code must never pass the
// array's own name to a kernel or a copy: on the host it is a stand-in).
static void* g_scratch_addr[kMaxDevices] = {};
static std::mutex g_scratch_mu;

int noalloc_setup(sde_ctx* ctx)
{
    if (ctx->device < 0 || ctx->device >= kMaxDevices)
        return fail(ctx, SDE_ERR_UNSUPPORTED, "device %d: beyond the %d devices the library tracks", ctx->device,
                    kMaxDevices);
    {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        if (!g_scratch_addr[ctx->device]) {
            void* ptr = nullptr;
            // the caller has made ctx->device current
            const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
            if (e != hipSuccess || !ptr)
                return fail(ctx, SDE_ERR_DEVICE, "hipGetSymbolAddress(scratch) failed: %s", hipGetErrorString(e));
            g_scratch_addr[ctx->device] = ptr;
        }
        ctx->noalloc_scratch = g_scratch_addr[ctx->device];
    }
    // the host image of a call's tables is staged here (pinned, so the copy
    // is asynchronous); it is never larger than the scratch
    SDE_HIP(ctx, hipHostMalloc(&ctx->noalloc_staging, kNoAllocScratchBytes, hipHostMallocDefault));
    SDE_HIP(ctx, hipEventCreateWithFlags(&ctx->noalloc_done, hipEventDisableTiming));
    return SDE_OK;
}

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

int jj_integrate_noalloc_impl(sde_ctx* ctx, const sde_jj_point* pts, uint32_t n_pts, const sde_run* run,
                              float* theta, int32_t* winding, float* v, double* acc, double* point_sums,
                              hipStream_t stream)
{
    if (!ctx->noalloc_scratch || !ctx->noalloc_staging || !ctx->noalloc_done)
        return fail(ctx, SDE_ERR_DEVICE, "the no-allocation scratch was not set up for this context");
    JJSetup<float> S;
    int st = jj_setup<float>(ctx, pts, n_pts, run, theta, winding, v, acc, point_sums, S);
    if (st) return st;
    // paths per lane: forced, else a choice the tuner cached, else the
    // default; never tuned here (tuning allocates)
    int choice = ctx->jj_ppt;
    if (!choice && !cached_choice(ctx, run, S, &choice)) choice = default_choice(ctx, S);

    // layout of the scratch; the tables [o_pts, o_part) are one host image
    JJLaunch L;
    JJPlan<float> plan;
    const size_t pts_bytes = S.P.size() * sizeof(JJPointDev), lut_bytes = S.lut.size() * sizeof(float);
    const size_t o_queue = 0, o_pts = align256(o_queue + kJJKinds * sizeof(uint32_t));
    const size_t o_items = align256(o_pts + pts_bytes);
    size_t items_bytes, o_lut, o_part, need;
    for (;;) {
        set_choice(L, choice);
        plan_items(S.P, S.kinds, L.ppt, plan);
        items_bytes = plan.items.size() * sizeof(JJItem);
        o_lut = align256(o_items + items_bytes);
        o_part = align256(o_lut + lut_bytes);
        need = o_part + (size_t)std::max(plan.n_chunks, 1u) * 2 * sizeof(double);
        if (need <= kNoAllocScratchBytes || ctx->jj_ppt || L.ppt != 1) break;
        choice = 2;  // one path per lane, not forced: half the chunks may fit
    }
    if (need > kNoAllocScratchBytes)
        return fail(ctx, SDE_ERR_INVALID,
                    "sde_jj_integrate_noalloc: %u points in %u path chunks need %zu bytes of scratch, the maximum "
                    "is %zu",
                    n_pts, plan.n_chunks, need, (size_t)kNoAllocScratchBytes);

    // the previous call's copy may still read the staging buffer
    if (ctx->noalloc_pending) {
        SDE_HIP(ctx, hipEventSynchronize(ctx->noalloc_done));
        ctx->noalloc_pending = false;
    }
    unsigned char* img = static_cast<unsigned char*>(ctx->noalloc_staging);
    std::memcpy(img, plan.pts.data(), pts_bytes);
    std::memcpy(img + (o_items - o_pts), plan.items.data(), items_bytes);
    std::memcpy(img + (o_lut - o_pts), S.lut.data(), lut_bytes);
    unsigned char* base = static_cast<unsigned char*>(ctx->noalloc_scratch);
    SDE_HIP(ctx, hipMemcpyAsync(base + o_pts, img, o_part - o_pts, hipMemcpyHostToDevice, stream));
    SDE_HIP(ctx, hipEventRecord(ctx->noalloc_done, stream));
    ctx->noalloc_pending = true;

    jj_fill_args<float>(ctx, run, S, theta, winding, v, acc, point_sums, L);
    L.queues = reinterpret_cast<uint32_t*>(base + o_queue);
    L.A.pts = base + o_pts;
    L.A.items = reinterpret_cast<const JJItem*>(base + o_items);
    L.A.lut = base + o_lut;
    L.A.partials = reinterpret_cast<double*>(base + o_part);
    std::copy(plan.kind_begin, plan.kind_begin + kJJKinds + 1, L.kind_begin);
    L.n_items = (uint32_t)plan.items.size();
    L.n_pts = (uint32_t)plan.pts.size();
    if ((st = jj_grids<float>(ctx, L))) return st;
    ctx->last.jj_paths_per_lane = L.ppt;
    ctx->last.work_items = plan.items.size();
    if ((st = jj_record<float>(ctx, L, stream))) return st;
    if (run->sync) return sync_and_check(ctx, stream);
    return SDE_OK;
}

int debug_philox_impl(sde_ctx* ctx, uint64_t seed, uint32_t tag, uint32_t a, uint32_t b, uint64_t c0,
                      uint64_t n, uint32_t* out, hipStream_t stream)
{
    if (!out || n == 0) return fail(ctx, SDE_ERR_INVALID, "null output or zero blocks");
    if (!aligned(out, 4)) return fail(ctx, SDE_ERR_INVALID, "misaligned output");
    const uint64_t blocks = (n + 255) / 256;
    if (blocks > 0x7fffffffu) return fail(ctx, SDE_ERR_INVALID, "too many blocks");
    hipLaunchKernelGGL(philox_dump_kernel, dim3((uint32_t)blocks), dim3(256), 0, stream, (uint32_t)seed,
                       (uint32_t)(seed >> 32), tag, a, b, c0, n, out);
    SDE_HIP(ctx, hipGetLastError());
    return SDE_OK;
}

int debug_gauss_impl(sde_ctx* ctx, uint64_t seed, uint32_t tag, uint32_t a, uint32_t b, uint64_t n0,
                     uint64_t n, float* out, hipStream_t stream)
{
    if (!out || n == 0) return fail(ctx, SDE_ERR_INVALID, "null output or zero count");
    if (!aligned(out, 4)) return fail(ctx, SDE_ERR_INVALID, "misaligned output");
    const uint64_t blocks = (n + 255) / 256;
    if (blocks > 0x7fffffffu) return fail(ctx, SDE_ERR_INVALID, "count too large");
    hipLaunchKernelGGL(gauss_dump_kernel, dim3((uint32_t)blocks), dim3(256), 0, stream, (uint32_t)seed,
                       (uint32_t)(seed >> 32), tag, a, b, n0, n, out);
    SDE_HIP(ctx, hipGetLastError());
    return SDE_OK;
}

}  // namespace sde
