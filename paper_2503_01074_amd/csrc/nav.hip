// Navigation sensors of Sec. III-A of arXiv 2503.01074 on gfx950: the
// barometer (pressure from the atmospheric pressure and the water density,
// optional Gaussian noise) and the four-beam Janus DVL (range-dependent
// measurement rate, dropout when too few beams return).  The paper prints no
// equations for either; the readings are stated in include/oceansim.h.
//
//   k_baro  one pressure per sample (elementwise, four samples per thread).
//   k_dvl   one workgroup per 64 instances (vehicles or Monte Carlo runs):
//           the ticks' ping periods in parallel, the measurement schedule
//           (which carries the time of the last measurement from tick to
//           tick) by one wave, the due measurements from a compacted list.
//   k_dvl_walk  one thread per instance, walking its ticks: few ticks or very
//           many instances (dvl_walks).
// Inputs are tick-major ([tick][instance]), so the loads of a tick are
// coalesced across the lanes of a wave.
#include <hip/hip_runtime.h>

#include <cmath>

#include "../../include/oceansim.h"
#include "device.hpp"
#include "host.hpp"
#include "launch.hpp"

namespace osim {
namespace {

constexpr int kNavThreads = 256;
constexpr int kBaroPerThread = 4;

// Standard normal from two words of a Philox block: Box-Muller, cosine branch.
__device__ __forceinline__ float gauss_of_words(uint32_t w0, uint32_t w1) {
    return __builtin_amdgcn_sqrtf(2.0f * neg_ln(unit_uniform(w0))) * cospif(2.0f * unit_uniform(w1));
}

struct BaroDev {
    double p_atm, rho_g, sigma;
    uint32_t seed_lo, seed_hi;
};

__global__ __launch_bounds__(kNavThreads) void k_baro(gptr<const float> depth, long long n, BaroDev p,
                                                      gptr<float> pressure) {
    const long long k0 = ((long long)blockIdx.x * kNavThreads * kBaroPerThread) + threadIdx.x;
#pragma unroll
    for (int u = 0; u < kBaroPerThread; ++u) {
        const long long k = k0 + (long long)u * kNavThreads;
        if (k >= n) return;
        const double d = (double)depth[k];
        double z = 0.0;
        if (p.sigma != 0.0) {
            const Words w = philox((uint32_t)k, (uint32_t)((unsigned long long)k >> 32), 3u, 0u, p.seed_lo, p.seed_hi);
            z = (double)gauss_of_words(w.w0, w.w1);
        }
        // the water column above the sensor (none above the surface)
        const double column = d > 0.0 ? p.rho_g * d : 0.0;
        pressure[k] = (float)(p.p_atm + column + p.sigma * z);
    }
}

struct DvlDev {
    double beam[4][3];          // unit beam directions (sensor frame)
    double range_min, range_max;
    double sigma_v;
    double pings_per_output, sound_speed, period_min;
    int min_beams;
    uint32_t seed_lo, seed_hi;
};

// A workgroup takes 64 neighbouring instances (one per lane) and walks their
// ticks in slabs of 32.  Only the measurement schedule is sequential, and it
// needs no more than each tick's ping period: all eight waves reduce a slab's
// ranges to periods and valid-beam bits (four ticks a wave, loaded a slab
// ahead); then wave 0 walks the schedule of that slab from LDS while the other
// seven write the slab before it: status, NaN where there is no velocity, and
// the due measurements (at 5-30 ms ticks and pings of 0.125 s and more, about
// one tick in fourteen), which each wave first lists, so that the draws and the
// least squares run on full lanes and read the velocity of those ticks alone.
// One barrier a slab; the buffers that cross it are double (periods, read by
// the schedule) or triple (beam bits and due bits, read a slab later).
// 256 ticks x 32768 instances: 82 us, 4.5 TB/s of the 44 B per tick and
// instance, 3.8 TB/s of the bytes it moves, since only the due ticks' velocities
// are read (374 us with one thread per instance walking its ticks: two waves
// per CU, one tick's loads in flight, the noise drawn under nearly every
// wave's branch; 95 us with the schedule and the writes in turn, four barriers
// a slab).  Bound by the slab's chain of loads, schedule and draws more than by
// HBM; 128 registers (the FP64 least squares) hold it to two workgroups a CU.
constexpr int kDvlInst = kWave;                       // instances per workgroup
constexpr int kDvlThreads = 512;
constexpr int kDvlWaves = kDvlThreads / kWave;
constexpr int kDvlSlab = 32;                          // ticks per round
constexpr int kDvlPerWave = kDvlSlab / kDvlWaves;     // ticks a wave reduces per round
constexpr int kDvlOut = (kDvlSlab + kDvlWaves - 2) / (kDvlWaves - 1);   // ticks a wave writes per round

// Least-squares velocity of a due measurement from the valid beams (bits of ok).
__device__ __forceinline__ void dvl_solve(const DvlDev &p, int k, int n, unsigned ok, double v0, double v1,
                                          double v2, float (&out)[3]) {
    // normal equations over the valid beams: A x = B^T u, A = sum b b^T
    Words w01{0u, 0u, 0u, 0u}, w23{0u, 0u, 0u, 0u};
    if (p.sigma_v != 0.0) {
        w01 = philox((uint32_t)k, (uint32_t)n, 4u, 0u, p.seed_lo, p.seed_hi);
        w23 = philox((uint32_t)k, (uint32_t)n, 4u, 1u, p.seed_lo, p.seed_hi);
    }
    double a00 = 0.0, a01 = 0.0, a02 = 0.0, a11 = 0.0, a12 = 0.0, a22 = 0.0;
    double q0 = 0.0, q1 = 0.0, q2 = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (!((ok >> i) & 1u)) continue;
        const double *b = p.beam[i];
        double z = 0.0;
        if (p.sigma_v != 0.0) {
            const Words &w = i < 2 ? w01 : w23;
            z = (double)gauss_of_words(pick(w, 2u * (i & 1)), pick(w, 2u * (i & 1) + 1u));
        }
        const double u = b[0] * v0 + b[1] * v1 + b[2] * v2 + p.sigma_v * z;   // along-beam Doppler velocity
        a00 += b[0] * b[0];
        a01 += b[0] * b[1];
        a02 += b[0] * b[2];
        a11 += b[1] * b[1];
        a12 += b[1] * b[2];
        a22 += b[2] * b[2];
        q0 += b[0] * u;
        q1 += b[1] * u;
        q2 += b[2] * u;
    }
    // x = adj(A) q / det(A) for the symmetric A
    const double c00 = a11 * a22 - a12 * a12, c01 = a02 * a12 - a01 * a22, c02 = a01 * a12 - a02 * a11;
    const double c11 = a00 * a22 - a02 * a02, c12 = a01 * a02 - a00 * a12, c22 = a00 * a11 - a01 * a01;
    const double inv_det = 1.0 / (a00 * c00 + a01 * c01 + a02 * c02);
    out[0] = (float)((c00 * q0 + c01 * q1 + c02 * q2) * inv_det);
    out[1] = (float)((c01 * q0 + c11 * q1 + c12 * q2) * inv_det);
    out[2] = (float)((c02 * q0 + c12 * q1 + c22 * q2) * inv_det);
}

__global__ __launch_bounds__(kDvlThreads, 4) void k_dvl(gptr<const double> t, gptr<const float4> ranges,
                                                     gptr<const float> vel, int n_ticks, int n_inst, DvlDev p,
                                                     gptr<float> vout, gptr<int> status) {
    __shared__ double period_s[2][kDvlSlab][kDvlInst];
    __shared__ unsigned char ok_s[3][kDvlSlab][kDvlInst];           // valid-beam bits
    __shared__ unsigned long long due_s[3][kDvlSlab];               // due instances of a tick
    __shared__ unsigned short items[kDvlWaves][kDvlOut * kDvlInst];   // tick in the slab << 6 | lane
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int n0 = blockIdx.x * kDvlInst;
    const int n = n0 + lane;
    const bool live = n < n_inst;
    const int nc = live ? n : n_inst - 1;
    float4 r4[kDvlPerWave];
    auto load_slab = [&](int s0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kDvlPerWave; ++u) {
            const int k = min(s0 + u * kDvlWaves + wave, n_ticks - 1);
            r4[u] = gload((gptr<const float4>)(ranges + ((long long)k * n_inst + nc)));
        }
    };
    // status and velocity of the slab from tick s0 on (buffer slot `b`), ticks w0, w0 + step, ...
    auto write_slab = [&](int s0, int b, int w0, int step) __attribute__((always_inline)) {
        unsigned short *list = items[wave];
        int total = 0;
        for (int i = w0; i < kDvlSlab && s0 + i < n_ticks; i += step) {
            const bool due = (due_s[b][i] >> lane) & 1ull;
            const bool meas = due && __popc((unsigned)ok_s[b][i][lane]) >= p.min_beams;
            const unsigned long long m = __ballot(meas);
            const long long row = (long long)(s0 + i) * n_inst + n;
            if (meas) {
                list[total + __popcll(m & ((1ull << lane) - 1ull))] = (unsigned short)(i * kDvlInst + lane);
            } else if (live) {
                const gptr<float> vo = vout + 3 * row;
                vo[0] = vo[1] = vo[2] = __builtin_nanf("");
            }
            if (live) status[row] = meas ? 1 : (due ? 2 : 0);
            total += __popcll(m);
        }
        // the wave's own list (no other wave touches it)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        for (int q = lane; q < total; q += kWave) {
            const int i = list[q] / kDvlInst, l = list[q] % kDvlInst;
            const long long row = (long long)(s0 + i) * n_inst + (n0 + l);
            const gptr<const float> v = vel + 3 * row;
            float o[3];
            dvl_solve(p, s0 + i, n0 + l, ok_s[b][i][l], v[0], v[1], v[2], o);
            const gptr<float> vo = vout + 3 * row;
            vo[0] = o[0];
            vo[1] = o[1];
            vo[2] = o[2];
        }
        __builtin_amdgcn_wave_barrier();
    };
    double t_last = 0.0;   // the schedule, carried by wave 0
    bool have_last = false;
    load_slab(0);
    int b3 = 0;   // slab index modulo 3
    for (int s0 = 0; s0 < n_ticks; s0 += kDvlSlab) {
        const int b2 = (s0 / kDvlSlab) & 1;
        // valid beams and ping period of each tick: two-way travel of the
        // farthest valid beam times the pings averaged into one output
#pragma unroll
        for (int u = 0; u < kDvlPerWave; ++u) {
            const float r[4] = {r4[u].x, r4[u].y, r4[u].z, r4[u].w};
            unsigned ok = 0u;
            double r_ref = 0.0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const double ri = (double)r[i];
                if (__builtin_isfinite(ri) && ri >= p.range_min && ri <= p.range_max) {
                    ok |= 1u << i;
                    r_ref = ri > r_ref ? ri : r_ref;
                }
            }
            if (ok == 0u) r_ref = p.range_max;
            double period = p.pings_per_output * 2.0 * r_ref / p.sound_speed;
            period = period < p.period_min ? p.period_min : period;
            period_s[b2][u * kDvlWaves + wave][lane] = period;
            ok_s[b3][u * kDvlWaves + wave][lane] = (unsigned char)ok;
        }
        if (s0 + kDvlSlab < n_ticks) load_slab(s0 + kDvlSlab);   // the next slab, under this one's work
        __syncthreads();
        const int prev3 = b3 == 0 ? 2 : b3 - 1;
        if (wave == 0) {
            const int cnt = min(kDvlSlab, n_ticks - s0);
            const double tl = t[s0 + min(lane, cnt - 1)];   // lane i: time of tick i
            const unsigned t_lo = (unsigned)__double_as_longlong(tl);
            const unsigned t_hi = (unsigned)(__double_as_longlong(tl) >> 32);
#pragma unroll 8
            for (int i = 0; i < cnt; ++i) {
                const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)t_lo, i);
                const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)t_hi, i);
                const double tk = __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
                const bool due = live && (!have_last || (tk - t_last >= period_s[b2][i][lane]));
                have_last |= due;
                t_last = due ? tk : t_last;
                const unsigned long long m = __ballot(due);
                if (lane == 0) due_s[b3][i] = m;
            }
        } else if (s0 > 0) {
            write_slab(s0 - kDvlSlab, prev3, wave - 1, kDvlWaves - 1);
        }
        b3 = b3 == 2 ? 0 : b3 + 1;
    }
    __syncthreads();
    const int last = (n_ticks - 1) / kDvlSlab * kDvlSlab;
    write_slab(last, b3 == 0 ? 2 : b3 - 1, wave, kDvlWaves);
}

// One thread per instance, walking its ticks.  Where there are waves enough to
// hide a tick's loads it is bound by HBM (8 ticks x 1048576 instances: 70 us,
// 5.3 TB/s), or by the solutions' VALU work where every tick is due.
__global__ __launch_bounds__(kNavThreads) void k_dvl_walk(gptr<const double> t, gptr<const float4> ranges,
                                                          gptr<const float> vel, int n_ticks, int n_inst, DvlDev p,
                                                          gptr<float> vout, gptr<int> status) {
    const int n = blockIdx.x * kNavThreads + threadIdx.x;
    if (n >= n_inst) return;
    double t_last = 0.0;
    bool have_last = false;
    // the next tick's inputs are loaded while this tick is processed (past
    // the last tick the loads re-read it)
    float4 r4n = gload((gptr<const float4>)(ranges + n));
    float vn0 = vel[3LL * n], vn1 = vel[3LL * n + 1], vn2 = vel[3LL * n + 2];
    for (int k = 0; k < n_ticks; ++k) {
        const long long row = (long long)k * n_inst + n;
        const float r[4] = {r4n.x, r4n.y, r4n.z, r4n.w};
        const double v0 = vn0, v1 = vn1, v2 = vn2;
        {
            const long long nrow = (long long)(k + 1 < n_ticks ? k + 1 : k) * n_inst + n;
            r4n = gload((gptr<const float4>)(ranges + nrow));
            vn0 = vel[3 * nrow];
            vn1 = vel[3 * nrow + 1];
            vn2 = vel[3 * nrow + 2];
        }
        unsigned ok = 0u;
        double r_ref = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const double ri = (double)r[i];
            if (__builtin_isfinite(ri) && ri >= p.range_min && ri <= p.range_max) {
                ok |= 1u << i;
                r_ref = ri > r_ref ? ri : r_ref;
            }
        }
        if (ok == 0u) r_ref = p.range_max;
        double period = p.pings_per_output * 2.0 * r_ref / p.sound_speed;
        period = period < p.period_min ? p.period_min : period;
        const double tk = t[k];
        const bool due = !have_last || (tk - t_last >= period);
        float o[3] = {__builtin_nanf(""), __builtin_nanf(""), __builtin_nanf("")};
        int s = 0;
        if (due) {
            have_last = true;
            t_last = tk;
            s = 2;
            if (__popc(ok) >= p.min_beams) {
                s = 1;
                dvl_solve(p, k, n, ok, v0, v1, v2, o);
            }
        }
        const gptr<float> vo = vout + 3 * row;
        vo[0] = o[0];
        vo[1] = o[1];
        vo[2] = o[2];
        status[row] = s;
    }
}

// Which calls walk.  k_dvl reduces slabs of 32 ticks whatever their number and
// gives up one wave of eight to the schedule; walking needs instances to fill
// the chip.  Walked / k_dvl, us, with about one tick in fourteen due (with
// every tick due):
//   49152 instances,  8 ticks  10 / 11 (14 / 13)     24 ticks   32 / 20 (37 / 26)
//   65536             8        10 / 13 (14 / 16)     24         32 / 24 (37 / 33)
//   98304            16        25 / 31 (34 / 35)     24         39 / 34 (49 / 48)
//   131072           32        54 / 51 (64 / 78)     64        121 / 92 (133 / 144)     128  246 / 155 (261 / 260)
//   262144           32        89 / 107 (111 / 161)  64        182 / 170 (217 / 275)    256  758 / 548 (842 / 956)
//   1048576           1        15 / 143 (14 / 143)    8         70 / 184 (102 / 237)     64  629 / 617 (797 / 1049)
// How many ticks are due is in the data, so the line lies where k_dvl is the
// faster one either way.
bool dvl_walks(int n_ticks, int n_inst) {
    if (n_inst >= 163840) return true;
    if (n_inst >= 114688) return n_ticks <= 64;
    return n_inst >= 49152 && n_ticks <= n_inst / 4096 - 4;
}

bool aligned_to(const void *p, size_t a) { return ((uintptr_t)p % a) == 0; }

}  // namespace
}  // namespace osim

using namespace osim;
using namespace osim::host;

extern "C" {

int oceansim_barometer(const float *depth_dev, int64_t n, const oceansim_baro_params *params, float *pressure_dev,
                       void *stream) {
    if (!params) return fail(OCEANSIM_E_INVALID_ARG, "params is NULL");
    if (n < 0) return fail(OCEANSIM_E_SHAPE, "n < 0");
    if (n > 0 && (!depth_dev || !pressure_dev)) return fail(OCEANSIM_E_INVALID_ARG, "NULL buffer");
    if (!aligned_to(depth_dev, 4) || !aligned_to(pressure_dev, 4))
        return fail(OCEANSIM_E_INVALID_ARG, "misaligned buffer");
    const oceansim_baro_params &q = *params;
    if (!(std::isfinite(q.p_atm) && std::isfinite(q.rho) && std::isfinite(q.g) && std::isfinite(q.sigma) &&
          q.rho >= 0.0 && q.g >= 0.0 && q.sigma >= 0.0))
        return fail(OCEANSIM_E_INVALID_ARG, "barometer parameters must be finite, rho, g and sigma >= 0");
    if (n == 0) return ok();
    BaroDev p{q.p_atm, q.rho * q.g, q.sigma, q.seed_lo, q.seed_hi};
    const long long per_block = (long long)kNavThreads * kBaroPerThread;
    const long long blocks = (n + per_block - 1) / per_block;
    if (blocks > 0x7fffffffLL) return fail(OCEANSIM_E_UNSUPPORTED, "too many samples");
    hipStream_t st = static_cast<hipStream_t>(stream);
    OSIM_LAUNCH("k_baro", k_baro, dim3((unsigned)blocks), dim3(kNavThreads), 0, st, gcast(depth_dev), (long long)n,
                p, gcast(pressure_dev));
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? ok() : hip_fail(e, "barometer launch");
}

int oceansim_dvl(const double *t_dev, const float *ranges_dev, const float *velocity_dev, int32_t n_ticks,
                 int32_t n_inst, const oceansim_dvl_params *params, float *velocity_out_dev, int32_t *status_dev,
                 void *stream) {
    if (!params) return fail(OCEANSIM_E_INVALID_ARG, "params is NULL");
    if (n_ticks < 0 || n_inst < 0) return fail(OCEANSIM_E_SHAPE, "n_ticks and n_inst must be >= 0");
    if ((long long)n_ticks * n_inst == 0) return ok();
    if (!t_dev || !ranges_dev || !velocity_dev || !velocity_out_dev || !status_dev)
        return fail(OCEANSIM_E_INVALID_ARG, "NULL buffer");
    if (!aligned_to(t_dev, 8) || !aligned_to(ranges_dev, 16) || !aligned_to(velocity_dev, 4) ||
        !aligned_to(velocity_out_dev, 4) || !aligned_to(status_dev, 4))
        return fail(OCEANSIM_E_INVALID_ARG, "misaligned buffer (ranges 16-byte, times 8-byte aligned)");
    const oceansim_dvl_params &q = *params;
    if (!(q.janus_angle > 0.0 && q.janus_angle < 1.5707963267948966))
        return fail(OCEANSIM_E_INVALID_ARG, "janus_angle must be in (0, pi/2)");
    if (!(std::isfinite(q.range_min) && std::isfinite(q.range_max) && q.range_min >= 0.0 &&
          q.range_max >= q.range_min))
        return fail(OCEANSIM_E_INVALID_ARG, "need finite 0 <= range_min <= range_max");
    if (q.min_beams != 3 && q.min_beams != 4)
        return fail(OCEANSIM_E_INVALID_ARG, "min_beams must be 3 or 4 (a velocity needs three beams)");
    if (!(std::isfinite(q.sigma_v) && q.sigma_v >= 0.0 && q.sound_speed > 0.0 && std::isfinite(q.sound_speed) &&
          q.pings_per_output > 0.0 && std::isfinite(q.pings_per_output) && q.period_min >= 0.0 &&
          std::isfinite(q.period_min)))
        return fail(OCEANSIM_E_INVALID_ARG, "sigma_v, sound_speed, pings_per_output, period_min out of range");
    DvlDev p;
    for (int i = 0; i < 4; ++i) {
        const double psi = 0.7853981633974483 + 1.5707963267948966 * i;
        p.beam[i][0] = std::sin(q.janus_angle) * std::cos(psi);
        p.beam[i][1] = std::sin(q.janus_angle) * std::sin(psi);
        p.beam[i][2] = -std::cos(q.janus_angle);
    }
    p.range_min = q.range_min;
    p.range_max = q.range_max;
    p.sigma_v = q.sigma_v;
    p.pings_per_output = q.pings_per_output;
    p.sound_speed = q.sound_speed;
    p.period_min = q.period_min;
    p.min_beams = q.min_beams;
    p.seed_lo = q.seed_lo;
    p.seed_hi = q.seed_hi;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool walk = dvl_walks(n_ticks, n_inst);
    const int per_block = walk ? kNavThreads : kDvlInst;
    const int blocks = (int)(((long long)n_inst + per_block - 1) / per_block);
    OSIM_LAUNCH("k_dvl", walk ? k_dvl_walk : k_dvl, dim3(blocks), dim3(walk ? kNavThreads : kDvlThreads), 0, st,
                gcast(t_dev), gcast(reinterpret_cast<const float4 *>(ranges_dev)), gcast(velocity_dev), (int)n_ticks,
                (int)n_inst, p, gcast(velocity_out_dev), gcast(status_dev));
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? ok() : hip_fail(e, "dvl launch");
}

}  // extern "C"
