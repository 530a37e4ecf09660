// Monte Carlo verification of a plan (Sec. 3, final phase; the system and
// localisation models of Sec. 4.1): many sampled flights of the plan, each a
// double integrator tracking the nominal trajectory with an LQR controller
// while a Kalman filter fuses a noisy accelerometer with position fixes taken
// where the mapped features are good enough.  Float64 state, counter-based
// normals (Philox4x32-10), blobs and boxes in LDS, one to sixteen lanes per
// flight (k_mc_rollout).
//
// The model, fixed where the paper gives only its structure:
//  * nominal: per edge the minimum-energy cubic between its two states --
//    2D/3D roadmaps: from rest to rest over 1.5 length / speed (peak speed
//    `speed`); 6D: the roadmap's states over the steering time (the
//    fixed-time minimum-energy trajectory); with velocity and acceleration;
//    samples at t_k = k dt, k = 0..K, K = ceil(duration / dt), clamped;
//  * per axis x = (p, v), x' = A x + B a, A = [[1, dt], [0, 1]],
//    B = [dt^2 / 2, dt]; applied a = u + sigma_w xi;
//  * u = (v_nom,k+1 - v_nom,k) / dt - k_p (p_hat - p_nom) - k_v (v_hat - v_nom):
//    the nominal velocity change over the step as feed-forward, the
//    steady-state discrete LQR gain for Q = diag(q_p, q_v), R = r_u (20,000
//    Riccati steps) as feedback;
//  * Kalman prediction with the measured acceleration a + sigma_a eta and
//    covariance sigma_a^2 B B^T; a position fix z = p + (sigma_v / sqrt(q)) zeta
//    at the new true position when its feature quality q >= q_min;
//  * start: p = p_nom + sigma_0 xi_0, v = v_nom, estimate nominal, covariance
//    diag(sigma_0^2, 0);
//  * per flight: the largest |p - p_hat| over k = 0..K, and whether a true
//    position lies in a closed box.
// Normals: Philox4x32-10 keyed by the seed, counter (step, flight, draw, 0)
// (step 0xffffffff at the start), two 53-bit uniforms per call and the
// Box-Muller pair; per step 3 dim normals in the order xi, eta, zeta.
#include "device_common.h"
#include "runtime_internal.h"

namespace {

constexpr int kMcGainSteps = 20000;
constexpr unsigned kMcStartStep = 0xffffffffu;

// Nominal at one step: position and velocity, and the feed-forward
// acceleration to the next step.
struct McStep {
    double p[3], v[3], ff[3];
};

// (read by uniform addresses: scalar loads)
typedef const __attribute__((address_space(4))) McStep *StepPtr;

struct McNominal {
    int K;
    int dim;       // workspace dimension (2 or 3)
    McStep *step;  // [K+1]
};

__device__ __forceinline__ void philox10(uint32_t c[4], uint32_t k0, uint32_t k1) {
    for (int r = 0; r < 10; ++r) {
        if (r > 0) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        const uint64_t p0 = (uint64_t)0xD2511F53u * c[0];
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c[2];
        const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
        const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
        const uint32_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
        c[0] = n0;
        c[1] = lo1;
        c[2] = n2;
        c[3] = lo0;
    }
}

// two standard normals for counter (step, flight, draw, 0)
__device__ __forceinline__ void normal2(uint32_t k0, uint32_t k1, uint32_t step, uint32_t flight,
                                        uint32_t draw, double &z0, double &z1) {
    uint32_t c[4] = {step, flight, draw, 0u};
    philox10(c, k0, k1);
    const uint64_t a = ((uint64_t)c[0] << 32) | c[1];
    const uint64_t b = ((uint64_t)c[2] << 32) | c[3];
    const double u1 = ((double)(a >> 11) + 0.5) * 0x1p-53;
    const double u2 = ((double)(b >> 11) + 0.5) * 0x1p-53;
    const double r = sqrt(-2.0 * log(u1));
    double sn, cs;
    sincospi(2.0 * u2, &sn, &cs);
    z0 = r * cs;
    z1 = r * sn;
}

// steady-state discrete LQR gain of the per-axis double integrator (one
// thread: a serial chain, 0.12 us a step).  The recursion ends early where a
// step leaves P as it was to the last bit: every later step would repeat it,
// so the gain is that of all kMcGainSteps (at the default weights after 1,274
// steps: 2,460 -> 160 us).
__global__ void k_mc_gain(double dt, double qp, double qv, double ru, double *gain) {
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    const double h = 0.5 * dt * dt;
    double P00 = qp, P01 = 0.0, P11 = qv;
    double kp = 0.0, kv = 0.0;
    for (int it = 0; it <= kMcGainSteps; ++it) {
        // B^T P B, B^T P A
        const double pb0 = P00 * h + P01 * dt, pb1 = P01 * h + P11 * dt;  // P B
        const double S = ru + (h * pb0 + dt * pb1);
        const double ba0 = pb0, ba1 = pb0 * dt + pb1;  // (P B)^T A
        kp = ba0 / S;
        kv = ba1 / S;
        if (it == kMcGainSteps) break;
        // A^T P A
        const double a00 = P00, a01 = P00 * dt + P01, a11 = (P00 * dt + P01) * dt + (P01 * dt + P11);
        // P <- Q + A^T P A - (A^T P B) K
        const double n00 = qp + a00 - ba0 * kp;
        const double n01 = a01 - ba0 * kv;
        const double n11 = qv + a11 - ba1 * kv;
        if (n00 == P00 && n01 == P01 && n11 == P11) break;
        P00 = n00;
        P01 = n01;
        P11 = n11;
    }
    gain[0] = kp;
    gain[1] = kv;
}

// duration and cumulative start time of every plan segment (one thread):
// polyline segments length / speed, or the steering time per edge
__global__ void k_mc_times(int m, int dim, const float *pos, const int *path, double speed,
                           double horizon, double *dur_out, double *tau) {
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    const int pw = dim;
    double t = 0.0;
    tau[0] = 0.0;
    for (int i = 0; i < m; ++i) {
        double dur;
        if (horizon > 0.0) {
            dur = horizon;
        } else {
            double l2 = 0.0;
            for (int k = 0; k < pw; ++k) {
                const double d = (double)pos[(size_t)path[i + 1] * pw + k] -
                                 (double)pos[(size_t)path[i] * pw + k];
                l2 = l2 + d * d;
            }
            dur = 1.5 * sqrt(l2) / speed;
        }
        dur_out[i] = dur;
        t = t + dur;
        tau[i + 1] = t;
    }
}

// nominal position and velocity at step k
__device__ __forceinline__ void nominal_at(int d, int m, const float *pos, const float *vel,
                                           const int *path, const double *dur, const double *tau,
                                           double dt, double horizon, int k, double *pp,
                                           double *vv) {
    const double t = fmin((double)k * dt, tau[m]);
    if (horizon > 0.0) {
        const double T = horizon;
        int i = (int)floor(t / T);
        i = min(max(i, 0), m - 1);
        const double s = t - (double)i * T;
        for (int c = 0; c < d; ++c) {
            const double p0 = pos[(size_t)path[i] * d + c], p1 = pos[(size_t)path[i + 1] * d + c];
            const double v0 = vel[(size_t)path[i] * 3 + c], v1 = vel[(size_t)path[i + 1] * 3 + c];
            const double c2 = (3.0 * (p1 - p0) - (2.0 * v0 + v1) * T) / (T * T);
            const double c3 = (2.0 * (p0 - p1) + (v0 + v1) * T) / (T * T * T);
            pp[c] = p0 + v0 * s + c2 * s * s + c3 * s * s * s;
            vv[c] = v0 + 2.0 * c2 * s + 3.0 * c3 * s * s;
        }
    } else {
        // last segment start <= t (searchsorted right, minus one), clamped
        int lo = 0, hi = m;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (tau[mid] <= t) lo = mid + 1; else hi = mid;
        }
        int i = min(max(lo - 1, 0), m - 1);
        const double s = t - tau[i];
        const double T = dur[i];
        for (int c = 0; c < d; ++c) {
            const double p0 = pos[(size_t)path[i] * d + c], p1 = pos[(size_t)path[i + 1] * d + c];
            const double c2 = (3.0 * (p1 - p0)) / (T * T);
            const double c3 = (2.0 * (p0 - p1)) / (T * T * T);
            pp[c] = p0 + c2 * s * s + c3 * s * s * s;
            vv[c] = 2.0 * c2 * s + 3.0 * c3 * s * s;
        }
    }
}

// the nominal's record of every step (one thread per step; the last step
// has no feed-forward), and 1 / (2 sigma^2) of every blob
__global__ void __launch_bounds__(256) k_mc_nominal(McNominal nm, int m, const float *pos,
                                                    const float *vel, const int *path,
                                                    const double *dur, const double *tau,
                                                    double dt, double horizon, int nblob,
                                                    const float *sig, double *inv2s) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    for (int j = k; j < nblob; j += gridDim.x * blockDim.x) {
        const double s = (double)sig[j];
        inv2s[j] = 1.0 / (2.0 * (s * s));
    }
    if (k > nm.K) return;
    const int d = nm.dim;
    McStep st{};
    double pn[3], vn[3];
    nominal_at(d, m, pos, vel, path, dur, tau, dt, horizon, k, st.p, st.v);
    if (k < nm.K) {
        nominal_at(d, m, pos, vel, path, dur, tau, dt, horizon, k + 1, pn, vn);
        for (int c = 0; c < d; ++c) st.ff[c] = (vn[c] - st.v[c]) / dt;
    }
    nm.step[k] = st;
}

struct McArgs {
    McNominal nm;
    int rollouts;
    double dt, sw, sa, sv, qmin, s0, bound;
    const double *gain;
    uint32_t k0, k1;
    int nblob;
    const float *mu, *sig, *amp;  // [nblob][dim], [nblob], [nblob]
    const double *inv2s;          // [nblob] 1 / (2 sigma^2)
    int nbox;
    const float *blo, *bhi;       // [nbox][dim]
    double *max_err;              // [rollouts]
    uint8_t *collided;            // [rollouts]
    unsigned long long *counts;   // [3]: within bound, collision free, both
    double *err_sum;              // [1]
    double roam;                  // how far an answer "no fix" holds (k_mc_rollout)
};

template <int D>
__device__ __forceinline__ bool in_box(const double (&x)[D], const float *lo, const float *hi) {
    bool in = true;
#pragma unroll
    for (int c = 0; c < D; ++c) in = in && x[c] >= (double)lo[c] && x[c] <= (double)hi[c];
    return in;
}

// sum over the G lanes of a flight
template <int G, typename T>
__device__ __forceinline__ T flight_sum(T v) {
#pragma unroll
    for (int o = 1; o < G; o <<= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Blobs in LDS: the centre, scale2 = log2(e) / (2 sigma^2) and the amplitude
// (the amplitudes of 3D blobs behind the others).
template <int D>
struct BlobLds {
    float *at;
    int n;
    __device__ __forceinline__ void put(int j, const float *mu, float scale2, float amp) const {
        float *b = at + 4 * j;
        for (int c = 0; c < D; ++c) b[c] = mu[c];
        b[D] = scale2;
        if constexpr (D == 2) b[3] = amp;
        else at[4 * n + j] = amp;
    }
    __device__ __forceinline__ void get(int j, float (&mu)[D], float &scale2, float &amp) const {
        const float4 b = *reinterpret_cast<const float4 *>(at + 4 * j);
        mu[0] = b.x;
        mu[1] = b.y;
        if constexpr (D == 2) {
            scale2 = b.z;
            amp = b.w;
        } else {
            mu[2] = b.z;
            scale2 = b.w;
            amp = at[4 * n + j];
        }
    }
};

// Squared distance of a float32 point to a blob.
template <int D>
__device__ __forceinline__ float dist2(const float (&x)[D], const float (&mu)[D]) {
    float d2 = 0.0f;
#pragma unroll
    for (int c = 0; c < D; ++c) {
        const float t = x[c] - mu[c];
        d2 = __builtin_fmaf(t, t, d2);
    }
    return d2;
}

// The quality q(x) in float64, the blobs shared by the flight's lanes.  Four
// blobs a step, so that their exponentials overlap; a step whose terms are
// all below 2^-end (far below the last bit of any q that counts) for every
// flight of the wave is left out (never for a NaN or a distance that float32
// cannot hold).
template <int G, int D>
__device__ __forceinline__ double quality(const double (&x)[D], const float (&xf)[D], int sub,
                                          const BlobLds<D> &bl, const double *inv2s, float end) {
    double acc = 0.0;
    for (int j0 = sub; j0 < bl.n; j0 += 4 * G) {
        float mu[4][D], amp[4];
        bool counts = false;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int j = j0 + i * G;
            float sc;
            bl.get(min(j, bl.n - 1), mu[i], sc, amp[i]);
            if (j >= bl.n) amp[i] = 0.0f;
            const float d2 = dist2<D>(xf, mu[i]);
            counts = counts || !(d2 * sc > end + __builtin_amdgcn_logf(fabsf(amp[i])) && d2 < MPAP_INF);
        }
        if (ballot64(counts) == 0) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            double d2 = 0.0;
#pragma unroll
            for (int c = 0; c < D; ++c) {
                const double t = x[c] - (double)mu[i][c];
                d2 = d2 + t * t;
            }
            const double e = exp(-d2 * inv2s[min(j0 + i * G, bl.n - 1)]);
            acc = acc + (double)amp[i] * e;
        }
    }
    return fmin(fmax(flight_sum<G>(acc), 0.0), 1.0);
}

// One flight per G lanes (neighbours in a wave): every lane carries the whole
// state, and the lanes share the normals of a step (lane i draws Philox call
// i), the blobs and the boxes.  Bound by float64 and transcendental issue
// when flights fill the chip, by the latency of one step's chain when they
// do not, hence G (launch_rollouts).
//
// A step does no more than its outcome needs:
//  * whether a position fix is taken (q >= qmin) is first asked in float32
//    on the hardware exponential.  The float32 sum is off by less than
//    m0 + m1 |x|; where it stays below qmin by that much the answer is
//    known to be no, and only undecided flights evaluate q in float64;
//  * that answer holds for a while: the same sum with every blob moved nearer
//    by `roam` bounds q within roam of x, so while it stays below qmin and
//    every flight of the wave within roam of where it was taken, nothing is
//    evaluated at all;
//  * the boxes within roam are listed (a bit mask per lane) at the same
//    point, and only those are tested until a flight leaves it;
//  * the normals of a fix are drawn only where a flight of the wave takes one.
// Measured, against one thread per flight with every blob in float64 at each
// step and every box tested: 70.2 -> 8.7 ms (3D, 80 blobs, 100 boxes, 100,000
// flights) and 11.9 -> 1.2 ms (2D, 30 blobs, 20 boxes, 4,096 flights).  The
// register budget is two waves per SIMD: three or four spill (8.9 and 11.4 ms).
template <int G, int D>
__global__ void __launch_bounds__(256, 2) k_mc_rollout(McArgs a) {
    extern __shared__ __align__(16) float env[];  // blobs (D + 2 words each), box lo, box hi
    const BlobLds<D> bl{env, a.nblob};
    float *blo = env + a.nblob * (D + 2), *bhi = blo + a.nbox * D;
    for (int i = threadIdx.x; i < a.nblob; i += blockDim.x) {
        const double scale = 0.8493218002880191 / (double)a.sig[i];  // sqrt(log2(e) / 2) / sigma
        bl.put(i, a.mu + i * D, (float)(scale * scale), a.amp[i]);
    }
    for (int i = threadIdx.x; i < a.nbox * D; i += blockDim.x) {
        blo[i] = a.blo[i];
        bhi[i] = a.bhi[i];
    }
    __syncthreads();
    // (by every wave for itself: all the LDS is the blobs' and boxes')
    float m0 = 0.0f, m1 = 0.0f;
    for (int i = lane_id(); i < a.nblob; i += 64) {
        float mu[D], sc, amp;
        bl.get(i, mu, sc, amp);
        // Error of one float32 term 2^-y, y = scale^2 |x - mu|^2: x rounds by
        // 2^-24 |x|, so y is off by 2 sqrt(y) scale |x| 2^-24 + 10 y 2^-24
        // and the term by ln 2 times that (at most 0.72 scale |x| + 4 units
        // of 2^-24) and by 2^-22 of the exponential itself: 0.72 scale |x| +
        // 8 units, and nblob units for the sum.  Twice that is taken.
        m0 += fabsf(amp) * (16.0f + 2.0f * (float)a.nblob) * 0x1p-24f;
        m1 += fabsf(amp) * 2.0f * __builtin_amdgcn_sqrtf(sc) * 0x1p-24f;
    }
    m0 = wave_sum(m0);
    m1 = wave_sum(m1);
    // q < qmin follows from the sum alone only for a positive qmin
    const float qcut = a.qmin > 0.0 ? (float)a.qmin : -MPAP_INF;
    // terms below 2^-62 qmin / nblob do not count
    const float end = a.qmin > 0.0 ? 62.0f + __builtin_amdgcn_logf((float)max(a.nblob, 1)) -
                                         __builtin_amdgcn_logf((float)a.qmin)
                                   : MPAP_INF;

    constexpr int kCalls = (3 * D + 1) / 2;     // Philox calls of a step
    constexpr int kAll = (kCalls + G - 1) / G;  // rounds of them, one call per lane
    constexpr int kMove = (D + G - 1) / G;      // rounds that hold the first 2 D normals
    const int lane = lane_id(), sub = lane % G, lead = lane - sub;
    const int r = blockIdx.x * (256 / G) + threadIdx.x / G;
    // (the lanes of a flight go the same way, and shuffles stay within them)
    const bool live = r < a.rollouts;
    const uint32_t flight = (uint32_t)r;
    const StepPtr steps = (StepPtr)a.nm.step;
    const double dt = a.dt, h = 0.5 * dt * dt;
    const double kp = a.gain[0], kv = a.gain[1];
    double p[D], v[D], ph[D], vh[D], z[kAll][2];
    auto draw = [&](uint32_t step, int first, int last) {
#pragma unroll
        for (int q = 0; q < kAll; ++q)
            if (q >= first && q < last)
                normal2(a.k0, a.k1, step, flight, (uint32_t)min(q * G + sub, kCalls - 1), z[q][0],
                        z[q][1]);
    };
    // normal i of the step: from lane (i / 2) mod G of the flight
    auto normal = [&](int i) -> double {
        const int call = i >> 1;
        const double own = z[call / G][i & 1];
        if constexpr (G == 1) return own;
        else return __shfl(own, lead + call % G, 64);
    };
    draw(kMcStartStep, 0, kMove);
    double e2 = 0.0;
#pragma unroll
    for (int c = 0; c < D; ++c) {
        p[c] = steps[0].p[c] + a.s0 * normal(c);
        v[c] = steps[0].v[c];
        ph[c] = steps[0].p[c];
        vh[c] = steps[0].v[c];
        const double e = p[c] - ph[c];
        e2 = e2 + e * e;
    }
    double P00 = a.s0 * a.s0, P01 = 0.0, P11 = 0.0;
    double merr = sqrt(e2);
    bool hit = false;
    for (int j = sub; j < a.nbox; j += G) hit = hit || in_box<D>(p, blo + j * D, bhi + j * D);
    const double qa = a.sa * a.sa;
    float at[D];            // where the box list and the last bound were taken
    bool holds = false;     // the bound rules out a fix within roam of there
    uint64_t near0 = 0, near1 = 0;  // boxes sub + i G within roam of there, i < 128
    // (finite, so that every flight is beyond it at first)
    const float roam = (float)a.roam, roam2 = fminf(0.98f * roam * roam, __FLT_MAX__);
#pragma unroll
    for (int c = 0; c < D; ++c) at[c] = MPAP_INF;
    for (int k = 0; k < a.nm.K; ++k) {
        draw((uint32_t)k, 0, kMove);
#pragma unroll
        for (int c = 0; c < D; ++c) {
            const double u = steps[k].ff[c] - kp * (ph[c] - steps[k].p[c]) -
                             kv * (vh[c] - steps[k].v[c]);
            const double acc = u + a.sw * normal(c);
            p[c] = p[c] + v[c] * dt + h * acc;
            v[c] = v[c] + dt * acc;
            const double am = acc + a.sa * normal(D + c);
            ph[c] = ph[c] + vh[c] * dt + h * am;
            vh[c] = vh[c] + dt * am;
        }
        const double n00 = P00 + 2.0 * dt * P01 + dt * dt * P11 + qa * h * h;
        const double n01 = P01 + dt * P11 + qa * h * dt;
        const double n11 = P11 + qa * dt * dt;
        P00 = n00;
        P01 = n01;
        P11 = n11;
        // is a fix possible?  (the negated comparisons are also true for NaN)
        float xf[D], xs = 0.0f;
#pragma unroll
        for (int c = 0; c < D; ++c) {
            xf[c] = (float)p[c];
            xs += fabsf(xf[c]);
        }
        const float marg = m0 + m1 * xs;
        if (ballot64(live && !(dist2<D>(xf, at) <= roam2))) {
            // (reach: and the roundings of x)
            const float reach = roam + xs * 0x1p-21f;
            float fu = 0.0f;
#pragma unroll 4
            for (int j = sub; j < a.nblob; j += G) {
                float mu[D], sc, amp;
                bl.get(j, mu, sc, amp);
                const float d = fmaxf(__builtin_amdgcn_sqrtf(dist2<D>(xf, mu)) - reach, 0.0f);
                fu = __builtin_fmaf(fmaxf(amp, 0.0f), __builtin_amdgcn_exp2f(-(d * d * sc)), fu);
            }
            holds = flight_sum<G>(fu) + marg < qcut;
            near0 = near1 = 0;
            const int n1 = min(a.nbox, 128 * G);
#pragma unroll 4
            for (int j = sub, i = 0; j < n1; j += G, ++i) {
                bool in = true;
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    const float lo = blo[j * D + c], hi = bhi[j * D + c];
                    const float w = reach + (fabsf(lo) + fabsf(hi)) * 0x1p-21f;
                    in = in && !(xf[c] < lo - w) && !(xf[c] > hi + w);
                }
                const uint64_t bit = in ? 1ull << (i & 63) : 0ull;
                if (i < 64) near0 |= bit;
                else near1 |= bit;
            }
#pragma unroll
            for (int c = 0; c < D; ++c) at[c] = xf[c];
        }
        if (ballot64(live && !holds)) {
            float fq = 0.0f;
#pragma unroll 4
            for (int j = sub; j < a.nblob; j += G) {
                float mu[D], sc, amp;
                bl.get(j, mu, sc, amp);
                fq = __builtin_fmaf(amp, __builtin_amdgcn_exp2f(-(dist2<D>(xf, mu) * sc)), fq);
            }
            fq = flight_sum<G>(fq);
            const bool maybe = live && !(fq + marg < qcut);
            if (ballot64(maybe)) {
                const double q = quality<G, D>(p, xf, sub, bl, a.inv2s, end);
                const bool fix = maybe && q >= a.qmin;
                if (ballot64(fix)) {
                    draw((uint32_t)k, kMove, kAll);
                    double zf[D];
#pragma unroll
                    for (int c = 0; c < D; ++c) zf[c] = normal(2 * D + c);
                    if (fix) {
                        const double Rv = a.sv * a.sv / q;
                        const double sd = a.sv / sqrt(q);
                        const double S = P00 + Rv;
                        const double K0 = P00 / S, K1 = P01 / S;
#pragma unroll
                        for (int c = 0; c < D; ++c) {
                            const double zp = p[c] + sd * zf[c];
                            const double innov = zp - ph[c];
                            ph[c] = ph[c] + K0 * innov;
                            vh[c] = vh[c] + K1 * innov;
                        }
                        const double u00 = (1.0 - K0) * P00, u01 = (1.0 - K0) * P01,
                                     u11 = P11 - K1 * P01;
                        P00 = u00;
                        P01 = u01;
                        P11 = u11;
                    }
                }
            }
        }
        e2 = 0.0;
#pragma unroll
        for (int c = 0; c < D; ++c) {
            const double e = p[c] - ph[c];
            e2 = e2 + e * e;
        }
        merr = fmax(merr, sqrt(e2));
        uint64_t m0n = near0, m1n = near1;
        while (m0n | m1n) {
            int i;
            if (m0n) {
                i = (int)__ffsll((unsigned long long)m0n) - 1;
                m0n &= m0n - 1;
            } else {
                i = 63 + (int)__ffsll((unsigned long long)m1n);
                m1n &= m1n - 1;
            }
            const int j = sub + i * G;
            hit = hit || in_box<D>(p, blo + j * D, bhi + j * D);
        }
        for (int j = sub + 128 * G; j < a.nbox; j += G)
            hit = hit || in_box<D>(p, blo + j * D, bhi + j * D);
    }
    hit = flight_sum<G>(hit ? 1 : 0) != 0;
    const bool first = live && sub == 0;
    bool within = false, free = false;
    if (first) {
        a.max_err[r] = merr;
        a.collided[r] = hit ? 1 : 0;
        within = merr <= a.bound;
        free = !hit;
    }
    // counts and the sum of the largest errors, one atomic per wave
    const unsigned long long bw = __popcll(ballot64(within)), bf = __popcll(ballot64(free)),
                             bb = __popcll(ballot64(within && free));
    const double es = wave_sum(first ? merr : 0.0);
    if (lane_id() == 0) {
        atomicAdd(&a.counts[0], bw);
        atomicAdd(&a.counts[1], bf);
        atomicAdd(&a.counts[2], bb);
        atomicAdd(a.err_sum, es);
    }
}

// Lanes per flight.  Few flights leave SIMDs idle, so a flight is spread over
// lanes until the chip holds about two waves per SIMD (131,072 lanes); with
// more flights the repeated state update costs more than the shorter chain
// gains.  Measured on the 3D plan (988 steps), lanes 16 / 8 / 4 / 2 / 1:
// 4,096 flights 1.87 / 2.05 / 2.55 / 4.14 / 6.55 ms; 8,192: 2.46 / 2.07 / 2.59;
// 32,768: - / 4.74 / 3.38 / 4.22 / 6.54; 65,536: - / - / 6.01 / 5.65 / 6.76;
// 100,000: - / - / 9.74 / 9.92 / 8.66.
template <int D>
void launch_rollouts(const McArgs &a, size_t lds, hipStream_t s) {
    const int R = a.rollouts;
    if (R <= 4096) k_mc_rollout<16, D><<<div_up(R, 16), 256, lds, s>>>(a);
    else if (R <= 8192) k_mc_rollout<8, D><<<div_up(R, 32), 256, lds, s>>>(a);
    else if (R <= 32768) k_mc_rollout<4, D><<<div_up(R, 64), 256, lds, s>>>(a);
    else if (R <= 65536) k_mc_rollout<2, D><<<div_up(R, 128), 256, lds, s>>>(a);
    else k_mc_rollout<1, D><<<div_up(R, 256), 256, lds, s>>>(a);
}

}  // namespace

extern "C" int mpap_mc_verify(const mpap_graph *g, const int32_t *nodes, int32_t n_nodes,
                              const mpap_mc_params *mp, void *stream, double *max_err,
                              uint8_t *collided, mpap_mc_stats *out) {
    if (!g || !nodes || !mp || !out) return fail(MPAP_ERR_INVAL, "null graph, plan, params or output");
    if (!g->pos || (g->dim != 2 && g->dim != 3 && g->dim != 6) || g->nq != 1)
        return fail(MPAP_ERR_INVAL, "a roadmap built by mpap_build_graph (one query)");
    if (mp->rollouts < 1) return fail(MPAP_ERR_INVAL, "rollouts must be >= 1");
    const float fpos[] = {mp->dt, mp->speed, mp->sigma_v, mp->r_u};
    for (float x : fpos)
        if (!(x > 0.0f) || !std::isfinite(x)) return fail(MPAP_ERR_INVAL, "dt, speed, sigma_v, r_u must be > 0");
    const float fnn[] = {mp->sigma_w, mp->sigma_a, mp->sigma0, mp->q_p, mp->q_v, mp->err_bound,
                         mp->q_min};
    for (float x : fnn)
        if (!(x >= 0.0f) || !std::isfinite(x))
            return fail(MPAP_ERR_INVAL, "noise levels, weights, bound and q_min must be >= 0");
    if (n_nodes < 2) return fail(MPAP_ERR_INVAL, "the plan has no edge");
    for (int32_t i = 0; i < n_nodes; ++i)
        if (nodes[i] < 0 || nodes[i] >= g->n) return fail(MPAP_ERR_INVAL, "plan node out of range");
    const int len = n_nodes;
    const int32_t *path_h = nodes;
    const int m = len - 1;
    const int d = g->dim == 6 ? 3 : g->dim;
    const double dt = mp->dt, speed = mp->speed;
    const double horizon = g->dim == 6 ? (double)g->horizon : 0.0;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    int *d_path = nullptr;
    double *segdur = nullptr;
    double *tau = nullptr, *gain = nullptr, *merr = nullptr, *esum = nullptr,
           *inv2s = nullptr;
    McStep *steps = nullptr;
    uint8_t *col = nullptr;
    unsigned long long *cnt = nullptr;
    auto cleanup = [&]() {
        dfree(d_path); dfree(segdur); dfree(tau); dfree(gain); dfree(steps); dfree(inv2s); dfree(merr);
        dfree(esum); dfree(col); dfree(cnt);
    };
    int rc;
    if ((rc = dalloc(&d_path, len)) || (rc = dalloc(&segdur, m)) || (rc = dalloc(&tau, m + 1)) ||
        (rc = dalloc(&gain, 2))) {
        cleanup();
        return rc;
    }
    HIP_TRY(hipMemcpyAsync(d_path, path_h, sizeof(int32_t) * len, hipMemcpyHostToDevice, s));
    k_mc_times<<<1, 64, 0, s>>>(m, d, g->pos, d_path, speed, horizon, segdur, tau);
    double total = 0.0;
    HIP_TRY(hipMemcpyAsync(&total, tau + m, sizeof(double), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    // (the gain's chain runs while the host sizes and allocates the rest)
    k_mc_gain<<<1, 64, 0, s>>>(dt, (double)mp->q_p, (double)mp->q_v, (double)mp->r_u, gain);
    const double kd = std::ceil(total / dt);
    if (!(kd < 1e8)) {
        cleanup();
        return fail(MPAP_ERR_INVAL, "the plan needs more than 1e8 time steps");
    }
    const int K = std::max(1, (int)kd);
    const int R = mp->rollouts;
    if ((rc = dalloc(&steps, (size_t)K + 1)) || (rc = dalloc(&inv2s, g->nblob)) || (rc = dalloc(&merr, R)) ||
        (rc = dalloc(&col, R)) || (rc = dalloc(&cnt, 3)) || (rc = dalloc(&esum, 1))) {
        cleanup();
        return rc;
    }
    McNominal nm{K, d, steps};
    k_mc_nominal<<<div_up(K + 1, 256), 256, 0, s>>>(nm, m, g->pos, g->vel, d_path, segdur, tau,
                                                     dt, horizon, g->nblob, g->bsig, inv2s);
    k_zero_i32<<<1, 64, 0, s>>>(reinterpret_cast<int *>(cnt), 6);
    k_zero_i32<<<1, 64, 0, s>>>(reinterpret_cast<int *>(esum), 2);
    McArgs a{};
    a.nm = nm;
    a.rollouts = R;
    a.dt = dt;
    a.sw = mp->sigma_w; a.sa = mp->sigma_a; a.sv = mp->sigma_v; a.qmin = mp->q_min;
    a.s0 = mp->sigma0; a.bound = mp->err_bound;
    a.gain = gain;
    a.k0 = (uint32_t)(mp->seed & 0xffffffffu);
    a.k1 = (uint32_t)(mp->seed >> 32);
    a.nblob = g->nblob; a.mu = g->bmu; a.sig = g->bsig; a.amp = g->bamp; a.inv2s = inv2s;
    a.nbox = g->nbox; a.blo = g->blo; a.bhi = g->bhi;
    a.max_err = merr; a.collided = col; a.counts = cnt; a.err_sum = esum;
    // eight steps at full speed
    a.roam = 8.0 * dt * (horizon > 0.0 ? 1.0 : speed);
    const size_t lds = sizeof(float) * ((size_t)g->nblob * (d + 2) + (size_t)g->nbox * 2 * d);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    HIP_TRY(hipEventCreate(&e0));
    HIP_TRY(hipEventCreate(&e1));
    HIP_TRY(hipEventRecord(e0, s));
    if (d == 2) launch_rollouts<2>(a, lds, s);
    else launch_rollouts<3>(a, lds, s);
    HIP_TRY(hipEventRecord(e1, s));
    HIP_TRY(hipGetLastError());
    unsigned long long hc[3] = {0, 0, 0};
    double hs = 0.0, hg[2] = {0, 0};
    HIP_TRY(hipMemcpyAsync(hc, cnt, sizeof(hc), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipMemcpyAsync(&hs, esum, sizeof(double), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipMemcpyAsync(hg, gain, sizeof(hg), hipMemcpyDeviceToHost, s));
    if (max_err) HIP_TRY(hipMemcpyAsync(max_err, merr, sizeof(double) * R, hipMemcpyDeviceToHost, s));
    if (collided) HIP_TRY(hipMemcpyAsync(collided, col, R, hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    float ms = 0.f;
    HIP_TRY(hipEventElapsedTime(&ms, e0, e1));
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    // the largest error over all flights (host, from the per-flight values
    // when they were asked for; else a device pass would be needed)
    double mx = 0.0;
    if (max_err)
        for (int i = 0; i < R; ++i) mx = std::max(mx, max_err[i]);
    out->rollouts = R;
    out->within_bound = (int64_t)hc[0];
    out->collision_free = (int64_t)hc[1];
    out->success = (int64_t)hc[2];
    out->steps = K;
    out->duration = total;
    out->mean_max_err = hs / R;
    out->max_max_err = max_err ? mx : -1.0;
    out->gain_p = hg[0];
    out->gain_v = hg[1];
    out->gpu_ms = ms;
    cleanup();
    return MPAP_OK;
}
