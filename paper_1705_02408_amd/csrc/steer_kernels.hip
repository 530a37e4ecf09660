// Double-integrator roadmap on the GPU (the state space of the quadrotor
// experiments, Sec. 4.1 and Sec. 5: position and velocity in 3D), built as
// BuildGraph does (Sec. 3, Alg. 2) with a steering cost for the neighbour
// relation, plus the per-edge drift inputs of the perception heuristic
// (Alg. 1 step 2).
//
// Steering (u -> v) is the minimum-energy control of p'' = a over the fixed
// time T: per axis, with a = (p_v - p_u) - v_u T and b = v_v - v_u, the control
// c0 + c1 t with c0 = 6a/T^2 - 2b/T and c1 = (6bT - 12a)/T^3, of energy
// J = 12a^2/T^3 - 12ab/T^2 + 4b^2/T (summed over the axes: the edge cost).
// The trajectory is checked at t_k = (k T)/K, k = 0..K: in the closed unit
// cube, in no closed box, speed at most 1.  Each state keeps the k_out
// reachable targets of least (J, id).  All of it in float32 with every
// operation rounded separately (-ffp-contract=off, correctly rounded
// division), so selection is reproducible bit for bit by any IEEE evaluation
// in the same order.
#include "device_common.h"
#include "graph_kernels.h"
#include "steer_kernels.h"

namespace {

__device__ __forceinline__ void load3(const float *a, int i, float *x) {
    x[0] = a[3 * i];
    x[1] = a[3 * i + 1];
    x[2] = a[3 * i + 2];
}

// energy J and control coefficients of the steer p0,v0 -> p1,v1 in time T
__device__ __forceinline__ float steer3(const float *p0, const float *v0, const float *p1,
                                        const float *v1, float T, float *c0, float *c1) {
    const float T2 = T * T, T3 = T2 * T;
    float ja[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float a = (p1[k] - p0[k]) - v0[k] * T;
        const float b = v1[k] - v0[k];
        ja[k] = ((12.0f * a) * a) / T3 - ((12.0f * a) * b) / T2 + ((4.0f * b) * b) / T;
        c0[k] = (6.0f * a) / T2 - (2.0f * b) / T;
        c1[k] = ((6.0f * b) * T - 12.0f * a) / T3;
    }
    return (ja[0] + ja[1]) + ja[2];
}

__device__ __forceinline__ float steer_cost(const float *p0, const float *v0, const float *p1,
                                            const float *v1, float T) {
    const float T2 = T * T, T3 = T2 * T;
    float ja[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float a = (p1[k] - p0[k]) - v0[k] * T;
        const float b = v1[k] - v0[k];
        ja[k] = ((12.0f * a) * a) / T3 - ((12.0f * a) * b) / T2 + ((4.0f * b) * b) / T;
    }
    return (ja[0] + ja[1]) + ja[2];
}

// The same cost for a steering time whose powers are powers of two: the
// quotients are then exact products with r1 = 1/T, r2 = 1/T^2, r3 = 1/T^3
// (or round once, below the normal range, as the quotients do).
__device__ __forceinline__ float steer_cost_scaled(const float *p0, const float *v0,
                                                   const float *p1, const float *v1, float T,
                                                   float r1, float r2, float r3) {
    float ja[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float a = (p1[k] - p0[k]) - v0[k] * T;
        const float b = v1[k] - v0[k];
        ja[k] = ((12.0f * a) * a) * r3 - ((12.0f * a) * b) * r2 + ((4.0f * b) * b) * r1;
    }
    return (ja[0] + ja[1]) + ja[2];
}

// position and velocity on the steered trajectory at time t (Horner order)
__device__ __forceinline__ void traj_at(const float *p0, const float *v0, const float *c0,
                                        const float *c1, float t, float *p, float *v) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float h2 = c0[k] * 0.5f, h3 = c1[k] / 6.0f, g1 = c1[k] * 0.5f;
        p[k] = p0[k] + t * (v0[k] + t * (h2 + t * h3));
        if (v) v[k] = v0[k] + t * (c0[k] + t * g1);
    }
}

__device__ __forceinline__ float check_time(int k, float T, int K) {
    return ((float)k * T) / (float)K;
}

// float order -> unsigned order (J + 0 turns -0 into +0)
__device__ __forceinline__ uint32_t ukey(float J) {
    const uint32_t b = __float_as_uint(J + 0.0f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float unkey(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

__device__ __forceinline__ float wave_max_f(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

// Reachability of the steer u -> v, decided by one wave (every lane returns
// the result).  sblo/sbhi: the boxes in LDS; wlist: per-wave LDS scratch of
// nbox ints.
__device__ bool wave_reachable(const SteerArgs &a, const float *p0, const float *v0, int v,
                               const float *sblo, const float *sbhi, int *wlist) {
    const int l = lane_id();
    float p1[3], v1[3], c0[3], c1[3];
    load3(a.pos, v, p1);
    load3(a.vel, v, v1);
    (void)steer3(p0, v0, p1, v1, a.T, c0, c1);
    float pts[4][3];
    bool ok = true;
    float lo[3] = {MPAP_INF, MPAP_INF, MPAP_INF}, hi[3] = {-MPAP_INF, -MPAP_INF, -MPAP_INF};
    int np = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int k = l + 64 * i;
        if (k <= a.K) {
            float p[3], vv[3];
            traj_at(p0, v0, c0, c1, check_time(k, a.T, a.K), p, vv);
            const float sp = (vv[0] * vv[0] + vv[1] * vv[1]) + vv[2] * vv[2];
            ok = ok && sp <= 1.0f;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                ok = ok && p[d] >= 0.0f && p[d] <= 1.0f;
                pts[i][d] = p[d];
                lo[d] = fminf(lo[d], p[d]);
                hi[d] = fmaxf(hi[d], p[d]);
            }
            np = i + 1;
        }
    }
    if (ballot64(!ok)) return false;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        lo[d] = wave_min(lo[d]);
        hi[d] = wave_max_f(hi[d]);
    }
    // boxes that meet the bounding box of the points
    int nl = 0;
    for (int j0 = 0; j0 < a.nbox; j0 += 64) {
        const int j = j0 + l;
        bool m = false;
        if (j < a.nbox)
            m = hi[0] >= sblo[3 * j] && lo[0] <= sbhi[3 * j] && hi[1] >= sblo[3 * j + 1] &&
                lo[1] <= sbhi[3 * j + 1] && hi[2] >= sblo[3 * j + 2] && lo[2] <= sbhi[3 * j + 2];
        const uint64_t bm = ballot64(m);
        if (m) wlist[nl + lanes_below(bm)] = j;
        nl += (int)__popcll(bm);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    bool hit = false;
    for (int i = 0; i < nl; ++i) {
        const int j = wlist[i];
        const float bl0 = sblo[3 * j], bl1 = sblo[3 * j + 1], bl2 = sblo[3 * j + 2];
        const float bh0 = sbhi[3 * j], bh1 = sbhi[3 * j + 1], bh2 = sbhi[3 * j + 2];
#pragma unroll
        for (int qi = 0; qi < 4; ++qi)
            if (qi < np)
                hit = hit || (pts[qi][0] >= bl0 && pts[qi][0] <= bh0 && pts[qi][1] >= bl1 &&
                              pts[qi][1] <= bh1 && pts[qi][2] >= bl2 && pts[qi][2] <= bh2);
    }
    const bool clear = ballot64(hit) == 0;
    __builtin_amdgcn_wave_barrier();  // wlist is reused by the next call
    return clear;
}

// LDS writes of the wave's lanes visible to its other lanes
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The bin (of 2048) where the running count of hist first reaches need
// (1-based); sres[0] = bin, sres[1] = count below it.  Every thread calls.
__device__ void find_bin(const int *hist, int need, int *scratch, int *sres) {
    const int t = threadIdx.x;
    int loc = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) loc += hist[8 * t + i];
    int total;
    const int ex = block_excl_scan(loc, scratch, &total);
    if (ex < need && need <= ex + loc) {
        int c = ex;
        for (int i = 0; i < 8; ++i) {
            const int h = hist[8 * t + i];
            if (c + h >= need) {
                sres[0] = 8 * t + i;
                sres[1] = c;
                break;
            }
            c += h;
        }
    }
    __syncthreads();
}

// A source's search ball in the grid: c is p_u + v_u T from the grid's corner,
// far2 the squared distance from there to the farthest position.
struct Ball {
    float c[3], reach, far2, h;
};
__device__ __forceinline__ Ball make_ball(const SteerArgs &a, const GridArgs &gr, const float *p0,
                                          const float *v0, const SteerBounds &sb) {
    Ball b;
    b.reach = sb.extent;
    b.far2 = 0.0f;
    b.h = 1.0f / gr.inv;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        b.c[k] = (p0[k] - gr.lo[k]) + v0[k] * a.T;
        b.reach += fabsf(v0[k]) * a.T;
        const float d = fmaxf(fabsf(b.c[k]), fabsf((sb.phi[k] - sb.plo[k]) - b.c[k]));
        b.far2 += d * d;
    }
    return b;
}

// Radius that holds every target of J <= tau (see k_steer_near); a ball of
// squared radius b.far2 or more holds every position.
__device__ __forceinline__ float ball_radius(const Ball &b, float T, float tau) {
    return sqrtf(tau * (T * T * T) * (1.0f / 3.0f)) * 1.0005f + 1e-6f * b.reach + 1e-3f * b.h;
}

// The ball of every target whose speed can be within the limit at the check
// time nearest T/2: there v = h (p1 - p0)/T + h10' v0 + h11' v1 (derivative of
// the Hermite cubic, h = h01'), so |v| <= 1 keeps p1 within sb.rho =
// (T/h)(1 + |h11'| max |v1|) of p0 - (T h10'/h) v0 (sb.vr = T h10'/h).
__device__ __forceinline__ Ball speed_ball(const Ball &b, const GridArgs &gr, const float *p0,
                                           const float *v0, const SteerBounds &sb, float &radius) {
    Ball s = b;
#pragma unroll
    for (int k = 0; k < 3; ++k) s.c[k] = (p0[k] - gr.lo[k]) - sb.vr * v0[k];
    radius = sb.rho * 1.0005f + 1e-6f * b.reach + 1e-3f * b.h;
    return s;
}

// f(first, last) for the run of sorted states in each row of cells that meets
// the ball (every row where all is set); rows are dealt out to `groups` callers
template <class F>
__device__ __forceinline__ void for_ball_rows(const GridArgs &gr, const Ball &b, float R, bool all,
                                              int group, int groups, F f) {
    const int gd[3] = {gr.gx, gr.gy, gr.gz};
    int lo[3], hi[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float top = (float)(gd[k] - 1);
        lo[k] = all ? 0 : (int)fminf(fmaxf(floorf((b.c[k] - R) * gr.inv), 0.0f), top);
        hi[k] = all ? gd[k] - 1 : (int)fminf(fmaxf(floorf((b.c[k] + R) * gr.inv), 0.0f), top);
    }
    // squared distance of the centre from the slab of cells i on axis k (the
    // border cells hold everything beyond them)
    auto slab2 = [&](int k, int i) -> float {
        const float a0 = (float)i * b.h, a1 = a0 + b.h;
        const float d = fmaxf(i > 0 ? a0 - b.c[k] : 0.0f, i < gd[k] - 1 ? b.c[k] - a1 : 0.0f);
        return d > 0.0f ? d * d : 0.0f;
    };
    const int ny = hi[1] - lo[1] + 1, rows = (hi[2] - lo[2] + 1) * ny;
    for (int q = group; q < rows; q += groups) {
        const int z = lo[2] + q / ny, y = lo[1] + q % ny;
        int x0 = lo[0], x1 = hi[0];
        if (!all) {
            const float rem = R * R - slab2(2, z) - slab2(1, y);
            if (rem < 0.0f) continue;
            const float hx = sqrtf(rem) * 1.0001f + 1e-3f * b.h, top = (float)(gr.gx - 1);
            x0 = max(x0, (int)fminf(fmaxf(floorf((b.c[0] - hx) * gr.inv), 0.0f), top));
            x1 = min(x1, (int)fminf(fmaxf(floorf((b.c[0] + hx) * gr.inv), 0.0f), top));
        }
        const int row = (z * gr.gy + y) * gr.gx;
        if (!f(gr.cstart[row + x0], gr.cstart[row + x1] + gr.ccount[row + x1])) return;
    }
}

// Can no target at all be reached from (p0, v0)?  At check time t the
// position is h00 p0 + h10 T v0 + h01 p1 + h11 T v1 (cubic Hermite basis in
// t/T), so over all targets of the bounding boxes of positions and velocities
// it stays in a small interval on each axis while t is small; if that lies
// outside the cube, or inside a box, at some check time, every trajectory
// fails there.  eps is far above the roundings of a checked point.  (The
// speed at t = 0 is |v0| whatever the target.)  Every lane returns the result.
__device__ bool wave_hopeless(const SteerArgs &a, const SteerBounds &sb, const float *p0,
                              const float *v0, const float *sblo, const float *sbhi) {
    const int l = lane_id();
    bool dead = !((v0[0] * v0[0] + v0[1] * v0[1]) + v0[2] * v0[2] <= 1.0f);
    for (int k0 = 0; k0 <= a.K; k0 += 64) {
        const int k = k0 + l;
        if (k <= a.K && !dead) {
            const float x = (float)k / (float)a.K, x2 = x * x, x3 = x2 * x;
            const float h00 = 2.0f * x3 - 3.0f * x2 + 1.0f, h10 = (x3 - 2.0f * x2 + x) * a.T;
            const float h01 = 3.0f * x2 - 2.0f * x3, h11 = (x3 - x2) * a.T;  // h01 >= 0 >= h11
            float lo[3], hi[3];
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const float m = h00 * p0[d] + h10 * v0[d];
                lo[d] = m + h01 * sb.plo[d] + h11 * sb.vhi[d] - sb.eps;
                hi[d] = m + h01 * sb.phi[d] + h11 * sb.vlo[d] + sb.eps;
                dead = dead || hi[d] < 0.0f || lo[d] > 1.0f;
            }
            for (int j = 0; j < a.nbox && !dead; ++j)
                dead = lo[0] >= sblo[3 * j] && hi[0] <= sbhi[3 * j] && lo[1] >= sblo[3 * j + 1] &&
                       hi[1] <= sbhi[3 * j + 1] && lo[2] >= sblo[3 * j + 2] &&
                       hi[2] <= sbhi[3 * j + 2];
        }
    }
    return ballot64(dead) != 0;
}

// Per-lane rejections before a trajectory is checked in full: the check
// points k = iK/16 of one candidate per lane against the cube and the speed
// limit (kBoxes false), or against the listed boxes (bounds in nlo / nhi).
// The points and tests are those of the full check, so a rejected candidate
// is unreachable.  (Two passes: the second sees the few that pass the first,
// listed densely.)
template <bool kBoxes>
__device__ __forceinline__ bool quick_inside(const SteerArgs &a, const float *p0, const float *v0,
                                             const float *p1, const float *v1, const float4 *nlo,
                                             const float4 *nhi, int nnear) {
    float c0[3], c1[3];
    (void)steer3(p0, v0, p1, v1, a.T, c0, c1);
    bool ok = true;
#pragma unroll 1
    for (int i = 0; i < 15; ++i) {
        // 8, 4, 12, 2, 6, 10, 14, 1, 3, .., 15
        const int sixteenth = (int)((0xFDB97531EA62C48ull >> (4 * i)) & 15);
        const int k = (sixteenth * a.K) >> 4;
        float p[3], v[3];
        traj_at(p0, v0, c0, c1, check_time(k, a.T, a.K), p, v);
        if constexpr (!kBoxes) {
            ok = ok && (v[0] * v[0] + v[1] * v[1]) + v[2] * v[2] <= 1.0f;
#pragma unroll
            for (int d = 0; d < 3; ++d) ok = ok && p[d] >= 0.0f && p[d] <= 1.0f;
        } else {
            bool in = false;
#pragma unroll 4
            for (int q = 0; q < nnear; ++q) {
                const float4 lo = nlo[q], hi = nhi[q];
                in = in || (p[0] >= lo.x && p[0] <= hi.x && p[1] >= lo.y && p[1] <= hi.y &&
                            p[2] >= lo.z && p[2] <= hi.z);
            }
            ok = ok && !in;
        }
        if (!ballot64(ok)) break;  // (of the lanes that came here)
    }
    return ok;
}

}  // namespace

// One wave per source, in cell order.  The cost J of a target is at least
// 3 |a|^2 / T^3, a = (p_v - p_u) - v_u T, so every target of J <= tau lies in
// the ball of radius sqrt(tau T^3 / 3) about p_u + v_u T (widened by far more
// than the roundings of J, which stay below 1e-5 of it, and of the cells).
// The wave evaluates the states in the cells of that ball, lists those of
// J <= tau0, ranks them by (J, id), and checks them in that order; where most
// were reachable it goes on with the shell up to a larger tau.  Sources that
// find fewer than k_out so are handed to k_steer_far, unless no target can be
// reached at all.
//
// Bound by the evaluation of J (about 3,000 states a source of 50,000) and by
// the checks (45 a source): 1.7 ms for 20,000 states, 3.6 ms for 50,000.
// (Selecting the 64th key among all states by four passes over them, a
// workgroup per source, took 45.9 and 300 ms.)
template <bool kPow2>
__global__ void __launch_bounds__(256) k_steer_near(SteerArgs a, GridArgs gr, SteerBounds sb,
                                                    const float4 *spos, const float4 *svel,
                                                    float tau0, int *nbr, float *ncost, int *ncnt,
                                                    SteerFar far) {
    extern __shared__ __align__(16) unsigned char lds[];
    float *keys = reinterpret_cast<float *>(lds);                  // 4 * kNearList
    int *ids = reinterpret_cast<int *>(keys + 4 * kNearList);      // 4 * kNearList
    float *sblo = reinterpret_cast<float *>(ids + 4 * kNearList);  // 3 * nbox
    float *sbhi = sblo + 3 * a.nbox;
    int *wlist = reinterpret_cast<int *>(sbhi + 3 * a.nbox);       // 4 * nbox
    for (int i = threadIdx.x; i < 3 * a.nbox; i += blockDim.x) {
        sblo[i] = a.blo[i];
        sbhi[i] = a.bhi[i];
    }
    __syncthreads();
    const int l = lane_id();
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int i0 = (int)blockIdx.x * 4 + w;
    if (i0 >= a.n) return;
    keys += w * kNearList;
    ids += w * kNearList;
    wlist += w * a.nbox;
    const float4 pu = spos[i0], vu = svel[i0];
    const int u = __float_as_int(pu.w);
    const float p0[3] = {pu.x, pu.y, pu.z}, v0[3] = {vu.x, vu.y, vu.z};
    const float r1 = 1.0f / a.T, r2 = 1.0f / (a.T * a.T), r3 = 1.0f / (a.T * a.T * a.T);
    const Ball ball = make_ball(a, gr, p0, v0, sb);
    float prev = -MPAP_INF, tau = tau0;
    int found = 0, listed = 0;
    bool ranked = true;
    for (int shell = 0; shell < kNearShells; ++shell) {
        const float R = ball_radius(ball, a.T, tau);
        int cnt = 0;
        for_ball_rows(gr, ball, R, !(R * R < ball.far2), 0, 1, [&](int b, int e) -> bool {
            for (int j0 = b; j0 < e; j0 += 64) {
                const int j = j0 + l;
                bool take = false;
                float J = 0.0f;
                int id = 0;
                if (j < e) {
                    const float4 pv = spos[j], vv = svel[j];
                    const float p1[3] = {pv.x, pv.y, pv.z}, v1[3] = {vv.x, vv.y, vv.z};
                    id = __float_as_int(pv.w);
                    J = kPow2 ? steer_cost_scaled(p0, v0, p1, v1, a.T, r1, r2, r3)
                              : steer_cost(p0, v0, p1, v1, a.T);
                    take = id != u && J > prev && J <= tau;
                }
                const uint64_t m = ballot64(take);
                const int slot = cnt + lanes_below(m);
                if (take && slot < kNearList) {
                    keys[slot] = J;
                    ids[slot] = id;
                }
                cnt += (int)__popcll(m);
                if (cnt > kNearList) return false;
            }
            return true;
        });
        ranked = cnt <= kNearList;
        if (!ranked) break;
        wave_sync();
        // (J, id) order: an entry's place is the number of smaller ones
        int ties = 0;
        float key[kNearList / 64];
        int id[kNearList / 64], rank[kNearList / 64];
#pragma unroll
        for (int t = 0; t < kNearList / 64; ++t) {
            const int i = t * 64 + l;
            rank[t] = -1;
            if (t * 64 < cnt && i < cnt) {
                key[t] = keys[i];
                id[t] = ids[i];
                int r = 0, same = 0;
                for (int j = 0; j < cnt; ++j) {
                    const float kj = keys[j];
                    r += kj < key[t] || (kj == key[t] && ids[j] < id[t]) ? 1 : 0;
                    same += kj == key[t] ? 1 : 0;
                }
                rank[t] = r;
                ties = max(ties, same);
            }
        }
        wave_sync();
#pragma unroll
        for (int t = 0; t < kNearList / 64; ++t)
            if (rank[t] >= 0) {
                keys[rank[t]] = key[t];
                ids[rank[t]] = id[t];
            }
        wave_sync();
        ranked = ballot64(ties > 64) == 0;
        if (!ranked) break;
        for (int i = 0; i < cnt && found < a.k_out; ++i) {
            const int v = __builtin_amdgcn_readfirstlane(ids[i]);
            if (wave_reachable(a, p0, v0, v, sblo, sbhi, wlist)) {
                if (l == 0) {
                    nbr[(size_t)u * a.k_out + found] = v;
                    ncost[(size_t)u * a.k_out + found] = keys[i] + 0.0f;  // -0 as +0
                }
                ++found;
            }
        }
        wave_sync();
        listed += cnt;
        prev = tau;
        // another shell where enough of the listed targets were reachable,
        // as wide as the rest needs at that rate (their number grows as
        // tau^3), a third more
        if (found >= a.k_out || 8 * found < listed) break;
        const float need = (float)(a.k_out - found) * (float)listed / (float)max(found, 1);
        tau *= fminf(cbrtf(1.0f + 1.33f * need / (float)max(listed, 1)), 2.0f);
    }
    if (l == 0) ncnt[u] = ranked ? found : 0;
    if (ranked && found >= a.k_out) return;
    if (ranked && found == 0 && wave_hopeless(a, sb, p0, v0, sblo, sbhi)) return;
    if (l == 0) {
        const int k = atomicAdd(far.count, 1);
        far.source[k] = u;
        far.tau[k] = ranked ? prev : -MPAP_INF;
    }
}

template __global__ void k_steer_near<true>(SteerArgs, GridArgs, SteerBounds, const float4 *,
                                            const float4 *, float, int *, float *, int *, SteerFar);
template __global__ void k_steer_near<false>(SteerArgs, GridArgs, SteerBounds, const float4 *,
                                             const float4 *, float, int *, float *, int *,
                                             SteerFar);

// The sources that k_steer_near did not finish, one workgroup each: shells of
// growing cost until k_out targets are found or every state that the speed
// limit allows has been looked at (about one source in twenty, near a wall or
// a box and heading for it).  Candidates are listed only if they pass
// quick_inside, so that shells can be wide; a shell that lists more than
// kFarList is thinned.  Bound by the quick tests: 3.5 ms for 20,000 states,
// 12 ms for 50,000.  A source whose candidates cannot be
// ranked so (65 and more of one cost in the first shell, shells that stay too
// full, kSteerShells of them) goes on to k_steer_select.
template <bool kPow2>
__global__ void __launch_bounds__(kFarThreads) k_steer_far(SteerArgs a, GridArgs gr, SteerBounds sb,
                                                           const float4 *spos, const float4 *svel,
                                                           float tau0, int *nbr, float *ncost,
                                                           int *ncnt, SteerFar far, int *left,
                                                           int *nleft) {
    constexpr int W = kFarThreads / 64;
    extern __shared__ __align__(16) unsigned char lds[];
    float *sblo = reinterpret_cast<float *>(lds);  // 3 * nbox
    float *sbhi = sblo + 3 * a.nbox;
    int *wlist = reinterpret_cast<int *>(sbhi + 3 * a.nbox);  // W * nbox
    __shared__ float keys[2][kFarList];  // [0]: in the cube; [1]: past the boxes; ranked: [0]
    __shared__ int ids[2][kFarList];
    __shared__ float4 nlo[kSteerNear], nhi[kSteerNear];
    __shared__ int s_cnt, s_past, s_near, s_ties, okf[W];
    for (int i = threadIdx.x; i < 3 * a.nbox; i += blockDim.x) {
        sblo[i] = a.blo[i];
        sbhi[i] = a.bhi[i];
    }
    const int l = lane_id();
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const float r1 = 1.0f / a.T, r2 = 1.0f / (a.T * a.T), r3 = 1.0f / (a.T * a.T * a.T);
    const int sources = *far.count;
    for (int si = blockIdx.x; si < sources; si += gridDim.x) {
        const int u = far.source[si];
        float p0[3], v0[3];
        load3(a.pos, u, p0);
        load3(a.vel, u, v0);
        const Ball ball = make_ball(a, gr, p0, v0, sb);
        float Rs, apart = 0.0f;  // the speed ball's radius; the distance of the two centres
        const Ball sball = speed_ball(ball, gr, p0, v0, sb, Rs);
#pragma unroll
        for (int k = 0; k < 3; ++k)
            apart += (ball.c[k] - sball.c[k]) * (ball.c[k] - sball.c[k]);
        apart = sqrtf(apart) * 1.0005f;
        float prev = far.tau[si], tau = prev > 0.0f ? 1.6f * prev : 0.25f * tau0;
        int found = ncnt[u], thin = 0;
        bool done = false;
        __syncthreads();  // the previous source's lists are done with
        if (threadIdx.x == 0) s_near = 0;
        __syncthreads();
        // boxes that a trajectory meets in its first half at full speed
        for (int j = threadIdx.x; j < a.nbox; j += blockDim.x) {
            bool m = true;
#pragma unroll
            for (int k = 0; k < 3; ++k)
                m = m && p0[k] >= sblo[3 * j + k] - 0.5f * a.T && p0[k] <= sbhi[3 * j + k] + 0.5f * a.T;
            if (!m) continue;
            const int q = atomicAdd(&s_near, 1);
            if (q < kSteerNear) {
                nlo[q] = make_float4(sblo[3 * j], sblo[3 * j + 1], sblo[3 * j + 2], 0.0f);
                nhi[q] = make_float4(sbhi[3 * j], sbhi[3 * j + 1], sbhi[3 * j + 2], 0.0f);
            }
        }
        __syncthreads();
        const int nnear = min(s_near, kSteerNear);
        for (int shell = 0; shell < kSteerShells; ++shell) {
            const bool first = !(prev > -MPAP_INF);
            const float R = ball_radius(ball, a.T, tau);
            // later shells look for reachable targets only: the smaller ball
            // of the two; once the shell's ball holds the other (or every
            // position) the last shell is all the rest
            const bool fast = !first && !(R < Rs);
            const bool all = !(R * R < ball.far2) && !(fast && Rs * Rs < ball.far2);
            if (!first && thin == 0 && (!(R * R < ball.far2) || R >= Rs + apart)) tau = MPAP_INF;
            if (threadIdx.x == 0) {
                s_cnt = 0;
                s_past = 0;
                s_ties = 0;
            }
            __syncthreads();
            for_ball_rows(gr, fast ? sball : ball, fast ? Rs : R, all, w, W, [&](int b, int e) -> bool {
                for (int j0 = b; j0 < e; j0 += 64) {
                    const int j = j0 + l;
                    bool take = false;
                    float J = 0.0f;
                    int id = 0;
                    if (j < e) {
                        const float4 pv = spos[j], vv = svel[j];
                        const float p1[3] = {pv.x, pv.y, pv.z}, v1[3] = {vv.x, vv.y, vv.z};
                        id = __float_as_int(pv.w);
                        J = kPow2 ? steer_cost_scaled(p0, v0, p1, v1, a.T, r1, r2, r3)
                                  : steer_cost(p0, v0, p1, v1, a.T);
                        take = id != u && J > prev && J <= tau;
                        if (take && !first)
                            take = quick_inside<false>(a, p0, v0, p1, v1, nlo, nhi, nnear);
                    }
                    const uint64_t m = ballot64(take);
                    int base = 0;
                    if (l == 0 && m) base = atomicAdd(&s_cnt, (int)__popcll(m));
                    base = __shfl(base, 0, 64);
                    const int slot = base + lanes_below(m);
                    if (take && slot < kFarList) {
                        keys[0][slot] = J;
                        ids[0][slot] = id;
                    }
                    if (base > kFarList) return false;
                }
                return true;
            });
            __syncthreads();
            const int cnt = s_cnt;
            if (cnt > kFarList) {
                // too many: a thinner shell
                const float base = fmaxf(prev, 0.0f);
                tau = tau < MPAP_INF ? base + 0.25f * (tau - base) : 4.0f * fmaxf(base, 1e-30f);
                __syncthreads();
                if (++thin > 24 || !(tau > prev)) break;
                continue;
            }
            for (int i0 = 64 * w; i0 < cnt; i0 += kFarThreads) {
                const int i = i0 + l;
                bool take = i < cnt;
                float J = 0.0f;
                int id = 0;
                if (take) {
                    J = keys[0][i];
                    id = ids[0][i];
                    float p1[3], v1[3];
                    load3(a.pos, id, p1);
                    load3(a.vel, id, v1);
                    if (!first) take = quick_inside<true>(a, p0, v0, p1, v1, nlo, nhi, nnear);
                }
                const uint64_t m = ballot64(take);
                int base = 0;
                if (l == 0 && m) base = atomicAdd(&s_past, (int)__popcll(m));
                base = __shfl(base, 0, 64);
                if (take) {
                    keys[1][base + lanes_below(m)] = J;
                    ids[1][base + lanes_below(m)] = id;
                }
            }
            __syncthreads();
            const int past = s_past;
            if (past <= kFarThreads) {
                // (J, id) order: an entry's place is the number of smaller ones
                const int i = threadIdx.x;
                if (i < past) {
                    const float key = keys[1][i];
                    const int id = ids[1][i];
                    int r = 0, same = 0;
#pragma unroll 4
                    for (int j = 0; j < past; ++j) {
                        const float kj = keys[1][j];
                        r += kj < key || (kj == key && ids[1][j] < id) ? 1 : 0;
                        same += kj == key ? 1 : 0;
                    }
                    keys[0][r] = key;
                    ids[0][r] = id;
                    if (same > 64) s_ties = 1;
                }
            } else {
                // longer lists: a bitonic sort
                int P = 1;
                while (P < past) P <<= 1;
                for (int i = threadIdx.x; i < P; i += kFarThreads) {
                    keys[0][i] = i < past ? keys[1][i] : MPAP_INF;
                    ids[0][i] = i < past ? ids[1][i] : 0x7fffffff;
                }
                __syncthreads();
                for (int k = 2; k <= P; k <<= 1)
                    for (int j = k >> 1; j > 0; j >>= 1) {
                        for (int i = threadIdx.x; i < P; i += kFarThreads) {
                            const int x = i ^ j;
                            if (x > i) {
                                const float ki = keys[0][i], kx = keys[0][x];
                                const int ii = ids[0][i], ix = ids[0][x];
                                const bool gt = ki > kx || (ki == kx && ii > ix);
                                if (gt == ((i & k) == 0)) {
                                    keys[0][i] = kx; keys[0][x] = ki;
                                    ids[0][i] = ix; ids[0][x] = ii;
                                }
                            }
                        }
                        __syncthreads();
                    }
                for (int i = threadIdx.x; i + 64 < past; i += kFarThreads)
                    if (keys[0][i] == keys[0][i + 64]) s_ties = 1;
            }
            __syncthreads();
            if (s_ties) break;
            for (int base = 0; base < past && found < a.k_out; base += W) {
                const int ci = base + w;
                const bool ok = ci < past && wave_reachable(a, p0, v0, ids[0][ci], sblo, sbhi,
                                                            wlist + w * a.nbox);
                if (l == 0) okf[w] = ok ? 1 : 0;
                __syncthreads();
                for (int i = 0; i < W && found < a.k_out; ++i)
                    if (okf[i]) {
                        if (threadIdx.x == 0) {
                            nbr[(size_t)u * a.k_out + found] = ids[0][base + i];
                            ncost[(size_t)u * a.k_out + found] = keys[0][base + i] + 0.0f;
                        }
                        ++found;
                    }
                __syncthreads();
            }
            if (found >= a.k_out || !(tau < MPAP_INF)) {
                done = true;
                break;
            }
            // the next shell: larger where this one listed few
            prev = tau;
            tau = fmaxf(tau * (cnt >= 1024 ? 1.26f : cnt >= 512 ? 1.6f : cnt >= 128 ? 2.5f : 4.0f), 1e-30f);
            thin = 0;
        }
        if (threadIdx.x == 0) {
            if (done) ncnt[u] = found;
            else left[atomicAdd(nleft, 1)] = u;
        }
    }
}

template __global__ void k_steer_far<true>(SteerArgs, GridArgs, SteerBounds, const float4 *,
                                           const float4 *, float, int *, float *, int *, SteerFar,
                                           int *, int *);
template __global__ void k_steer_far<false>(SteerArgs, GridArgs, SteerBounds, const float4 *,
                                            const float4 *, float, int *, float *, int *, SteerFar,
                                            int *, int *);

// positions (with the id in w) and velocities in cell order
__global__ void __launch_bounds__(256) k_steer_scatter(SteerArgs a, GridArgs gr, const int *cell,
                                                       const int *slot, float4 *spos,
                                                       float4 *svel) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= a.n) return;
    const int i = gr.cstart[cell[u]] + slot[u];
    float p[3], v[3];
    load3(a.pos, u, p);
    load3(a.vel, u, v);
    spos[i] = make_float4(p[0], p[1], p[2], __int_as_float(u));
    svel[i] = make_float4(v[0], v[1], v[2], 0.0f);
}

// The sources that k_steer_far left, one workgroup each: the candidates'
// keys ranked by radix passes over all states.
__global__ void __launch_bounds__(kSteerThreads) k_steer_select(SteerArgs a, const int *left,
                                                                const int *nleft, int *nbr,
                                                                float *ncost, int *ncnt,
                                                                int *err) {
    extern __shared__ __align__(16) unsigned char lds[];
    int *hist = reinterpret_cast<int *>(lds);                          // 2048
    uint32_t *bkey = reinterpret_cast<uint32_t *>(hist + 2048);       // 2 * W
    int *bid = reinterpret_cast<int *>(bkey + 2 * kSteerMaxWidth);    // 2 * W
    float *sblo = reinterpret_cast<float *>(bid + 2 * kSteerMaxWidth);  // 3 * nbox
    float *sbhi = sblo + 3 * a.nbox;
    int *wlist = reinterpret_cast<int *>(sbhi + 3 * a.nbox);          // 4 * nbox
    __shared__ int scratch[kSteerThreads / 64 + 1];
    __shared__ int sres[2];
    __shared__ int s_cnt, s_found;
    __shared__ int out_id[kSteerMaxOut];
    __shared__ uint32_t out_key[kSteerMaxOut];
    __shared__ int okf[kSteerThreads / 64];

    for (int i = threadIdx.x; i < 3 * a.nbox; i += blockDim.x) {
        sblo[i] = a.blo[i];
        sbhi[i] = a.bhi[i];
    }
    const int w = threadIdx.x >> 6;
    const int sources = *nleft;
    for (int si = blockIdx.x; si < sources; si += gridDim.x) {
    const int u = left[si];
    float p0[3], v0[3];
    load3(a.pos, u, p0);
    load3(a.vel, u, v0);
    if (threadIdx.x == 0) s_found = 0;
    __syncthreads();

    uint32_t prev_key = 0u;
    int prev_id = -1;
    bool first = true;
    int width = 64;
    int found = 0;
    auto eligible = [&](int v, uint32_t k) {
        return v != u && (first || k > prev_key || (k == prev_key && v > prev_id));
    };
    auto key_of = [&](int v) {
        float p1[3], v1[3];
        load3(a.pos, v, p1);
        load3(a.vel, v, v1);
        return ukey(steer_cost(p0, v0, p1, v1, a.T));
    };
    while (found < a.k_out) {
        // radix select of the width-th smallest eligible key: 11 + 11 + 10 bits
        uint32_t tau = 0xffffffffu;
        int total = 0;
        {
            int need = width;
            uint32_t prefix = 0u;
            const int shifts[3] = {21, 10, 0};
            const uint32_t masks[3] = {2047u, 2047u, 1023u};
            for (int pass = 0; pass < 3; ++pass) {
                for (int i = threadIdx.x; i < 2048; i += blockDim.x) hist[i] = 0;
                __syncthreads();
                for (int v = threadIdx.x; v < a.n; v += blockDim.x) {
                    const uint32_t k = key_of(v);
                    if (!eligible(v, k)) continue;
                    if (pass > 0 && (k >> (shifts[pass - 1])) != prefix) continue;
                    atomicAdd(&hist[(k >> shifts[pass]) & masks[pass]], 1);
                }
                __syncthreads();
                if (pass == 0) {
                    int loc = 0;
                    for (int i = 0; i < 8; ++i) loc += hist[8 * threadIdx.x + i];
                    block_excl_scan(loc, scratch, &total);
                    if (total <= width) break;  // every eligible candidate fits
                }
                find_bin(hist, need, scratch, sres);
                const int bin = sres[0];
                need -= sres[1];
                prefix = (prefix << (pass == 0 ? 11 : (pass == 1 ? 11 : 10))) | (uint32_t)bin;
                if (pass == 2) tau = prefix;
                __syncthreads();
            }
        }
        if (total == 0) break;
        // gather the eligible keys <= tau, sort them by (key, id)
        if (threadIdx.x == 0) s_cnt = 0;
        __syncthreads();
        const int cap = 2 * width;
        for (int v = threadIdx.x; v < a.n; v += blockDim.x) {
            const uint32_t k = key_of(v);
            if (!eligible(v, k) || k > tau) continue;
            const int slot = atomicAdd(&s_cnt, 1);
            if (slot < cap) {
                bkey[slot] = k;
                bid[slot] = v;
            }
        }
        __syncthreads();
        int m = s_cnt;
        if (m > cap) {
            if (threadIdx.x == 0) atomicOr(err, 1);
            m = cap;
        }
        int P = 1;
        while (P < m) P <<= 1;
        for (int i = m + threadIdx.x; i < P; i += blockDim.x) {
            bkey[i] = 0xffffffffu;
            bid[i] = 0x7fffffff;
        }
        __syncthreads();
        for (int k = 2; k <= P; k <<= 1)
            for (int j = k >> 1; j > 0; j >>= 1) {
                for (int i = threadIdx.x; i < P; i += blockDim.x) {
                    const int x = i ^ j;
                    if (x > i) {
                        const bool up = (i & k) == 0;
                        const uint32_t ki = bkey[i], kx = bkey[x];
                        const int ii = bid[i], ix = bid[x];
                        const bool gt = ki > kx || (ki == kx && ii > ix);
                        if (gt == up) {
                            bkey[i] = kx; bkey[x] = ki;
                            bid[i] = ix; bid[x] = ii;
                        }
                    }
                }
                __syncthreads();
            }
        const int cnt = min(m, width);
        // check the ranked candidates in order, one wave each
        for (int base = 0; base < cnt && found < a.k_out; base += kSteerThreads / 64) {
            const int ci = base + w;
            bool ok = false;
            if (ci < cnt) ok = wave_reachable(a, p0, v0, bid[ci], sblo, sbhi, wlist + w * a.nbox);
            if (lane_id() == 0) okf[w] = ok ? 1 : 0;
            __syncthreads();
            if (threadIdx.x == 0) {
                int f = s_found;
                for (int i = 0; i < kSteerThreads / 64 && base + i < cnt && f < a.k_out; ++i)
                    if (okf[i]) {
                        out_id[f] = bid[base + i];
                        out_key[f] = bkey[base + i];
                        ++f;
                    }
                s_found = f;
            }
            __syncthreads();
            found = s_found;
        }
        if (cnt == 0 || total <= width) break;  // every eligible candidate was ranked
        prev_key = bkey[cnt - 1];
        prev_id = bid[cnt - 1];
        first = false;
        width = min(2 * width, kSteerMaxWidth);
        __syncthreads();
    }
    for (int i = threadIdx.x; i < found; i += blockDim.x) {
        nbr[(size_t)u * a.k_out + i] = out_id[i];
        ncost[(size_t)u * a.k_out + i] = unkey(out_key[i]);
    }
    if (threadIdx.x == 0) ncnt[u] = found;
    __syncthreads();
    }
}

// one wave per row (at most 64 targets): a target's place is the number of
// smaller ids (distinct in a row)
__global__ void __launch_bounds__(256) k_steer_compact(int n, int k_out, const int *row_ptr,
                                                       const int *nbr, const float *ncost,
                                                       const int *ncnt, int *col, float *cost) {
    const int u = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (u >= n) return;
    const int l = lane_id();
    const int o = row_ptr[u], c = ncnt[u];
    const int id = l < c ? nbr[(size_t)u * k_out + l] : 0x7fffffff;
    int rank = 0;
    for (int i = 0; i < c; ++i) rank += __shfl(id, i, 64) < id ? 1 : 0;
    if (l < c) {
        col[o + rank] = id;
        cost[o + rank] = ncost[(size_t)u * k_out + l];
    }
}

namespace {

// From here on the exponential counts as zero (e^-700 is 1e-304); and where
// the plain one becomes zero.
constexpr double kExpEnd = 700.0, kExpZero = 745.1332191019412;

// exp(-x), x >= 0, by table: -x = k ln 2 / 64 + r, |r| <= ln 2 / 128, so
// exp(-x) = 2^(k div 64) 2^((k mod 64)/64) e^r, with e^r - 1 by its series to
// r^5 (the next term is below 2^-55 of the result) (Tang, "Table-driven
// implementation of the exponential function in IEEE floating-point
// arithmetic", ACM TOMS 15, 1989).  pow[j] = 2^(j/64).  k is rounded by
// adding 1.5 2^52, whose low word then holds it; its power of two goes
// into the table entry's exponent.  Zero beyond `end` (at most kExpEnd: there
// the exponent would leave its range), NaN for NaN.  Off by at most 2.2e-16 of
// the result (2 million points).
__device__ __forceinline__ double exp_neg(double x, double end, const double *pow) {
    const double big = 6755399441055744.0;
    const double kb = __builtin_fma(x, -92.33248261689366, big);
    const int k = __double2loint(kb);
    const double kd = kb - big;
    // (ln 2 / 64 in two parts)
    double r = __builtin_fma(kd, -0.010830424696249145, -x);
    r = __builtin_fma(kd, -3.623510646634843e-19, r);
    const double t0 = pow[k & 63];
    const double t = __hiloint2double(__double2hiint(t0) + ((k >> 6) << 20), __double2loint(t0));
    double p = __builtin_fma(r, 1.0 / 120.0, 1.0 / 24.0);
    p = __builtin_fma(r, p, 1.0 / 6.0);
    p = __builtin_fma(r, p, 0.5);
    p = __builtin_fma(r * r, p, r);
    return x > end ? 0.0 : __builtin_fma(t, p, t);
}

}  // namespace

// A blob in float64, read by uniform addresses (scalar loads).
typedef const __attribute__((address_space(4))) SteerBlob *BlobPtr;

__global__ void __launch_bounds__(256) k_steer_blobs(int nblob, const float *mu, const float *sig,
                                                     const float *amp, SteerBlob *out) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= nblob) return;
    const double s = (double)sig[j];
    SteerBlob b{};
    for (int d = 0; d < 3; ++d) b.mu[d] = (double)mu[3 * j + d];
    b.inv = 1.0 / (2.0 * (s * s));
    b.amp = (double)amp[j];
    // an infinite amplitude counts at every point whose plain exponential is
    // not zero, and gives NaN (so q = 0) elsewhere: only where it ends matters
    if (isinf(amp[j])) b.inv *= kExpEnd / kExpZero;
    b.end = fmin(kExpEnd, log(fabs(b.amp)) + 65.0 * 0.6931471805599453);
    out[j] = b;
}

// Drift of every edge: sum over the K chords of the checked points of |chord|
// (1 - q(chord midpoint)), the terms in float64 from the float32 check
// points, summed in chord order and rounded once to float32; elen = float32
// sum of |chord| (the trajectory length of the surrogate's inputs).
//
// One wave per source row, the chords of several of its edges side by side
// so that all lanes have one (K = 100 leaves 28 of 128 idle otherwise), their
// terms in LDS and summed by one lane per edge.  Bound by the float64
// exponential of each chord and blob: blobs whose centre is too far from the
// hull of the edges' Bezier control points to reach the last bit of q are
// left out (a value below 2^-66; each lane drops those below 2^-65 itself, so
// an edge's drift does not depend on the edges beside it), the exponent is scaled by 1 / (2 sigma^2) instead of divided, the
// exponential is exp_neg, and the blobs, the same for the whole wave, come
// through scalar loads four at a time.  Measured, 20,000 states (100 blobs,
// 569,000 edges): 5.6 ms (14.2 ms with one edge at a time and the general
// exponential; 8.8 ms with that here; 7.1 ms with twice the terms in LDS and
// two workgroups instead of five per CU).
__global__ void __launch_bounds__(256) k_traj_drift(SteerArgs a, const SteerBlob *blobs,
                                                    const int *row_ptr, const int *col,
                                                    float *drift, float *elen) {
    // per wave: terms, chord lengths, edge coefficients, bits of the blobs in reach
    extern __shared__ __align__(16) unsigned char lds[];
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int words = (a.nblob + 63) >> 6;
    double *term = reinterpret_cast<double *>(lds) + w * kTrajTerms;
    float *clen = reinterpret_cast<float *>(lds + 4 * kTrajTerms * 8) + w * kTrajTerms;
    float *coef = reinterpret_cast<float *>(lds + 4 * kTrajTerms * 12) + w * kSteerMaxOut * 6;
    uint64_t *mask = reinterpret_cast<uint64_t *>(lds + 4 * kTrajTerms * 12 + 4 * kSteerMaxOut * 24) +
                     w * words;
    const BlobPtr blob = (BlobPtr)blobs;
    __shared__ double pow[64];
    if (threadIdx.x < 64) pow[threadIdx.x] = exp2((double)threadIdx.x * (1.0 / 64.0));
    __syncthreads();
    const int u = (int)blockIdx.x * 4 + w;
    if (u >= a.n) return;
    const int l = lane_id();
    float p0[3], v0[3];
    load3(a.pos, u, p0);
    load3(a.vel, u, v0);
    const int end = row_ptr[u + 1];
    const int group = max(1, kTrajTerms / a.K);  // edges side by side
    for (int e0 = row_ptr[u]; e0 < end; e0 += group) {
        const int ne = min(group, end - e0);
        // coefficients, and the box of the control points p0, p0 + v0 T/3,
        // p1 - v1 T/3, p1 (widened by far more than the points' roundings)
        float lo[3] = {MPAP_INF, MPAP_INF, MPAP_INF}, hi[3] = {-MPAP_INF, -MPAP_INF, -MPAP_INF};
        if (l < ne) {
            float p1[3], v1[3], c0[3], c1[3];
            load3(a.pos, col[e0 + l], p1);
            load3(a.vel, col[e0 + l], v1);
            (void)steer3(p0, v0, p1, v1, a.T, c0, c1);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                coef[l * 6 + d] = c0[d];
                coef[l * 6 + 3 + d] = c1[d];
                const float q0 = p0[d] + v0[d] * a.T * (1.0f / 3.0f);
                const float q1 = p1[d] - v1[d] * a.T * (1.0f / 3.0f);
                const float wide = 1e-4f * (fabsf(p0[d]) + fabsf(p1[d]) + fabsf(q0) + fabsf(q1));
                lo[d] = fminf(fminf(p0[d], p1[d]), fminf(q0, q1)) - wide;
                hi[d] = fmaxf(fmaxf(p0[d], p1[d]), fmaxf(q0, q1)) + wide;
            }
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            lo[d] = wave_min(lo[d]);
            hi[d] = wave_max_f(hi[d]);
        }
        for (int g = 0; g < words; ++g) {
            const int j = g * 64 + l;
            bool keep = j < a.nblob;
            if (keep) {
                float d2 = 0.0f;
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    const float m = a.mu[3 * j + d];
                    const float t = fmaxf(lo[d] - m, m - hi[d]);
                    if (!(t <= 0.0f)) d2 = __builtin_fmaf(t, t, d2);
                }
                const float sg = a.sig[j];
                // base-two exponent at the hull, against the one whose value
                // is below 2^-66 (NaN and what float32 cannot hold stay in)
                const float y = 0.7213f * d2 * __builtin_amdgcn_rcpf(sg * sg);
                keep = !(y > 66.0f + __builtin_amdgcn_logf(fabsf(a.amp[j])) && d2 < MPAP_INF);
            }
            const uint64_t m = ballot64(keep);
            if (l == 0) mask[g] = m;
        }
        wave_sync();
        const int chords = ne * a.K;
        int ei = l / a.K, k = l % a.K;
        for (int c0_ = 0; c0_ < chords; c0_ += 64) {
            const int c = c0_ + l;
            // (lanes beyond the last chord repeat chord 0)
            const bool on = c < chords;
            const int ej = on ? ei : 0, kj = on ? k : 0;
            float c0[3], c1[3], pa[3], pb[3];
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                c0[d] = coef[ej * 6 + d];
                c1[d] = coef[ej * 6 + 3 + d];
            }
            traj_at(p0, v0, c0, c1, check_time(kj, a.T, a.K), pa, nullptr);
            traj_at(p0, v0, c0, c1, check_time(kj + 1, a.T, a.K), pb, nullptr);
            const float fx = pb[0] - pa[0], fy = pb[1] - pa[1], fz = pb[2] - pa[2];
            double sq = 0.0, mid[3];
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const double t = (double)pb[d] - (double)pa[d];
                sq = sq + t * t;
                mid[d] = 0.5 * ((double)pb[d] + (double)pa[d]);
            }
            double acc = 0.0;
            for (int g = 0; g < words; ++g) {
                const uint64_t own = mask[g];
                uint64_t m = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(own >> 32)) << 32) |
                             (uint32_t)__builtin_amdgcn_readfirstlane((int)(own & 0xffffffffu));
                while (m) {
                    // up to four blobs at once (fewer: the last again, as nothing)
                    int j[4];
                    bool real[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        real[i] = m != 0;
                        j[i] = real[i] ? 64 * g + (int)__builtin_ctzll(m) : j[max(i - 1, 0)];
                        m &= m - 1;
                        if (!real[i]) m = 0;
                    }
                    double e[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        double d2 = 0.0;
#pragma unroll
                        for (int d = 0; d < 3; ++d) {
                            const double t = mid[d] - blob[j[i]].mu[d];
                            d2 = __builtin_fma(t, t, d2);
                        }
                        e[i] = exp_neg(d2 * blob[j[i]].inv, blob[j[i]].end, pow);
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (real[i]) acc = __builtin_fma(blob[j[i]].amp, e[i], acc);
                }
            }
            if (on) {
                clen[c] = sqrtf((fx * fx + fy * fy) + fz * fz);
                term[c] = sqrt(sq) * (1.0 - fmin(fmax(acc, 0.0), 1.0));
            }
            k += 64;
            while (k >= a.K) {
                k -= a.K;
                ++ei;
            }
        }
        wave_sync();
        if (l < ne) {
            double acc = 0.0;
            for (int i = 0; i < a.K; ++i) acc = acc + term[l * a.K + i];
            drift[e0 + l] = (float)acc;
        }
        if (elen)
            for (int e = 0; e < ne; ++e) {
                float len = 0.0f;
                for (int i = l; i < a.K; i += 64) len = len + clen[e * a.K + i];
                len = wave_sum(len);
                if (l == 0) elen[e0 + e] = len;
            }
        wave_sync();  // the next group writes the terms again
    }
}

// drift (and, elen not null, the trajectory length) of every edge
void launch_traj_drift(const SteerArgs &a, const SteerBlob *blobs, const int *row_ptr,
                       const int *col, float *drift, float *elen, hipStream_t s) {
    const size_t lds = 4 * (size_t)kTrajTerms * 12 + 4 * (size_t)kSteerMaxOut * 24 +
                       4 * 8 * (size_t)((a.nblob + 63) / 64);
    k_traj_drift<<<(unsigned)((a.n + 3) / 4), 256, lds, s>>>(a, blobs, row_ptr, col, drift, elen);
}

// one thread per edge of the row: p_u (3), p_v (3), trajectory length,
// 1 - q at t = (k + 1/2) T / 8, k = 0..7, and 1 - q(p_v); base = the
// speed-weighted mean of the eight 1 - q values (arc-length weighting)
__global__ void __launch_bounds__(256) k_traj_features(SteerArgs a, const int *row_ptr,
                                                       const int *col, const float *elen,
                                                       uint16_t *X, float *base) {
    extern __shared__ float blob[];
    for (int i = threadIdx.x; i < 3 * a.nblob; i += blockDim.x) blob[i] = a.mu[i];
    for (int i = threadIdx.x; i < a.nblob; i += blockDim.x) {
        blob[3 * a.nblob + i] = a.sig[i];
        blob[4 * a.nblob + i] = a.amp[i];
    }
    __syncthreads();
    BuildArgs q{};
    q.dim = 3;
    q.nblob = a.nblob;
    q.mu = blob;
    q.sig = blob + 3 * a.nblob;
    q.amp = blob + 4 * a.nblob;
    // one thread per edge; its source u: last row with row_ptr[u] <= e
    const int m = row_ptr[a.n];
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= m) return;
    int lo = 0, hi = a.n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (row_ptr[mid] <= e) lo = mid; else hi = mid - 1;
    }
    const int u = lo;
    float p0[3], v0[3];
    load3(a.pos, u, p0);
    load3(a.vel, u, v0);
    {
        float p1[3], v1[3], c0[3], c1[3];
        load3(a.pos, col[e], p1);
        load3(a.vel, col[e], v1);
        (void)steer3(p0, v0, p1, v1, a.T, c0, c1);
        uint16_t *f = X + (size_t)e * 16;
        for (int d = 0; d < 3; ++d) {
            f[d] = f2bf(p0[d]);
            f[3 + d] = f2bf(p1[d]);
        }
        f[6] = f2bf(elen[e]);
        float sw = 0.0f, ss = 0.0f, sm = 0.0f;
        for (int j = 0; j < 8; ++j) {
            const float t = (((float)j + 0.5f) * a.T) / 8.0f;
            float p[3], vv[3];
            traj_at(p0, v0, c0, c1, t, p, vv);
            const float wq = 1.0f - blob_quality(q, p);
            const float sp = sqrtf((vv[0] * vv[0] + vv[1] * vv[1]) + vv[2] * vv[2]);
            f[7 + j] = f2bf(wq);
            sw = sw + sp * wq;
            ss = ss + sp;
            sm = sm + wq;
        }
        f[15] = f2bf(1.0f - blob_quality(q, p1));
        if (base) base[e] = ss > 0.0f ? sw / ss : sm * 0.125f;
    }
}
