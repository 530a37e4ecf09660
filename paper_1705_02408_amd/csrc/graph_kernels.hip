// Roadmap construction on the GPU: Sec. 3 Alg. 2 (BuildGraph: Near within
// r_n, then Collision against axis-aligned boxes as in Sec. 4.2) and the
// per-edge / per-node inputs of the perception heuristic (Alg. 1 step 2):
// drift increment = length * (1 - mean feature quality over the collision
// sub-steps) and the relocalisation flag q(x) > threshold (Sec. 4.1 drift
// reading with a feature-density quality q).
//
// Every float32 operation on the geometry is rounded separately (built with
// -ffp-contract=off), so neighbour sets and edge lengths are reproducible
// bit for bit by any IEEE float32 evaluation of the same formulas.
#include "device_common.h"
#include "graph_kernels.h"

namespace {

__device__ __forceinline__ float sqdist(const float *a, const float *b, int dim) {
    float dx = b[0] - a[0];
    float s = dx * dx;
    for (int k = 1; k < dim; ++k) {
        float d = b[k] - a[k];
        s = s + d * d;
    }
    return s;
}

// cell coordinate on one axis: floor((x - lo) / h), clamped to the grid
// (monotone in x, so cells of points less than one cell apart differ by at
// most one)
__device__ __forceinline__ int cell_axis(float x, float lo, float inv, int cells) {
    const float t = floorf((x - lo) * inv);
    return (int)fminf(fmaxf(t, 0.0f), (float)(cells - 1));
}

__device__ __forceinline__ int cell_coords(const GridArgs &gr, const float *x, int dim, int &cx,
                                           int &cy, int &cz) {
    cx = cell_axis(x[0], gr.lo[0], gr.inv, gr.gx);
    cy = cell_axis(x[1], gr.lo[1], gr.inv, gr.gy);
    cz = dim == 3 ? cell_axis(x[2], gr.lo[2], gr.inv, gr.gz) : 0;
    return (cz * gr.gy + cy) * gr.gx + cx;
}

// f(b, e) for every run [b, e) of sorted slots of the cells adjacent to
// (cx, cy, cz), the cell itself included: one per (y, z) row of cells
template <class F>
__device__ __forceinline__ void for_adjacent(const GridArgs &gr, int cx, int cy, int cz, F f) {
    const int x0 = max(cx - 1, 0), x1 = min(cx + 1, gr.gx - 1);
    const int z1 = min(cz + 1, gr.gz - 1), y1 = min(cy + 1, gr.gy - 1);
    for (int z = max(cz - 1, 0); z <= z1; ++z)
        for (int y = max(cy - 1, 0); y <= y1; ++y) {
            const int row = (z * gr.gy + y) * gr.gx;
            const int b = gr.cstart[row + x0];
            const int e = gr.cstart[row + x1] + gr.ccount[row + x1];
            f(b, e);
        }
}

// source row (the last u with uptr[u] <= t) of the t-th id-ordered pair (a, b),
// a < b, of a symmetric roadmap for the lanes of a wave, t rising with the lane:
// the wave finds the rows of its first and last pair together (64 probes a
// step), each lane its own between them
__device__ __forceinline__ int wave_pair_row(const int *uptr, int n, int t) {
    const int l = lane_id();
    int ends[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int ti = __shfl(t, i == 0 ? 0 : 63, 64);
        int lo = 0, span = n;  // the row is in [lo, lo + span)
        while (span > 1) {
            const int step = (span + 63) >> 6;
            const int at = lo + l * step;
            const uint64_t below = ballot64(l * step < span && uptr[min(at, n - 1)] <= ti);
            const int last = 63 - (int)__clzll((unsigned long long)below);
            lo += last * step;
            span = min(step, span - last * step);
        }
        ends[i] = lo;
    }
    int lo = ends[0], hi = ends[1];
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (uptr[mid] <= t) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// index of edge v -> u in row v (rows sorted by target id), -1 if absent
__device__ __forceinline__ int reverse_edge(const int *row_ptr, const int *col, int v, int u) {
    const int end = row_ptr[v + 1];
    int lo = row_ptr[v], hi = end;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (col[mid] < u) lo = mid + 1; else hi = mid;
    }
    return (lo < end && col[lo] == u) ? lo : -1;
}

// blob parameters staged in LDS (mu[nblob*dim], sig[nblob], amp[nblob]);
// returns g reading them from there
__device__ __forceinline__ BuildArgs stage_blobs(const BuildArgs &g, float *blob) {
    for (int i = threadIdx.x; i < g.nblob * g.dim; i += blockDim.x) blob[i] = g.mu[i];
    for (int i = threadIdx.x; i < g.nblob; i += blockDim.x) {
        blob[g.nblob * g.dim + i] = g.sig[i];
        blob[g.nblob * g.dim + g.nblob + i] = g.amp[i];
    }
    __syncthreads();
    BuildArgs gl = g;
    gl.mu = blob;
    gl.sig = blob + g.nblob * g.dim;
    gl.amp = blob + g.nblob * g.dim + g.nblob;
    return gl;
}

// midpoints whose quality sums one pass over the blobs holds in registers, and
// the place of a run's anchor among them
constexpr int kDriftRun = 16;
constexpr int kDriftMid = 8;

// 1 / n!, n <= 18
constexpr double inv_factorial(int n) {
    double f = 1.0;
    for (int i = 2; i <= n; ++i) f *= (double)i;
    return 1.0 / f;
}
// e^(-u - v) - 1, e^(u - v) - 1 and e^-2v - 1 for 0 <= v <= 1/128, from the
// series of sinh u (to u^13), cosh u - 1 (to u^14) and e^-v - 1 (to v^6)
__device__ __forceinline__ void expm1_both(double u, double v, double &down, double &up,
                                           double &twice) {
    const double z = u * u;
    double sh = inv_factorial(13), ch = inv_factorial(14), m = inv_factorial(6);
#pragma unroll
    for (int n = 11; n >= 3; n -= 2) sh = __builtin_fma(z, sh, inv_factorial(n));
#pragma unroll
    for (int n = 12; n >= 4; n -= 2) ch = __builtin_fma(z, ch, inv_factorial(n));
#pragma unroll
    for (int n = 5; n >= 2; --n) m = __builtin_fma(-v, m, inv_factorial(n));
    sh = __builtin_fma(z * u, sh, u);
    ch = z * __builtin_fma(z, ch, 0.5);
    m = __builtin_fma(v * v, m, -v);
    const double a = ch - sh, b = ch + sh;
    down = __builtin_fma(a, m, a + m);
    up = __builtin_fma(b, m, b + m);
    twice = __builtin_fma(m, m, 2.0 * m);
}

// sum over the four lanes of a quad, in each of them (every lane of the wave calls)
template <int kPerm>
__device__ __forceinline__ double quad_perm(double v) {
    return __hiloint2double(
        __builtin_amdgcn_update_dpp(0, __double2hiint(v), kPerm, 0xf, 0xf, false),
        __builtin_amdgcn_update_dpp(0, __double2loint(v), kPerm, 0xf, 0xf, false));
}
__device__ __forceinline__ double quad_sum(double v) {
    v += quad_perm<0xb1>(v);         // lanes 1, 0, 3, 2
    return v + quad_perm<0x4e>(v);   // lanes 2, 3, 0, 1
}

// lanes that share a pair's blobs (a quad)
constexpr int kDriftLanes = 4;

// Drift of the id-ordered pair (a, b) of length len: sum_j (len/K)(1 - q(mid_j))
// over the K sub-step midpoints x_a + ((j + 1/2)/K)(x_b - x_a), in float64
// in j order from the float32 positions and length, rounded once to float32.
//
// Bound by float64 issue.  Along a segment a blob's exponent is quadratic in
// j, so its values at successive midpoints follow from the one at a run's
// middle, the ratio to its neighbour on either side and the constant ratio of
// ratios: three operations a midpoint instead of an exponential (about 45
// operations) each.  The ratios are carried less one, so a step adds one
// rounding of the value, and at most eight steps lie between a midpoint and
// its run's middle.  Against 128-bit sums the mean relative error is 3.1e-16
// (2D) and 4.2e-16 (3D) at the workloads' blobs, 5.3e-16 and 4.8e-16 with an
// exponential a midpoint; where q is within 1e-7 of one, 1.6e-10 and 1.5e-10
// (1.8e-10 and 1.4e-10).  A blob narrower than eight steps, or many widths
// away, is evaluated point by point, and blobs too far from the segment to
// reach the last bit of q are left out.
//
// What a lane adds depends on its pair alone (a wave leaves out what all its
// lanes leave out) and the blobs are dealt out and summed in one way, so a
// pair has the same drift in every roadmap with the same blobs.  Every lane
// of the wave calls (live: it holds a pair).
template <int D>
__device__ __forceinline__ float pair_drift(const BuildArgs &gl, int a, int b, float len,
                                            bool live) {
    const int sub = lane_id() % kDriftLanes;
    double xa[D], df[D], dl[D], c2 = 0.0;  // dl: the step between midpoints, c2 its square
    float xaf[D];
    int K = (int)ceilf(len / gl.step);
    if (K < 1) K = 1;
    const double dK = (double)K, rK = 1.0 / dK;
    const double w = (double)len / dK;
#pragma unroll
    for (int k = 0; k < D; ++k) {
        xaf[k] = gl.pos[a * D + k];
        xa[k] = (double)xaf[k];
        df[k] = (double)gl.pos[b * D + k] - xa[k];
        dl[k] = df[k] * rK;
        c2 = __builtin_fma(dl[k], dl[k], c2);
    }
    // runs of equal length; the wave goes through those of its longest pair
    const int runs = live ? (K - 1) / kDriftRun + 1 : 0;
    const int run = live ? (K - 1) / runs + 1 : 0;
    const int most = __builtin_amdgcn_readfirstlane(wave_max_i(runs));
    const int longest = __builtin_amdgcn_readfirstlane(wave_max_i(run));
    const int back = longest / 2, ahead = (longest - 1) / 2;  // steps from a run's middle
    // every point lies within len (and the roundings) of x_a
    const float reach = len * 1.0001f;
    double acc = 0.0;
    for (int r = 0; r < most; ++r) {
        const bool mine = r < runs;
        const int j0 = r * run, jc = j0 + run / 2, j1 = min(j0 + run, K);
        const double sc = ((double)jc + 0.5) / dK;
        double q[kDriftRun];
#pragma unroll
        for (int i = 0; i < kDriftRun; ++i) q[i] = 0.0;
        for (int j = sub; j < gl.nblob; j += kDriftLanes) {
            const float sg = gl.sig[j], am = gl.amp[j];
            float d2f = 0.0f, xs = 0.0f;
#pragma unroll
            for (int k = 0; k < D; ++k) {
                const float mu = gl.mu[j * D + k];
                const float t = xaf[k] - mu;
                d2f = __builtin_fmaf(t, t, d2f);
                xs += fabsf(xaf[k]) + fabsf(mu);
            }
            // exponent (base 2) at the nearest the segment can come, low by
            // far more than its roundings, against the one whose value is
            // below 2^-66 (NaN and what float32 cannot hold stay in)
            const float gap = __builtin_amdgcn_sqrtf(d2f) * 0.9999f - reach - xs * 0x1p-20f;
            const float near = gap < 0.0f ? 0.0f : gap;
            const float y = 0.7213f * __builtin_amdgcn_rcpf(sg * sg) * (near * near);
            const float end = 66.0f + __builtin_amdgcn_logf(fabsf(am));
            const bool in = mine && !(y > end && d2f < MPAP_INF);
            if (ballot64(in) == 0) continue;
            const double s = (double)sg, amp = (double)am;
            const double two_s2 = 2.0 * (s * s);
            // 1 / (2 sigma^2) by two Newton steps (NaN where that fails: the
            // run is then evaluated point by point, with the division)
            double inv = __builtin_amdgcn_rcp(two_s2);
            inv = __builtin_fma(__builtin_fma(-two_s2, inv, 1.0), inv, inv);
            inv = __builtin_fma(__builtin_fma(-two_s2, inv, 1.0), inv, inv);
            double d2 = 0.0, g = 0.0;
#pragma unroll
            for (int k = 0; k < D; ++k) {
                const double t = __builtin_fma(sc, df[k], xa[k] - (double)gl.mu[j * D + k]);
                d2 = __builtin_fma(t, t, d2);
                g = __builtin_fma(t, dl[k], g);
            }
            // exponent at i steps from the middle: e + slope i + curve i^2
            const double e = d2 * inv, slope = 2.0 * g * inv, curve = c2 * inv;
            // (the run's least exponent is at least this)
            const float least = 1.4425f * (float)(e - (double)kDriftMid * fabs(slope));
            const bool near_run = in && !(least > end);
            const bool smooth = e <= 690.0 && fabs(slope) <= 2.0 && curve <= 0x1p-7 &&
                                fabsf(am) < MPAP_INF;
            if (ballot64(near_run && smooth)) {
                const bool use = near_run && smooth;
                double C, Rf, Rb;
                // (the others add nothing)
                expm1_both(use ? slope : 0.0, use ? curve : 0.0, Rf, Rb, C);
                const double C1 = 1.0 + C;
                double Ef = use ? amp * exp(-e) : 0.0, Eb = Ef;
                q[kDriftMid] += Ef;
                auto behind = [&](int i) {
                    Eb = __builtin_fma(Eb, Rb, Eb);
                    Rb = __builtin_fma(Rb, C1, C);
                    q[kDriftMid - i] += Eb;
                };
                auto before = [&](int i) {
                    Ef = __builtin_fma(Ef, Rf, Ef);
                    Rf = __builtin_fma(Rf, C1, C);
                    q[kDriftMid + i] += Ef;
                };
#pragma unroll
                for (int i = 1; i <= kDriftMid; ++i) {
                    if (i % 2 == 1 && longest < 2 * i) break;
                    behind(i);
                    if (i < kDriftMid) before(i);
                }
            }
            if (ballot64(near_run && !smooth)) {
                const bool use = near_run && !smooth;
                int first = jc - kDriftMid;
                asm volatile("" : "+v"(first));  // (no points kept from blob to blob: registers)
#pragma unroll
                for (int i = 0; i < kDriftRun; ++i) {
                    if (i < kDriftMid - back || i > kDriftMid + ahead) continue;
                    const double si = ((double)(first + i) + 0.5) / dK;
                    double t2 = 0.0;
#pragma unroll
                    for (int k = 0; k < D; ++k) {
                        const double t = xa[k] + si * df[k] - (double)gl.mu[j * D + k];
                        t2 = t2 + t * t;
                    }
                    q[i] += use ? amp * exp(-t2 / two_s2) : 0.0;

                }
            }
        }
#pragma unroll
        for (int i = 0; i < kDriftRun; ++i) {
            if (i < kDriftMid - back || i > kDriftMid + ahead) continue;
            const double v = quad_sum(q[i]);
            const int j = jc + i - kDriftMid;
            if (mine && j >= j0 && j < j1) acc = acc + w * (1.0 - fmin(fmax(v, 0.0), 1.0));
        }
    }
    return (float)acc;
}

// Blobs staged for the float32 quality: 2 sigma^2 in the place of sigma and,
// for plain blobs (see launch_edge_features), its reciprocal behind the
// amplitudes.
template <bool kPlain, int D>
__device__ __forceinline__ void stage_quality_blobs(const BuildArgs &g, float *blob) {
    for (int i = threadIdx.x; i < g.nblob * D; i += blockDim.x) blob[i] = g.mu[i];
    for (int i = threadIdx.x; i < g.nblob; i += blockDim.x) {
        const float s = g.sig[i];
        const float b = 2.0f * s * s;
        blob[g.nblob * D + i] = b;
        blob[g.nblob * (D + 1) + i] = g.amp[i];
        if constexpr (kPlain) blob[g.nblob * (D + 2) + i] = 1.0f / b;
    }
    __syncthreads();
}

// q at P points (blob_quality's float32 sums, bit for bit).  Bound by
// instruction issue: distance, division and exponential.  For plain blobs the
// division d2 / b is three operations with r = 1 / b rounded: q = d2 r, then
// q + r (d2 - q b), each in one fused operation.  This rounds as the division
// itself: q is off by less than 1.5 units in the last place, and by half a unit
// wherever the quotient lies so near the middle between two floats that it
// matters (d2 r is off by less than one unit before it is rounded, so q is one
// of the two floats); there d2 - q b is exact, and r's rounding moves the
// corrected value by less than the quotient's distance from the middle, which
// two 24-bit significands keep at 1/(2 b) units or more (Markstein, "Computation
// of elementary functions on the IBM RISC System/6000 processor", 1990, theorem
// 8.4, for a q within one unit).  Checked over random and over nearest
// quotients.
template <bool kPlain, int D, int P>
__device__ __forceinline__ void quality_points(const float *blob, int nblob,
                                               const float (&x)[P][D], float (&q)[P]) {
    const float *two_s2 = blob + nblob * D, *amp = two_s2 + nblob, *inv = amp + nblob;
#pragma unroll
    for (int i = 0; i < P; ++i) q[i] = 0.0f;
#pragma unroll 2
    for (int j = 0; j < nblob; ++j) {
        const float b = two_s2[j], am = amp[j];
#pragma unroll
        for (int i = 0; i < P; ++i) {
            float d2 = 0.0f;
#pragma unroll
            for (int k = 0; k < D; ++k) {
                const float t = x[i][k] - blob[j * D + k];
                d2 = d2 + t * t;
            }
            float y;
            if constexpr (kPlain) {
                const float r = inv[j];
                const float q0 = d2 * r;
                y = __builtin_fmaf(__builtin_fmaf(-q0, b, d2), r, q0);
            } else {
                y = d2 / b;
            }
            q[i] = q[i] + am * expf(-y);
        }
    }
#pragma unroll
    for (int i = 0; i < P; ++i) q[i] = fminf(fmaxf(q[i], 0.0f), 1.0f);
}

}  // namespace

// Grid Near, step 1: each node's cell and its slot among the cell's nodes.
__global__ void __launch_bounds__(256) k_grid_bin(BuildArgs g, GridArgs gr, int *cell, int *slot) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= g.n) return;
    float x[3] = {0.f, 0.f, 0.f};
    for (int k = 0; k < g.dim; ++k) x[k] = g.pos[u * g.dim + k];
    int cx, cy, cz;
    const int c = cell_coords(gr, x, g.dim, cx, cy, cz);
    cell[u] = c;
    slot[u] = atomicAdd(&gr.ccount[c], 1);
}

// Step 2 (after the scan of the cell counts): nodes and positions in cell
// order.
__global__ void __launch_bounds__(256) k_grid_scatter(BuildArgs g, GridArgs gr, const int *cell,
                                                      const int *slot) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= g.n) return;
    float x[3] = {0.f, 0.f, 0.f};
    for (int k = 0; k < g.dim; ++k) x[k] = g.pos[u * g.dim + k];
    const int i = gr.cstart[cell[u]] + slot[u];
    gr.sid[i] = u;
    gr.spos[i] = make_float4(x[0], x[1], x[2], 0.0f);
}

// Step 3: the Near count of each node (the same test as the all-pairs
// kernel on the candidates of the adjacent cells); kNearLanes lanes share a
// node's candidates, and nodes are taken in cell order so the lanes of a wave
// scan the same cells.  A thread per node was bound by its chain of loads:
// 33 us for 50,000 samples in 3D (125), 9 for 2,000 in 2D (32); step 4
// 37 (137) and 8 (35).  max_cnt gets the longest row.
__global__ void __launch_bounds__(256) k_near_count_grid(BuildArgs g, GridArgs gr, int *cnt,
                                                         int *max_cnt) {
    const int i = (int)((blockIdx.x * blockDim.x + threadIdx.x) / kNearLanes);
    const int sub = (int)threadIdx.x % kNearLanes;
    int c = 0;
    if (i < g.n) {
        const int u = gr.sid[i];
        const float4 p = gr.spos[i];
        const float xu[3] = {p.x, p.y, p.z};
        int cx, cy, cz;
        cell_coords(gr, xu, g.dim, cx, cy, cz);
        for_adjacent(gr, cx, cy, cz, [&](int j0, int j1) {
            for (int j = j0 + sub; j < j1; j += kNearLanes) {
                const float4 q = gr.spos[j];
                const float xv[3] = {q.x, q.y, q.z};
                const float cost = sqrtf(sqdist(xu, xv, g.dim));
                c += (cost < g.r && gr.sid[j] != u) ? 1 : 0;
            }
        });
        for (int o = kNearLanes / 2; o > 0; o >>= 1) c += __shfl_xor(c, o);
        if (sub == 0) cnt[u] = c;
    }
    for (int o = 32; o >= kNearLanes; o >>= 1) c = max(c, __shfl_xor(c, o));
    // (atomics at one address wait for each other, 12 ns each: only those
    // that may raise it)
    if ((threadIdx.x & 63) == 0 &&
        c > __hip_atomic_load(max_cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(max_cnt, c);
}

// Step 4: the candidates of each node written to its row at off[u] (step 5
// orders them).
__global__ void __launch_bounds__(256) k_near_fill_grid(BuildArgs g, GridArgs gr, const int *off,
                                                        int *cand_u, int *cand_v, float *cand_c) {
    const int i = (int)((blockIdx.x * blockDim.x + threadIdx.x) / kNearLanes);
    const int sub = (int)threadIdx.x % kNearLanes;
    if (i >= g.n) return;
    const int u = gr.sid[i];
    const float4 p = gr.spos[i];
    const float xu[3] = {p.x, p.y, p.z};
    int cx, cy, cz;
    cell_coords(gr, xu, g.dim, cx, cy, cz);
    // the node's lanes within the wave, and those below this one
    const int first = lane_id() - sub;
    const uint64_t lanes = ((1ull << kNearLanes) - 1ull) << first;
    const uint64_t below = ((1ull << sub) - 1ull) << first;
    int o = off[u];
    for_adjacent(gr, cx, cy, cz, [&](int j0, int j1) {
        for (int jb = j0; jb < j1; jb += kNearLanes) {
            const int j = jb + sub;
            bool take = j < j1;
            int v = u;
            float cost = 0.f;
            if (take) {
                v = gr.sid[j];
                const float4 q = gr.spos[j];
                const float xv[3] = {q.x, q.y, q.z};
                cost = sqrtf(sqdist(xu, xv, g.dim));
                take = cost < g.r && v != u;
            }
            // (a node's lanes stay together: the same cells and trips)
            const uint64_t tk = __ballot(take) & lanes;
            if (take) {
                const int at = o + (int)__popcll(tk & below);
                cand_u[at] = u;
                cand_v[at] = v;
                cand_c[at] = cost;
            }
            o += (int)__popcll(tk);
        }
    });
}

// Step 5: each row put in target-id order, one wave per row (rows of at
// most kGridSortMax entries, staged in LDS): an entry's place is the number
// of smaller ids in its row (the ids of a row are distinct), so the rows
// equal the all-pairs kernel's.
__global__ void __launch_bounds__(256) k_sort_rows(int n, const int *off, const int *cnt,
                                                   int *cand_v, float *cand_c) {
    __shared__ int sv[4][kGridSortMax];
    __shared__ float sc[4][kGridSortMax];
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const int u = blockIdx.x * 4 + w;
    const int o = u < n ? off[u] : 0;
    const int d = u < n ? min(cnt[u], kGridSortMax) : 0;
    for (int i = l; i < d; i += 64) {
        sv[w][i] = cand_v[o + i];
        sc[w][i] = cand_c[o + i];
    }
    __syncthreads();
    for (int i = l; i < d; i += 64) {
        const int v = sv[w][i];
        int rank = 0;
        for (int j = 0; j < d; ++j) rank += sv[w][j] < v ? 1 : 0;
        cand_v[o + rank] = v;
        cand_c[o + rank] = sc[w][i];
    }
}

// Near: number of v != u with Cost(u, v) < r.  Positions are staged in LDS
// tiles shared by the block.
__global__ void __launch_bounds__(256) k_near_count(BuildArgs g, int *cnt) {
    __shared__ float tile[256 * 3];
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    float xu[3] = {0.f, 0.f, 0.f};
    if (u < g.n)
        for (int k = 0; k < g.dim; ++k) xu[k] = g.pos[u * g.dim + k];
    int c = 0;
    for (int t0 = 0; t0 < g.n; t0 += 256) {
        __syncthreads();
        const int v = t0 + threadIdx.x;
        if (v < g.n)
            for (int k = 0; k < g.dim; ++k) tile[threadIdx.x * 3 + k] = g.pos[v * g.dim + k];
        __syncthreads();
        const int m = min(256, g.n - t0);
        if (u < g.n)
            for (int i = 0; i < m; ++i) {
                const float cost = sqrtf(sqdist(xu, &tile[i * 3], g.dim));
                c += (cost < g.r && t0 + i != u) ? 1 : 0;
            }
    }
    if (u < g.n) cnt[u] = c;
}

__global__ void __launch_bounds__(256) k_near_fill(BuildArgs g, const int *off, int *cand_u,
                                                   int *cand_v, float *cand_c) {
    __shared__ float tile[256 * 3];
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    float xu[3] = {0.f, 0.f, 0.f};
    if (u < g.n)
        for (int k = 0; k < g.dim; ++k) xu[k] = g.pos[u * g.dim + k];
    int o = (u < g.n) ? off[u] : 0;
    for (int t0 = 0; t0 < g.n; t0 += 256) {
        __syncthreads();
        const int v = t0 + threadIdx.x;
        if (v < g.n)
            for (int k = 0; k < g.dim; ++k) tile[threadIdx.x * 3 + k] = g.pos[v * g.dim + k];
        __syncthreads();
        const int m = min(256, g.n - t0);
        if (u < g.n)
            for (int i = 0; i < m; ++i) {
                const float cost = sqrtf(sqdist(xu, &tile[i * 3], g.dim));
                if (cost < g.r && t0 + i != u) {
                    cand_u[o] = u;
                    cand_v[o] = t0 + i;
                    cand_c[o] = cost;
                    ++o;
                }
            }
    }
}

// Collision(a, b), (a, b) the candidate pair in id order: points
// x_a + (k/K)(x_b - x_a), k = 0..K, K = ceil(cost/step), against closed boxes.
// Where rows are long a wave's 64 candidates have few sources (about four of 20
// neighbours in 2D, two or three of 40 in 3D) and lie within the radius of
// them: the boxes that miss the wave's common range are left out 64 at a time
// (3D, 2.0 million candidates, 100 boxes: 63 us, each candidate against each box
// 476; 2D, 1.2 million, 20 boxes: 17 and 56; the edges that are left against
// five new boxes 23 and 48, 13 and 23).  Sources far apart make the range wide
// and the gain small, whatever their number; the result is the same.
template <int D>
__global__ void __launch_bounds__(256) k_collide(BuildArgs g, long long m, const int *cand_u,
                                                 const int *cand_v, const float *cand_c,
                                                 int *keep) {
    extern __shared__ float boxes[];  // lo[nbox*dim], hi[nbox*dim]
    for (int i = threadIdx.x; i < g.nbox * D; i += blockDim.x) {
        boxes[i] = g.blo[i];
        boxes[g.nbox * D + i] = g.bhi[i];
    }
    __syncthreads();
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const bool in_list = e < m;
    float xa[D] = {}, df[D] = {}, fK = 1.0f;
    // Each rounded coordinate xa + t df is monotone in s (t = s/K rounded,
    // t = 1 at s = K), so the points lie between the first (xa) and the
    // last (xa + df rounded) on every axis: a box missing that range on an
    // axis holds none of them.  The boxes are taken one at a time and only
    // those meeting the range are tested point by point (the same set of
    // point-in-box tests, grouped by box).
    float plo[D], phi[D];
    for (int k = 0; k < D; ++k) {
        plo[k] = MPAP_INF;  // (meets no box)
        phi[k] = -MPAP_INF;
    }
    int K = 1;
    if (in_list) {
        const int u = cand_u[e], v = cand_v[e];
        const int a = min(u, v), b = max(u, v);
        for (int k = 0; k < D; ++k) {
            xa[k] = g.pos[a * D + k];
            df[k] = g.pos[b * D + k] - xa[k];
            const float last = xa[k] + df[k];
            plo[k] = fminf(xa[k], last);
            phi[k] = fmaxf(xa[k], last);
        }
        K = (int)ceilf(cand_c[e] / g.step);
        if (K < 1) K = 1;
        fK = (float)K;
    }
    float wlo[D], whi[D];
    for (int k = 0; k < D; ++k) {
        wlo[k] = wave_min(plo[k]);
        whi[k] = -wave_min(-phi[k]);
    }
    bool hit = false;
    for (int j0 = 0; j0 < g.nbox; j0 += 64) {
        const int jl = j0 + lane_id();
        bool near = jl < g.nbox;
        if (near)
            for (int k = 0; k < D; ++k)
                near = near && whi[k] >= boxes[jl * D + k] &&
                       wlo[k] <= boxes[g.nbox * D + jl * D + k];
        uint64_t todo = ballot64(near);
        while (todo) {
            const int j = j0 + (int)__ffsll((unsigned long long)todo) - 1;
            todo &= todo - 1;
            float lo[D], hi[D];
            bool meets = !hit;
            for (int k = 0; k < D; ++k) {
                lo[k] = boxes[j * D + k];
                hi[k] = boxes[g.nbox * D + j * D + k];
                meets = meets && phi[k] >= lo[k] && plo[k] <= hi[k];
            }
            if (!meets) continue;
            for (int s = 0; s <= K && !hit; ++s) {
                const float t = (float)s / fK;
                bool in = true;
                for (int k = 0; k < D; ++k) {
                    const float p = xa[k] + t * df[k];
                    in = in && (p >= lo[k]) && (p <= hi[k]);
                }
                hit = in;
            }
        }
    }
    if (in_list) keep[e] = hit ? 0 : 1;
}
void launch_collide(const BuildArgs &g, long long m, const int *cand_u, const int *cand_v,
                    const float *cand_c, int *keep, hipStream_t s) {
    const size_t lds = sizeof(float) * 2 * (size_t)g.nbox * g.dim;
    const unsigned blocks = (unsigned)((m + 255) / 256);
    if (g.dim == 2) k_collide<2><<<blocks, 256, lds, s>>>(g, m, cand_u, cand_v, cand_c, keep);
    else k_collide<3><<<blocks, 256, lds, s>>>(g, m, cand_u, cand_v, cand_c, keep);
}

__global__ void __launch_bounds__(256) k_compact_edges(long long m, const int *keep,
                                                       const int *kscan, const int *cand_v,
                                                       const float *cand_c, int *col,
                                                       float *cost) {
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= m || !keep[e]) return;
    const int o = kscan[e];
    col[o] = cand_v[e];
    cost[o] = cand_c[e];
}

__global__ void __launch_bounds__(256) k_row_ptr(int n, long long m, const int *cand_off,
                                                 const int *kscan, const int *keep,
                                                 int *row_ptr) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    if (u > n) return;
    const long long o = (u < n) ? cand_off[u] : m;
    row_ptr[u] = (o < m) ? kscan[o] : (m > 0 ? kscan[m - 1] + keep[m - 1] : 0);
}

// The drift of every edge of a symmetric roadmap (rows sorted by target id,
// the same value both ways), a quad of lanes per id-ordered pair: the t-th
// pair's value is evaluated once and written to both of its edges.  uptr[u]
// counts the entries v > u of the rows before u (uptr[n] pairs in all).
// Measured against one thread per pair and an exponential per midpoint:
// 2,164 -> 548 us (3D, 50,000 samples, 80 blobs, 968,000 pairs), 1,113 -> 229
// (368,000 pairs), 860 -> 115 (82,000 pairs) and 109 -> 16 (2D, 2,000
// samples, 30 blobs, 21,000 pairs); widths of 0.01 to 0.03, most runs point by
// point, 1,107 -> 568 (3D, 12,000 samples).  One number of lanes for all sizes,
// since it fixes the order of the sums; with 1 / 2 / 4 / 8 lanes: 3D, 9,000
// pairs 151 / 84 / 49 / 41 us; 82,000 pairs 157 / 116 / 115 / 120; 968,000
// pairs 500 / 522 / 553 / 654; 2D, 21,000 pairs 26 / 17 / 16 / 16; 601,000
// pairs 128 / 134 / 165 / 221.
template <int D>
__global__ void __launch_bounds__(256, 3) k_edge_drift_pairs(BuildArgs g, int n, const int *row_ptr,
                                                          const int *col, const float *cost,
                                                          const int *uptr, float *drift) {
    extern __shared__ float blob[];
    const BuildArgs gl = stage_blobs(g, blob);
    const int pairs = uptr[n];
    const int i = (int)((blockIdx.x * 256ll + threadIdx.x) / kDriftLanes);
    // (whole waves: the lanes beyond the last pair repeat it)
    if ((int)((blockIdx.x * 256ll + (threadIdx.x & ~63)) / kDriftLanes) >= pairs) return;
    const bool live = i < pairs;
    const int t = min(i, pairs - 1);
    const int u = wave_pair_row(uptr, n, t);
    const int e = row_ptr[u + 1] - (uptr[u + 1] - t);
    const int v = col[e];
    const float d = pair_drift<D>(gl, u, v, cost[e], live);
    if (!live || lane_id() % kDriftLanes) return;
    drift[e] = d;
    const int r = reverse_edge(row_ptr, col, v, u);
    if (r >= 0) drift[r] = d;
}

// uptr helper: cnt[u] = entries v > u of row u (u < n), cnt[n] = 0; rows
// sorted by target id, no self loops
__global__ void __launch_bounds__(256) k_upper_count(int n, const int *row_ptr, const int *col,
                                                     int *cnt) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    if (u > n) return;
    if (u == n) {
        cnt[n] = 0;
        return;
    }
    const int end = row_ptr[u + 1];
    int lo = row_ptr[u], hi = end;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (col[mid] < u) lo = mid + 1; else hi = mid;
    }
    cnt[u] = end - lo;
}

__global__ void __launch_bounds__(256) k_node_flags(BuildArgs g, uint8_t *flag) {
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= g.n) return;
    float x[3] = {0.f, 0.f, 0.f};
    double xd[3] = {0.0, 0.0, 0.0};
    for (int k = 0; k < g.dim; ++k) {
        x[k] = g.pos[v * g.dim + k];
        xd[k] = (double)x[k];
    }
    uint8_t f = 0;
    if (blob_quality_f64(g, xd) > (double)g.reset_q) f |= 1u;
    float gg[3] = {g.goal[0], g.goal[1], g.goal[2]};
    const float r = g.goal_r;
    if (sqdist(gg, x, g.dim) <= r * r) f |= 2u;
    flag[v] = f;
}

// In-edge rows of a directed roadmap, each in the order of the sources (the
// order of the out-edge rows).  Three passes over the edges: count per target
// (and *bad = the least 2 k + 0 (cost) or + 1 (drift) of an edge k whose value
// a search can't take), any slot of the target's row, then the slot by the rank of
// the edge's index in the row.  A roadmap of 20,000 states with 24 out-edges
// each: 30 us; by the host, with both copies, 4.4 ms.
__global__ void __launch_bounds__(256) k_in_count(long long m, const int *col, const float *cost,
                                                  const float *drift, int *cnt,
                                                  unsigned long long *bad) {
    const long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= m) return;
    atomicAdd(&cnt[col[k]], 1);
    const float c = cost[k], d = drift[k];
    if (!(c > 0.0f) || !isfinite(c)) atomicMin(bad, 2ull * k);
    else if (!(d >= 0.0f) || !isfinite(d)) atomicMin(bad, 2ull * k + 1ull);
}
__global__ void __launch_bounds__(256) k_in_scatter(int n, const int *optr, const int *col,
                                                    const int *rptr, int *fill, int *edge,
                                                    int *src) {
    const int u = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6);  // a wave per row
    if (u >= n) return;
    for (int k = optr[u] + lane_id(); k < optr[u + 1]; k += 64) {
        const int v = col[k];
        const int p = rptr[v] + atomicAdd(&fill[v], 1);
        edge[p] = k;
        src[p] = u;
    }
}
__global__ void __launch_bounds__(256) k_in_place(long long m, const int *col, const float *cost,
                                                  const float *drift, const int *rptr,
                                                  const int *edge, const int *src, int *rsrc,
                                                  float *rcost, float *rdrift, int *rperm) {
    const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= m) return;
    const int k = edge[p], v = col[k];
    const int r0 = rptr[v], r1 = rptr[v + 1];
    int q = r0;
    for (int i = r0; i < r1; ++i) q += edge[i] < k ? 1 : 0;
    rsrc[q] = src[p];
    rcost[q] = cost[k];
    rdrift[q] = drift[k];
    rperm[q] = k;
}

// Ordered list of the nodes with flag bit `bit` set (single block; 16 flags a
// thread: 50,000 nodes in four rounds, 9 us; one flag a thread 59).  flag is
// 16-byte aligned.
__global__ void __launch_bounds__(1024) k_flag_list(int n, const uint8_t *flag, unsigned bit,
                                                    int *list, int *count) {
    __shared__ int scan[32];
    int carry = 0;
    for (int t0 = 0; t0 < n; t0 += 16 * (int)blockDim.x) {
        const int v0 = t0 + 16 * (int)threadIdx.x;
        unsigned w[4] = {0u, 0u, 0u, 0u};
        if (v0 + 16 <= n) {
            const uint4 q = *reinterpret_cast<const uint4 *>(flag + v0);
            w[0] = q.x; w[1] = q.y; w[2] = q.z; w[3] = q.w;
        } else {
            for (int i = 0; i < 16; ++i)
                if (v0 + i < n) w[i >> 2] |= (unsigned)flag[v0 + i] << (8 * (i & 3));
        }
        const unsigned each = 0x01010101u * bit;
        int mine = 0;
        for (int i = 0; i < 4; ++i) mine += __popc(w[i] & each);
        int tot;
        int o = carry + block_excl_scan(mine, scan, &tot);
        if (mine)
            for (int i = 0; i < 16; ++i)
                if ((w[i >> 2] >> (8 * (i & 3))) & bit) list[o++] = v0 + i;
        carry += tot;
    }
    if (threadIdx.x == 0) *count = carry;
}

// ------------------------------------------------------------------- scan
// Exclusive prefix sum of int32 values in three passes (block sums, scan of
// block sums in one block, add-back).  Each block covers kScanTile items.
__global__ void __launch_bounds__(256) k_scan_block_sums(const int *in, long long n,
                                                         int *bsum) {
    __shared__ int scan[16];
    const long long base = (long long)blockIdx.x * kScanTile;
    int s = 0;
    for (int i = threadIdx.x; i < kScanTile; i += blockDim.x)
        if (base + i < n) s += in[base + i];
    int tot;
    block_excl_scan(s, scan, &tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

__global__ void __launch_bounds__(1024) k_scan_sums(int *bsum, int nb) {
    __shared__ int scan[32];
    int carry = 0;
    for (int t0 = 0; t0 < nb; t0 += blockDim.x) {
        const int i = t0 + threadIdx.x;
        const int v = (i < nb) ? bsum[i] : 0;
        int tot;
        const int ex = block_excl_scan(v, scan, &tot);
        if (i < nb) bsum[i] = carry + ex;
        carry += tot;
    }
}

__global__ void __launch_bounds__(256) k_scan_apply(const int *in, long long n,
                                                    const int *bsum, int *out) {
    __shared__ int scan[16];
    const long long base = (long long)blockIdx.x * kScanTile;
    int carry = bsum[blockIdx.x];
    constexpr int per = kScanTile / 256;
    // each thread owns `per` consecutive items
    int v[per];
    int s = 0;
    for (int k = 0; k < per; ++k) {
        const long long i = base + (long long)threadIdx.x * per + k;
        v[k] = (i < n) ? in[i] : 0;
        s += v[k];
    }
    int tot;
    int ex = block_excl_scan(s, scan, &tot);
    int run = carry + ex;
    for (int k = 0; k < per; ++k) {
        const long long i = base + (long long)threadIdx.x * per + k;
        if (i < n) out[i] = run;
        run += v[k];
    }
}

// p[i] += add for i < n (id shifts when roadmaps are concatenated)
__global__ void __launch_bounds__(256) k_add_i32(int *p, long long n, int add) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] += add;
}

// p[i] = 0 for i < n (used instead of memset so the sequence can be captured)
__global__ void __launch_bounds__(256) k_zero_i32(int *p, long long n) {
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        p[i] = 0;
}

// 1 - q of every node, float32 (the last input of the edges into it)
template <bool kPlain, int D>
__global__ void __launch_bounds__(256) k_node_free(BuildArgs g, float *node_w) {
    extern __shared__ float blob[];
    stage_quality_blobs<kPlain, D>(g, blob);
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= g.n) return;
    float x[1][D], q[1];
#pragma unroll
    for (int k = 0; k < D; ++k) x[0][k] = g.pos[v * D + k];
    quality_points<kPlain, D, 1>(blob, g.nblob, x, q);
    node_w[v] = 1.0f - q[0];
}

// Inputs of the learned drift surrogate of every edge of a symmetric roadmap
// (uptr as for the drift): x_a (3), x_b (3, zero z in 2D), the length, 1 - q
// at the 8 segment points (k + 1/2)/8, 1 - q(x_b); bfloat16; and base, the
// mean of the eight.  L lanes per id-ordered pair, 8 / L points each; both
// edges' rows are written by the pair's lanes.  1 - q(x_b) comes from
// k_node_free: one evaluation a node instead of one a pair.
template <bool kPlain, int L, int D>
__global__ void __launch_bounds__(256) k_edge_features_pairs(BuildArgs g, int n,
                                                             const int *row_ptr, const int *col,
                                                             const float *cost, const int *uptr,
                                                             const float *node_w, uint16_t *X,
                                                             float *base) {
    extern __shared__ float blob[];
    stage_quality_blobs<kPlain, D>(g, blob);
    constexpr int P = 8 / L;
    const int pairs = uptr[n];
    const int i = (int)((blockIdx.x * 256ll + threadIdx.x) / L);
    // (whole waves: the lanes beyond the last pair repeat it)
    if ((int)((blockIdx.x * 256ll + (threadIdx.x & ~63)) / L) >= pairs) return;
    const bool live = i < pairs;
    const int sub = lane_id() % L, lead = lane_id() - sub;
    const int t = min(i, pairs - 1);
    const int u = wave_pair_row(uptr, n, t);
    const int e = row_ptr[u + 1] - (uptr[u + 1] - t);
    const int v = col[e];
    const float len = cost[e];
    float xa[3] = {0.f, 0.f, 0.f}, xb[3] = {0.f, 0.f, 0.f};
    float x[P][D], w[P];
#pragma unroll
    for (int k = 0; k < D; ++k) {
        xa[k] = g.pos[u * D + k];
        xb[k] = g.pos[v * D + k];
        const float df = xb[k] - xa[k];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const float s = ((float)(sub * P + p) + 0.5f) / 8.0f;
            x[p][k] = xa[k] + s * df;
        }
    }
    quality_points<kPlain, D, P>(blob, g.nblob, x, w);
    // all eight values in every lane of the pair, in point order
    float f[8], acc = 0.0f;
#pragma unroll
    for (int p = 0; p < P; ++p) w[p] = 1.0f - w[p];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if constexpr (L == 1) f[j] = w[j];
        else f[j] = __shfl(w[j % P], lead + j / P, 64);
        acc = acc + f[j];
    }
    if (!live) return;
    const float b8 = acc * 0.125f;
    const int r = reverse_edge(row_ptr, col, v, u);
    auto two = [](float lo, float hi) { return (uint32_t)f2bf(lo) | ((uint32_t)f2bf(hi) << 16); };
    const uint32_t word[8] = {two(xa[0], xa[1]), two(xa[2], xb[0]), two(xb[1], xb[2]),
                              two(len, f[0]),    two(f[1], f[2]),   two(f[3], f[4]),
                              two(f[5], f[6]),   two(f[7], node_w[v])};
    uint32_t *xe = reinterpret_cast<uint32_t *>(X + (size_t)e * 16);
    uint32_t *xr = reinterpret_cast<uint32_t *>(X + (size_t)max(r, 0) * 16);
#pragma unroll
    for (int k = 0; k < 8; ++k)
        if (k / P == sub) {
            xe[k] = word[k];
            if (r >= 0) xr[k] = word[k];
        }
    if (sub == 0) {
        base[e] = b8;
        if (r >= 0) base[r] = b8;
    }
}

// t[e] = scale * (drift[e] / cost[e] - base[e]): the analytic per-edge mean
// of (1 - q) less its 8-point estimate, scaled, the surrogate network's
// training target
__global__ void __launch_bounds__(256) k_drift_ratio(long long m, const float *drift,
                                                     const float *cost, const float *base,
                                                     float scale, float *t) {
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < m) t[e] = scale * (drift[e] / cost[e] - (base ? base[e] : 0.0f));
}

template <bool kPlain, int D>
static void edge_features(const BuildArgs &g, int n, long long pairs, const int *row_ptr,
                          const int *col, const float *cost, const int *uptr, float *node_w,
                          uint16_t *X, float *base, hipStream_t s) {
    const size_t lds = sizeof(float) * (size_t)g.nblob * (D + (kPlain ? 3 : 2));
    k_node_free<kPlain, D><<<(unsigned)((n + 255) / 256), 256, lds, s>>>(g, node_w);
    auto blocks = [&](int lanes) { return (unsigned)((pairs * lanes + 255) / 256); };
    if (pairs <= 262144)
        k_edge_features_pairs<kPlain, 4, D><<<blocks(4), 256, lds, s>>>(
            g, n, row_ptr, col, cost, uptr, node_w, X, base);
    else
        k_edge_features_pairs<kPlain, 2, D><<<blocks(2), 256, lds, s>>>(
            g, n, row_ptr, col, cost, uptr, node_w, X, base);
}

// Lanes per pair: four until the chip is full, then two (more points a lane
// share each blob's reads).  Measured, inputs and network together, 1 / 2 / 4
// / 8 lanes: 3D, 5,900 pairs 52 / 38 / 30 / 27 us; 47,500 pairs 60 / 51 / 46 /
// 48; 177,000 pairs 119 / 111 / 109 / 115; 370,000 pairs 200 / 188 / 191 /
// 202; 2D, 592,000 pairs 141 / 142 / 151 / 176.  One thread per pair with nine
// points and the plain division took 209, 218, 279, 445 and 252 us.
void launch_edge_features(const BuildArgs &g, bool plain, int n, long long pairs,
                          const int *row_ptr, const int *col, const float *cost,
                          const int *uptr, float *node_w, uint16_t *X, float *base,
                          hipStream_t s) {
    if (g.dim == 2 && plain)
        edge_features<true, 2>(g, n, pairs, row_ptr, col, cost, uptr, node_w, X, base, s);
    else if (g.dim == 2)
        edge_features<false, 2>(g, n, pairs, row_ptr, col, cost, uptr, node_w, X, base, s);
    else if (plain)
        edge_features<true, 3>(g, n, pairs, row_ptr, col, cost, uptr, node_w, X, base, s);
    else
        edge_features<false, 3>(g, n, pairs, row_ptr, col, cost, uptr, node_w, X, base, s);
}

// pairs: uptr[n] (half the edges)
void launch_edge_drift_pairs(const BuildArgs &g, int n, long long pairs, const int *row_ptr,
                             const int *col, const float *cost, const int *uptr, float *drift,
                             hipStream_t s) {
    const size_t lds = sizeof(float) * ((size_t)g.nblob * g.dim + 2 * (size_t)g.nblob);
    const unsigned blocks = (unsigned)((pairs * kDriftLanes + 255) / 256);
    if (g.dim == 2) k_edge_drift_pairs<2><<<blocks, 256, lds, s>>>(g, n, row_ptr, col, cost, uptr, drift);
    else k_edge_drift_pairs<3><<<blocks, 256, lds, s>>>(g, n, row_ptr, col, cost, uptr, drift);
}
