// Kernels of the double-integrator roadmap (position and velocity in 3D):
// minimum-energy fixed-time steering costs, selection of each state's
// cheapest reachable targets, and the drift increment along each trajectory.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "graph_kernels.h"

constexpr int kSteerThreads = 256;
constexpr int kSteerMaxWidth = 1024;  // candidates ranked per selection round
constexpr int kSteerMaxSteps = 255;   // check steps per trajectory (K + 1 <= 256 points)
constexpr int kSteerMaxOut = 64;      // out-degree limit
constexpr int kSteerMaxBoxes = 4096;
constexpr int kNearList = 256;        // candidates one wave lists and ranks (k_steer_near)
constexpr int kNearShells = 4;        // shells a wave lists for a source
constexpr int kFarThreads = 512;
constexpr int kFarList = 4096;        // candidates one workgroup lists and ranks (k_steer_far)
constexpr int kTrajTerms = 512;       // chord terms a wave holds (at least kSteerMaxSteps)
constexpr int kSteerNear = 64;        // boxes near a source that the quick test looks at
constexpr int kSteerShells = 4096;    // shells (thinned ones counted) tried for a source

struct SteerArgs {
    int n;
    const float *pos;  // [n][3]
    const float *vel;  // [n][3]
    int nbox;
    const float *blo;  // [nbox][3]
    const float *bhi;
    int nblob;
    const float *mu;   // [nblob][3]
    const float *sig;
    const float *amp;
    float T;           // steering time
    int K;             // check steps (K + 1 points)
    int k_out;         // out-degree
};

// bounding boxes of the states, the sum of the position box's edges, a
// margin far above the roundings of a trajectory point, and the speed ball's
// offset and radius (speed_ball; infinite when no check time lies inside)
struct SteerBounds {
    float plo[3], phi[3], vlo[3], vhi[3], extent, eps, vr, rho;
};
// sources that k_steer_near did not finish, and the cost up to which it ranked
struct SteerFar {
    int *source;  // [n]
    float *tau;   // [n]
    int *count;
};

// Per source u: the first k_out reachable targets in ascending (J, id) order
// -> nbr[u * k_out + i], ncost (J), ncnt[u], from the states of a uniform
// grid in cell order.  tau0: cost below which a typical source has about 64
// targets; kPow2: T is a power of two (within 2^-40..2^40).
template <bool kPow2>
__global__ void k_steer_near(SteerArgs a, GridArgs gr, SteerBounds sb, const float4 *spos,
                             const float4 *svel, float tau0, int *nbr, float *ncost, int *ncnt,
                             SteerFar far);
template <bool kPow2>
__global__ void k_steer_far(SteerArgs a, GridArgs gr, SteerBounds sb, const float4 *spos,
                            const float4 *svel, float tau0, int *nbr, float *ncost, int *ncnt,
                            SteerFar far, int *left, int *nleft);
__global__ void k_steer_scatter(SteerArgs a, GridArgs gr, const int *cell, const int *slot,
                                float4 *spos, float4 *svel);
// The same for the sources of `left`, by ranking all states.  *err |= 1 when
// more than the ranking buffer's worth of candidates share one steering cost
// (the selection cannot order them).
__global__ void k_steer_select(SteerArgs a, const int *left, const int *nleft, int *nbr,
                               float *ncost, int *ncnt, int *err);
// rows of the CSR, each sorted by target id
__global__ void k_steer_compact(int n, int k_out, const int *row_ptr, const int *nbr,
                                const float *ncost, const int *ncnt, int *col, float *cost);
// a blob widened to float64: centre, 1 / (2 sigma^2), amplitude, and the
// exponent beyond which its value counts as zero (below 2^-65)
struct SteerBlob {
    double mu[3], inv, amp, end, pad[2];
};
__global__ void k_steer_blobs(int nblob, const float *mu, const float *sig, const float *amp,
                              SteerBlob *out);
// drift increment and (elen nullable) polyline length of every edge; blobs
// from k_steer_blobs
void launch_traj_drift(const SteerArgs &a, const SteerBlob *blobs, const int *row_ptr,
                       const int *col, float *drift, float *elen, hipStream_t s);
// surrogate inputs of every edge along its trajectory, and the 8-point base
__global__ void k_traj_features(SteerArgs a, const int *row_ptr, const int *col,
                                const float *elen, uint16_t *X, float *base);
