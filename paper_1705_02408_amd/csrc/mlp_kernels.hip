// Learned per-edge drift surrogate on the gfx950 matrix cores.
//
// Network: y = w3 . relu(W2^T h1 + b2) + b3,  h1 = bf16(relu(W1^T x + b1)),
// 16 -> 64 -> 64 -> 1, x and the weights in bfloat16, float32 accumulation
// (v_mfma_f32_32x32x16_bf16).  The prediction is the edge's mean
// "1 - quality" along its length; the drift increment is length * clamp(y, 0, 1).
//
// Layout.  One wave computes 32 edges at a time as transposed products
// (hidden x edges), so every lane owns one edge (lane % 32) and the
// accumulator registers of one layer can feed the B operand of the next
// directly.  For the 32x32 MFMA, accumulator register v of lane l holds row
// 8*(v/4) + 4*(l/32) + v%4 and column l%32; operand slot e of lane l holds
// K index 8*(l/32) + e.  Hidden units reach layer 2 in that row order, and the
// layer-2 weight fragments are loaded in the same permuted order.
//
// Training: one kernel a batch takes rows forward, back through layer 2 and
// into the weight gradients (matrix products with the rows as the K dimension,
// their operands transposed in LDS), one more sums the workgroups' partial
// gradients in a fixed order (deterministic) and applies Adam.
#include "device_common.h"
#include "mlp_kernels.h"

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short short8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

namespace {

__device__ __forceinline__ bf16x8 load8(const uint16_t *p) {
    const uint4 q = *reinterpret_cast<const uint4 *>(p);
    return __builtin_bit_cast(bf16x8, q);
}
__device__ __forceinline__ bf16x8 zero8() {
    const uint4 q = make_uint4(0u, 0u, 0u, 0u);
    return __builtin_bit_cast(bf16x8, q);
}
__device__ __forceinline__ bf16x8 pack8(const uint16_t *v) {
    short8 s;
#pragma unroll
    for (int e = 0; e < 8; ++e) s[e] = (short)v[e];
    return __builtin_bit_cast(bf16x8, s);
}
__device__ __forceinline__ f32x16 mfma(const bf16x8 &a, const bf16x8 &b, const f32x16 &c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// accumulator register v of a lane in half h holds tile row rowmap(v, h)
__device__ __forceinline__ int rowmap(int v, int h) { return 8 * (v >> 2) + 4 * h + (v & 3); }

struct Frags {
    bf16x8 a1[2];        // W1^T, hidden tile t
    bf16x8 a2[2][2][2];  // W2^T, output tile, input tile, K half
};

// where parameter W1[f][j] and W2[i][o] lie in the lanes' order: lane
// 32 h + c of a fragment, slot e
__device__ __forceinline__ int frag_w1(int f, int j) {
    return (((j >> 5) * 64 + 32 * (f >> 3) + (j & 31)) << 3) + (f & 7);
}
__device__ __forceinline__ int frag_w2(int i, int o) {
    const int r = i & 31, hs = r >> 4, h = (r >> 2) & 1, e = 4 * ((r >> 3) & 1) + (r & 3);
    const int frag = ((o >> 5) * 2 + (i >> 5)) * 2 + hs;
    return ((frag * 64 + 32 * h + (o & 31)) << 3) + e;
}

__device__ __forceinline__ void load_frags(const MlpDev &d, int l, Frags &f) {
#pragma unroll
    for (int t = 0; t < 2; ++t) f.a1[t] = load8(d.pb + kBfW1 + (t * 64 + l) * 8);
#pragma unroll
    for (int to = 0; to < 2; ++to)
#pragma unroll
        for (int ti = 0; ti < 2; ++ti)
#pragma unroll
            for (int hs = 0; hs < 2; ++hs)
                f.a2[to][ti][hs] = load8(d.pb + kBfW2F + ((((to * 2 + ti) * 2 + hs) * 64) + l) * 8);
}

// Forward of the 32 edges whose features the lane pair holds in bx.  Returns
// the output (both halves), the layer-1 accumulators (pre-bias) and the
// layer-2 pre-activations z2.
__device__ __forceinline__ float forward32(const Frags &f, const bf16x8 &bx, const float *sb1,
                                           const float *sb2, const float *sw3, float sb3,
                                           int h, f32x16 (&d1)[2], uint16_t (&h1)[2][16],
                                           f32x16 (&z2)[2]) {
    const f32x16 zero = {};
    d1[0] = mfma(f.a1[0], bx, zero);
    d1[1] = mfma(f.a1[1], bx, zero);
    bf16x8 bh[2][2];
#pragma unroll
    for (int ti = 0; ti < 2; ++ti) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
            h1[ti][v] = f2bf(fmaxf(d1[ti][v] + sb1[32 * ti + rowmap(v, h)], 0.0f));
        bh[ti][0] = pack8(&h1[ti][0]);
        bh[ti][1] = pack8(&h1[ti][8]);
    }
    float y = 0.0f;
#pragma unroll
    for (int to = 0; to < 2; ++to) {
        f32x16 acc = {};
#pragma unroll
        for (int ti = 0; ti < 2; ++ti)
#pragma unroll
            for (int hs = 0; hs < 2; ++hs) acc = mfma(f.a2[to][ti][hs], bh[ti][hs], acc);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int o = 32 * to + rowmap(v, h);
            const float z = acc[v] + sb2[o];
            z2[to][v] = z;
            y += sw3[o] * fmaxf(z, 0.0f);
        }
    }
    y += __shfl_xor(y, 32, 64);
    return y + sb3;
}

// the bfloat16 copies of parameter i
__device__ __forceinline__ void store_bf16(uint16_t *pb, int i, float p) {
    const uint16_t q = f2bf(p);
    if (i < kOffB1) {
        pb[kBfW1 + frag_w1((i - kOffW1) / kMlpH, (i - kOffW1) % kMlpH)] = q;
    } else if (i >= kOffW2 && i < kOffB2) {
        pb[kBfW2 + (i - kOffW2)] = q;
        pb[kBfW2F + frag_w2((i - kOffW2) / kMlpH, (i - kOffW2) % kMlpH)] = q;
    } else if (i >= kOffW3 && i < kOffB3) {
        pb[kBfW3 + (i - kOffW3)] = q;
    }
}

__device__ __forceinline__ void load_small(const MlpDev &d, float *sb1, float *sb2, float *sw3,
                                           float *sb3) {
    for (int i = threadIdx.x; i < kMlpH; i += blockDim.x) {
        sb1[i] = d.p[kOffB1 + i];
        sb2[i] = d.p[kOffB2 + i];
        sw3[i] = bf2f(d.pb[kBfW3 + i]);
    }
    if (threadIdx.x == 0) *sb3 = d.p[kOffB3];
    __syncthreads();
}

// sums over the 32 lanes of each half: lane c's result is that of v[c] (each
// step hands half of the values over: 31 exchanges instead of 160)
template <int K>
__device__ __forceinline__ float half_sums(float (&v)[2 * K], int c) {
    const bool up = (c & K) != 0;
    float u[K];
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const float keep = up ? v[i + K] : v[i], send = up ? v[i] : v[i + K];
        u[i] = keep + __shfl_xor(send, K, 64);
    }
    if constexpr (K == 1) return u[0];
    else return half_sums<K / 2>(u, c);
}

}  // namespace

// y = network(X[i]) and drift = len * clamp(base + y / kResidualScale, 0, 1).
__global__ void __launch_bounds__(256) k_mlp_infer(MlpDev d, const uint16_t *X, long long n,
                                                   const float *len, const float *base, float *y,
                                                   float *drift) {
    __shared__ float sb1[kMlpH], sb2[kMlpH], sw3[kMlpH], sb3;
    load_small(d, sb1, sb2, sw3, &sb3);
    const int l = lane_id(), h = l >> 5, c = l & 31;
    Frags f;
    load_frags(d, l, f);
    const long long waves = (long long)gridDim.x * (blockDim.x >> 6);
    for (long long tile = (long long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
         tile * 32 < n; tile += waves) {
        const long long i = tile * 32 + c;
        const bool valid = i < n;
        const bf16x8 bx = valid ? load8(X + i * kMlpIn + 8 * h) : zero8();
        f32x16 d1[2], z2[2];
        uint16_t h1[2][16];
        const float out = forward32(f, bx, sb1, sb2, sw3, sb3, h, d1, h1, z2);
        if (h == 0 && valid) {
            if (y) y[i] = out;
            if (drift) {
                const float r = (base ? base[i] : 0.0f) + out * (1.0f / kResidualScale);
                drift[i] = len[i] * fminf(fmaxf(r, 0.0f), 1.0f);
            }
        }
    }
}

__global__ void __launch_bounds__(256) k_mlp_loss(MlpDev d, const uint16_t *X, const float *t,
                                                  const long long *idx, long long n,
                                                  float *acc) {
    __shared__ float sb1[kMlpH], sb2[kMlpH], sw3[kMlpH], sb3, red[16];
    load_small(d, sb1, sb2, sw3, &sb3);
    const int l = lane_id(), h = l >> 5, c = l & 31;
    Frags f;
    load_frags(d, l, f);
    const long long waves = (long long)gridDim.x * (blockDim.x >> 6);
    float s = 0.0f;
    for (long long tile = (long long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
         tile * 32 < n; tile += waves) {
        const long long i = tile * 32 + c;
        const bool valid = i < n;
        const long long row = valid ? idx[i] : 0;
        const bf16x8 bx = valid ? load8(X + row * kMlpIn + 8 * h) : zero8();
        const float want = valid ? t[row] : 0.0f;
        f32x16 d1[2], z2[2];
        uint16_t h1[2][16];
        const float e = forward32(f, bx, sb1, sb2, sw3, sb3, h, d1, h1, z2) - want;
        if (h == 0 && valid) s += e * e;
    }
    s = wave_sum(s);
    if (l == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < (int)(blockDim.x >> 6); ++w) s += red[w];
        atomicAdd(acc, s);
    }
}

// One training batch over the rows t.idx[0..B): outputs and the partial sums
// of every parameter's gradient.  A workgroup takes kTrainRows rows at a time,
// a wave 32 of them: forward, dZ2 = dy w3 (where z2 > 0), dZ1 = W2 dZ2 (where
// z1 > 0) with the accumulators of one product as the operand of the next.
// The weight gradients
//   dW2^T[o][j] = sum_b dZ2T[o][b] H1T[j][b],  dW1^T[j][f] = sum_b dZ1T[j][b] XT[f][b]
// need these values with the rows as K: they go through LDS, transposed, and
// each wave sums one 32x32 tile of dW2 (the first two one of dW1) over the
// workgroup's rows.  Bounded by the latency of this chain: a batch of 4,096
// rows is 128 waves, 12.2 us.  (Three kernels with the activations in memory
// and each wave its own partial sums took 43 us; each value's sum over the rows
// by itself, 160 exchanges for 32 values, and operands gathered two bytes at a
// time were a good part of it.)
__global__ void __launch_bounds__(256) k_mlp_train(MlpDev d, MlpTrain t) {
    constexpr int kRow = kTrainRows + 8;  // (16-byte loads of 32 rows spread over the banks)
    __shared__ __align__(16) uint16_t sx[kMlpIn][kRow], sh1[kMlpH][kRow], sdz1[kMlpH][kRow],
        sdz2[kMlpH][kRow];
    __shared__ float sb1[kMlpH], sb2[kMlpH], sw3[kMlpH], sb3, red[4][3][kMlpH], redb[4];
    const int l = lane_id(), h = l >> 5, c = l & 31;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int k = 32 * w + c;  // the lane pair's row of the workgroup's
    // a group's index, then its inputs: two trips to memory, begun before the
    // weights are waited for
    bool valid;  // (whole waves)
    bf16x8 bx;
    float want;
    auto fetch = [&](int b) {
        valid = b < t.B;
        const long long row = valid ? t.idx[b] : 0;
        bx = valid ? load8(t.X + row * kMlpIn + 8 * h) : zero8();
        want = valid ? t.t[row] : 0.0f;
    };
    fetch((int)blockIdx.x * kTrainRows + k);
    Frags f;
    load_frags(d, l, f);
    // W2 with rows hidden, K over the outputs in the accumulators' order
    bf16x8 aw[2][2][2];
#pragma unroll
    for (int th = 0; th < 2; ++th)
#pragma unroll
        for (int to = 0; to < 2; ++to)
#pragma unroll
            for (int hs = 0; hs < 2; ++hs) {
                const uint16_t *row = d.pb + kBfW2 + (32 * th + c) * kMlpH + 32 * to + 16 * hs + 4 * h;
                const uint2 a = *reinterpret_cast<const uint2 *>(row);
                const uint2 b = *reinterpret_cast<const uint2 *>(row + 8);
                aw[th][to][hs] = __builtin_bit_cast(bf16x8, make_uint4(a.x, a.y, b.x, b.y));
            }
    load_small(d, sb1, sb2, sw3, &sb3);
    const float inv = 2.0f / (float)t.B;
    f32x16 g2 = {}, g1 = {};  // this wave's tile of dW2^T and dW1^T
    float s3 = 0.0f, s2 = 0.0f, s1 = 0.0f, gb3 = 0.0f;
    for (int r0 = (int)blockIdx.x * kTrainRows; r0 < t.B; r0 += (int)gridDim.x * kTrainRows) {
        const int b = r0 + k;
        {
            const uint4 raw = __builtin_bit_cast(uint4, bx);
            const uint32_t x[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
            for (int e = 0; e < 8; ++e)
                sx[8 * h + e][k] = (uint16_t)(x[e >> 1] >> (16 * (e & 1)));
        }
        f32x16 d1[2], z2[2];
        uint16_t h1[2][16];
        const float y = forward32(f, bx, sb1, sb2, sw3, sb3, h, d1, h1, z2);
        const float dy = valid ? inv * (y - want) : 0.0f;
        if (h == 0) gb3 += dy;
        float v3[32], v2[32], v1[32];
        bf16x8 bz[2][2];
#pragma unroll
        for (int to = 0; to < 2; ++to) {
            uint16_t dzb[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int o = 32 * to + rowmap(v, h);
                const float z = z2[to][v];
                const float pass = dy * sw3[o];  // (read by every lane: no branch)
                const float dz = z > 0.0f ? pass : 0.0f;
                dzb[v] = f2bf(dz);
                sdz2[o][k] = dzb[v];
                sh1[o][k] = h1[to][v];
                v3[16 * to + v] = dy * fmaxf(z, 0.0f);
                v2[16 * to + v] = dz;
            }
            bz[to][0] = pack8(&dzb[0]);
            bz[to][1] = pack8(&dzb[8]);
        }
#pragma unroll
        for (int th = 0; th < 2; ++th) {
            f32x16 acc = {};
#pragma unroll
            for (int to = 0; to < 2; ++to)
#pragma unroll
                for (int hs = 0; hs < 2; ++hs) acc = mfma(aw[th][to][hs], bz[to][hs], acc);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int hid = 32 * th + rowmap(v, h);
                const float dz = d1[th][v] + sb1[hid] > 0.0f ? acc[v] : 0.0f;
                sdz1[hid][k] = f2bf(dz);
                v1[16 * th + v] = dz;
            }
        }
        s3 += half_sums<16>(v3, c);
        s2 += half_sums<16>(v2, c);
        s1 += half_sums<16>(v1, c);
        __syncthreads();
#pragma unroll
        for (int kk = 8 * h; kk < kTrainRows; kk += 16) {
            g2 = mfma(load8(&sdz2[32 * (w >> 1) + c][kk]), load8(&sh1[32 * (w & 1) + c][kk]), g2);
            if (w < 2)
                g1 = mfma(load8(&sdz1[32 * w + c][kk]), c < kMlpIn ? load8(&sx[c][kk]) : zero8(), g1);
        }
        __syncthreads();
        // (not before: a barrier waits for stores on their way)
        if (h == 0 && valid) t.y[b] = y;
        fetch(b + (int)gridDim.x * kTrainRows);
    }
    float *part = t.part + (size_t)blockIdx.x * kGradWords;
#pragma unroll
    for (int v = 0; v < 16; v += 4) {
        const int o = 32 * (w >> 1) + rowmap(v, h), j = 32 * (w & 1) + c;
        *reinterpret_cast<float4 *>(part + kOffW2 + j * kMlpH + o) =
            make_float4(g2[v], g2[v + 1], g2[v + 2], g2[v + 3]);
        if (w < 2 && c < kMlpIn)
            *reinterpret_cast<float4 *>(part + kOffW1 + c * kMlpH + 32 * w + rowmap(v, h)) =
                make_float4(g1[v], g1[v + 1], g1[v + 2], g1[v + 3]);
    }
    const int o = 32 * (c >> 4) + rowmap(c & 15, h);
    red[w][0][o] = s3;
    red[w][1][o] = s2;
    red[w][2][o] = s1;
    gb3 = wave_sum(gb3);
    if (l == 0) redb[w] = gb3;
    __syncthreads();
    if (threadIdx.x < 3 * kMlpH) {
        const int q = (int)threadIdx.x / kMlpH, i = (int)threadIdx.x % kMlpH;
        part[(q == 0 ? kOffW3 : q == 1 ? kOffB2 : kOffB1) + i] =
            (red[0][q][i] + red[1][q][i]) + (red[2][q][i] + red[3][q][i]);
    } else if (threadIdx.x == 3 * kMlpH) {
        part[kOffB3] = (redb[0] + redb[1]) + (redb[2] + redb[3]);
    }
}

// Sum the workgroups' partials in a fixed order, then (optionally) one Adam
// step on the float32 masters and a refresh of the bfloat16 copies.  64
// parameters a block, each by eight threads: 3.9 us a batch of 4,096 rows (16.3
// with a thread a parameter, all partials one after the other).
__global__ void __launch_bounds__(512) k_mlp_adam(MlpAdam a) {
    __shared__ float red[8][64];
    const int l = lane_id(), w = (int)threadIdx.x >> 6;
    const int i = blockIdx.x * 64 + l;
    float gs = 0.0f;
    if (i < kMlpParams)
        for (int g = w; g < a.nparts; g += 8) gs += a.part[(size_t)g * kGradWords + i];
    red[w][l] = gs;
    __syncthreads();
    if (w != 0 || i >= kMlpParams) return;
    gs = ((red[0][l] + red[1][l]) + (red[2][l] + red[3][l])) +
         ((red[4][l] + red[5][l]) + (red[6][l] + red[7][l]));
    if (a.grad_out) a.grad_out[i] = gs;
    if (!a.apply) return;
    const float m = a.beta1 * a.m[i] + (1.0f - a.beta1) * gs;
    const float v = a.beta2 * a.v[i] + (1.0f - a.beta2) * gs * gs;
    a.m[i] = m;
    a.v[i] = v;
    const float p = a.p[i] - a.lr * (m / a.c1) / (sqrtf(v / a.c2) + a.eps);
    a.p[i] = p;
    store_bf16(a.pb, i, p);
}

__global__ void __launch_bounds__(256) k_mlp_to_bf16(const float *p, uint16_t *pb) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kMlpParams) store_bf16(pb, i, p[i]);
}
