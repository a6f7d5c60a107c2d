// Learned CG preconditioner kernels: node features over the 1-ring, the
// per-node MLP 12 -> 64 -> 64 -> 3 (softplus) on bf16 matrix cores, and its
// training (forward + backward, Adam).
//
// Preconditioner (per node i, N(i) = nodes sharing an element with i):
//   g_i = D_i^-1 r_i (0 on prescribed DOFs), s_i = 1-ring RMS of g,
//   z_i = g_i + s_i * MLP(f_i), prescribed DOFs -> 0, with the 12 features
//   f = [g_i/s_i, mean_N(i) g/s_i, log(D_i / mean_{N(i)+i} D), prescribed
//   fraction of i, of N(i), |N(i)|/26].
// Weights and every layer input are rounded to bfloat16; accumulation is FP32.
#include "efem_mlp.h"

namespace efem {

typedef short s4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

// float -> bfloat16 bits, round to nearest even (one hardware conversion on gfx950)
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
__device__ __forceinline__ float bfr(float f) { return bf2f(f2bf(f)); }

// two bfloat16 values, a in the low half (one conversion for both)
typedef __bf16 bf2_t __attribute__((ext_vector_type(2)));
typedef float f2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf(float a, float b)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f2_t){a, b}, bf2_t));
}

// softplus(x) = max(x, 0) + ln(1 + t), t = e^-|x| in (0, 1], with the
// hardware base-2 exponential and logarithm (the exponent is <= 0 and the
// logarithm's argument lies in [1, 2], so neither needs range reduction).
// For x < 0 softplus is ln(1 + t) alone, so that term needs relative
// accuracy, which the logarithm of the rounded u = 1 + t lacks for small t
// (off by up to 2^-24 / t relative: several bfloat16 ulps once x < -12).
// The rounding error e = (1 + t) - u = t - (u - 1) is exact (u - 1 is exact
// for u in [1, 2], and t and u - 1 differ by at most an ulp of u), and
// ln(1 + t) = ln u + ln(1 + e/u) = ln u + e to within 2^-24 relative
// (|e| <= 2^-24, u >= 1); where 1 + t rounds to 1 this gives t itself.
__device__ __forceinline__ float softplus(float x)
{
    const float t = __builtin_amdgcn_exp2f(-fabsf(x) * 1.4426950408889634f);
    const float u = 1.f + t;
    const float e = t - (u - 1.f);
    return fmaxf(x, 0.f) + fmaf(0.6931471805599453f, __builtin_amdgcn_logf(u), e);
}

// ------------------------------------------------------------------ features

// Static features of node i into slots 6..15: its diagonal di, the sums sd over
// its closed 1-ring, its own prescribed components and its neighbours' (sm).
__device__ __forceinline__ void store_static(uint16_t *__restrict__ X, int64_t i, int deg, const double di[3],
                                             const double sd[3], int mi, int sm)
{
    uint16_t x[10];
#pragma unroll
    for (int c = 0; c < 3; ++c) x[c] = f2bf((float)log(di[c] / (sd[c] / (deg + 1))));
    x[3] = f2bf((float)mi / 3.f);
    x[4] = f2bf((float)sm / (3.f * (float)max(deg, 1)));
    x[5] = f2bf((float)deg / 26.f);
    x[6] = x[7] = x[8] = x[9] = 0;
    uint32_t *o = reinterpret_cast<uint32_t *>(X + i * kInPad + 6);
#pragma unroll
    for (int k = 0; k < 5; ++k) o[k] = (uint32_t)x[2 * k] | (uint32_t)x[2 * k + 1] << 16;
}

// Dynamic features of node i into slots 0..5 and its scale: its g, the sums s of
// its neighbours' g, and q = |g|^2 over its closed 1-ring.
__device__ __forceinline__ void store_dynamic(uint16_t *__restrict__ X, float *__restrict__ s_out, int64_t i, int deg,
                                              const float4 gi, float s0, float s1, float s2, float q)
{
    const float s = sqrtf(q / (3.f * (float)(deg + 1)));
    uint16_t *x = X + i * kInPad;
    if (s > 0.f) {
        const float rs = 1.f / s, rd = rs / (float)max(deg, 1);
        x[0] = f2bf(gi.x * rs), x[1] = f2bf(gi.y * rs), x[2] = f2bf(gi.z * rs);
        x[3] = f2bf(s0 * rd), x[4] = f2bf(s1 * rd), x[5] = f2bf(s2 * rd);
    } else {
        x[0] = x[1] = x[2] = x[3] = x[4] = x[5] = 0;
    }
    s_out[i] = s;
}

// Static features (depend on the Jacobi diagonal and the mask only): slots
// 6..15.  Bound by the gather of the neighbours' diagonals from L2.  The
// 1-ring comes column-major (ell, as in k_feat_dyn), so each step's indices are
// one coalesced load, and eight neighbours are in flight at once: 18.6 us for
// 274,625 nodes of 26 neighbours (24.7 us with four loads between waits; 63 us
// by row-wise lists, where every lane walked its own range).
template <bool MASK>
__global__ void __launch_bounds__(256) k_feat_static(int64_t n, const int64_t *__restrict__ ptr,
                                                     const int32_t *__restrict__ ell,
                                                     const double *__restrict__ diag,
                                                     const uint8_t *__restrict__ nmask, uint16_t *__restrict__ X)
{
    constexpr int kB = 8;   // neighbours in flight
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int deg = (int)(ptr[i + 1] - ptr[i]);
    const double di[3] = {diag[3 * i], diag[3 * i + 1], diag[3 * i + 2]};
    double sd[3] = {di[0], di[1], di[2]};
    int sm = 0, k = 0;
    for (; k + kB <= deg; k += kB) {
        int64_t j[kB];
        double d[kB][3];
        int m[kB];
#pragma unroll
        for (int b = 0; b < kB; ++b) j[b] = ell[(int64_t)(k + b) * n + i];
#pragma unroll
        for (int b = 0; b < kB; ++b) {
            d[b][0] = diag[3 * j[b]], d[b][1] = diag[3 * j[b] + 1], d[b][2] = diag[3 * j[b] + 2];
            m[b] = MASK ? nmask[j[b]] : 0;
        }
#pragma unroll
        for (int b = 0; b < kB; ++b) {
            sd[0] += d[b][0], sd[1] += d[b][1], sd[2] += d[b][2];
            if (MASK) sm += __popc(m[b]);
        }
    }
    for (; k < deg; ++k) {
        const int64_t j = ell[(int64_t)k * n + i];
        sd[0] += diag[3 * j], sd[1] += diag[3 * j + 1], sd[2] += diag[3 * j + 2];
        if (MASK) sm += __popc(nmask[j]);
    }
    store_static(X, i, deg, di, sd, MASK ? __popc(nmask[i]) : 0, sm);
}

// g = D^-1 r per node with |g|^2, one 16-byte record each, so that the
// 1-ring gather of the features reads one vector per neighbour.
__global__ void k_g4(int64_t n, const float *__restrict__ r, const float *__restrict__ dinv,
                     float4 *__restrict__ g4)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float a = r[3 * i] * dinv[3 * i], b = r[3 * i + 1] * dinv[3 * i + 1], c = r[3 * i + 2] * dinv[3 * i + 2];
    g4[i] = make_float4(a, b, c, a * a + b * b + c * c);
}

// Dynamic features (slots 0..5) and the scale s from g4 = (D^-1 r, |D^-1 r|^2)
// (dinv = 0 on prescribed DOFs).  The 1-ring comes column-major (ell[k][i],
// padded with the zero record g4[n]), so every neighbour slot is one
// coalesced index load; slots are taken two at a time.
__global__ void k_feat_dyn(int64_t n, const int64_t *__restrict__ ptr, const int32_t *__restrict__ ell,
                           int max_deg, const float4 *__restrict__ g4, uint16_t *__restrict__ X,
                           float *__restrict__ s_out)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int deg = (int)(ptr[i + 1] - ptr[i]);
    const float4 gi = g4[i];
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, q = gi.w;
    int k = 0;
    for (; k + 8 <= max_deg; k += 8) {   // four pairs in flight
        int32_t j[8];
        float4 v[8];
#pragma unroll
        for (int b = 0; b < 8; ++b) j[b] = ell[(int64_t)(k + b) * n + i];
#pragma unroll
        for (int b = 0; b < 8; ++b) v[b] = g4[j[b]];
#pragma unroll
        for (int b = 0; b < 8; b += 2) {
            s0 += v[b].x + v[b + 1].x;
            s1 += v[b].y + v[b + 1].y;
            s2 += v[b].z + v[b + 1].z;
            q += v[b].w + v[b + 1].w;
        }
    }
    for (; k + 2 <= max_deg; k += 2) {
        const float4 a = g4[ell[(int64_t)k * n + i]], b = g4[ell[(int64_t)(k + 1) * n + i]];
        s0 += a.x + b.x;
        s1 += a.y + b.y;
        s2 += a.z + b.z;
        q += a.w + b.w;
    }
    if (k < max_deg) {
        const float4 a = g4[ell[(int64_t)k * n + i]];
        s0 += a.x;
        s1 += a.y;
        s2 += a.z;
        q += a.w;
    }
    store_dynamic(X, s_out, i, deg, gi, s0, s1, s2, q);
}

// Both at once, for an apply or training rows at a new diagonal: the 1-ring's
// indices are read once, and a neighbour's diagonal, mask and g4 are in flight
// together.  The sums run in the order of the two kernels above.  Bound by the
// gather's loads (41 bytes in four loads a neighbour): 25 us for 274,625 nodes of
// 26 neighbours, 30.5 us for the two kernels; the same within 1 us with two to
// eight neighbours in flight (eight: 3 waves per SIMD with 64-bit indices, 33 us).
template <bool MASK>
__global__ void __launch_bounds__(256) k_feat_all(int64_t n, const int64_t *__restrict__ ptr,
                                                  const int32_t *__restrict__ ell, int max_deg,
                                                  const double *__restrict__ diag, const uint8_t *__restrict__ nmask,
                                                  const float4 *__restrict__ g4, uint16_t *__restrict__ X,
                                                  float *__restrict__ s_out)
{
    constexpr int kB = 4;   // neighbours in flight
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int deg = (int)(ptr[i + 1] - ptr[i]);
    const float4 gi = g4[i];
    const double di[3] = {diag[3 * i], diag[3 * i + 1], diag[3 * i + 2]};
    double sd[3] = {di[0], di[1], di[2]};
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, q = gi.w;
    int sm = 0;
    auto add = [&](const float4 *v, const double (*d)[3], const int *m, int b) {
        s0 += v[b].x + v[b + 1].x;
        s1 += v[b].y + v[b + 1].y;
        s2 += v[b].z + v[b + 1].z;
        q += v[b].w + v[b + 1].w;
#pragma unroll
        for (int e = b; e < b + 2; ++e) {
            sd[0] += d[e][0], sd[1] += d[e][1], sd[2] += d[e][2];
            if (MASK) sm += __popc(m[e]);
        }
    };
    // one neighbour's values; past the node's own ring (j = n) all are zero
    auto load = [&](int32_t j, float4 &v, double d[3], int &m) {
        v = g4[j];
        const bool in = j < n;
        const int32_t jj = in ? j : (int32_t)i;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double t = diag[3 * (int64_t)jj + c];
            d[c] = in ? t : 0.0;
        }
        const int t = MASK ? nmask[jj] : 0;
        m = in ? t : 0;
    };
    for (int k = 0; k < max_deg; k += kB) {
        int32_t j[kB];
        float4 v[kB];
        double d[kB][3];
        int m[kB];
#pragma unroll
        for (int b = 0; b < kB; ++b) j[b] = k + b < max_deg ? ell[(int64_t)(k + b) * n + i] : (int32_t)n;
#pragma unroll
        for (int b = 0; b < kB; ++b) load(j[b], v[b], d[b], m[b]);
#pragma unroll
        for (int b = 0; b < kB; b += 2) add(v, d, m, b);
    }
    store_static(X, i, deg, di, sd, MASK ? __popc(nmask[i]) : 0, sm);
    store_dynamic(X, s_out, i, deg, gi, s0, s1, s2, q);
}

// ------------------------------------------------------------- MLP forward

// One wave evaluates 16 nodes per step on 16x16x16 bf16 matrix cores, nodes on
// the N dimension: D[h][node] = sum_k W[h][k] H[k][node].  The accumulator
// layout (lane = node + 16*(h/4), element h%4) is the B-operand layout of the
// next layer, so activations never leave registers.  Lane l holds
//   A[m][k]: m = l%16, k = 4(l/16)+v;  B[k][n]: n = l%16, k = 4(l/16)+v;
//   D[m][n]: n = l%16, m = 4(l/16)+v.
struct MlpRegs {
    s4 A1[4], A2[4][4], A3[4];
    float B1[4][4], B2[4][4], B3[4];
};

// Four consecutive parameters per load: every operand and bias of a lane starts
// at a multiple of four in the parameter vector (kOff* and the row lengths 12
// and 64 are), and W is the context's own 256-byte aligned copy.
__device__ __forceinline__ void load_weights(const uint16_t *__restrict__ W, MlpRegs &R)
{
    static_assert(kIn % 4 == 0 && kHid % 4 == 0 && kOffB1 % 4 == 0 && kOffW2 % 4 == 0 && kOffB2 % 4 == 0
                      && kOffW3 % 4 == 0, "four-wide weight loads");
    const int lane = threadIdx.x & 63, col = lane & 15, quad = lane >> 4;
    const s4 none = {0, 0, 0, 0};
    auto at = [&](int k) { return *reinterpret_cast<const s4 *>(W + k); };
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        R.A1[t] = quad < 3 ? at(kOffW1 + (16 * t + col) * kIn + 4 * quad) : none;
        R.A3[t] = col < kOut ? at(kOffW3 + col * kHid + 16 * t + 4 * quad) : none;
        const s4 b1 = at(kOffB1 + 16 * t + 4 * quad), b2 = at(kOffB2 + 16 * t + 4 * quad);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            R.B1[t][v] = bf2f((uint16_t)b1[v]);
            R.B2[t][v] = bf2f((uint16_t)b2[v]);
        }
#pragma unroll
        for (int t2 = 0; t2 < 4; ++t2) R.A2[t2][t] = at(kOffW2 + (16 * t2 + col) * kHid + 16 * t + 4 * quad);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) R.B3[v] = (4 * quad + v < kOut) ? bf2f(W[kOffB3 + 4 * quad + v]) : 0.f;
}

// The bf16 activations of one hidden layer for this lane's node: hidden
// units 16 t + 4 quad + (0..3) of tile t, one 8-byte store per tile
// (H [n][64], only where node < n).
__device__ __forceinline__ void store_layer(uint16_t *__restrict__ H, const s4 h[4], int64_t node, int64_t n)
{
    if (node >= n) return;
    const int quad = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int t = 0; t < 4; ++t) *reinterpret_cast<s4 *>(H + node * kHid + 16 * t + 4 * quad) = h[t];
}

// four activations, bf16(softplus(d + b))
__device__ __forceinline__ s4 act4(const f4 d, const float b[4])
{
    uint2 w;
    w.x = pack_bf(softplus(d[0] + b[0]), softplus(d[1] + b[1]));
    w.y = pack_bf(softplus(d[2] + b[2]), softplus(d[3] + b[3]));
    return __builtin_bit_cast(s4, w);
}

// out[v] for v < 3 is valid in lanes 0..15 (node = lane).  LAYERS: the two
// hidden layers' bf16 activations also go to H1 and H2 ([n][64]) for this
// lane's node.
template <bool LAYERS = false>
__device__ __forceinline__ f4 mlp16(const MlpRegs &R, s4 xb, uint16_t *H1 = nullptr, uint16_t *H2 = nullptr,
                                    int64_t node = 0, int64_t n = 0)
{
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    s4 hb[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const f4 d = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(R.A1[t], xb, zero, 0, 0, 0);
        hb[t] = act4(d, R.B1[t]);
    }
    if constexpr (LAYERS) store_layer(H1, hb, node, n);
    s4 h2[4];
#pragma unroll
    for (int t2 = 0; t2 < 4; ++t2) {
        f4 d = zero;
#pragma unroll
        for (int t = 0; t < 4; ++t) d = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(R.A2[t2][t], hb[t], d, 0, 0, 0);
        h2[t2] = act4(d, R.B2[t2]);
    }
    if constexpr (LAYERS) store_layer(H2, h2, node, n);
    f4 o = zero;
#pragma unroll
    for (int t = 0; t < 4; ++t) o = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(R.A3[t], h2[t], o, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 4; ++v) o[v] += R.B3[v];
    return o;
}

__device__ __forceinline__ s4 load_x(const uint16_t *__restrict__ X, int64_t node, int64_t n)
{
    const int quad = (threadIdx.x & 63) >> 4;
    if (node >= n) return s4{0, 0, 0, 0};
    return *reinterpret_cast<const s4 *>(X + node * kInPad + 4 * quad);
}

// out [n, 3] = MLP(X); LAYERS: the hidden activations to H1, H2 as well
template <bool LAYERS>
__global__ void __launch_bounds__(256) k_mlp_forward(int64_t n, const uint16_t *__restrict__ X,
                                                     const uint16_t *__restrict__ W,
                                                     float *__restrict__ out, uint16_t *__restrict__ H1,
                                                     uint16_t *__restrict__ H2)
{
    MlpRegs R;
    load_weights(W, R);
    const int lane = threadIdx.x & 63;
    const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
    const int64_t nw = ((int64_t)gridDim.x * blockDim.x) >> 6;
    // the next group's features are loaded while this group is evaluated
    s4 xn = load_x(X, wave * 16 + (lane & 15), n);
    for (int64_t g0 = wave * 16; g0 < n; g0 += nw * 16) {
        const int64_t node = g0 + (lane & 15);
        const s4 xb = xn;
        xn = load_x(X, node + nw * 16, n);
        const f4 o = mlp16<LAYERS>(R, xb, H1, H2, node, n);
        if (lane < 16 && node < n) {
            out[3 * node] = o[0];
            out[3 * node + 1] = o[1];
            out[3 * node + 2] = o[2];
        }
    }
}

// z = g + s * MLP(X) with g = dinv r; z = 0 where dinv = 0 or s = 0;
// per-workgroup partials of r.z
__global__ void __launch_bounds__(256) k_mlp_apply(int64_t n, const uint16_t *__restrict__ X,
                                                   const uint16_t *__restrict__ W,
                                                   const float *__restrict__ r,
                                                   const float *__restrict__ dinv,
                                                   const float *__restrict__ s,
                                                   float *__restrict__ z, double *__restrict__ prz)
{
    __shared__ double red[256];
    MlpRegs R;
    load_weights(W, R);
    const int lane = threadIdx.x & 63;
    const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
    const int64_t nw = ((int64_t)gridDim.x * blockDim.x) >> 6;
    double rz = 0.0;
    // the next group's features are loaded while this group is evaluated
    s4 xn = load_x(X, wave * 16 + (lane & 15), n);
    for (int64_t g0 = wave * 16; g0 < n; g0 += nw * 16) {
        const int64_t node = g0 + (lane & 15);
        const s4 xb = xn;
        xn = load_x(X, node + nw * 16, n);
        const f4 o = mlp16(R, xb);
        if (lane < 16 && node < n) {
            // z = g + gamma c with g = D^-1 r, c = s MLP; gamma < 1 only where
            // r_i.z_i would fall below half of r_i.g_i, so r.z >= r.D^-1 r / 2
            const float si = s[node];
            float ri[3], gi[3], ci[3], a = 0.f, b = 0.f;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const float di = dinv[3 * node + c];
                ri[c] = r[3 * node + c];
                gi[c] = ri[c] * di;
                ci[c] = (di == 0.f || si == 0.f) ? 0.f : si * o[c];
                a += ri[c] * gi[c];
                b += ri[c] * ci[c];
            }
            const float gam = (a + b < 0.5f * a) ? (-0.5f * a) / b : 1.f;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const float zi = gi[c] + gam * ci[c];
                z[3 * node + c] = zi;
                rz += (double)ri[c] * (double)zi;
            }
        }
    }
    red[threadIdx.x] = rz;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) prz[blockIdx.x] = red[0];
}

// ------------------------------------------------- energy-norm training rows

// Block sum of one double per thread (256 threads); thread 0 gets the total.
__device__ __forceinline__ double block_sum256(double v, double *red)
{
    red[threadIdx.x] = v;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    const double t = red[0];
    __syncthreads();
    return t;
}

// z = m (g + s out) for one sample's rows aux = [g(3), t(3), m(3), s, w, 0];
// partials of r . g (the Jacobi share, which normalises the sample).
__global__ void __launch_bounds__(256) k_energy_z(int64_t n, const float *__restrict__ r,
                                                  const float *__restrict__ out,
                                                  const float *__restrict__ aux, float *__restrict__ z,
                                                  double *__restrict__ part)
{
    __shared__ double red[256];
    double rg = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const float *a = aux + i * kAux;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            z[3 * i + c] = a[6 + c] * (a[c] + a[9] * out[3 * i + c]);
            rg += (double)r[3 * i + c] * (double)a[c];
        }
    }
    const double t = block_sum256(rg, red);
    if (threadIdx.x == 0) part[blockIdx.x] = t;
}

// With w = 1 / (n_samples r.g): aux w = w, aux t = (g + s out) - (K z - r), so
// that the target-fit loss gradient of the rows equals the gradient of
// w (z.Kz - 2 r.z); partials of that energy term.
__global__ void __launch_bounds__(256) k_energy_target(int64_t n, const float *__restrict__ r,
                                                       const float *__restrict__ out,
                                                       const float *__restrict__ z,
                                                       const float *__restrict__ kz, float *__restrict__ aux,
                                                       const double *__restrict__ rgpart, int G,
                                                       double n_samples, double *__restrict__ part)
{
    __shared__ double red[256];
    double rg = 0.0;
    for (int k = threadIdx.x; k < G; k += blockDim.x) rg += rgpart[k];
    rg = block_sum256(rg, red);
    const double w = rg > 0.0 ? 1.0 / (n_samples * rg) : 0.0;
    double e = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        float *a = aux + i * kAux;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const float ri = r[3 * i + c], zi = z[3 * i + c], ki = kz[3 * i + c];
            a[3 + c] = (a[c] + a[9] * out[3 * i + c]) - (ki - ri);
            e += (double)zi * (double)ki - 2.0 * (double)ri * (double)zi;
        }
        a[10] = (float)w;
    }
    const double t = block_sum256(e, red);
    if (threadIdx.x == 0) part[blockIdx.x] = w * t;
}

__global__ void __launch_bounds__(256) k_energy_acc(const double *__restrict__ part, int G,
                                                    double *__restrict__ energy)
{
    __shared__ double red[256];
    double e = 0.0;
    for (int k = threadIdx.x; k < G; k += blockDim.x) e += part[k];
    e = block_sum256(e, red);
    if (threadIdx.x == 0) *energy += e;
}

// ------------------------------------------------------------------ training

// Training rows of one sample: X (features of b), aux = [g(3), t(3), m(3), s, w, 0]
// with m = 1 on free DOFs, w = 1 / (|t|^2 n_total).  tt = |t|^2 (device scalar).
__global__ void k_rows_aux(int64_t n, const float *__restrict__ b, const float *__restrict__ dinv,
                           const float *__restrict__ t, const float *__restrict__ s,
                           const double *__restrict__ tt, double n_total, float *__restrict__ aux)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    float *a = aux + i * kAux;
    const float w = (float)(1.0 / (tt[0] * n_total));
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const float d = dinv[3 * i + c];
        a[c] = b[3 * i + c] * d;
        a[3 + c] = t[3 * i + c];
        a[6 + c] = d == 0.f ? 0.f : 1.f;
    }
    a[9] = s[i];
    a[10] = w;
    a[11] = 0.f;
}

// ---- gradient of the training loss, on the matrix cores
//
// 16 rows per wave step (rows on the N dimension).  The forward runs on the
// FP32 matrix instruction, which adds its four products one after another, as
// four FMAs would: with the contraction in ascending order from the bias, the
// sums are those of the plain FP32 loop bit for bit, so no activation rounds to
// another bfloat16 than it would there.
// The backward treats the forward's roundings as identity.  Its four
// contractions run on bf16 matrix cores at FP32 accuracy: one factor of each
// (W3, W2, the layer inputs x, h1, h2) is a bfloat16 number to begin with, and
// the other (the FP32 deltas) is split into three bfloat16 terms hi + mid + lo
// that together hold its 24 bits, so every product is exact and only the FP32
// accumulation rounds.
//   delta chain:       dz2[h][row] = sum_c W3[c][h] do[c][row] * sigmoid(a2),
//                      dz1[j][row] = sum_h W2[h][j] dz2[h][row] * sigmoid(a1):
//                      the accumulator layout is again the B-operand layout;
//   weight gradients:  dW2[h][j] += sum_row dz2[h][row] h1[row][j] and the same
//                      for W1, W3: the contraction is over rows, so both
//                      operands go through a per-wave LDS transpose (planes
//                      [unit][16 rows]).  b1 rides as a feature that is 1.
// What bounds it: issue and latency at 2 waves per SIMD (the gradient's 112
// accumulators take the registers of a third): 1,650 VALU instructions, 208
// matrix instructions (4,800 cycles) and 185 LDS instructions per 16 rows.
// Weight fragments lie in LDS in lane order.  Loss and gradient of 179,685 rows,
// with the reduction below: 79 us, of 16 rows 21 (latency: the parameters to LDS,
// their fragments, one step, the sums of the four waves), of 2,048 rows 22; 944,
// 22 and 56 for a form on the vector units whose weight reads met 16-way LDS bank
// conflicts.  The gradient's error against float64 is unchanged.
typedef uint32_t __attribute__((may_alias)) u32a;
typedef s4 __attribute__((may_alias)) s4a;
typedef f4 __attribute__((may_alias)) f4a;

constexpr int kPlane = kHid * 32 + (kHid / 8) * 16;   // bytes of a [64 units][16 rows] bf16 plane
// plane row of a unit: 32 bytes, 16 more after every 8 units (bank spread)
__device__ __forceinline__ int plane_off(int unit) { return unit * 32 + (unit >> 3) * 16; }
constexpr int kSmallPlane = 16 * 32 + 2 * 16;         // 16 units
constexpr int kGradWaves = 4;
constexpr int kFrags = 4 + 16 + 4 + 4 + 16;           // W1, W2, W3, W3^T, W2^T
constexpr int kFragBytes = kFrags * 512;
constexpr int kBiasBytes = (2 * kHid + 4) * 4;
constexpr int kWaveBytes = 5 * kPlane + 2 * kSmallPlane;   // three delta planes, h1, h2, x, do
constexpr int kGradLds = kFragBytes + kBiasBytes + kGradWaves * kWaveBytes;
static_assert(2 * kP * 4 <= kFragBytes + kBiasBytes + kGradWaves * kWaveBytes, "two sets of gradient sums share the LDS");
static_assert((kP + 2 * kHid) * 2 <= kGradWaves * kWaveBytes, "the parameters are staged in the planes' space");
static_assert(kFrags == 44 && kGradWaves == 4, "eleven fragments a wave");

// orders LDS accesses within the wave for the compiler (the LDS itself serves
// a wave's accesses in order)
__device__ __forceinline__ void wave_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// four consecutive units of this lane's row into a plane: lane pairs (rows
// 2k, 2k + 1) swap values so that each lane writes two rows of two units at
// once.  p: the plane row of the first unit, plus 4 (row / 2), plus 32 in odd lanes
__device__ __forceinline__ void put_rows(unsigned char *p, uint2 own, uint32_t sel)
{
    uint2 nb;   // the neighbouring row's (lane ^ 1) values
    nb.x = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)own.x, 0xB1, 0xF, 0xF, false);
    nb.y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)own.y, 0xB1, 0xF, 0xF, false);
    *reinterpret_cast<u32a *>(p) = __builtin_amdgcn_perm(nb.x, own.x, sel);
    *reinterpret_cast<u32a *>(p + 64) = __builtin_amdgcn_perm(nb.y, own.y, sel);
}
// byte selections: even lanes write units 0 and 2 (low halves: own, neighbour),
// odd lanes units 1 and 3 (high halves: neighbour, own)
constexpr uint32_t kSelEven = 0x05040100u, kSelOdd = 0x03020706u;

__device__ __forceinline__ float lo_bf(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_bf(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ s4 as_s4(uint2 w) { return __builtin_bit_cast(s4, w); }

// x = hi + mid + lo in bfloat16.  An infinite x is hi alone: the median of
// (NaN, NaN, 0) is 0, and of (r, r, 0) it is r.
__device__ __forceinline__ void split2(float x, float y, uint32_t &hi, uint32_t &mid, uint32_t &lo)
{
    hi = pack_bf(x, y);
    const float dx = x - lo_bf(hi), dy = y - hi_bf(hi);
    const float rx = __builtin_amdgcn_fmed3f(dx, dx, 0.f), ry = __builtin_amdgcn_fmed3f(dy, dy, 0.f);
    mid = pack_bf(rx, ry);
    lo = pack_bf(rx - lo_bf(mid), ry - hi_bf(mid));
}
__device__ __forceinline__ void split3(const float x[4], uint2 &hi, uint2 &mid, uint2 &lo)
{
    split2(x[0], x[1], hi.x, mid.x, lo.x);
    split2(x[2], x[3], hi.y, mid.y, lo.y);
}

// softplus(x) (as softplus()) and its derivative 1 / (1 + e^-x) from the same exponential
__device__ __forceinline__ float softplus_d(float x, float &dx)
{
    const float t = __builtin_amdgcn_exp2f(-fabsf(x) * 1.4426950408889634f);
    const float u = 1.f + t;
    const float e = t - (u - 1.f);
    const float r = __builtin_amdgcn_rcpf(u);
    dx = x >= 0.f ? r : t * r;
    return fmaxf(x, 0.f) + fmaf(0.6931471805599453f, __builtin_amdgcn_logf(u), e);
}

__device__ __forceinline__ f4 mfma16(s4 a, s4 b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0); }

__device__ __forceinline__ f4 mfma4(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// one value of a plane: unit `u` of row `row`
typedef uint16_t __attribute__((may_alias)) u16a;
__device__ __forceinline__ float unit_row(const unsigned char *p, int u, int row)
{
    return bf2f(*reinterpret_cast<const u16a *>(p + plane_off(u) + 2 * row));
}

__global__ void __launch_bounds__(64 * kGradWaves, 2) k_mlp_grad(int64_t rows, const uint16_t *__restrict__ X,
                                                  const float *__restrict__ aux,
                                                  const float *__restrict__ params,
                                                  float *__restrict__ gpart, double *__restrict__ lpart)
{
    __shared__ __align__(16) unsigned char smem[kGradLds];
    __shared__ double lred[kGradWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 15, quad = lane >> 4;
    s4a *F1 = reinterpret_cast<s4a *>(smem), *F2 = F1 + 4 * 64, *F3 = F2 + 16 * 64, *F3T = F3 + 4 * 64,
        *F2T = F3T + 4 * 64;
    float *bias = reinterpret_cast<float *>(smem + kFragBytes);   // b1, b2, b3 (padded to 4)
    unsigned char *mine = smem + kFragBytes + kBiasBytes + wave * kWaveBytes;
    unsigned char *pd = mine, *ph1 = mine + 3 * kPlane, *ph2 = ph1 + kPlane, *px = ph2 + kPlane, *pdo = px + kSmallPlane;
    // operand fragments: entry f * 64 + l holds lane l's four values, for the
    // forward (W1, W2, W3) those of four FP32 steps v (m = l % 16, k = 4 v +
    // l / 16 of its 16), else one bf16 operand (m = l % 16, k = 4 (l / 16) + v).
    // They are gathered from a copy of the parameters in the planes' space, whose
    // W2 rows are two apart of 64 (rows 128 bytes apart lie on the same banks).
    // Wave w gathers fragments w, w + 4, ...: four of a kind at a time, so that the
    // eleven rounds are one straight run of independent reads (a loop that looked up
    // each fragment's kind took 5.4 us, as long as 16 rows).
    auto at = [](int k) { return k < kOffW2 ? k : (k < kOffB2 ? k + 2 * ((k - kOffW2) >> 6) : k + 2 * kHid); };
    uint16_t *pl = reinterpret_cast<uint16_t *>(smem + kFragBytes + kBiasBytes);
    constexpr int kU = 10;   // loads in flight
    for (int k0 = tid; k0 < kP; k0 += kU * 64 * kGradWaves) {
        float t[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) t[u] = params[min(k0 + u * 64 * kGradWaves, kP - 1)];
#pragma unroll
        for (int u = 0; u < kU; ++u)
            if (k0 + u * 64 * kGradWaves < kP) pl[at(k0 + u * 64 * kGradWaves)] = f2bf(t[u]);
    }
    __syncthreads();
    {
        constexpr int kRow = kHid + 2;   // of W2's copy
        const uint16_t *w1 = pl + (16 * wave + col) * kIn, *w2 = pl + kOffW2, *w3 = pl + at(kOffW3);
        s4 f[kFrags / 4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int k = 4 * quad + v, kf = 4 * v + quad;
            const short a = (short)w1[kOffW1 + min(kf, kIn - 1)], b = (short)w3[min(col, kOut - 1) * kHid + 16 * wave + kf],
                        c = (short)w3[(k % 3) * kHid + 16 * wave + col];
            f[0][v] = kf < kIn ? a : (short)0;      // W1, tile `wave`
            f[5][v] = col < kOut ? b : (short)0;    // W3, group `wave`
            f[6][v] = k < 9 ? c : (short)0;         // W3^T, tile `wave`: k = 3 term + c
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                f[1 + g][v] = (short)w2[(16 * wave + col) * kRow + 16 * g + kf];   // W2: group g, tile `wave`
                f[7 + g][v] = (short)w2[(16 * wave + k) * kRow + 16 * g + col];    // W2^T: tile g of t1, t = `wave`
            }
        }
#pragma unroll
        for (int r = 0; r < kFrags / 4; ++r) F1[(4 * r + wave) * 64 + lane] = f[r];
    }
    if (tid < kHid) {
        bias[tid] = bf2f(pl[at(kOffB1 + tid)]);
        bias[kHid + tid] = bf2f(pl[at(kOffB2 + tid)]);
    }
    if (tid < 4) bias[2 * kHid + tid] = tid < kOut ? bf2f(pl[at(kOffB3 + tid)]) : 0.f;
    __syncthreads();
    // rows 9..15 of the output-delta plane stay 0
    for (int i = lane; i < kSmallPlane / 4; i += 64) *reinterpret_cast<u32a *>(pdo + 4 * i) = 0u;
    __syncthreads();

    const uint32_t sel = (lane & 1) ? kSelOdd : kSelEven;
    // this lane's place in a plane for put_rows (of the units 4 quad + ...) and
    // for an operand read (unit l % 16 of a tile, rows 4 quad + ...)
    const int wr = plane_off(4 * quad) + (col >> 1) * 4 + (lane & 1) * 32, rd = plane_off(col) + 8 * quad;
    constexpr int kTile = 16 * 32 + 2 * 16;   // bytes of a plane's tile of 16 units
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    f4 g2[4][4], g1[4], g3[4];      // dW2 [h tile][j tile], dW1 (and b1), dW3 (three terms)
    float gb2[4][4], gb3[kOut] = {0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        g1[t] = g3[t] = zero;
#pragma unroll
        for (int j = 0; j < 4; ++j) g2[t][j] = zero, gb2[t][j] = 0.f;
    }
    double loss = 0.0;
    const int64_t nw = (int64_t)gridDim.x * kGradWaves, first = (int64_t)blockIdx.x * kGradWaves + wave;
    s4 xn = load_x(X, first * 16 + col, rows);
    for (int64_t r0 = first * 16; r0 < rows; r0 += nw * 16) {
        const int64_t row = r0 + col;
        s4 xb = xn;
        xn = load_x(X, row + nw * 16, rows);
        // this row's training data, used by the quad that holds the outputs
        float ax[11];
        const bool mine_out = quad == 0 && row < rows;
#pragma unroll
        for (int k = 0; k < 11; ++k) ax[k] = mine_out ? aux[row * kAux + k] : 0.f;
        if (quad == 3) xb[0] = 0x3f80;   // feature 12 = 1: its weight is 0, its gradient that of b1
        put_rows(px + wr, __builtin_bit_cast(uint2, xb), sel);
        wave_fence();
        // forward
        float s1[4][4], s2[4][4];
        f4 a[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) a[t] = *reinterpret_cast<const f4a *>(bias + 16 * t + 4 * quad);
#pragma unroll
        for (int v = 0; v < kIn / 4; ++v) {
            const float b = unit_row(px, 4 * v + quad, col);
#pragma unroll
            for (int t = 0; t < 4; ++t) a[t] = mfma4(bf2f((uint16_t)F1[t * 64 + lane][v]), b, a[t]);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            float h[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) h[v] = softplus_d(a[t][v], s1[t][v]);
            put_rows(ph1 + t * kTile + wr, make_uint2(pack_bf(h[0], h[1]), pack_bf(h[2], h[3])), sel);
        }
        wave_fence();
#pragma unroll
        for (int t = 0; t < 4; ++t) a[t] = *reinterpret_cast<const f4a *>(bias + kHid + 16 * t + 4 * quad);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            s4 w[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) w[t] = F2[(4 * g + t) * 64 + lane];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float b = unit_row(ph1, 16 * g + 4 * v + quad, col);
#pragma unroll
                for (int t = 0; t < 4; ++t) a[t] = mfma4(bf2f((uint16_t)w[t][v]), b, a[t]);
            }
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            float h[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) h[v] = softplus_d(a[t][v], s2[t][v]);
            put_rows(ph2 + t * kTile + wr, make_uint2(pack_bf(h[0], h[1]), pack_bf(h[2], h[3])), sel);
        }
        wave_fence();
        f4 o = *reinterpret_cast<const f4a *>(bias + 2 * kHid);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const s4 w = F3[g * 64 + lane];
#pragma unroll
            for (int v = 0; v < 4; ++v)
                o = mfma4(bf2f((uint16_t)w[v]), unit_row(ph2, 16 * g + 4 * v + quad, col), o);
        }
        // loss and output deltas (quad 0 holds outputs 0..2 of its row)
        float dout[4] = {0.f, 0.f, 0.f, 0.f};
        if (mine_out) {
#pragma unroll
            for (int c = 0; c < kOut; ++c) {
                const float z = ax[6 + c] * (ax[c] + ax[9] * o[c]);
                const float e = z - ax[6 + c] * ax[3 + c];
                loss += (double)ax[10] * (double)e * (double)e;
                dout[c] = 2.f * ax[10] * ax[9] * ax[6 + c] * e;
                gb3[c] += dout[c];
            }
        }
        uint2 dh, dm, dl;
        split3(dout, dh, dm, dl);
        // the three terms of the three outputs in k = 3 term + c order: quad q
        // gets k = 4 q .. 4 q + 3 of its row
        uint2 db;
        {
            const uint32_t w[5] = {dh.x, dh.y | dm.x << 16, dm.x >> 16 | dm.y << 16, dl.x, dl.y};
            uint32_t g[5];
#pragma unroll
            for (int k = 0; k < 5; ++k) g[k] = (uint32_t)__shfl((int)w[k], col, 64);
            db.x = quad == 0 ? g[0] : quad == 1 ? g[2] : quad == 2 ? g[4] : 0u;
            db.y = quad == 0 ? g[1] : quad == 1 ? g[3] : 0u;
        }
        put_rows(pdo + wr, db, sel);
        // dz2 = (W3^T do) sigmoid(a2), its terms to the planes
        uint2 dz[3][4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const f4 d = mfma16(F3T[t * 64 + lane], as_s4(db), zero);
            float z[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                z[v] = d[v] * s2[t][v];
                gb2[t][v] += z[v];
            }
            split3(z, dz[0][t], dz[1][t], dz[2][t]);
#pragma unroll
            for (int k = 0; k < 3; ++k) put_rows(pd + k * kPlane + t * kTile + wr, dz[k][t], sel);
        }
        wave_fence();
        // dW3 += do h2, dW2 += dz2 h1: units on both sides, contraction over the 16 rows
        const s4 ado = *reinterpret_cast<const s4a *>(pdo + rd);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            g3[t] = mfma16(ado, *reinterpret_cast<const s4a *>(ph2 + t * kTile + rd), g3[t]);
        }
        s4 bh1[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) bh1[t] = *reinterpret_cast<const s4a *>(ph1 + t * kTile + rd);
#pragma unroll
        for (int t2 = 0; t2 < 4; ++t2)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const s4 ad = *reinterpret_cast<const s4a *>(pd + k * kPlane + t2 * kTile + rd);
#pragma unroll
                for (int t = 0; t < 4; ++t) g2[t2][t] = mfma16(ad, bh1[t], g2[t2][t]);
            }
        wave_fence();
        // dz1 = (W2^T dz2) sigmoid(a1), its terms to the planes
#pragma unroll
        for (int t1 = 0; t1 < 4; ++t1) {
            f4 d = zero;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const s4 w = F2T[(4 * t1 + t) * 64 + lane];
#pragma unroll
                for (int k = 2; k >= 0; --k) d = mfma16(w, as_s4(dz[k][t]), d);
            }
            float z[4];
            uint2 e[3];
#pragma unroll
            for (int v = 0; v < 4; ++v) z[v] = d[v] * s1[t1][v];
            split3(z, e[0], e[1], e[2]);
#pragma unroll
            for (int k = 0; k < 3; ++k) put_rows(pd + k * kPlane + t1 * kTile + wr, e[k], sel);
        }
        wave_fence();
        const s4 bx = *reinterpret_cast<const s4a *>(px + rd);
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int k = 0; k < 3; ++k)
                g1[t] = mfma16(*reinterpret_cast<const s4a *>(pd + k * kPlane + t * kTile + rd), bx,
                               g1[t]);
        wave_fence();
    }

    // the wave's sums of the row-wise parts
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) gb2[t][v] += __shfl_xor(gb2[t][v], off, 64);
#pragma unroll
        for (int c = 0; c < kOut; ++c) gb3[c] += __shfl_xor(gb3[c], off, 64);
        loss += __shfl_xor(loss, off, 64);
    }
    if (lane == 0) lred[wave] = loss;
    // dW3: the terms of output c lie in rows c, 3 + c, 6 + c (quads 0, 1, 2)
    float w3[4][kOut];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        float q1[4], q2;
#pragma unroll
        for (int v = 0; v < 4; ++v) q1[v] = __shfl(g3[t][v], col + 16, 64);
        q2 = __shfl(g3[t][0], col + 32, 64);
        w3[t][0] = g3[t][0] + (g3[t][3] + q1[2]);
        w3[t][1] = g3[t][1] + (q1[0] + q1[3]);
        w3[t][2] = g3[t][2] + (q1[1] + q2);
    }
    // the four waves' sums in a fixed order, (0 + 1) + (2 + 3), through two sets in LDS:
    // the odd waves store theirs, the even ones add, a tile's entries all read before
    // the first is stored (read and stored one by one, 5.2 us)
    float *gs = reinterpret_cast<float *>(smem) + (wave >> 1) * kP;
    auto each = [&](int t, auto f) {   // the lane's entries of tile t: f(n, index, value)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int h = 16 * t + 4 * quad + v;
            if (col <= kIn) f(v, col < kIn ? kOffW1 + h * kIn + col : kOffB1 + h, g1[t][v]);
#pragma unroll
            for (int j = 0; j < 4; ++j) f(4 + 4 * v + j, kOffW2 + h * kHid + 16 * j + col, g2[t][j][v]);
            if (col == 0) f(20 + v, kOffB2 + h, gb2[t][v]);
        }
        if (quad == 0)
#pragma unroll
            for (int c = 0; c < kOut; ++c) f(24 + c, kOffW3 + c * kHid + 16 * t + col, w3[t][c]);
        if (t == 0 && lane == 0)
#pragma unroll
            for (int c = 0; c < kOut; ++c) f(27 + c, kOffB3 + c, gb3[c]);
    };
    __syncthreads();
    if (wave & 1)
#pragma unroll
        for (int t = 0; t < 4; ++t) each(t, [&](int, int k, float g) { gs[k] = g; });
    __syncthreads();
    if (!(wave & 1))
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            float sum[27 + kOut];
            each(t, [&](int n, int k, float g) { sum[n] = g + gs[k]; });
            each(t, [&](int n, int k, float) { gs[k] = sum[n]; });
        }
    __syncthreads();
    gs = reinterpret_cast<float *>(smem);
    for (int k = tid; k < kP; k += 64 * kGradWaves) gpart[(int64_t)blockIdx.x * kP + k] = gs[k] + gs[kP + k];
    if (tid == 0) lpart[blockIdx.x] = (lred[0] + lred[1]) + (lred[2] + lred[3]);
}

// Column sums of gpart [G][kP] and the loss partials, in a fixed order: 16
// columns per workgroup, 64 threads per column, so that every CU pulls its share
// and a column's partials are all in flight at once (one thread per column read
// them one after another: 299 us for 1024 partials; for 512, 64 columns on 80
// workgroups 12 us, 32 columns 8, 16 columns 6.5).  The last workgroup sums the loss.
constexpr int kReduceCols = 16;
__global__ void __launch_bounds__(1024) k_grad_reduce(int G, const float *__restrict__ gpart,
                                                      const double *__restrict__ lpart,
                                                      float *__restrict__ grad, double *__restrict__ loss)
{
    constexpr int kC = kReduceCols, kQ = 1024 / kC, kLoads = kGradBlocks / kQ;
    __shared__ double red[kQ][kC];
    const int c = threadIdx.x % kC, q = threadIdx.x / kC;
    double s = 0.0;
    if (blockIdx.x == gridDim.x - 1) {
        for (int b = threadIdx.x; b < G; b += 1024) s += lpart[b];
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) s += __shfl_xor(s, off, 64);
        double *waves = &red[0][0];
        if ((threadIdx.x & 63) == 0) waves[threadIdx.x >> 6] = s;
        __syncthreads();
        if (threadIdx.x == 0) {
            double t = 0.0;
            for (int k = 0; k < 16; ++k) t += waves[k];
            *loss = t;
        }
        return;
    }
    const int k = blockIdx.x * kC + c;
    if (k < kP) {   // G <= kGradBlocks: all loads in flight at once
        float p[kLoads];
#pragma unroll
        for (int j = 0; j < kLoads; ++j) p[j] = q + kQ * j < G ? gpart[(int64_t)(q + kQ * j) * kP + k] : 0.f;
#pragma unroll
        for (int j = 0; j < kLoads; ++j) s += p[j];
    }
    red[q][c] = s;
    __syncthreads();
    if (q == 0 && k < kP) {
        double t = 0.0;
#pragma unroll
        for (int j = 0; j < kQ; ++j) t += red[j][c];
        grad[k] = (float)t;
    }
}

__global__ void k_adam(float *__restrict__ p, float *__restrict__ m, float *__restrict__ v,
                       const float *__restrict__ g, float lr, float b1, float b2, float eps, int t)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= kP) return;
    const float gk = g[k];
    const float mk = b1 * m[k] + (1.f - b1) * gk;
    const float vk = b2 * v[k] + (1.f - b2) * gk * gk;
    m[k] = mk;
    v[k] = vk;
    const float mh = mk / (1.f - powf(b1, (float)t)), vh = vk / (1.f - powf(b2, (float)t));
    p[k] -= lr * mh / (sqrtf(vh) + eps);
}

__global__ void k_to_bf16(const float *__restrict__ p, int n, uint16_t *__restrict__ out)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) out[k] = f2bf(p[k]);
}

// |t|^2 of a float vector (one workgroup)
__global__ void k_norm2_f32(int64_t n, const float *__restrict__ t, double *__restrict__ out)
{
    __shared__ double red[256];
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) s += (double)t[i] * (double)t[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = red[0];
}

__global__ void k_dinv_f32(int64_t n, const double *__restrict__ diag, const uint8_t *__restrict__ nmask,
                           float *__restrict__ dinv)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const bool fixed = nmask && ((nmask[i / 3] >> (i % 3)) & 1);
    dinv[i] = fixed ? 0.f : (float)(1.0 / diag[i]);
}

// dinv of the diagonal and g4 of r in one pass over the nodes (the values of
// k_dinv_f32 and k_g4): an apply at a new diagonal starts with one launch
__global__ void __launch_bounds__(256) k_dinv_g4(int64_t n, const double *__restrict__ diag,
                                                 const uint8_t *__restrict__ nmask, const float *__restrict__ r,
                                                 float *__restrict__ dinv, float4 *__restrict__ g4)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int m = nmask ? nmask[i] : 0;
    float g[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const float d = (m >> c) & 1 ? 0.f : (float)(1.0 / diag[3 * i + c]);
        dinv[3 * i + c] = d;
        g[c] = r[3 * i + c] * d;
    }
    g4[i] = make_float4(g[0], g[1], g[2], g[0] * g[0] + g[1] * g[1] + g[2] * g[2]);
}

// ---------------------------------------------------------------- launchers

static unsigned g256(int64_t n) { return (unsigned)((n + 255) / 256); }
// The MLP kernels load the weights once per wave; a grid of about the
// resident wave count (3 waves per SIMD) spreads that over many node groups.
static unsigned mlp_grid(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 63) / 64, 768)); }

hipError_t mlp_features_static(hipStream_t s, const MlpState &M, int64_t n, const double *diag,
                               const uint8_t *nmask, uint16_t *X)
{
    auto kern = nmask ? k_feat_static<true> : k_feat_static<false>;
    hipLaunchKernelGGL(kern, dim3(g256(n)), dim3(256), 0, s, n, M.ptr, M.ell, diag, nmask, X);
    return hipGetLastError();
}

hipError_t mlp_features(hipStream_t s, const MlpState &M, int64_t n, const double *diag, const uint8_t *nmask,
                        const float *r, uint16_t *X)
{
    hipLaunchKernelGGL(k_dinv_g4, dim3(g256(n)), dim3(256), 0, s, n, diag, nmask, r, M.dinv, M.g4);
    auto kern = nmask ? k_feat_all<true> : k_feat_all<false>;
    hipLaunchKernelGGL(kern, dim3(g256(n)), dim3(256), 0, s, n, M.ptr, M.ell, M.max_deg, diag, nmask, M.g4, X, M.scale);
    return hipGetLastError();
}

hipError_t mlp_features_dyn(hipStream_t s, const MlpState &M, int64_t n, const float *r,
                            const float *dinv, uint16_t *X, float *scale, float4 *g4)
{
    hipLaunchKernelGGL(k_g4, dim3(g256(n)), dim3(256), 0, s, n, r, dinv, g4);
    hipLaunchKernelGGL(k_feat_dyn, dim3(g256(n)), dim3(256), 0, s, n, M.ptr, M.ell, M.max_deg, g4, X, scale);
    return hipGetLastError();
}

hipError_t mlp_forward(hipStream_t s, const uint16_t *W, int64_t n, const uint16_t *X, float *out, uint16_t *H1,
                       uint16_t *H2)
{
    if (H1 && H2)
        hipLaunchKernelGGL(k_mlp_forward<true>, dim3(mlp_grid(n)), dim3(256), 0, s, n, X, W, out, H1, H2);
    else
        hipLaunchKernelGGL(k_mlp_forward<false>, dim3(mlp_grid(n)), dim3(256), 0, s, n, X, W, out, H1, H2);
    return hipGetLastError();
}

int mlp_apply_grid(int64_t n) { return (int)mlp_grid(n); }

hipError_t mlp_apply(hipStream_t s, const uint16_t *W, int64_t n, const uint16_t *X, const float *r,
                     const float *dinv, const float *scale, float *z, double *prz)
{
    hipLaunchKernelGGL(k_mlp_apply, dim3(mlp_grid(n)), dim3(256), 0, s, n, X, W, r, dinv, scale, z, prz);
    return hipGetLastError();
}

hipError_t mlp_rows_aux(hipStream_t s, int64_t n, const float *b, const float *dinv, const float *t,
                        const float *scale, double *tt, double n_total, float *aux)
{
    hipLaunchKernelGGL(k_norm2_f32, dim3(1), dim3(256), 0, s, 3 * n, t, tt);
    hipLaunchKernelGGL(k_rows_aux, dim3(g256(n)), dim3(256), 0, s, n, b, dinv, t, scale, tt, n_total, aux);
    return hipGetLastError();
}

hipError_t mlp_loss_grad(hipStream_t s, int64_t rows, const uint16_t *X, const float *aux,
                         const float *params, float *gpart, double *lpart, int G, float *grad,
                         double *loss)
{
    hipLaunchKernelGGL(k_mlp_grad, dim3(G), dim3(64 * kGradWaves), 0, s, rows, X, aux, params, gpart, lpart);
    hipLaunchKernelGGL(k_grad_reduce, dim3((kP + kReduceCols - 1) / kReduceCols + 1), dim3(1024), 0, s, G, gpart,
                       lpart, grad, loss);
    return hipGetLastError();
}

hipError_t mlp_energy_z(hipStream_t s, int64_t n, const float *r, const float *out, const float *aux,
                        float *z, double *part, int G)
{
    hipLaunchKernelGGL(k_energy_z, dim3(G), dim3(256), 0, s, n, r, out, aux, z, part);
    return hipGetLastError();
}

hipError_t mlp_energy_target(hipStream_t s, int64_t n, const float *r, const float *out, const float *z,
                             const float *kz, float *aux, const double *rgpart, double n_samples,
                             double *part, int G, double *energy)
{
    hipLaunchKernelGGL(k_energy_target, dim3(G), dim3(256), 0, s, n, r, out, z, kz, aux, rgpart, G,
                       n_samples, part);
    hipLaunchKernelGGL(k_energy_acc, dim3(1), dim3(256), 0, s, part, G, energy);
    return hipGetLastError();
}

hipError_t mlp_adam(hipStream_t s, float *p, float *m, float *v, const float *g, float lr, float b1,
                    float b2, float eps, int t)
{
    hipLaunchKernelGGL(k_adam, dim3(g256(kP)), dim3(256), 0, s, p, m, v, g, lr, b1, b2, eps, t);
    return hipGetLastError();
}

hipError_t mlp_to_bf16(hipStream_t s, const float *p, uint16_t *out)
{
    hipLaunchKernelGGL(k_to_bf16, dim3(g256(kP)), dim3(256), 0, s, p, kP, out);
    return hipGetLastError();
}

hipError_t mlp_dinv_f32(hipStream_t s, int64_t n, const double *diag, const uint8_t *nmask, float *dinv)
{
    hipLaunchKernelGGL(k_dinv_f32, dim3(g256(n)), dim3(256), 0, s, n, diag, nmask, dinv);
    return hipGetLastError();
}

}  // namespace efem
