// HIP kernels and C ABI (include/mlp.h) of the flow-curve surrogate network:
// a 3 -> 64 -> 64 -> 1 tanh multilayer perceptron trained by full-batch Adam.
//
// Lane j of a wavefront owns hidden unit j of both layers: the 64-wide layers map
// one-to-one onto the 64-lane wavefront.  A wavefront takes one training row and
// a block eight, those of one partial gradient; the weights sit in LDS, W2 in both
// orientations so that the forward and the backward contraction read consecutive
// addresses.  The partial gradients go to global memory and a second kernel adds
// them up in a fixed order and applies Adam, so training is deterministic.  The
// network is small (4481 parameters, a few MFLOP per epoch): it is latency-bound
// and uses no matrix cores (their order of summation is not the one the results
// have).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>

#include "../../include/mlp.h"

namespace mlpk {

constexpr int H = 64;
constexpr int NP = MLP_NPARAM;
constexpr int NPL = NP + 1;           // partial row: gradient + loss
constexpr int OFF_W1 = 0, OFF_B1 = OFF_W1 + 3 * H, OFF_W2 = OFF_B1 + H, OFF_B2 = OFF_W2 + H * H,
              OFF_W3 = OFF_B2 + H, OFF_B3 = OFF_W3 + H;
constexpr int PROWS = 8;               // rows of a partial gradient
constexpr int WAVES = PROWS;           // wavefronts per block, one a row
constexpr int W2T = H + 1;             // row length of the transposed W2 (its writes spread over the banks)
constexpr int BLOCKS = 1024;           // blocks of a launch at most, four per compute unit

// Partials of n rows, and row i of partial p: each 32 rows are dealt to four.
constexpr int partials(int n) { return (n + 31) / 32 * 4; }
__device__ __forceinline__ int row_of(int p, int i) { return p / 4 * 32 + p % 4 + 4 * i; }

struct Norm {
    float in_mean[3], in_std[3], out_mean, out_std;
};

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

struct Lds {
    alignas(16) float w2[H * H];
    alignas(16) float a1[PROWS][H];
    float w2t[H * W2T], lo[OFF_W2], hi[NP - OFF_B2];   // lo: W1, b1; hi: b2, W3, b3
    __device__ __forceinline__ float w1(int i) const { return lo[OFF_W1 + i]; }
    __device__ __forceinline__ float b1(int i) const { return lo[OFF_B1 + i]; }
    __device__ __forceinline__ float b2(int i) const { return hi[i]; }
    __device__ __forceinline__ float w3(int i) const { return hi[OFF_W3 - OFF_B2 + i]; }
    __device__ __forceinline__ float b3() const { return hi[OFF_B3 - OFF_B2]; }
};

// The parameters into LDS, every load in flight at once (a block of 64 WAVES threads).
__device__ __forceinline__ void load_params(Lds& L, const float* __restrict__ th)
{
    constexpr int T = 64 * WAVES, Q = H * H / 4 / T;
    static_assert(Q * T * 4 == H * H && 3 * H + 2 * H + H + 1 <= T, "a thread's share of the parameters");
    // W1, b1 and b2, W3, b3: the parameters before and after W2 (OFF_W2 is a multiple of four)
    const int t = threadIdx.x, lo = OFF_W2, hi = NP - OFF_B2;
    float4 w[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) w[q] = *reinterpret_cast<const float4*>(th + OFF_W2 + 4 * (q * T + t));
    const float x = t < lo ? th[t] : (t < lo + hi ? th[OFF_B2 + t - lo] : 0.f);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int i = 4 * (q * T + t), c = i % H, r = i / H;
        *reinterpret_cast<float4*>(&L.w2[i]) = w[q];
        L.w2t[c * W2T + r] = w[q].x;
        L.w2t[(c + 1) * W2T + r] = w[q].y;
        L.w2t[(c + 2) * W2T + r] = w[q].z;
        L.w2t[(c + 3) * W2T + r] = w[q].w;
    }
    if (t < lo) L.lo[t] = x;
    else if (t < lo + hi) L.hi[t - lo] = x;
    __syncthreads();
}

// Standardised inputs of row r.
__device__ __forceinline__ void load_row(const Norm& nm, const float* __restrict__ X, int r, float (&xs)[3])
{
#pragma unroll
    for (int c = 0; c < 3; ++c) xs[c] = (X[3 * r + c] - nm.in_mean[c]) / nm.in_std[c];
}

// s plus the sum over k of m[k * stride + j] v[k], k ascending: the contraction of
// both directions.
__device__ __forceinline__ float contract(const float* m, int stride, const float (&v)[H], int j, float s)
{
#pragma unroll 8
    for (int k = 0; k < H; k += 4) {
        const float4 x = *reinterpret_cast<const float4*>(&v[k]);
        s += m[k * stride + j] * x.x;
        s += m[(k + 1) * stride + j] * x.y;
        s += m[(k + 2) * stride + j] * x.z;
        s += m[(k + 3) * stride + j] * x.w;
    }
    return s;
}

// Forward pass of wave w's row: lane j returns a1_j, a2_j; all lanes return the
// standardised output.
__device__ __forceinline__ float forward_row(Lds& L, int w, int j, const float (&xs)[3], float& a1, float& a2)
{
    const float z1 = L.w1(3 * j) * xs[0] + L.w1(3 * j + 1) * xs[1] + L.w1(3 * j + 2) * xs[2] + L.b1(j);
    a1 = tanhf(z1);
    L.a1[w][j] = a1;
    __builtin_amdgcn_wave_barrier();
    a2 = tanhf(contract(L.w2t, W2T, L.a1[w], j, L.b2(j)));
    return wave_sum(L.w3(j) * a2) + L.b3();
}

// Forward + backward over the rows: a partial gradient and loss sum per eight.  A
// wave takes a row; the sums over the eight rows, in their order, are then split
// over the waves.  A partial keeps the gradient of W2 transposed, [k][j], so that
// its stores are consecutive.  1800 rows: 25.3 us a launch with 57 blocks of four
// waves that took eight rows each in turn, 9.1 us now.
__global__ void __launch_bounds__(64 * WAVES)
k_fwdbwd(const float* __restrict__ th, Norm nm, const float* __restrict__ X, const float* __restrict__ Y,
         int n, float* __restrict__ part)
{
    __shared__ Lds L;
    __shared__ alignas(16) float D2[PROWS][H];
    __shared__ float A2[PROWS][H], D1[PROWS][H], XS[PROWS][3], D[PROWS], RES[PROWS];
    const int w = threadIdx.x / 64, j = threadIdx.x % 64;
    const float inv_n = 1.0f / (float)n;
    const int np = partials(n);
    bool loaded = false;
    for (int p = blockIdx.x; p < np; p += gridDim.x) {
        const int r = min(row_of(p, w), n - 1);        // a row past the last: computed, not added
        float xs[3], a1, a2;
        load_row(nm, X, r, xs);
        const float ys = (Y[r] - nm.out_mean) / nm.out_std;
        if (!loaded) load_params(L, th);
        loaded = true;
        const float out = forward_row(L, w, j, xs, a1, a2);
        const float res = out - ys;
        const float d = 2.0f * res * inv_n;
        const float d2 = d * L.w3(j) * (1.0f - a2 * a2);
        D2[w][j] = d2;
        __builtin_amdgcn_wave_barrier();
        const float s = contract(L.w2, H, D2[w], j, 0.f);
        const float d1 = s * (1.0f - a1 * a1);
        A2[w][j] = a2;
        D1[w][j] = d1;
        if (j < 3) XS[w][j] = j == 0 ? xs[0] : (j == 1 ? xs[1] : xs[2]);
        if (j == 0) {
            D[w] = d;
            RES[w] = res;
        }
        __syncthreads();
        float* row = part + (size_t)p * NPL;
        const int k0 = w * (H / WAVES);
        float g[H / WAVES], v = 0.f;
#pragma unroll
        for (int k = 0; k < H / WAVES; ++k) g[k] = 0.f;
#pragma unroll
        for (int i = 0; i < PROWS; ++i) {
            if (row_of(p, i) >= n) break;
            const float dj = D2[i][j];
#pragma unroll
            for (int k = 0; k < H / WAVES; ++k) g[k] += dj * L.a1[i][k0 + k];
            if (w < 3) v += D1[i][j] * XS[i][w];
            else if (w == 3) v += D1[i][j];
            else if (w == 4) v += dj;
            else if (w == 5) v += D[i] * A2[i][j];
            else if (w == 6) v += D[i];
            else v += RES[i] * RES[i];
        }
#pragma unroll
        for (int k = 0; k < H / WAVES; ++k) row[OFF_W2 + (k0 + k) * H + j] = g[k];
        if (w < 3) row[OFF_W1 + 3 * j + w] = v;
        else if (w < 6) row[(w == 3 ? OFF_B1 : (w == 4 ? OFF_B2 : OFF_W3)) + j] = v;
        else if (j == 0) row[w == 6 ? OFF_B3 : NP] = v;
        __syncthreads();
    }
}

// Sum of the partial rows in a fixed order; optional Adam update.  A block takes 64
// entries; its waves fetch RROWS rows into LDS at once and the first adds them up one
// after the other, so that the order costs no memory latency (a thread that read its
// entry of the rows in turn took 52 us over 228 of them, this 4.6 us).
constexpr int RWAVES = 16, RROWS = 256;
__global__ void __launch_bounds__(64 * RWAVES)
k_reduce_adam(const float* __restrict__ part, int nparts, float* __restrict__ th, float* __restrict__ m,
              float* __restrict__ v, float* __restrict__ gout, float* __restrict__ loss_out, float inv_n,
              int update, float lr, float c1, float c2)
{
    __shared__ float rows[RROWS][64];
    const int w = threadIdx.x / 64, j = threadIdx.x % 64;
    const int e = blockIdx.x * 64 + j;     // entry of the partial rows
    // its parameter: the gradient of W2 is transposed
    const int q = e - OFF_W2;
    const int p = (q >= 0 && q < H * H) ? OFF_W2 + (q % H) * H + q / H : e;
    float m0 = 0.f, v0 = 0.f, th0 = 0.f;
    if (w == 0 && update && p < NP) { m0 = m[p]; v0 = v[p]; th0 = th[p]; }
    float g = 0.f;
    for (int b0 = 0; b0 < nparts; b0 += RROWS) {
        float x[RROWS / RWAVES];
#pragma unroll
        for (int i = 0; i < RROWS / RWAVES; ++i) {
            const int b = b0 + i * RWAVES + w;
            x[i] = (b < nparts && e < NPL) ? part[(size_t)b * NPL + e] : 0.f;
        }
#pragma unroll
        for (int i = 0; i < RROWS / RWAVES; ++i) rows[i * RWAVES + w][j] = x[i];
        __syncthreads();
        if (w == 0) {
            const int nb = min(RROWS, nparts - b0);
#pragma unroll 16
            for (int b = 0; b < nb; ++b) g += rows[b][j];
        }
        __syncthreads();
    }
    if (w != 0 || e >= NPL) return;
    if (e == NP) {
        *loss_out = g * inv_n;
        return;
    }
    gout[p] = g;
    if (update) {
        const float mm = 0.9f * m0 + 0.1f * g;
        const float vv = 0.999f * v0 + 0.001f * g * g;
        m[p] = mm;
        v[p] = vv;
        th[p] = th0 - lr * (mm * c1) / (sqrtf(vv * c2) + 1e-8f);
    }
}

__global__ void __launch_bounds__(64 * WAVES)
k_infer(const float* __restrict__ th, Norm nm, const float* __restrict__ X, int n, float* __restrict__ Y)
{
    __shared__ Lds L;
    const int w = threadIdx.x / 64, j = threadIdx.x % 64;
    bool loaded = false;
    for (int r0 = blockIdx.x * WAVES; r0 < n; r0 += gridDim.x * WAVES) {
        const int r = min(r0 + w, n - 1);
        float xs[3], a1, a2;
        load_row(nm, X, r, xs);
        if (!loaded) load_params(L, th);
        loaded = true;
        const float out = forward_row(L, w, j, xs, a1, a2);
        if (j == 0 && r0 + w < n) Y[r] = out * nm.out_std + nm.out_mean;
        __builtin_amdgcn_wave_barrier();
    }
}

__global__ void k_zero(float* __restrict__ p, size_t n)
{
    for (size_t k = blockIdx.x * (size_t)blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x) p[k] = 0.f;
}

}  // namespace mlpk

// ---------------------------------------------------------------- runtime --

// The library's thread-local error message (lb_last_error), set in lb_capi.hip.
void lbi_set_error(const char* msg);

namespace {

lb_status mfail(lb_status code, const char* fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    lbi_set_error(buf);
    return code;
}

size_t al(size_t v) { return (v + 255) / 256 * 256; }

struct MLayout {
    size_t th, m, v, g, loss, X, Y, Xi, Yi, part, total;
};

MLayout mlayout(int rows)
{
    MLayout L;
    size_t o = 0;
    L.th = o; o += al(sizeof(float) * mlpk::NP);
    L.m = o; o += al(sizeof(float) * mlpk::NP);
    L.v = o; o += al(sizeof(float) * mlpk::NP);
    L.g = o; o += al(sizeof(float) * mlpk::NP);
    L.loss = o; o += al(sizeof(float));
    L.X = o; o += al(sizeof(float) * 3 * rows);
    L.Y = o; o += al(sizeof(float) * rows);
    L.Xi = o; o += al(sizeof(float) * 3 * rows);
    L.Yi = o; o += al(sizeof(float) * rows);
    L.part = o; o += al(sizeof(float) * (size_t)mlpk::partials(rows) * mlpk::NPL);
    L.total = o;
    return L;
}

}  // namespace


struct mlp_handle {
    char* base = nullptr;
    MLayout lay;
    int max_rows = 0, n = 0;
    long long t = 0;    // Adam step count
    hipStream_t stream = nullptr;
    // pinned host rows of short inferences, inputs then outputs (null: none granted); its
    // allocation makes a new handle 80 us dearer, which seven inferences earn back
    static constexpr int PIN_ROWS = 4096;
    float* pin = nullptr;
    mlpk::Norm norm;
    float* p(size_t off) { return (float*)(base + off); }
};

#define MHIP(call)                                                                            \
    do {                                                                                      \
        hipError_t e_ = (call);                                                               \
        if (e_ != hipSuccess) return mfail(LB_EDEVICE, "%s failed: %s", #call, hipGetErrorString(e_)); \
    } while (0)

namespace {

lb_status fill_zero(mlp_handle* h, size_t off, size_t count)
{
    hipLaunchKernelGGL(mlpk::k_zero, dim3((unsigned)std::min<size_t>((count + 255) / 256, mlpk::BLOCKS)), dim3(256), 0,
                       h->stream, h->p(off), count);
    MHIP(hipGetLastError());
    return LB_OK;
}

// One forward/backward over the uploaded data; optionally one Adam step.
lb_status fwdbwd(mlp_handle* h, bool update, float lr)
{
    if (h->n < 1) return mfail(LB_ESTATE, "no training data uploaded (mlp_set_data)");
    const int np = mlpk::partials(h->n);
    hipLaunchKernelGGL(mlpk::k_fwdbwd, dim3(std::min(np, mlpk::BLOCKS)), dim3(64 * mlpk::WAVES), 0, h->stream, h->p(h->lay.th), h->norm,
                       h->p(h->lay.X), h->p(h->lay.Y), h->n, h->p(h->lay.part));
    MHIP(hipGetLastError());
    float c1 = 1.f, c2 = 1.f;
    if (update) {
        h->t += 1;
        c1 = (float)(1.0 / (1.0 - std::pow(0.9, (double)h->t)));
        c2 = (float)(1.0 / (1.0 - std::pow(0.999, (double)h->t)));
    }
    hipLaunchKernelGGL(mlpk::k_reduce_adam, dim3((mlpk::NPL + 63) / 64), dim3(64 * mlpk::RWAVES), 0, h->stream,
                       h->p(h->lay.part), np, h->p(h->lay.th), h->p(h->lay.m), h->p(h->lay.v), h->p(h->lay.g),
                       h->p(h->lay.loss), 1.0f / (float)h->n, update ? 1 : 0, lr, c1, c2);
    MHIP(hipGetLastError());
    return LB_OK;
}

}  // namespace

extern "C" {

lb_status mlp_state_bytes(int32_t max_rows, size_t* bytes)
{
    if (!bytes || max_rows < 1 || max_rows > (1 << 22)) return mfail(LB_EINVAL, "max_rows must be in [1, 2^22]");
    *bytes = mlayout(max_rows).total;
    return LB_OK;
}

lb_status mlp_init(void* dev_state, size_t bytes, int32_t max_rows, void* stream, mlp_handle** out)
{
    if (!out) return mfail(LB_EINVAL, "null output handle");
    *out = nullptr;
    size_t need = 0;
    lb_status st = mlp_state_bytes(max_rows, &need);
    if (st != LB_OK) return st;
    if (!dev_state || ((uintptr_t)dev_state) % 256) return mfail(LB_EINVAL, "device state must be 256-byte aligned");
    if (bytes < need) return mfail(LB_ENOMEM, "device state of %zu bytes is smaller than the %zu required", bytes, need);
    mlp_handle* h = new (std::nothrow) mlp_handle();
    if (!h) return mfail(LB_ENOMEM, "host allocation failed");
    h->base = (char*)dev_state;
    h->lay = mlayout(max_rows);
    h->max_rows = max_rows;
    h->stream = (hipStream_t)stream;
    for (int c = 0; c < 3; ++c) { h->norm.in_mean[c] = 0.f; h->norm.in_std[c] = 1.f; }
    h->norm.out_mean = 0.f;
    h->norm.out_std = 1.f;
    st = fill_zero(h, 0, h->lay.Y / sizeof(float));
    if (st != LB_OK) { delete h; return st; }
    if (hipStreamSynchronize(h->stream) != hipSuccess) { delete h; return mfail(LB_EDEVICE, "device state not writable"); }
    const size_t pinned = sizeof(float) * 4 * (size_t)std::min<int>(max_rows, mlp_handle::PIN_ROWS);
    if (hipHostMalloc(reinterpret_cast<void**>(&h->pin), pinned, hipHostMallocDefault) != hipSuccess) {
        h->pin = nullptr;
        (void)hipGetLastError();
    }
    *out = h;
    return LB_OK;
}

lb_status mlp_set_params(mlp_handle* h, const float* theta)
{
    if (!h || !theta) return mfail(LB_EINVAL, "null argument");
    for (int i = 0; i < mlpk::NP; ++i)
        if (!std::isfinite(theta[i])) return mfail(LB_EINVAL, "non-finite parameter %d", i);
    MHIP(hipMemcpyAsync(h->p(h->lay.th), theta, sizeof(float) * mlpk::NP, hipMemcpyHostToDevice, h->stream));
    h->t = 0;
    lb_status st = fill_zero(h, h->lay.m, mlpk::NP);
    if (st == LB_OK) st = fill_zero(h, h->lay.v, mlpk::NP);
    if (st != LB_OK) return st;
    MHIP(hipStreamSynchronize(h->stream));
    return LB_OK;
}

lb_status mlp_get_params(mlp_handle* h, float* theta)
{
    if (!h || !theta) return mfail(LB_EINVAL, "null argument");
    MHIP(hipMemcpyAsync(theta, h->p(h->lay.th), sizeof(float) * mlpk::NP, hipMemcpyDeviceToHost, h->stream));
    MHIP(hipStreamSynchronize(h->stream));
    return LB_OK;
}

lb_status mlp_set_norm(mlp_handle* h, const float in_mean[3], const float in_std[3], float out_mean, float out_std)
{
    if (!h || !in_mean || !in_std) return mfail(LB_EINVAL, "null argument");
    for (int c = 0; c < 3; ++c)
        if (!(in_std[c] > 0.f) || !std::isfinite(in_mean[c])) return mfail(LB_EINVAL, "bad input standardisation");
    if (!(out_std > 0.f) || !std::isfinite(out_mean)) return mfail(LB_EINVAL, "bad output standardisation");
    for (int c = 0; c < 3; ++c) { h->norm.in_mean[c] = in_mean[c]; h->norm.in_std[c] = in_std[c]; }
    h->norm.out_mean = out_mean;
    h->norm.out_std = out_std;
    return LB_OK;
}

lb_status mlp_set_data(mlp_handle* h, const float* X, const float* y, int32_t n)
{
    if (!h || !X || !y) return mfail(LB_EINVAL, "null argument");
    if (n < 1 || n > h->max_rows) return mfail(LB_EINVAL, "row count %d outside [1, %d]", n, h->max_rows);
    for (int i = 0; i < 3 * n; ++i)
        if (!std::isfinite(X[i])) return mfail(LB_EINVAL, "non-finite input");
    for (int i = 0; i < n; ++i)
        if (!std::isfinite(y[i])) return mfail(LB_EINVAL, "non-finite target");
    MHIP(hipMemcpyAsync(h->p(h->lay.X), X, sizeof(float) * 3 * n, hipMemcpyHostToDevice, h->stream));
    MHIP(hipMemcpyAsync(h->p(h->lay.Y), y, sizeof(float) * n, hipMemcpyHostToDevice, h->stream));
    MHIP(hipStreamSynchronize(h->stream));
    h->n = n;
    return LB_OK;
}

lb_status mlp_loss_grad(mlp_handle* h, float* loss, float* grad)
{
    if (!h) return mfail(LB_EINVAL, "null handle");
    lb_status st = fwdbwd(h, false, 0.f);
    if (st != LB_OK) return st;
    if (loss) MHIP(hipMemcpyAsync(loss, h->p(h->lay.loss), sizeof(float), hipMemcpyDeviceToHost, h->stream));
    if (grad) MHIP(hipMemcpyAsync(grad, h->p(h->lay.g), sizeof(float) * mlpk::NP, hipMemcpyDeviceToHost, h->stream));
    MHIP(hipStreamSynchronize(h->stream));
    return LB_OK;
}

lb_status mlp_train(mlp_handle* h, int32_t iters, float lr, float* loss)
{
    if (!h) return mfail(LB_EINVAL, "null handle");
    if (iters < 0 || !(lr > 0.f) || !std::isfinite(lr)) return mfail(LB_EINVAL, "need iters >= 0 and lr > 0");
    for (int k = 0; k < iters; ++k) {
        lb_status st = fwdbwd(h, true, lr);
        if (st != LB_OK) return st;
    }
    if (loss) MHIP(hipMemcpyAsync(loss, h->p(h->lay.loss), sizeof(float), hipMemcpyDeviceToHost, h->stream));
    MHIP(hipStreamSynchronize(h->stream));
    return LB_OK;
}

lb_status mlp_infer(mlp_handle* h, const float* X, int32_t n, float* y)
{
    if (!h || !X || !y) return mfail(LB_EINVAL, "null argument");
    if (n < 1 || n > h->max_rows) return mfail(LB_EINVAL, "row count %d outside [1, %d]", n, h->max_rows);
    // Up to PIN_ROWS rows the kernel reads its inputs from pinned host memory and writes its
    // outputs there: a copy each way took longer than it (512 rows: 31 us a call with the
    // copies, 20 us without).
    const bool pinned = h->pin && n <= std::min<int>(h->max_rows, mlp_handle::PIN_ROWS);
    float* xi = pinned ? h->pin : h->p(h->lay.Xi);
    float* yi = pinned ? h->pin + 3 * (size_t)n : h->p(h->lay.Yi);
    if (pinned) std::memcpy(xi, X, sizeof(float) * 3 * n);
    else MHIP(hipMemcpyAsync(xi, X, sizeof(float) * 3 * n, hipMemcpyHostToDevice, h->stream));
    const int nb = std::min((n + mlpk::WAVES - 1) / mlpk::WAVES, mlpk::BLOCKS);
    hipLaunchKernelGGL(mlpk::k_infer, dim3(nb), dim3(64 * mlpk::WAVES), 0, h->stream, h->p(h->lay.th), h->norm,
                       xi, n, yi);
    MHIP(hipGetLastError());
    if (!pinned) MHIP(hipMemcpyAsync(y, yi, sizeof(float) * n, hipMemcpyDeviceToHost, h->stream));
    MHIP(hipStreamSynchronize(h->stream));
    if (pinned) std::memcpy(y, yi, sizeof(float) * n);
    return LB_OK;
}

lb_status mlp_destroy(mlp_handle* h)
{
    if (h && h->pin) (void)hipHostFree(h->pin);
    delete h;
    return LB_OK;
}

}  // extern "C"
