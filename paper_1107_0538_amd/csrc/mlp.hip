// Multilayer perceptron of the learned warm start: forward, backward and Adam
// on the GPU with hand-written kernels.
//
// Network: hidden layers h = silu(W h_prev + b), linear output, loss =
// sum((Y - T)^2) / (B * out), Adam with bias correction.  W_l is (out x in)
// row-major; batches are (B x features) row-major.  Two precisions:
//   FP32  every operand FP32;
//   BF16  weights and hidden activations held as BF16 copies (FP32 master
//         weights updated by Adam), products accumulated in FP32, gradients
//         FP32.
// Where 64 x 64 output tiles would not fill the chip, a layer is one launch in
// either direction (the small-network kernels below).  Otherwise the products
// are one tiled GEMM kernel (64 x 64 output tiles, 16-deep LDS
// stages, 4 x 4 outputs per thread, FP32 accumulation) with optional
// transposed operands and a split of the reduction dimension whose partials
// are summed in fixed order (weight gradients reduce over the batch).
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>
#include <vector>

#include "context.hpp"

namespace jpcg {

using bf16 = uint16_t;

__device__ __forceinline__ float to_f(float v) { return v; }
__device__ __forceinline__ float to_f(bf16 v) { return __uint_as_float((uint32_t)v << 16); }

// Round to nearest even (ties to even), NaN kept quiet.
__device__ __forceinline__ bf16 f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (bf16)0x7fc0;
    u += 0x7fffu + ((u >> 16) & 1u);
    return (bf16)(u >> 16);
}
template <typename T>
__device__ __forceinline__ T from_f(float v);
template <>
__device__ __forceinline__ float from_f<float>(float v) { return v; }
template <>
__device__ __forceinline__ bf16 from_f<bf16>(float v) { return f2bf(v); }

constexpr int GT = 64, GK = 16;
constexpr int kSmallTiles = 256;  // see small_net

// C_z (M x N, row-major, ldc) = sum over k in split z of A(m,k) B(k,n).
// A(m,k) = TA ? A[k*lda + m] : A[m*lda + k];  B(k,n) = TB ? B[n*ldb + k] : B[k*ldb + n].
template <typename XA, typename XB, bool TA, bool TB>
__global__ __launch_bounds__(256) void k_mgemm(int M, int N, int K, const XA* __restrict__ A, int lda,
                                               const XB* __restrict__ B, int ldb, float* __restrict__ C, int ldc,
                                               int kchunk)
{
    __shared__ float As[GK][GT + 1];
    __shared__ float Bs[GK][GT + 1];
    const int mb = blockIdx.x * GT, nb = blockIdx.y * GT, z = blockIdx.z;
    const int k_lo = z * kchunk, k_hi = min(K, k_lo + kchunk);
    const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
    float acc[4][4] = {};
    for (int k0 = k_lo; k0 < k_hi; k0 += GK) {
        for (int e = threadIdx.x; e < GT * GK; e += 256) {
            const int kk = e / GT, mm = e % GT;
            const int m = mb + mm, k = k0 + kk;
            float av = 0.f;
            if (m < M && k < k_hi) av = to_f(TA ? A[(size_t)k * lda + m] : A[(size_t)m * lda + k]);
            As[kk][mm] = av;
            const int n = nb + mm;
            float bv = 0.f;
            if (n < N && k < k_hi) bv = to_f(TB ? B[(size_t)n * ldb + k] : B[(size_t)k * ldb + n]);
            Bs[kk][mm] = bv;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < GK; ++kk) {
            float av[4], bv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                av[u] = As[kk][ty * 4 + u];
                bv[u] = Bs[kk][tx * 4 + u];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[u][v] = __builtin_fmaf(av[u], bv[v], acc[u][v]);
        }
        __syncthreads();
    }
    float* out = C + (size_t)z * M * ldc;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int m = mb + ty * 4 + u;
        if (m >= M) continue;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int n = nb + tx * 4 + v;
            if (n < N) out[(size_t)m * ldc + n] = acc[u][v];
        }
    }
}

__global__ void k_sum_splits(const float* __restrict__ part, int splits, int64_t count, float* __restrict__ out)
{
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < count; e += (int64_t)gridDim.x * blockDim.x) {
        float s = 0.f;
        for (int z = 0; z < splits; ++z) s += part[(size_t)z * count + e];
        out[e] = s;
    }
}

__device__ __forceinline__ float sigmoidf_(float u) { return 1.f / (1.f + __expf(-u)); }

// U = C + bias (pre-activation, FP32); H = silu(U) (hidden) or U (output).
template <typename TH>
__global__ void k_bias_act(int Bn, int N, const float* __restrict__ C, const float* __restrict__ bias,
                           float* __restrict__ U, TH* __restrict__ H, int act)
{
    const int64_t count = (int64_t)Bn * N;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < count; e += (int64_t)gridDim.x * blockDim.x) {
        const float u = C[e] + bias[e % N];
        U[e] = u;
        H[e] = from_f<TH>(act ? u * sigmoidf_(u) : u);
    }
}

// D = 2 (Y - T) / (B * m); per-block partial sums of (Y - T)^2.
__global__ void k_mse(int64_t count, const float* __restrict__ Y, const float* __restrict__ T, float scale,
                      float* __restrict__ D, double* __restrict__ loss_part)
{
    __shared__ double red[256];
    double l = 0.0;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < count; e += (int64_t)gridDim.x * blockDim.x) {
        const float d = Y[e] - T[e];
        D[e] = 2.f * d * scale;
        l += (double)d * (double)d;
    }
    red[threadIdx.x] = l;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int i = 0; i < (int)blockDim.x; ++i) s += red[i];
        loss_part[blockIdx.x] = s;
    }
}

// D_out = D_in * silu'(U).
__global__ void k_silu_back(int64_t count, const float* __restrict__ Din, const float* __restrict__ U,
                            float* __restrict__ Dout)
{
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < count; e += (int64_t)gridDim.x * blockDim.x) {
        const float u = U[e], s = sigmoidf_(u);
        Dout[e] = Din[e] * (s * (1.f + u * (1.f - s)));
    }
}

// db[o] = sum over the batch of D[b, o], in batch order.
__global__ void k_colsum(int Bn, int N, const float* __restrict__ D, float* __restrict__ db)
{
    const int o = blockIdx.x * blockDim.x + threadIdx.x;
    if (o >= N) return;
    float s = 0.f;
    for (int b = 0; b < Bn; ++b) s += D[(size_t)b * N + o];
    db[o] = s;
}

// Adam on the FP32 master parameters; refresh the BF16 copies.
struct AdamArgs {
    float *p, *g, *m, *v;
    bf16* pb;
    float lr, b1, b2, eps, c1, c2;
    int update;  // 0: the gradient is stored, 1: Adam's step is taken
};
struct AdamState {
    float p, m, v;
    __device__ __forceinline__ void load(const AdamArgs& a, int64_t i)
    {
        p = a.p[i];
        m = a.m[i];
        v = a.v[i];
    }
    __device__ __forceinline__ void step(const AdamArgs& a, int64_t i, float gi) const
    {
        const float mi = __builtin_fmaf(1.f - a.b1, gi, a.b1 * m);
        const float vi = __builtin_fmaf((1.f - a.b2) * gi, gi, a.b2 * v);
        a.m[i] = mi;
        a.v[i] = vi;
        const float pi = p - a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
        a.p[i] = pi;
        if (a.pb) a.pb[i] = f2bf(pi);
    }
};
__global__ void k_adam(int64_t n, AdamArgs a)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        AdamState w;
        w.load(a, i);
        w.step(a, i, a.g[i]);
    }
}

__global__ void k_to_bf16(int64_t n, const float* __restrict__ in, bf16* __restrict__ out)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        out[i] = f2bf(in[i]);
}

// ---------------------------------------------------------------------------
// Small networks: one launch per layer and direction.
//
// A 64 x 64 output tile gives a 256 x 256 layer 16 workgroups, each walking the
// whole reduction in stages of 16, and the sums over the batch, the bias, the
// activation and its derivative, the splits' sum and Adam were launches of their
// own: 22 a step, 410 us with a batch and hidden layers of 256 (24 inputs, 64
// outputs); 46 as it is, in six launches.  Here a workgroup forms 16 x 16 outputs, an output per thread, from
// panels of 256 along the reduction held in LDS, and applies what follows in
// registers.  What bounds it is latency: a panel's loads, the chain of
// additions, the launch.
//
// Every sum keeps the order of the kernels above: k ascending, the weight
// gradients' reduction over the batch in the same chunks, which are added in
// order, the bias gradients in batch order.
// ---------------------------------------------------------------------------
constexpr int ST = 16, SK = 256, SP = SK + 4;  // pitch: 16 rows' 16-byte reads fall on different banks

struct SmallPanels {
    float a[ST][SP];
    float b[ST][SP];
};

// p[r][k] = f(r, k) for r < rows and k < kn, else 0 (k to a multiple of 16).
// Neighbouring threads take neighbouring k (ALONG) or neighbouring rows,
// whichever lie together in memory.  A panel's loads are sent one after the
// other from addresses that are always good, and looked at when all are sent:
// a conversion or a branch at each would wait for it (a layer of 256 forward 10.5
// us, backward 16.5; with the loads apart from their use 6.6 and 8.4).
template <typename T>
struct SmallLoads {
    T v[ST];
    template <bool ALONG, typename F>
    __device__ __forceinline__ void send(int rows, int kn, F f)
    {
        const int t = threadIdx.x;
        if (ALONG) {
            const int k = min(t, kn - 1);
#pragma unroll
            for (int r = 0; r < ST; ++r) v[r] = f(min(r, rows - 1), k);
        } else {
            const int r = min(t % ST, rows - 1);
#pragma unroll
            for (int j = 0; j < SK / ST; ++j) v[j] = f(r, min(t / ST + ST * j, kn - 1));
        }
    }
    template <bool ALONG, typename C>
    __device__ __forceinline__ void keep(float (&p)[ST][SP], int rows, int kn, C convert) const
    {
        const int t = threadIdx.x;
        if (ALONG) {
#pragma unroll
            for (int r = 0; r < ST; ++r) p[r][t] = r < rows && t < kn ? convert(v[r], r, t) : 0.f;
        } else {
            const int r = t % ST;
#pragma unroll
            for (int j = 0; j < SK / ST; ++j) {
                const int k = t / ST + ST * j;
                p[r][k] = r < rows && k < kn ? convert(v[j], r, k) : 0.f;
            }
        }
    }
};
static_assert(SK == 256 && SK / ST == ST, "a thread holds 16 of a panel's values either way");

// acc += sum over k_lo <= k < kn of a[m][k] b[n][k], k ascending (k_lo a multiple of 16).
__device__ __forceinline__ float small_dot(const SmallPanels& s, int m, int n, int k_lo, int kn, float acc)
{
    for (int k = k_lo; k < kn; k += 16) {
        float4 av[4], bv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            av[u] = *(const float4*)&s.a[m][k + 4 * u];
            bv[u] = *(const float4*)&s.b[n][k + 4 * u];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            acc = __builtin_fmaf(av[u].x, bv[u].x, acc);
            acc = __builtin_fmaf(av[u].y, bv[u].y, acc);
            acc = __builtin_fmaf(av[u].z, bv[u].z, acc);
            acc = __builtin_fmaf(av[u].w, bv[u].w, acc);
        }
    }
    return acc;
}

// One layer forward: U = H W' + b, the activation; for the last layer with
// targets also D = 2 (U - T) scale and the workgroup's sum of (U - T)^2.
template <typename TW>
struct SmallForward {
    int M, N, K;
    const float* X;  // the first layer: the caller's batch, kept in H0 as the network keeps activations
    TW* H0;
    const TW* in;    // other layers
    const TW* W;
    const float* bias;
    float* U;
    TW* H;         // hidden layers: silu(U)
    float* Y;      // the last layer's output
    const float* T;
    float scale;
    float* D;
    double* loss;
};
template <typename TW>
__global__ __launch_bounds__(256) void k_small_forward(SmallForward<TW> f)
{
    __shared__ SmallPanels s;
    __shared__ double red[256];
    const int mb = blockIdx.x * ST, nb = blockIdx.y * ST;
    const int m = threadIdx.x / ST, n = threadIdx.x % ST;
    float acc = 0.f;
    for (int k0 = 0; k0 < f.K; k0 += SK) {
        const int kn = min(SK, f.K - k0);
        SmallLoads<TW> la, lb;
        SmallLoads<float> lx;
        auto at = [&](int r, int k) { return (int64_t)(mb + r) * f.K + k0 + k; };
        if (f.X) lx.template send<true>(f.M - mb, kn, [&](int r, int k) { return f.X[at(r, k)]; });
        else la.template send<true>(f.M - mb, kn, [&](int r, int k) { return f.in[at(r, k)]; });
        lb.template send<true>(f.N - nb, kn, [&](int r, int k) { return f.W[(int64_t)(nb + r) * f.K + k0 + k]; });
        if (k0) __syncthreads();
        if (f.X) {
            lx.template keep<true>(s.a, f.M - mb, kn, [&](float x, int r, int k) {
                const TW v = from_f<TW>(x);
                if (nb == 0) f.H0[at(r, k)] = v;
                return to_f(v);
            });
        } else {
            la.template keep<true>(s.a, f.M - mb, kn, [](TW v, int, int) { return to_f(v); });
        }
        lb.template keep<true>(s.b, f.N - nb, kn, [](TW v, int, int) { return to_f(v); });
        __syncthreads();
        acc = small_dot(s, m, n, 0, kn, acc);
    }
    double l = 0.0;
    if (mb + m < f.M && nb + n < f.N) {
        const int64_t e = (int64_t)(mb + m) * f.N + nb + n;
        const float u = acc + f.bias[nb + n];
        f.U[e] = u;
        if (f.H) f.H[e] = from_f<TW>(u * sigmoidf_(u));
        if (f.Y) f.Y[e] = u;
        if (f.T) {
            const float d = u - f.T[e];
            f.D[e] = 2.f * d * f.scale;
            l = (double)d * (double)d;
        }
    }
    if (!f.T) return;
    red[threadIdx.x] = l;
    for (int w = 128; w > 0; w /= 2) {
        __syncthreads();
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    }
    if (threadIdx.x == 0) f.loss[blockIdx.y * gridDim.x + blockIdx.x] = red[0];
}

// Dn = (D W) silu'(U): the gradient through a layer and the activation before it.
template <typename TW>
struct SmallThrough {
    int M, N, K;  // batch, inputs, outputs of the layer
    int tiles;    // 0: none
    const float* D;
    const TW* W;
    const float* U;
    float* Dn;
};
// dW = D' H and db over the batch in chunks, and what is done with them.
template <typename TW>
struct SmallWeights {
    int M, N, K;  // outputs, inputs, batch
    int tiles;
    int chunk, splits;
    const float* D;
    const TW* in;
    int64_t at;  // of the layer's weights in the parameters, its biases behind them
};
// Several at once where none waits for another: a layer's gradient through its
// weights, and the weights of up to two layers whose gradients are known and
// whose weights nothing reads any more.
template <typename TW>
struct SmallBackward {
    SmallThrough<TW> through;
    SmallWeights<TW> w[2];
    AdamArgs adam;
};
template <typename TW>
__global__ __launch_bounds__(256) void k_small_backward(SmallBackward<TW> f)
{
    __shared__ SmallPanels s;
    const int m = threadIdx.x / ST, n = threadIdx.x % ST;
    int tile = blockIdx.x;
    if (tile < f.through.tiles) {
        const SmallThrough<TW>& t = f.through;
        const int across = (t.N + ST - 1) / ST, mb = tile / across * ST, nb = tile % across * ST;
        const float u = t.U[(int64_t)min(mb + m, t.M - 1) * t.N + min(nb + n, t.N - 1)];
        float acc = 0.f;
        for (int k0 = 0; k0 < t.K; k0 += SK) {
            const int kn = min(SK, t.K - k0);
            SmallLoads<float> la;
            SmallLoads<TW> lb;
            la.template send<true>(t.M - mb, kn, [&](int r, int k) { return t.D[(int64_t)(mb + r) * t.K + k0 + k]; });
            lb.template send<false>(t.N - nb, kn, [&](int r, int k) { return t.W[(int64_t)(k0 + k) * t.N + nb + r]; });
            if (k0) __syncthreads();
            la.template keep<true>(s.a, t.M - mb, kn, [](float v, int, int) { return v; });
            lb.template keep<false>(s.b, t.N - nb, kn, [](TW v, int, int) { return to_f(v); });
            __syncthreads();
            acc = small_dot(s, m, n, 0, kn, acc);
        }
        if (mb + m < t.M && nb + n < t.N) {
            const int64_t e = (int64_t)(mb + m) * t.N + nb + n;
            const float sg = sigmoidf_(u);
            t.Dn[e] = acc * (sg * (1.f + u * (1.f - sg)));
        }
        return;
    }
    tile -= f.through.tiles;
    const bool second = tile >= f.w[0].tiles;
    if (second) tile -= f.w[0].tiles;
    const SmallWeights<TW>& t = second ? f.w[1] : f.w[0];
    const int across = (t.N + ST - 1) / ST, mb = tile / across * ST, nb = tile % across * ST;
    const bool mine = mb + m < t.M && nb + n < t.N;
    const bool biases = nb == 0 && threadIdx.x < ST && mb + (int)threadIdx.x < t.M;
    // The parameters' state is on its way while the sums are formed.
    AdamState w, wb;
    const int64_t iw = t.at + (int64_t)(mb + m) * t.N + nb + n, ib = t.at + (int64_t)t.M * t.N + mb + threadIdx.x;
    if (f.adam.update && mine) w.load(f.adam, iw);
    if (f.adam.update && biases) wb.load(f.adam, ib);
    float sum = 0.f, db = 0.f;
    auto panel = [&](int k0, int kn) {
        SmallLoads<float> la;
        SmallLoads<TW> lb;
        la.template send<false>(t.M - mb, kn, [&](int r, int k) { return t.D[(int64_t)(k0 + k) * t.M + mb + r]; });
        lb.template send<false>(t.N - nb, kn, [&](int r, int k) { return t.in[(int64_t)(k0 + k) * t.N + nb + r]; });
        __syncthreads();
        la.template keep<false>(s.a, t.M - mb, kn, [](float v, int, int) { return v; });
        lb.template keep<false>(s.b, t.N - nb, kn, [](TW v, int, int) { return to_f(v); });
        __syncthreads();
        if (biases) {
            int k = 0;
            for (; k + 16 <= kn; k += 16) {
                float v[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) v[u] = s.a[threadIdx.x][k + u];
#pragma unroll
                for (int u = 0; u < 16; ++u) db += v[u];
            }
            for (; k < kn; ++k) db += s.a[threadIdx.x][k];
        }
    };
    // One panel for the whole batch where its chunks begin at multiples of 16.
    const bool whole = t.K <= SK && t.chunk % 16 == 0;
    if (whole) panel(0, t.K);
    for (int z = 0; z < t.splits; ++z) {
        const int k1 = min(t.K, (z + 1) * t.chunk);
        float acc = 0.f;
        if (whole) {
            acc = small_dot(s, m, n, z * t.chunk, k1, acc);
        } else {
            for (int k0 = z * t.chunk; k0 < k1; k0 += SK) {
                const int kn = min(SK, k1 - k0);
                panel(k0, kn);
                acc = small_dot(s, m, n, 0, kn, acc);
            }
        }
        sum = t.splits > 1 ? sum + acc : acc;
    }
    if (f.adam.update) {
        if (mine) w.step(f.adam, iw, sum);
        if (biases) wb.step(f.adam, ib, db);
    } else {
        if (mine) f.adam.g[iw] = sum;
        if (biases) f.adam.g[ib] = db;
    }
}

static int grid_for(int64_t count) { return (int)std::min<int64_t>(2048, std::max<int64_t>(1, (count + 255) / 256)); }

}  // namespace jpcg

struct mlp_net {
    hipStream_t stream = nullptr;
    int L = 0;                  // layers
    std::vector<int> dims;      // L + 1
    int precision = 0;          // 0 FP32, 1 BF16
    int max_batch = 0;
    int64_t nparam = 0;
    std::vector<int64_t> woff;  // offset of W_l in the flat parameter vector (b_l follows)
    float* p = nullptr;         // FP32 master parameters
    float* g = nullptr;         // gradients
    float* m = nullptr;         // Adam moments
    float* v = nullptr;
    jpcg::bf16* pb = nullptr;   // BF16 copies (BF16 mode)
    std::vector<void*> H;       // activations per layer input (L + 1): FP32 or BF16 (input and hidden), FP32 output
    std::vector<float*> U;      // pre-activations per layer
    float* D0 = nullptr;        // gradient buffers (max_batch x max width)
    float* D1 = nullptr;
    float* D2 = nullptr;
    float* C = nullptr;         // GEMM output / split partials
    size_t c_cap = 0;
    double* loss_part = nullptr;
    double* hloss = nullptr;
    int t = 0;                  // Adam step count
};

namespace jpcg {

static void free_mlp(mlp_net* n)
{
    if (!n) return;
    void* ptrs[] = {n->p, n->g, n->m, n->v, n->pb, n->D0, n->D1, n->D2, n->C, n->loss_part};
    for (void* q : ptrs)
        if (q) (void)hipFree(q);
    for (void* q : n->H)
        if (q) (void)hipFree(q);
    for (float* q : n->U)
        if (q) (void)hipFree(q);
    if (n->hloss) (void)hipHostFree(n->hloss);
    delete n;
}

// C = op(A) op(B) with the reduction split in `splits` fixed chunks.
template <typename XA, typename XB, bool TA, bool TB>
static void gemm(mlp_net* n, int M, int N, int K, const XA* A, int lda, const XB* B, int ldb, float* out, int splits)
{
    const int kchunk = (K + splits - 1) / splits;
    splits = (K + kchunk - 1) / kchunk;
    float* dst = splits > 1 ? n->C : out;
    if (splits > 1 && (size_t)splits * M * N > n->c_cap) throw HipError{hipErrorInvalidValue, "gemm scratch"};
    dim3 grid((M + GT - 1) / GT, (N + GT - 1) / GT, splits);
    k_mgemm<XA, XB, TA, TB><<<grid, 256, 0, n->stream>>>(M, N, K, A, lda, B, ldb, dst, N, kchunk);
    JPCG_HIP(hipGetLastError());
    if (splits > 1) {
        const int64_t count = (int64_t)M * N;
        k_sum_splits<<<grid_for(count), 256, 0, n->stream>>>(n->C, splits, count, out);
        JPCG_HIP(hipGetLastError());
    }
}

template <typename TW>
static const TW* weights(mlp_net* n, int l);
template <>
const float* weights<float>(mlp_net* n, int l) { return n->p + n->woff[l]; }
template <>
const bf16* weights<bf16>(mlp_net* n, int l) { return n->pb + n->woff[l]; }

// Fixed chunks of the batch that the weight gradients are summed in.
static int batch_splits(int Bn) { return std::max(1, std::min(16, Bn / 128)); }

static int64_t tiles_of(int a, int b) { return (int64_t)((a + GT - 1) / GT) * ((b + GT - 1) / GT); }

// The small-network kernels serve networks and batches no layer of which fills
// the chip with 64 x 64 tiles: up to 256 of them per product.  24-256-256-64 in
// BF16, a step with batches of 32, 256 and 4096: 35, 45 and 343 us against 207,
// 410 and 2831; hidden layers of 1024 with 1024 (256 tiles): 674 us against 1198;
// with 2048 (512 tiles) about equal.
static bool small_net(const mlp_net* n, int Bn)
{
    for (int l = 0; l < n->L; ++l)
        if (tiles_of(Bn, n->dims[l + 1]) > kSmallTiles || tiles_of(n->dims[l], n->dims[l + 1]) > kSmallTiles) return false;
    return true;
}

// A forward pass by itself: a layer of K inputs and t tiles takes 5 + 0.02 t + 0.15 K
// us in large tiles and 4.5 + 0.02 t + 0.00068 t K here (K = 64 to 1024, t = 64 to
// 256; 256 tiles of 64, 256 and 1024 inputs: 20, 48, 160 us and 21, 49, 184), so
// layers of over 220 tiles are better off in large ones.
static bool small_pass(const mlp_net* n, int Bn)
{
    double more = -735.0 * n->L;  // 0.00068 t K - 0.15 K - 0.5, in units of 0.00068 us
    for (int l = 0; l < n->L; ++l) more += n->dims[l] * (tiles_of(Bn, n->dims[l + 1]) - 220.0);
    return more <= 0.0 && small_net(n, Bn);
}

// The forward pass of a small network; with targets also the last layer's
// gradient, into n->D0, and the loss partials (their number is returned).
template <typename TW>
static int small_forward(mlp_net* n, const float* X, int Bn, float* Y, const float* T)
{
    int partials = 0;
    for (int l = 0; l < n->L; ++l) {
        const int in = n->dims[l], out = n->dims[l + 1];
        const bool last = l == n->L - 1;
        SmallForward<TW> f{};
        f.M = Bn;
        f.N = out;
        f.K = in;
        f.X = l == 0 ? X : nullptr;
        f.H0 = (TW*)n->H[0];
        f.in = (const TW*)n->H[l];
        f.W = weights<TW>(n, l);
        f.bias = n->p + n->woff[l] + (int64_t)out * in;
        f.U = n->U[l];
        f.H = last ? nullptr : (TW*)n->H[l + 1];
        f.Y = last ? (Y ? Y : (float*)n->H[l + 1]) : nullptr;
        f.T = last ? T : nullptr;
        f.scale = 1.f / (float)((int64_t)Bn * out);
        f.D = n->D0;
        f.loss = n->loss_part;
        const dim3 grid((Bn + ST - 1) / ST, (out + ST - 1) / ST);
        k_small_forward<TW><<<grid, 256, 0, n->stream>>>(f);
        JPCG_HIP(hipGetLastError());
        partials = (int)(grid.x * grid.y);
    }
    return partials;
}

template <typename TW>
static void small_backward(mlp_net* n, int Bn, const AdamArgs& adam)
{
    float* D[3] = {n->D0, n->D1, n->D2};  // layer l's gradient in D[(L - 1 - l) % 3]
    const int L = n->L;
    auto tiles = [](int a, int b) { return ((a + ST - 1) / ST) * ((b + ST - 1) / ST); };
    auto weight_job = [&](int l) {
        SmallWeights<TW> w{};
        if (l >= L) return w;
        const int splits = batch_splits(Bn);
        w.M = n->dims[l + 1];
        w.N = n->dims[l];
        w.K = Bn;
        w.tiles = tiles(w.M, w.N);
        w.chunk = (Bn + splits - 1) / splits;
        w.splits = (Bn + w.chunk - 1) / w.chunk;
        w.D = D[(L - 1 - l) % 3];
        w.in = (const TW*)n->H[l];
        w.at = n->woff[l];
        return w;
    };
    for (int l = L - 1; l >= 0; --l) {
        // Layer l's weights wait for the launch after the one that reads them;
        // the last launch takes the first two layers'.
        SmallBackward<TW> f{};
        f.adam = adam;
        f.w[0] = weight_job(l + 1);
        if (l > 0) {
            SmallThrough<TW>& t = f.through;
            t.M = Bn;
            t.N = n->dims[l];
            t.K = n->dims[l + 1];
            t.tiles = tiles(t.M, t.N);
            t.D = D[(L - 1 - l) % 3];
            t.W = weights<TW>(n, l);
            t.U = n->U[l - 1];
            t.Dn = D[(L - l) % 3];
        } else {
            f.w[1] = weight_job(0);
        }
        k_small_backward<TW><<<f.through.tiles + f.w[0].tiles + f.w[1].tiles, 256, 0, n->stream>>>(f);
        JPCG_HIP(hipGetLastError());
    }
}

template <typename TW>
static void forward_t(mlp_net* n, const float* X, int Bn, float* Y)
{
    hipStream_t st = n->stream;
    if (Y && small_pass(n, Bn)) {
        // A single layer reads X while it writes its output, which may be X.
        small_forward<TW>(n, X, Bn, n->L > 1 ? Y : nullptr, nullptr);
        if (n->L > 1) return;
        JPCG_HIP(hipMemcpyAsync(Y, n->H[1], sizeof(float) * (int64_t)Bn * n->dims[1], hipMemcpyDeviceToDevice, st));
        return;
    }
    const int64_t in0 = (int64_t)Bn * n->dims[0];
    if constexpr (sizeof(TW) == 2) {
        k_to_bf16<<<grid_for(in0), 256, 0, st>>>(in0, X, (bf16*)n->H[0]);
    } else {
        JPCG_HIP(hipMemcpyAsync(n->H[0], X, sizeof(float) * in0, hipMemcpyDeviceToDevice, st));
    }
    for (int l = 0; l < n->L; ++l) {
        const int in = n->dims[l], out = n->dims[l + 1];
        const bool last = l == n->L - 1;
        gemm<TW, TW, false, true>(n, Bn, out, in, (const TW*)n->H[l], in, weights<TW>(n, l), in, n->C, 1);
        const float* bias = n->p + n->woff[l] + (int64_t)out * in;
        const int64_t count = (int64_t)Bn * out;
        if (last) {
            k_bias_act<float><<<grid_for(count), 256, 0, st>>>(Bn, out, n->C, bias, n->U[l], (float*)n->H[l + 1], 0);
        } else {
            k_bias_act<TW><<<grid_for(count), 256, 0, st>>>(Bn, out, n->C, bias, n->U[l], (TW*)n->H[l + 1], 1);
        }
        JPCG_HIP(hipGetLastError());
    }
    if (Y) {
        JPCG_HIP(hipMemcpyAsync(Y, n->H[n->L], sizeof(float) * (int64_t)Bn * n->dims[n->L], hipMemcpyDeviceToDevice,
                                st));
    }
}

// Forward, loss, and gradients: into n->g, or Adam's step with them.  Returns the
// loss (host, after sync if want_loss).
template <typename TW>
static double backward_t(mlp_net* n, const float* X, const float* T, int Bn, bool want_loss, const AdamArgs& adam)
{
    hipStream_t st = n->stream;
    auto loss = [&](int partials) {
        if (!want_loss) return 0.0;
        JPCG_HIP(hipMemcpyAsync(n->hloss, n->loss_part, sizeof(double) * partials, hipMemcpyDeviceToHost, st));
        JPCG_HIP(hipStreamSynchronize(st));
        double s = 0.0;
        for (int i = 0; i < partials; ++i) s += n->hloss[i];
        return s / (double)((int64_t)Bn * n->dims[n->L]);
    };
    if (small_net(n, Bn)) {
        const int partials = small_forward<TW>(n, X, Bn, nullptr, T);
        small_backward<TW>(n, Bn, adam);
        return loss(partials);
    }
    forward_t<TW>(n, X, Bn, nullptr);
    const int L = n->L;
    const int m = n->dims[L];
    const int64_t cnt = (int64_t)Bn * m;
    const int lg = grid_for(cnt);
    k_mse<<<lg, 256, 0, st>>>(cnt, (const float*)n->H[L], T, 1.f / (float)cnt, n->D0, n->loss_part);
    JPCG_HIP(hipGetLastError());
    float* D = n->D0;
    float* Dn = n->D1;
    for (int l = L - 1; l >= 0; --l) {
        const int in = n->dims[l], out = n->dims[l + 1];
        float* gW = n->g + n->woff[l];
        float* gb = gW + (int64_t)out * in;
        // dW = D' H_l (out x in), reduced over the batch in fixed chunks.
        const int splits = batch_splits(Bn);
        gemm<float, TW, true, false>(n, out, in, Bn, D, out, (const TW*)n->H[l], in, gW, splits);
        k_colsum<<<(out + 255) / 256, 256, 0, st>>>(Bn, out, D, gb);
        JPCG_HIP(hipGetLastError());
        if (l > 0) {
            // dH = D W_l (B x in), then through the SiLU of layer l-1.
            gemm<float, TW, false, false>(n, Bn, in, out, D, out, weights<TW>(n, l), in, Dn, 1);
            const int64_t c2 = (int64_t)Bn * in;
            k_silu_back<<<grid_for(c2), 256, 0, st>>>(c2, Dn, n->U[l - 1], Dn);
            JPCG_HIP(hipGetLastError());
            std::swap(D, Dn);
        }
    }
    if (adam.update) {
        k_adam<<<grid_for(n->nparam), 256, 0, st>>>(n->nparam, adam);
        JPCG_HIP(hipGetLastError());
    }
    return loss(lg);
}

}  // namespace jpcg

using namespace jpcg;

extern "C" {

int mlp_create(int32_t nlayers, const int32_t* dims, int32_t precision, int32_t max_batch, void* stream,
               mlp_net** out)
{
    if (!out) return CG_EINVAL;
    *out = nullptr;
    if (nlayers < 1 || !dims || (precision != 0 && precision != 1) || max_batch < 1) return CG_EINVAL;
    for (int l = 0; l <= nlayers; ++l)
        if (dims[l] < 1) return CG_EINVAL;
    mlp_net* n = nullptr;
    try {
        n = new mlp_net();
        n->stream = (hipStream_t)stream;
        n->L = nlayers;
        n->dims.assign(dims, dims + nlayers + 1);
        n->precision = precision;
        n->max_batch = max_batch;
        int64_t o = 0;
        int wmax = 0;
        for (int l = 0; l < nlayers; ++l) {
            n->woff.push_back(o);
            o += (int64_t)dims[l] * dims[l + 1] + dims[l + 1];
        }
        for (int l = 0; l <= nlayers; ++l) wmax = std::max(wmax, dims[l]);
        n->nparam = o;
        for (float** q : {&n->p, &n->g, &n->m, &n->v}) JPCG_HIP(hipMalloc((void**)q, sizeof(float) * o));
        JPCG_HIP(hipMemsetAsync(n->p, 0, sizeof(float) * o, n->stream));
        JPCG_HIP(hipMemsetAsync(n->m, 0, sizeof(float) * o, n->stream));
        JPCG_HIP(hipMemsetAsync(n->v, 0, sizeof(float) * o, n->stream));
        if (precision == 1) {
            JPCG_HIP(hipMalloc((void**)&n->pb, sizeof(bf16) * o));
            JPCG_HIP(hipMemsetAsync(n->pb, 0, sizeof(bf16) * o, n->stream));
        }
        const size_t act_bytes = precision == 1 ? sizeof(bf16) : sizeof(float);
        n->H.assign(nlayers + 1, nullptr);
        n->U.assign(nlayers, nullptr);
        for (int l = 0; l <= nlayers; ++l) {
            const size_t eb = l == nlayers ? sizeof(float) : act_bytes;
            JPCG_HIP(hipMalloc(&n->H[l], eb * (size_t)max_batch * dims[l]));
        }
        for (int l = 0; l < nlayers; ++l) JPCG_HIP(hipMalloc((void**)&n->U[l], sizeof(float) * (size_t)max_batch * dims[l + 1]));
        JPCG_HIP(hipMalloc((void**)&n->D0, sizeof(float) * (size_t)max_batch * wmax));
        JPCG_HIP(hipMalloc((void**)&n->D1, sizeof(float) * (size_t)max_batch * wmax));
        JPCG_HIP(hipMalloc((void**)&n->D2, sizeof(float) * (size_t)max_batch * wmax));
        n->c_cap = std::max<size_t>((size_t)max_batch * wmax, (size_t)16 * wmax * wmax);
        JPCG_HIP(hipMalloc((void**)&n->C, sizeof(float) * n->c_cap));
        JPCG_HIP(hipMalloc((void**)&n->loss_part, sizeof(double) * std::max(2048, 16 * kSmallTiles)));
        JPCG_HIP(hipHostMalloc((void**)&n->hloss, sizeof(double) * std::max(2048, 16 * kSmallTiles), hipHostMallocDefault));
        JPCG_HIP(hipStreamSynchronize(n->stream));
        *out = n;
        return 0;
    } catch (const HipError& e) {
        free_mlp(n);
        return e.code == hipErrorOutOfMemory ? CG_ENOMEM : CG_EHIP;
    } catch (const std::bad_alloc&) {
        free_mlp(n);
        return CG_ENOMEM;
    }
}

int64_t mlp_param_count(const mlp_net* n) { return n ? n->nparam : CG_EINVAL; }

int mlp_set_params(mlp_net* n, const float* host)
{
    if (!n || !host) return CG_EINVAL;
    try {
        JPCG_HIP(hipMemcpyAsync(n->p, host, sizeof(float) * n->nparam, hipMemcpyHostToDevice, n->stream));
        if (n->pb) k_to_bf16<<<grid_for(n->nparam), 256, 0, n->stream>>>(n->nparam, n->p, n->pb);
        JPCG_HIP(hipMemsetAsync(n->m, 0, sizeof(float) * n->nparam, n->stream));
        JPCG_HIP(hipMemsetAsync(n->v, 0, sizeof(float) * n->nparam, n->stream));
        JPCG_HIP(hipStreamSynchronize(n->stream));
        n->t = 0;
        return 0;
    } catch (const HipError&) {
        return CG_EHIP;
    }
}

int mlp_get_params(mlp_net* n, float* host)
{
    if (!n || !host) return CG_EINVAL;
    try {
        JPCG_HIP(hipMemcpyAsync(host, n->p, sizeof(float) * n->nparam, hipMemcpyDeviceToHost, n->stream));
        JPCG_HIP(hipStreamSynchronize(n->stream));
        return 0;
    } catch (const HipError&) {
        return CG_EHIP;
    }
}

int mlp_forward(mlp_net* n, const float* X, int32_t batch, float* Y)
{
    if (!n || !X || !Y || batch < 1 || batch > n->max_batch) return CG_EINVAL;
    try {
        if (n->precision == 1) forward_t<bf16>(n, X, batch, Y);
        else forward_t<float>(n, X, batch, Y);
        return 0;
    } catch (const HipError&) {
        return CG_EHIP;
    }
}

int mlp_gradients(mlp_net* n, const float* X, const float* T, int32_t batch, float* grads_host, double* loss)
{
    if (!n || !X || !T || batch < 1 || batch > n->max_batch) return CG_EINVAL;
    try {
        AdamArgs adam{};
        adam.g = n->g;
        const double l = n->precision == 1 ? backward_t<bf16>(n, X, T, batch, true, adam)
                                           : backward_t<float>(n, X, T, batch, true, adam);
        if (loss) *loss = l;
        if (grads_host) {
            JPCG_HIP(hipMemcpyAsync(grads_host, n->g, sizeof(float) * n->nparam, hipMemcpyDeviceToHost, n->stream));
            JPCG_HIP(hipStreamSynchronize(n->stream));
        }
        return 0;
    } catch (const HipError&) {
        return CG_EHIP;
    }
}

int mlp_train_step(mlp_net* n, const float* X, const float* T, int32_t batch, float lr, float beta1, float beta2,
                   float eps, double* loss)
{
    if (!n || !X || !T || batch < 1 || batch > n->max_batch || !(lr > 0.f)) return CG_EINVAL;
    try {
        const int t = n->t + 1;
        const float c1 = 1.f - std::pow(beta1, (float)t), c2 = 1.f - std::pow(beta2, (float)t);
        const AdamArgs adam{n->p, n->g, n->m, n->v, n->pb, lr, beta1, beta2, eps, c1, c2, 1};
        const double l = n->precision == 1 ? backward_t<bf16>(n, X, T, batch, loss != nullptr, adam)
                                           : backward_t<float>(n, X, T, batch, loss != nullptr, adam);
        n->t = t;
        if (loss) *loss = l;
        return 0;
    } catch (const HipError&) {
        return CG_EHIP;
    }
}

void mlp_destroy(mlp_net* n)
{
    if (!n) return;
    (void)hipStreamSynchronize(n->stream);
    free_mlp(n);
}

}  // extern "C"
