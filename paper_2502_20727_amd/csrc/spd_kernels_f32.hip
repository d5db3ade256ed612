// fp32 path: small, plain kernels in natural layouts (used by the toy-sized configuration and
// as the library's generic rank-sum), plus helpers shared by both paths.
#include <mutex>

#include "spd_internal.h"

namespace {

constexpr int TB = 256;

__global__ void k_rank_sum(const float *__restrict__ base, const float *__restrict__ slots, int n_slots,
                           int64_t n, float *__restrict__ out, const float *__restrict__ bias, int h) {
    // partials are summed in ascending slot order, the base is added last
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float acc = 0.0f;
    if (n_slots > 0) {
        acc = slots[i];
        for (int s = 1; s < n_slots; ++s) acc += slots[(int64_t)s * n + i];
    }
    if (base) acc = base[i] + acc;
    if (bias) acc += bias[i % h];          // the output projection's bias, once, after the sum
    out[i] = acc;
}

__global__ void k_rank_sum4(const float4 *__restrict__ base, const float4 *__restrict__ slots, int n_slots,
                            int64_t n4, float4 *__restrict__ out, const float4 *__restrict__ bias, int h4) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n4) return;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    if (n_slots > 0) {
        acc = slots[i];
        for (int s = 1; s < n_slots; ++s) {
            const float4 v = slots[(int64_t)s * n4 + i];
            acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
        }
    }
    if (base) {
        const float4 b = base[i];
        acc.x = b.x + acc.x; acc.y = b.y + acc.y; acc.z = b.z + acc.z; acc.w = b.w + acc.w;
    }
    if (bias) {
        const float4 b = bias[i % h4];
        acc.x += b.x; acc.y += b.y; acc.z += b.z; acc.w += b.w;
    }
    out[i] = acc;
}

__global__ void k_fill_zero(uint32_t *p, size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// y[m][:] = x[m][:] * rsqrt(mean(x^2) + eps) * g      one workgroup per row
__global__ void k_rmsnorm(const float *__restrict__ x, const float *__restrict__ g, float *__restrict__ y, int h,
                          float eps) {
    __shared__ float red[TB];
    const float *xr = x + (size_t)blockIdx.x * h;
    float s = 0.f;
    for (int i = threadIdx.x; i < h; i += TB) s += xr[i] * xr[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = TB / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    const float rs = 1.0f / sqrtf(red[0] / (float)h + eps);
    float *yr = y + (size_t)blockIdx.x * h;
    for (int i = threadIdx.x; i < h; i += TB) yr[i] = xr[i] * rs * g[i];
}

// C[M][N] (ldc) = A[M][K] (lda) * W[K][N] (ldw) (+ add[M][N], ldc).  32x32 tiles, 2x2 per thread.
__global__ void k_gemm(const float *__restrict__ A, int lda, const float *__restrict__ W, int ldw,
                       const float *__restrict__ add, float *__restrict__ C, int ldc, int M, int N, int K) {
    __shared__ float As[32][33];
    __shared__ float Ws[32][33];
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int m0 = blockIdx.y * 32, n0 = blockIdx.x * 32;
    float acc[2][2] = {{0.f, 0.f}, {0.f, 0.f}};
    for (int k0 = 0; k0 < K; k0 += 32) {
        for (int i = threadIdx.x; i < 1024; i += TB) {
            const int r = i >> 5, c = i & 31;
            As[r][c] = (m0 + r < M && k0 + c < K) ? A[(size_t)(m0 + r) * lda + k0 + c] : 0.f;
            Ws[r][c] = (k0 + r < K && n0 + c < N) ? W[(size_t)(k0 + r) * ldw + n0 + c] : 0.f;
        }
        __syncthreads();
#pragma unroll 8
        for (int k = 0; k < 32; ++k) {
            const float a0 = As[ty][k], a1 = As[ty + 16][k];
            const float b0 = Ws[k][tx], b1 = Ws[k][tx + 16];
            acc[0][0] += a0 * b0; acc[0][1] += a0 * b1;
            acc[1][0] += a1 * b0; acc[1][1] += a1 * b1;
        }
        __syncthreads();
    }
    for (int i = 0; i < 2; ++i)
        for (int j = 0; j < 2; ++j) {
            const int m = m0 + ty + 16 * i, n = n0 + tx + 16 * j;
            if (m < M && n < N) {
                const size_t o = (size_t)m * ldc + n;
                C[o] = add ? add[o] + acc[i][j] : acc[i][j];
            }
        }
}

// Rotate queries (in place in the qkv buffer) and keys, append keys and values to the cache.
// qkv: [M][nqkv] = [Q heads | K heads | V heads].  One thread per (token, head, j < d/2).
__global__ void k_rope_append(float *__restrict__ qkv, float *__restrict__ kc, float *__restrict__ vc,
                              const float *__restrict__ cosT, const float *__restrict__ sinT, spd_positions P, int M,
                              int q_len, int q, int kv, int d, int nqkv, int max_ctx) {
    const int half = d >> 1;
    const int per_tok = (q + kv) * half;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)M * per_tok) return;
    const int m = (int)(i / per_tok), r = (int)(i % per_tok);
    const int head = r / half, j = r % half;
    const int b = m / q_len, pos = P.pos[b] + (m % q_len);
    const float c = cosT[(size_t)pos * half + j], s = sinT[(size_t)pos * half + j];
    float *v = qkv + (size_t)m * nqkv + head * d;
    const float lo = v[j], hi = v[j + half];
    const float rlo = lo * c - hi * s, rhi = hi * c + lo * s;
    if (head < q) {
        v[j] = rlo;
        v[j + half] = rhi;
    } else {
        const int kh = head - q;
        const size_t o = (((size_t)b * kv + kh) * max_ctx + pos) * d;
        kc[o + j] = rlo;
        kc[o + j + half] = rhi;
        const float *vv = qkv + (size_t)m * nqkv + (q + kv + kh) * d;
        vc[o + j] = vv[j];
        vc[o + j + half] = vv[j + half];
    }
}

// Small products (at most ROWS_MAX_M rows, ROWS_MAX_K contraction elements): bound by latency, not by work, so a kernel does
// as much as it can between two launches.  A workgroup of 16 waves owns 1 to 8 rows of A and 64 columns of W: it loads
// its rows once (optionally applying the RMS norm: the whole row is there), wave w contracts the w-th sixteenth of K
// with lane = column, the waves' sums meet in LDS in wave order and an epilogue finishes the tile.  Toy model (hidden
// 256, two ranks side by side), us for 1 / 32 tokens: norm + QKV + rotation 5.2 / 5.9, O 3.9 / 4.2, fold + norm + gate + up + SwiGLU 5.0 / 6.0,
// down 4.8 / 5.3 (an almost empty launch 1.5; 8 rows per workgroup at any size, a row's elements apart in the LDS and the weights of K = 344
// in two goes 7.3, 4.8, 8.6, 7.4 for one token and rank).
constexpr int RW = 16, RN = 64;
constexpr int ROWS_MAX_M = 64, ROWS_MAX_K = 1024;
// Every group of 8 rows reads the weights again, so a very wide product is left to the 32 x 32 tiles.  hidden 1024, two layers,
// us, tiles / rows by workgroups of the gate/up launch: 64 rows 1024 2119 / 1752, 2048 3605 / 3323, 4096 8422 / 8457, 8192 16821 / 17845;
// 32 rows 2048 8537 / 8280, 3072 12412 / 12626; hidden 256: 64 rows 2048 3157 / 3108, 4096 6358 / 6394
constexpr int ROWS_MAX_WGS = 2048;

// What the rows of a product are made of: a[m][k], or a sum over ranks on top of it, a + (slot_0 + slot_1 + ...) [+ bias], which the first
// column block of the first rank leaves in `out` (no workgroup of the launch reads `out`).  So a sync point, and the SPD block's
// local fold X + Y_r [+ b] (one slot, the rank's own), need no launch of their own.  grid.z is the rank: all ranks a call
// emulates run side by side, `*_rank` being the distances between their buffers.
// (Rows of A and W follow each other without gaps.)
struct RowsIn {
    const float *a;
    int a_rank;
    const float *gain;           // RMS norm of the row with this gain, or NULL
    float eps;
    int w_rank;                  // distance between two ranks' weights (gain included)
    const float *slots = nullptr;
    size_t slot_stride = 0, slot_rank = 0;
    int n_slots = 0;
    const float *bias = nullptr;
    float *out = nullptr;
};

// Epilogues: one thread per element.  What does not depend on the product is requested ahead of it, by where() before the weights and by
// pre() (what needs where()'s result) behind them.
struct RowsQKV {       // queries and keys rotated, keys and values appended to the cache; needs whole heads per tile (64 % d == 0)
    static constexpr bool kDual = false;
    float *qkv, *kc, *vc;
    size_t qkv_rank, kv_rank;
    const float *cosT, *sinT;
    int q, kv, d, dlog, nqkv, max_ctx;         // d = 2^dlog (it divides 64)
    Divider by_qlen;
    spd_positions P;
    struct Pre { float c, s; int b, pos; };
    __device__ __forceinline__ int where(int m) const { return P.pos[by_qlen.div(m)]; }
    __device__ __forceinline__ Pre pre(int first, int, int m, int n) const {
        const int half = d >> 1, j = n & (d - 1), jj = j < half ? j : j - half;
        Pre p;
        p.b = by_qlen.div(m);
        p.pos = first + by_qlen.mod(m);
        p.c = cosT[(size_t)p.pos * half + jj];
        p.s = sinT[(size_t)p.pos * half + jj];
        return p;
    }
    __device__ __forceinline__ void operator()(const float *tile, const float *, int r, int cl, int m, int n, int z, const Pre &p) const {
        const int half = d >> 1, head = n >> dlog, j = n & (d - 1);
        float v = tile[r * RN + cl];
        if (head < q + kv) {
            const float o = tile[r * RN + (j < half ? cl + half : cl - half)];
            v = j < half ? v * p.c - o * p.s : v * p.c + o * p.s;
        }
        if (head < q) {
            qkv[z * qkv_rank + (size_t)m * nqkv + n] = v;
        } else {
            const int kh = head < q + kv ? head - q : head - q - kv;
            (head < q + kv ? kc : vc)[z * kv_rank + (((size_t)p.b * kv + kh) * max_ctx + p.pos) * d + j] = v;
        }
    }
};
struct RowsO {         // y = the partial product; r_out (optional) = x + y [+ bias], the SPD block's local fold
    static constexpr bool kDual = false;
    float *y, *r_out;
    size_t y_rank;
    const float *x, *bias;
    int ld;
    struct Pre { float x, b; };
    __device__ __forceinline__ int where(int) const { return 0; }
    __device__ __forceinline__ Pre pre(int, int, int m, int n) const {
        return Pre{r_out ? x[(size_t)m * ld + n] : 0.f, r_out && bias ? bias[n] : 0.f};
    }
    __device__ __forceinline__ void operator()(const float *tile, const float *, int r, int cl, int m, int n, int z, const Pre &p) const {
        const size_t o = (size_t)m * ld + n;
        const float v = tile[r * RN + cl];
        y[z * y_rank + o] = v;
        if (r_out) r_out[o] = bias ? (p.x + v) + p.b : p.x + v;
    }
};
struct RowsGU {        // silu(gate) * up
    static constexpr bool kDual = true;
    float *u;
    size_t u_rank;
    int ld;
    struct Pre {};
    __device__ __forceinline__ int where(int) const { return 0; }
    __device__ __forceinline__ Pre pre(int, int, int, int) const { return Pre(); }
    __device__ __forceinline__ void operator()(const float *tile, const float *tile2, int r, int cl, int m, int n, int z, const Pre &) const {
        const float x = tile[r * RN + cl];
        u[z * u_rank + (size_t)m * ld + n] = x / (1.0f + expf(-x)) * tile2[r * RN + cl];
    }
};
struct RowsDown {      // out = [add +] z  (add may be out itself)
    static constexpr bool kDual = false;
    float *out;
    const float *add;
    size_t out_rank;   // also the distance between two ranks' `add`
    int ld;
    struct Pre { float a; };
    __device__ __forceinline__ int where(int) const { return 0; }
    __device__ __forceinline__ Pre pre(int, int z, int m, int n) const { return Pre{add ? add[z * out_rank + (size_t)m * ld + n] : 0.f}; }
    __device__ __forceinline__ void operator()(const float *tile, const float *, int r, int cl, int m, int n, int z, const Pre &p) const {
        const float v = tile[r * RN + cl];
        out[z * out_rank + (size_t)m * ld + n] = add ? p.a + v : v;
    }
};

template <int RM>
struct alignas(RM * 4 < 16 ? RM * 4 : 16) RowsOf { float v[RM]; };

// The product of a workgroup's rows in the LDS, xs [K][RM], with its 64 columns and the epilogue: wave w contracts k0 .. k1 - 1 (the first U
// weights are on their way, `load` requests U more), the waves' sums meet in `red`, [NB][RW][RM][RN].
template <int RM, int U, class Epi, int U2, class Load>
__device__ __forceinline__ void rows_product(const float *xs, float *red, float (*tile)[RM * RN], int k0, int k1, float (&w0)[U], float (&w1)[U2],
                                             const Load &load, const Epi &epi, bool elem, int er, int cl, int em, int en, int z,
                                             const typename Epi::Pre &pre) {
    constexpr int NB = Epi::kDual ? 2 : 1;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float acc[NB][RM];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < RM; ++r) acc[b][r] = 0.f;
    for (int kb = k0; kb < k1; kb += U) {
        if (kb > k0) load(kb);
        auto use = [&](int u) {
            const RowsOf<RM> x = *(const RowsOf<RM> *)&xs[(kb + u) * RM];
#pragma unroll
            for (int r = 0; r < RM; ++r) {
                acc[0][r] += x.v[r] * w0[u];
                if constexpr (NB == 2) acc[1][r] += x.v[r] * w1[u];
            }
        };
        // (uniform branches, four rows' reads from the LDS between two of them)
#pragma unroll
        for (int u0 = 0; u0 < U; u0 += 4) {
            if (kb + u0 + 4 <= k1) {
#pragma unroll
                for (int u = u0; u < u0 + 4; ++u) use(u);
            } else {
#pragma unroll
                for (int u = u0; u < u0 + 3; ++u)
                    if (kb + u < k1) use(u);
            }
        }
    }
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < RM; ++r) red[((b * RW + wave) * RM + r) * RN + lane] = acc[b][r];
    __syncthreads();
    if (threadIdx.x < NB * RM * RN) {                   // (at most all 1024 threads)
        const int b = threadIdx.x / (RM * RN), e = threadIdx.x % (RM * RN);
        float t = red[(b * RW) * RM * RN + e];
#pragma unroll
        for (int w = 1; w < RW; ++w) t += red[(b * RW + w) * RM * RN + e];
        tile[b][e] = t;
    }
    __syncthreads();
    if (elem) epi(tile[0], tile[NB - 1], er, cl, em, en, z, pre);
}

// (What the first loads need comes as arguments of its own, which are in registers when a kernel starts: see build.py.  `in` for the rest.)
template <int RM, int KMAX, class Epi>      // RM rows of at most KMAX elements per workgroup
__global__ void __launch_bounds__(RW * 64) k_rows(const float *__restrict__ a, const float *__restrict__ W, const float *__restrict__ W2,
                                                  const float *__restrict__ gain, int K, int N, int M, int n_slots, int a_rank, int w_rank,
                                                  RowsIn in, Epi epi) {
    constexpr int NB = Epi::kDual ? 2 : 1;
    constexpr int P = RW / RM;                          // waves that load a row together
    constexpr int V = KMAX / P > 64 ? KMAX / P / 64 : 1;      // pieces of 64 elements of a wave's part of a row
    constexpr int U = KMAX / RW < 32 ? KMAX / RW : 32;  // weight rows that a wave requests at once
    // rows, transposed: [K][RM], so that what a wave multiplies with one weight is side by side; then the waves' sums
    // [NB][RW][RM][RN]
    extern __shared__ __attribute__((aligned(16))) float rows_lds[];
    __shared__ float ssq[RM][P];
    __shared__ float tile[NB][RM * RN];
    float *xs = rows_lds, *red = rows_lds + RM * K;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n0 = blockIdx.x * RN, m0 = blockIdx.y * RM, z = blockIdx.z;
    const int n = n0 + lane < N ? n0 + lane : N - 1;    // (columns past the matrix repeat its last one and are dropped)
    // Everything a workgroup reads is requested up front: a launch of this kind is its start and one trip to the memory.
    // rows: wave w takes part w % P of row w / P (past its end the last element again, not used)
    const int row = wave / P, hk = (K + P - 1) / P, rb = (wave % P) * hk, re = rb + hk < K ? rb + hk : K;
    const bool valid = m0 + row < M;
    float v[V], gn[V], bs[V], sl[V];
    size_t ro[V];
#pragma unroll
    for (int t = 0; t < V; ++t) {
        const int k = rb + t * 64 + lane;
        ro[t] = k < re ? k : K - 1;
        gn[t] = gain ? gain[(size_t)z * w_rank + ro[t]] : 1.f;
        bs[t] = in.bias ? in.bias[ro[t]] : 0.f;
        ro[t] += (size_t)(valid ? m0 + row : 0) * K;
        v[t] = a[(size_t)z * a_rank + ro[t]];
    }
    const float *slots = in.slots + z * in.slot_rank;
#pragma unroll
    for (int t = 0; t < V; ++t) sl[t] = n_slots > 0 ? slots[ro[t]] : 0.f;
    const int er = (threadIdx.x / RN) % RM, em = m0 + er, en = n0 + (int)threadIdx.x % RN;
    const bool elem = threadIdx.x < RM * RN && em < M && en < N;
    const int first = epi.where(em < M ? em : M - 1);
    const int k0 = (wave * K) / RW, k1 = ((wave + 1) * K) / RW, klast = k1 > k0 ? k1 - 1 : k0;
    float w0[U], w1[NB == 2 ? U : 1];
    auto load = [&](int kb) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = kb + u < klast ? kb + u : klast;
            w0[u] = W[(size_t)z * w_rank + (size_t)k * N + n];
            if constexpr (NB == 2) w1[u] = W2[(size_t)z * w_rank + (size_t)k * N + n];
        }
    };
    load(k0);
    typename Epi::Pre pre;
    {
        // the slots in ascending order, then what they join, then the bias
        for (int s = 1; s < n_slots; ++s) {
#pragma unroll
            for (int t = 0; t < V; ++t) sl[t] += slots[s * in.slot_stride + ro[t]];
        }
        float sq = 0.f;
#pragma unroll
        for (int t = 0; t < V; ++t) {
            const int k = rb + t * 64 + lane;
            if (n_slots > 0) v[t] += sl[t];
            if (in.bias) v[t] += bs[t];
            if (in.out && blockIdx.x == 0 && z == 0 && valid && k < re) in.out[ro[t]] = v[t];
            if (!valid || k >= re) v[t] = 0.f;
            sq += v[t] * v[t];
        }
        if (elem) pre = epi.pre(first, z, em, en);
        float rs = 1.f;
        if (gain) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
            if (lane == 0) ssq[row][wave % P] = sq;
            __syncthreads();
            // (the parts in pairs: the factor is common to the whole row, and with the parts of one token one after the other its rounding
            // showed in the results, 2.29e-7 instead of 2.16e-7 from 64 bits)
            float part[P];
#pragma unroll
            for (int i = 0; i < P; ++i) part[i] = ssq[row][i];
#pragma unroll
            for (int n = P / 2; n > 0; n /= 2)
#pragma unroll
                for (int i = 0; i < n; ++i) part[i] += part[i + n];
            rs = 1.0f / sqrtf(part[0] / (float)K + in.eps);
        }
#pragma unroll
        for (int t = 0; t < V; ++t) {
            const int k = rb + t * 64 + lane;
            if (k < re) xs[k * RM + row] = gain ? v[t] * rs * gn[t] : v[t];
        }
    }
    __syncthreads();
    rows_product<RM, U>(xs, red, tile, k0, k1, w0, w1, load, epi, elem, er, en - n0, em, en, z, pre);
}

bool rows_fit(int M, int N, int K) {
    return M <= ROWS_MAX_M && K <= ROWS_MAX_K && K >= 1 && (int64_t)((N + RN - 1) / RN) * ((M + 7) / 8) <= ROWS_MAX_WGS;
}

template <int RM, int KMAX, class Epi>
hipError_t launch_rows_as(hipStream_t s, const RowsIn &in, const float *W, const float *W2, int M, int N, int K, const Epi &epi,
                          int n_ranks) {
    constexpr int RED = (Epi::kDual ? 2 : 1) * RW * RM * RN * 4;
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [] {
        attr_err = hipFuncSetAttribute((const void *)k_rows<RM, KMAX, Epi>, hipFuncAttributeMaxDynamicSharedMemorySize, RED + RM * KMAX * 4);
    });
    if (attr_err != hipSuccess) return attr_err;
    hipLaunchKernelGGL((k_rows<RM, KMAX, Epi>), dim3((N + RN - 1) / RN, (M + RM - 1) / RM, n_ranks), dim3(RW * 64), RED + RM * K * 4, s, in.a, W,
                       W2, in.gain, K, N, M, in.n_slots, in.a_rank, in.w_rank, in, epi);
    return hipGetLastError();
}
template <int RM, class Epi>
hipError_t launch_rows_rm(hipStream_t s, const RowsIn &in, const float *W, const float *W2, int M, int N, int K, const Epi &epi,
                          int n_ranks) {
    if (K <= 256) return launch_rows_as<RM, 256>(s, in, W, W2, M, N, K, epi, n_ranks);
    if (K <= 512) return launch_rows_as<RM, 512>(s, in, W, W2, M, N, K, epi, n_ranks);
    return launch_rows_as<RM, ROWS_MAX_K>(s, in, W, W2, M, N, K, epi, n_ranks);
}
// The fewest rows per workgroup with which the launch is one round of the chip: a workgroup's vector work grows with its rows (8 rows of
// 344 elements: 1.3 us), and every group of rows reads the weights again.  Toy model, us per call, 8 rows
// always / this: 1 token 55.8 / 48.0, 32 tokens 59.2 / 50.5.
int rows_per_wg(int M, int N, int n_ranks) {
    const int64_t cols = (int64_t)((N + RN - 1) / RN) * n_ranks;
    return cols * M <= 256 ? 1 : (cols * ((M + 1) / 2) <= 256 ? 2 : (cols * ((M + 3) / 4) <= 256 ? 4 : 8));
}
template <class Epi>
hipError_t launch_rows(hipStream_t s, const RowsIn &in, const float *W, const float *W2, int M, int N, int K, const Epi &epi,
                       int n_ranks = 1) {
    switch (rows_per_wg(M, N, n_ranks)) {
        case 1: return launch_rows_rm<1>(s, in, W, W2, M, N, K, epi, n_ranks);
        case 2: return launch_rows_rm<2>(s, in, W, W2, M, N, K, epi, n_ranks);
        case 4: return launch_rows_rm<4>(s, in, W, W2, M, N, K, epi, n_ranks);
        default: return launch_rows_rm<8>(s, in, W, W2, M, N, K, epi, n_ranks);
    }
}

// The O projection of rows whose attention fits a workgroup: it does that attention itself, for its RM rows and all heads of the rank, instead
// of a launch in between (every block of 64 columns again).  The 16 waves share out the (row, head) items, `wpi` waves an item; eight lanes
// take a key, D / 8 features each, up to ROWS_ATT_PASSES keys per group of lanes, and everything is requested up front, the weights included.  The waves' softmax
// states meet in the LDS.  Toy model (two layers, two ranks, 11 -> 9 launches), us per call, launch of its own / this: 1 token 47.4 / 42.5, 32 tokens
// 48.7 / 45.8.
constexpr int ROWS_ATT_PASSES = 2;
template <int RM, int KMAX, int D>
__global__ void __launch_bounds__(RW * 64) k_rows_att(const float *__restrict__ qkv, const float *__restrict__ kc, const float *__restrict__ vc,
                                                      const float *__restrict__ W, int q, int kv, int nqkv, int max_ctx, int M, int N,
                                                      int wpi, int qkv_rank, int w_rank, Divider by_wpi, Divider by_q, Divider by_qlen, Divider by_group,
                                                      size_t kv_rank, spd_positions P, RowsO epi) {
    constexpr int NP = ROWS_ATT_PASSES, F = D / 8;
    constexpr int U = KMAX / RW < 32 ? KMAX / RW : 32;
    __shared__ __attribute__((aligned(16))) float xs[KMAX * RM];      // (read as RowsOf<RM>)
    __shared__ float red[RW * RM * RN];
    __shared__ float tile[1][RM * RN];
    __shared__ float so[RW][D], sml[RW][2];
    const int K = q * D;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n0 = blockIdx.x * RN, m0 = blockIdx.y * RM, z = blockIdx.z;
    const int n = n0 + lane < N ? n0 + lane : N - 1;
    const int item = min(by_wpi.div(wave), RM * q - 1), part = by_wpi.mod(wave);      // (a wave too many repeats the last item and is not used)
    const int row = by_q.div(item), head = by_q.mod(item), m = m0 + row < M ? m0 + row : M - 1, b = by_qlen.div(m);
    const int n_keys = P.pos[b] + by_qlen.mod(m) + 1;                                  // causal
    const size_t c0 = z * kv_rank + ((size_t)b * kv + by_group.div(head)) * max_ctx * D + (lane & 7) * F;
    struct Piece { float v[F]; };
    auto piece = [](const float *p) { Piece r; __builtin_memcpy(&r, p, sizeof(r)); return r; };       // (the cache is aligned to its elements only)
    const Piece qv = piece(qkv + (size_t)z * qkv_rank + (size_t)m * nqkv + head * D + (lane & 7) * F);
    Piece kk[NP], vv[NP];
    bool live[NP];
#pragma unroll
    for (int t = 0; t < NP; ++t) {
        const int key = (t * wpi + part) * 8 + (lane >> 3);
        live[t] = key < n_keys;
        const size_t o = c0 + (size_t)(live[t] ? key : n_keys - 1) * D;
        kk[t] = piece(kc + o);
        vv[t] = piece(vc + o);
    }
    const int er = (threadIdx.x / RN) % RM, em = m0 + er, en = n0 + (int)threadIdx.x % RN;
    const bool elem = threadIdx.x < RM * RN && em < M && en < N;
    const int k0 = (wave * K) / RW, k1 = ((wave + 1) * K) / RW, klast = k1 > k0 ? k1 - 1 : k0;
    float w0[U], w1[1];
    auto load = [&](int kb) {
#pragma unroll
        for (int u = 0; u < U; ++u) w0[u] = W[(size_t)z * w_rank + (size_t)(kb + u < klast ? kb + u : klast) * N + n];
    };
    load(k0);
    RowsO::Pre pre;
    if (elem) pre = epi.pre(0, z, em, en);
    const float scale = 1.0f / sqrtf((float)D);
    float s[NP], mx = -INFINITY;
#pragma unroll
    for (int t = 0; t < NP; ++t) {
        s[t] = 0.f;
#pragma unroll
        for (int f = 0; f < F; ++f) s[t] += qv.v[f] * kk[t].v[f];
#pragma unroll
        for (int o = 1; o < 8; o <<= 1) s[t] += __shfl_xor(s[t], o, 64);
        s[t] = live[t] ? s[t] * scale : -INFINITY;
        mx = fmaxf(mx, s[t]);
    }
#pragma unroll
    for (int o = 8; o < 64; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    // (a wave without keys, or whose keys all have no score, which a maximum passes over: the state is 0 for the one and NaN for the other)
    const float top = mx == -INFINITY ? 0.f : mx;
    float sum = 0.f, out[F];
#pragma unroll
    for (int f = 0; f < F; ++f) out[f] = 0.f;
#pragma unroll
    for (int t = 0; t < NP; ++t) {
        const float p = live[t] ? expf(s[t] - top) : 0.f;
        sum += p;
#pragma unroll
        for (int f = 0; f < F; ++f) out[f] += live[t] ? p * vv[t].v[f] : 0.f;
    }
#pragma unroll
    for (int o = 8; o < 64; o <<= 1) {
        sum += __shfl_xor(sum, o, 64);
#pragma unroll
        for (int f = 0; f < F; ++f) out[f] += __shfl_xor(out[f], o, 64);
    }
    if (lane < 8) {
#pragma unroll
        for (int f = 0; f < F; ++f) so[wave][lane * F + f] = out[f];
    }
    if (lane == 0) {
        sml[wave][0] = mx;
        sml[wave][1] = sum;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < RM * K; e += RW * 64) {
        const int it = e / D, f = e % D;
        float mm = -INFINITY, den = 0.f, num = 0.f;
        for (int w = it * wpi; w < (it + 1) * wpi; ++w) mm = fmaxf(mm, sml[w][0]);
        for (int w = it * wpi; w < (it + 1) * wpi; ++w) {
            const float sc = expf(sml[w][0] - mm);               // (0 for a wave without keys)
            den += sml[w][1] * sc;
            num += so[w][f] * sc;
        }
        xs[(by_q.mod(it) * D + f) * RM + by_q.div(it)] = num / den;
    }
    __syncthreads();
    rows_product<RM, U>(xs, red, tile, k0, k1, w0, w1, load, epi, elem, er, en - n0, em, en, z, pre);
}

// One workgroup of 4 waves per (token, query head): causal softmax attention over the cache.  A thread takes a key at a time
// for the scores; for the output wave w takes keys w, w + 4, ... with lane = feature, and the four sums meet in LDS.
__global__ void __launch_bounds__(TB) k_attention(const float *__restrict__ qkv, const float *__restrict__ kc, const float *__restrict__ vc,
                                                  int q_len, int q, int kv, int d, int nqkv, int max_ctx, float *__restrict__ out,
                                                  size_t qkv_rank, size_t kv_rank, size_t out_rank, spd_positions P) {
    qkv += blockIdx.y * qkv_rank;          // (grid.y: the rank)
    kc += blockIdx.y * kv_rank;
    vc += blockIdx.y * kv_rank;
    out += blockIdx.y * out_rank;
    extern __shared__ float sc[];          // [n_keys] scores, then probabilities
    __shared__ float part[4][64];
    __shared__ float qs[256];
    __shared__ float red[2][4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = blockIdx.x / q, j = blockIdx.x % q;
    const int b = m / q_len, pos = P.pos[b] + (m % q_len);
    const int n_keys = pos + 1;            // causal: key position <= query position
    const int kh = j / (q / kv);
    for (int c = threadIdx.x; c < d; c += TB) qs[c] = qkv[(size_t)m * nqkv + j * d + c];
    const float *K = kc + ((size_t)b * kv + kh) * max_ctx * d;
    const float *V = vc + ((size_t)b * kv + kh) * max_ctx * d;
    const float scale = 1.0f / sqrtf((float)d);
    __syncthreads();
    float mx = -INFINITY;
    for (int t = threadIdx.x; t < n_keys; t += TB) {
        const float *kr = K + (size_t)t * d;
        float s = 0.f;
        int c = 0;
        for (; c + 32 <= d; c += 32) {     // 32 loads in flight
            float kk[32];
#pragma unroll
            for (int u = 0; u < 32; ++u) kk[u] = kr[c + u];
#pragma unroll
            for (int u = 0; u < 32; ++u) s += qs[c + u] * kk[u];
        }
        for (; c < d; ++c) s += qs[c] * kr[c];
        s *= scale;
        sc[t] = s;
        mx = fmaxf(mx, s);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    if (lane == 0) red[0][wave] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(red[0][0], red[0][1]), fmaxf(red[0][2], red[0][3]));
    float sum = 0.f;
    for (int t = threadIdx.x; t < n_keys; t += TB) {
        const float e = expf(sc[t] - mx);
        sc[t] = e;
        sum += e;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    if (lane == 0) red[1][wave] = sum;
    __syncthreads();
    const float inv = 1.0f / (((red[1][0] + red[1][1]) + red[1][2]) + red[1][3]);
    for (int c0 = 0; c0 < d; c0 += 64) {
        const int c = c0 + lane < d ? c0 + lane : d - 1;
        float a = 0.f;
        for (int t0 = wave; t0 < n_keys; t0 += 32) {
            float vv[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int t = t0 + 4 * u < n_keys ? t0 + 4 * u : n_keys - 1;
                vv[u] = V[(size_t)t * d + c];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (t0 + 4 * u < n_keys) a += sc[t0 + 4 * u] * vv[u];
        }
        part[wave][lane] = a;
        __syncthreads();
        if (wave == 0 && c0 + lane < d)
            out[(size_t)m * (q * d) + j * d + c0 + lane] = (((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane]) * inv;
        __syncthreads();
    }
}

__global__ void k_swiglu(const float *__restrict__ g, const float *__restrict__ u, float *__restrict__ out, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float x = g[i];
    out[i] = x / (1.0f + expf(-x)) * u[i];
}

__global__ void k_copy2d(const float *__restrict__ src, int lds, float *__restrict__ dst, int ldd, int rows, int cols) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)rows * cols) return;
    const int r = (int)(i / cols), c = (int)(i % cols);
    dst[(size_t)r * ldd + c] = src[(size_t)r * lds + c];
}

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + TB - 1) / TB); }

hipError_t gemm(const float *A, int lda, const float *W, int ldw, const float *add, float *C, int ldc, int M, int N,
                int K, hipStream_t s) {
    dim3 grid((N + 31) / 32, (M + 31) / 32);
    hipLaunchKernelGGL(k_gemm, grid, dim3(TB), 0, s, A, lda, W, ldw, add, C, ldc, M, N, K);
    return hipGetLastError();
}

}  // namespace

namespace spd_common {

hipError_t rank_sum(const float *base, const float *slots, int n_slots, int64_t n, float *out, hipStream_t s,
                    const float *bias, int h) {
    if (n <= 0) return hipSuccess;
    const bool al = ((((uintptr_t)base) | ((uintptr_t)slots) | ((uintptr_t)out) | ((uintptr_t)bias)) & 15) == 0 &&
                    (n % 4) == 0 && (!bias || h % 4 == 0);
    if (al)
        hipLaunchKernelGGL(k_rank_sum4, dim3(blocks_for(n / 4)), dim3(TB), 0, s, (const float4 *)base,
                           (const float4 *)slots, n_slots, n / 4, (float4 *)out, (const float4 *)bias, h / 4);
    else
        hipLaunchKernelGGL(k_rank_sum, dim3(blocks_for(n)), dim3(TB), 0, s, base, slots, n_slots, n, out, bias, h);
    return hipGetLastError();
}

hipError_t fill_zero_u32(uint32_t *p, size_t n, hipStream_t s) {
    if (!n) return hipSuccess;
    hipLaunchKernelGGL(k_fill_zero, dim3(blocks_for((int64_t)n)), dim3(TB), 0, s, p, n);
    return hipGetLastError();
}

hipError_t copy2d(const float *src, int lds, float *dst, int ldd, int rows, int cols, hipStream_t s) {
    if (rows <= 0 || cols <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_copy2d, dim3(blocks_for((int64_t)rows * cols)), dim3(TB), 0, s, src, lds, dst, ldd, rows, cols);
    return hipGetLastError();
}

}  // namespace spd_common

namespace spd_f32 {

#define SPD_TRY(x)                        \
    do {                                  \
        hipError_t e_ = (x);              \
        if (e_ != hipSuccess) return e_;  \
    } while (0)

static RowsQKV rows_qkv(const spd_call &c, float *qkv, size_t qkv_rank, char *kvc) {
    const spd_dims &D = *c.D;
    RowsQKV e;
    e.qkv = qkv; e.qkv_rank = qkv_rank;
    e.kc = (float *)kvc; e.vc = (float *)(kvc + D.kv_v); e.kv_rank = D.kv_bytes / 4;
    e.cosT = (const float *)(c.ws + D.ws_cos); e.sinT = (const float *)(c.ws + D.ws_sin);
    e.by_qlen = Divider::by(c.q_len); e.q = D.q; e.kv = D.kv; e.d = D.d; e.dlog = __builtin_ctz(D.d); e.nqkv = D.nqkv; e.max_ctx = D.max_ctx; e.P = c.pos;
    return e;
}
static RowsIn rows_in(const spd_call &c, const float *a, size_t a_rank, const float *gain) {
    RowsIn in;
    in.a = a; in.a_rank = (int)a_rank; in.gain = gain; in.eps = c.D->eps; in.w_rank = (int)(c.D->weight_bytes / 4);      // (of a few rows: see rows_fit())
    return in;
}

bool ranks_fit(const spd_call &c, int n_ranks) {
    const spd_dims &D = *c.D;
    const int M = c.M, qd = D.q * D.d;
    return rows_fit(M, D.nqkv, D.h) && RN % D.d == 0 && rows_fit(M, D.h, qd) && rows_fit(M, D.f, D.h) && rows_fit(M, D.h, D.f) &&
           (n_ranks == 1 || (n_ranks <= D.rk_ranks && M <= D.rk_rows));
}

// A sum over the ranks that a product's rows are made of: in the product's launch, whose every column block then reads the slots of
// its rows, one slot after the other, or, where that is too much, by a launch of its own ahead of it (the same additions in the same order).
// us per call of two layers with both sync points, sums in the products / ahead of them: up to 4 MiB of slots read by a launch the first
// gains (2 ranks, hidden 256, 1 token 48.0 / 49.5; 16, hidden 1024, 4 tokens 72.7 / 77.9; 256, hidden 64, 4 tokens 138 / 155), at
// 8 to 16 MiB with up to 32 slots too (8, hidden 1024, 16 tokens 72.0 / 77.5; 16 MiB of 8 ranks side by side 103.8 / 110.5), with
// more of them no longer (64, hidden 1024, 6 MiB 96.9 / 89.4; 128, 8 MiB 143 / 117); from 24 MiB on it loses (16, 24 MiB 82.1 /
// 79.7; 16 side by side 256 MiB 427 / 249, 1 GiB 1370 / 675).
constexpr int64_t SUM_INSIDE = (int64_t)16 << 20, SUM_INSIDE_MANY = (int64_t)4 << 20;
constexpr int SUM_MANY_SLOTS = 32;
static hipError_t sum_ahead(const spd_call &c, RowsIn &in, int N, int n_ranks) {
    const spd_dims &D = *c.D;
    const int64_t bytes = (int64_t)((N + RN - 1) / RN) * n_ranks * in.n_slots * c.M * D.h * 4;
    if (bytes <= (in.n_slots <= SUM_MANY_SLOTS ? SUM_INSIDE : SUM_INSIDE_MANY)) return hipSuccess;
    if (c.on(SPD_STAGE_PREP)) {
        spd_stage_scope prof(c, SPD_STAGE_PREP);
        SPD_TRY(spd_common::rank_sum(in.a, in.slots, in.n_slots, (int64_t)in.slot_stride, in.out, c.s, in.bias, D.h));
    }
    in.a = in.out;
    in.n_slots = 0;
    in.slots = in.bias = nullptr;
    in.out = nullptr;
    return hipSuccess;
}

// Does the O projection of a small call do the attention itself?  Heads of 32 or 64 features, at most 16 (row, head) items a workgroup and as
// many keys as its lanes take in ROWS_ATT_PASSES rounds.  Returns the waves per item, 0 for a launch of its own.
static int att_in_o(const spd_call &c, int n_ranks) {
    const spd_dims &D = *c.D;
    const int items = rows_per_wg(c.M, D.h, n_ranks) * D.q;
    if ((D.d != 32 && D.d != 64) || items > RW) return 0;
    return c.max_pos_end <= RW / items * 8 * ROWS_ATT_PASSES ? RW / items : 0;
}
template <int RM>
static hipError_t launch_rows_att_rm(const spd_call &c, const float *qkv, size_t qkv_rank, const char *kvc, const char *w, const RowsO &epi,
                                     int n, int wpi) {
    const spd_dims &D = *c.D;
    const dim3 grid((D.h + RN - 1) / RN, (c.M + RM - 1) / RM, n);
#define SPD_ROWS_ATT(KMAX, DD)                                                                                                              \
    hipLaunchKernelGGL((k_rows_att<RM, KMAX, DD>), grid, dim3(RW * 64), 0, c.s, qkv, (const float *)kvc, (const float *)(kvc + D.kv_v),      \
                       (const float *)(w + D.w_o), D.q, D.kv, D.nqkv, D.max_ctx, c.M, D.h, wpi, (int)qkv_rank, (int)(D.weight_bytes / 4),    \
                       Divider::by(wpi), Divider::by(D.q), Divider::by(c.q_len), Divider::by(D.group), D.kv_bytes / 4, c.pos, epi)
    // (at most 16 / RM heads)
    if (D.d == 32) SPD_ROWS_ATT(RW / RM * 32, 32);
    else if (D.q * 64 <= 256 || RM > 2) SPD_ROWS_ATT(256, 64);
    else SPD_ROWS_ATT(RW / RM * 64, 64);
#undef SPD_ROWS_ATT
    return hipGetLastError();
}
static hipError_t launch_rows_att(const spd_call &c, const float *qkv, size_t qkv_rank, const char *kvc, const char *w, const RowsO &epi, int n,
                                  int wpi) {
    switch (rows_per_wg(c.M, c.D->h, n)) {
        case 1: return launch_rows_att_rm<1>(c, qkv, qkv_rank, kvc, w, epi, n, wpi);
        case 2: return launch_rows_att_rm<2>(c, qkv, qkv_rank, kvc, w, epi, n, wpi);
        case 4: return launch_rows_att_rm<4>(c, qkv, qkv_rank, kvc, w, epi, n, wpi);
        default: return launch_rows_att_rm<8>(c, qkv, qkv_rank, kvc, w, epi, n, wpi);
    }
}

// One block of `n` ranks side by side in five launches (23 -> 11 of a two-layer model with two ranks).  X is x->base, or the sum
// *x describes, which is written to x->out; the sum that ends the block is left to the reader of its slots: *x describes it
// on return.  R: where a TP block's kept sync point puts X + sum of the slots.  Toy model (hidden 256, two layers, two ranks), us per call, one
// rank after the other with launches of their own for the sums / side by side: 1 token 137 / 50, 32 tokens 142 / 51.
hipError_t block_ranks(const spd_call &c, const char *w, char *kvc, int n, int spd, float *slot0, const float *slots, spd_sum *x, float *R,
                       const float *bo) {
    const spd_dims &D = *c.D;
    const int M = c.M, qd = D.q * D.d, f = D.f;
    const size_t mr = n > 1 ? D.rk_rows : D.m_pad;
    float *qkv = (float *)(c.ws + (n > 1 ? D.ws_rk_qkv : D.ws_qkv)), *att = (float *)(c.ws + (n > 1 ? D.ws_rk_ahat : D.ws_ahat)),
          *u = (float *)(c.ws + (n > 1 ? D.ws_rk_uhat : D.ws_uhat));
    const size_t slot_n = c.slot_stride;
    const float *X = x->n ? x->out : x->base;

    RowsIn in = rows_in(c, x->base, 0, (const float *)(w + D.w_g1));
    in.slots = x->slots; in.slot_stride = slot_n; in.n_slots = x->n; in.bias = x->bias; in.out = x->out;
    SPD_TRY(sum_ahead(c, in, D.nqkv, n));
    if (c.on(SPD_STAGE_QKV)) {
        spd_stage_scope prof(c, SPD_STAGE_QKV);
        SPD_TRY(launch_rows(c.s, in, (const float *)(w + D.w_qkv), nullptr, M, D.nqkv, D.h, rows_qkv(c, qkv, mr * D.nqkv, kvc), n));
    }
    // (a call of one of the two stages alone keeps a launch for each)
    const int wpi = att_in_o(c, n);
    const bool fused = wpi > 0 && c.on(SPD_STAGE_ATTN) && c.on(SPD_STAGE_O);
    if (c.on(SPD_STAGE_ATTN) && (!fused || c.taps)) {      // (a tapped call also wants what the O projection would keep to itself)
        spd_stage_scope prof(c, SPD_STAGE_ATTN);
        hipLaunchKernelGGL(k_attention, dim3(M * D.q, n), dim3(TB), (size_t)c.max_pos_end * sizeof(float), c.s, qkv, (const float *)kvc,
                           (const float *)(kvc + D.kv_v), c.q_len, D.q, D.kv, D.d, D.nqkv, D.max_ctx, att, mr * D.nqkv, D.kv_bytes / 4, mr * qd,
                           c.pos);
        SPD_TRY(hipGetLastError());
    }
    if (c.on(SPD_STAGE_O)) {
        RowsO eo;                          // Y_r into the rank's slot
        eo.y = slot0; eo.y_rank = slot_n; eo.r_out = nullptr; eo.x = nullptr; eo.bias = nullptr; eo.ld = D.h;
        spd_stage_scope prof(c, SPD_STAGE_O);
        if (fused) SPD_TRY(launch_rows_att(c, qkv, mr * D.nqkv, kvc, w, eo, n, wpi));
        else SPD_TRY(launch_rows(c.s, rows_in(c, att, mr * qd, nullptr), (const float *)(w + D.w_o), nullptr, M, D.h, qd, eo, n));
    }
    if (c.taps) {                          // (of several ranks the last one's)
        const size_t r = n - 1;
        if (c.taps->q) SPD_TRY(spd_common::copy2d(qkv + r * mr * D.nqkv, D.nqkv, c.taps->q, qd, M, qd, c.s));
        if (c.taps->attn) SPD_TRY(spd_common::copy2d(att + r * mr * qd, qd, c.taps->attn, qd, M, qd, c.s));
        if (c.taps->y) SPD_TRY(spd_common::copy2d(slot0 + r * slot_n, D.h, c.taps->y, D.h, M, D.h, c.s));
    }
    in = rows_in(c, X, 0, (const float *)(w + D.w_g2));
    in.bias = bo;
    if (spd) {                             // R_r = X + Y_r [+ b] (Sec. 4.1.1), needed by this product only
        in.slots = slot0; in.slot_rank = slot_n; in.n_slots = 1;
    } else {                               // the kept sync point
        in.slots = slots; in.slot_stride = slot_n; in.n_slots = D.tp; in.out = R;
        SPD_TRY(sum_ahead(c, in, f, n));
    }
    if (c.on(SPD_STAGE_GATEUP)) {
        RowsGU eg;
        eg.u = u; eg.u_rank = mr * f; eg.ld = f;
        spd_stage_scope prof(c, SPD_STAGE_GATEUP);
        SPD_TRY(launch_rows(c.s, in, (const float *)(w + D.w_g), (const float *)(w + D.w_u), M, f, D.h, eg, n));
    }
    if (c.taps && c.taps->u) SPD_TRY(spd_common::copy2d(u + (size_t)(n - 1) * mr * f, f, c.taps->u, f, M, f, c.s));
    if (c.on(SPD_STAGE_DOWN)) {
        RowsDown ed;                       // slot = Z_r, or Y_r + Z_r
        ed.out = slot0; ed.add = spd ? slot0 : nullptr; ed.out_rank = slot_n; ed.ld = D.h;
        spd_stage_scope prof(c, SPD_STAGE_DOWN);
        SPD_TRY(launch_rows(c.s, rows_in(c, u, mr * f, nullptr), (const float *)(w + D.w_d), nullptr, M, D.h, f, ed, n));
    }
    x->base = spd ? X : R;
    x->slots = slots;
    x->n = D.tp;
    x->bias = spd ? bo : nullptr;
    return hipSuccess;
}

// r_out (may be NULL) <- x + Y_r [+ bias], the local fold of an SPD block
hipError_t attention_half(const spd_call &c, const char *w, char *kvc, const float *x, float *y_out, float *r_out, const float *bias) {
    const spd_dims &D = *c.D;
    const int M = c.M, qd = D.q * D.d;
    float *xn = (float *)(c.ws + D.ws_xhat), *qkv = (float *)(c.ws + D.ws_qkv), *att = (float *)(c.ws + D.ws_ahat);
    const float *cosT = (const float *)(c.ws + D.ws_cos), *sinT = (const float *)(c.ws + D.ws_sin);
    float *kc = (float *)kvc, *vc = (float *)(kvc + D.kv_v);
    if (rows_fit(M, D.nqkv, D.h) && RN % D.d == 0) {
        SPD_TRY(launch_rows(c.s, rows_in(c, x, 0, (const float *)(w + D.w_g1)), (const float *)(w + D.w_qkv), nullptr, M, D.nqkv, D.h,
                            rows_qkv(c, qkv, 0, kvc)));
    } else {
        hipLaunchKernelGGL(k_rmsnorm, dim3(M), dim3(TB), 0, c.s, x, (const float *)(w + D.w_g1), xn, D.h, D.eps);
        SPD_TRY(hipGetLastError());
        SPD_TRY(gemm(xn, D.h, (const float *)(w + D.w_qkv), D.nqkv, nullptr, qkv, D.nqkv, M, D.nqkv, D.h, c.s));
        const int64_t nro = (int64_t)M * (D.q + D.kv) * (D.d / 2);
        hipLaunchKernelGGL(k_rope_append, dim3(blocks_for(nro)), dim3(TB), 0, c.s, qkv, kc, vc, cosT, sinT, c.pos, M,
                           c.q_len, D.q, D.kv, D.d, D.nqkv, D.max_ctx);
        SPD_TRY(hipGetLastError());
    }
    hipLaunchKernelGGL(k_attention, dim3(M * D.q), dim3(TB), (size_t)c.max_pos_end * sizeof(float), c.s, qkv, kc, vc, c.q_len, D.q, D.kv, D.d,
                       D.nqkv, D.max_ctx, att, (size_t)0, (size_t)0, (size_t)0, c.pos);
    SPD_TRY(hipGetLastError());
    if (rows_fit(M, D.h, qd)) {
        RowsO e;
        e.y = y_out; e.y_rank = 0; e.r_out = r_out; e.x = x; e.bias = bias; e.ld = D.h;
        SPD_TRY(launch_rows(c.s, rows_in(c, att, 0, nullptr), (const float *)(w + D.w_o), nullptr, M, D.h, qd, e));
    } else {
        SPD_TRY(gemm(att, qd, (const float *)(w + D.w_o), D.h, nullptr, y_out, D.h, M, D.h, qd, c.s));
        if (r_out) SPD_TRY(spd_common::rank_sum(x, y_out, 1, (int64_t)M * D.h, r_out, c.s, bias, D.h));
    }
    if (c.taps) {
        if (c.taps->q) SPD_TRY(spd_common::copy2d(qkv, D.nqkv, c.taps->q, qd, M, qd, c.s));
        if (c.taps->attn) SPD_TRY(spd_common::copy2d(att, qd, c.taps->attn, qd, M, qd, c.s));
        if (c.taps->y) SPD_TRY(spd_common::copy2d(y_out, D.h, c.taps->y, D.h, M, D.h, c.s));
    }
    return hipSuccess;
}

hipError_t mlp_half(const spd_call &c, const char *w, const float *r_in, const float *add, float *out) {
    const spd_dims &D = *c.D;
    const int M = c.M, f = D.f;
    float *xn = (float *)(c.ws + D.ws_xhat), *gu = (float *)(c.ws + D.ws_gu), *u = (float *)(c.ws + D.ws_uhat);
    if (rows_fit(M, f, D.h)) {
        RowsGU e;
        e.u = u; e.u_rank = 0; e.ld = f;
        SPD_TRY(launch_rows(c.s, rows_in(c, r_in, 0, (const float *)(w + D.w_g2)), (const float *)(w + D.w_g), (const float *)(w + D.w_u),
                            M, f, D.h, e));
    } else {
        hipLaunchKernelGGL(k_rmsnorm, dim3(M), dim3(TB), 0, c.s, r_in, (const float *)(w + D.w_g2), xn, D.h, D.eps);
        SPD_TRY(hipGetLastError());
        SPD_TRY(gemm(xn, D.h, (const float *)(w + D.w_g), f, nullptr, gu, f, M, f, D.h, c.s));
        SPD_TRY(gemm(xn, D.h, (const float *)(w + D.w_u), f, nullptr, gu + (size_t)M * f, f, M, f, D.h, c.s));
        hipLaunchKernelGGL(k_swiglu, dim3(blocks_for((int64_t)M * f)), dim3(TB), 0, c.s, gu, gu + (size_t)M * f, u,
                           (int64_t)M * f);
        SPD_TRY(hipGetLastError());
    }
    if (rows_fit(M, D.h, f)) {
        RowsDown e;
        e.out = out; e.add = add; e.out_rank = 0; e.ld = D.h;
        SPD_TRY(launch_rows(c.s, rows_in(c, u, 0, nullptr), (const float *)(w + D.w_d), nullptr, M, D.h, f, e));
    } else {
        SPD_TRY(gemm(u, f, (const float *)(w + D.w_d), D.h, add, out, D.h, M, D.h, f, c.s));
    }
    if (c.taps && c.taps->u) SPD_TRY(spd_common::copy2d(u, f, c.taps->u, f, M, f, c.s));
    return hipSuccess;
}

}  // namespace spd_f32
