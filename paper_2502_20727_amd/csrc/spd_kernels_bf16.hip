// bf16 path: MFMA (16x16x32 bf16, fp32 accumulate) kernels for gfx950 over the packed
// fragment layouts described in spd_internal.h.
//
// Orientation used everywhere: the *weights* (or keys / values) are the first MFMA operand,
// the *activations* (or queries / probabilities) the second, so an accumulator tile is
// D[output feature][token]: lane l holds token (l % 16) and the 4 consecutive output
// features 4*(l/16) .. 4*(l/16)+3.  Four consecutive features per lane is exactly what the
// next contraction wants as its packed operand, so every epilogue stores 8-byte pieces
// straight into the next kernel's fragment layout.
//
// "Split" activations: an activation buffer may carry a second plane holding, for every
// element, the rounding error of the first plane (x = hi + lo up to 2^-17 relative).
// Contractions then run over both planes.
//
// Operand format.  The projections contract fp16 operands (v_mfma_f32_16x16x32_f16): activations are
// rounded to fp16's 11 significant bits, and the packed shard holds every weight w as
// round_fp16(2^k w), one power of two per matrix, undone in the epilogue (`wsc`).  The bf16 weights the
// library is given fit that encoding exactly (8 significant bits; the power of two puts the matrix's
// largest magnitude just below 2^15, so every weight within 2^-29 of it is a normal fp16 number).
// Attention contracts bf16: the KV cache holds bf16 values, queries and probabilities are bf16 pairs.
// fp16 and bf16 fragments are 16-bit elements in the same order, so everything that only moves data
// is typed as bf16.
#include <mutex>
#include <type_traits>

#include "spd_internal.h"

namespace {

#define SPD_TRY(x)                       \
    do {                                 \
        hipError_t e_ = (x);             \
        if (e_ != hipSuccess) return e_; \
    } while (0)

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));

#define MFMA(a, b, c) __builtin_amdgcn_mfma_f32_16x16x32_bf16((a), (b), (c), 0, 0, 0)
// fp16 operands held in registers typed as bf16 (raw 16-bit elements)
#define MFMA16(a, b, c) \
    __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, (a)), __builtin_bit_cast(f16x8, (b)), (c), 0, 0, 0)

// bf16 (attention operands: queries, keys, values, probabilities)
__device__ __forceinline__ bf16x4 cvt4(float a, float b, float c, float d) {
    bf16x4 r;
    r[0] = (__bf16)a; r[1] = (__bf16)b; r[2] = (__bf16)c; r[3] = (__bf16)d;
    return r;
}
// rounding error of cvt4, itself rounded to bf16
__device__ __forceinline__ bf16x4 cvt4_lo(float a, float b, float c, float d, bf16x4 hi) {
    return cvt4(a - (float)hi[0], b - (float)hi[1], c - (float)hi[2], d - (float)hi[3]);
}
// An fp16 activation as raw 16 bits typed __bf16 (the type the data-moving code uses).
__device__ __forceinline__ __bf16 act_one(float v) { return __builtin_bit_cast(__bf16, (_Float16)v); }
__device__ __forceinline__ float act_back(__bf16 r) { return (float)__builtin_bit_cast(_Float16, r); }
__device__ __forceinline__ bf16x4 cvt4h(float a, float b, float c, float d) {
    bf16x4 r;
    r[0] = act_one(a); r[1] = act_one(b); r[2] = act_one(c); r[3] = act_one(d);
    return r;
}
// fp16(x g) of four elements, each product rounded once: the compiler makes one mixed-precision instruction of a product and its conversion,
// but not where it finds two conversions side by side for its packed one (elements of a vector, say): the halves are put together
// as integers.  A product rounded to 32 bits first is a tie of fp16 for one in 17 000 elements of an N(0, 1) input and then goes the wrong way
// half of the time.
__device__ __forceinline__ bf16x4 mul4h(float4 x, float4 g) {
    auto one = [](float a, float b) { return (unsigned)__builtin_bit_cast(unsigned short, (_Float16)(a * b)); };
    const uint2 r = make_uint2(one(x.x, g.x) | one(x.y, g.y) << 16, one(x.z, g.z) | one(x.w, g.w) << 16);
    return __builtin_bit_cast(bf16x4, r);
}
// rounding error of cvt4h, itself rounded to fp16
__device__ __forceinline__ bf16x4 cvt4h_lo(float a, float b, float c, float d, bf16x4 hi) {
    return cvt4h(a - act_back(hi[0]), b - act_back(hi[1]), c - act_back(hi[2]), d - act_back(hi[3]));
}
__device__ __forceinline__ float shfl_xor_f(float v, int mask) { return __shfl_xor(v, mask, 64); }
// Sum / maximum over the four lanes l, l^16, l^32, l^48 (the lanes that share a token or an attention column),
// left in all four.  gfx950's row swaps (v_permlane16_swap: the odd 16-lane rows of one operand against the even
// rows of the other; v_permlane32_swap: the same for the halves) do it in the vector ALU; with both operands the
// same register the two results hold "my row pair's even row" and "its odd row".  The additions are those of
// x += shfl_xor(x, 16); x += shfl_xor(x, 32) in the same order (fp addition commutes), so the bits are the same.
__device__ __forceinline__ float quad_sum(float x) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float s = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
__device__ __forceinline__ float quad_max(float x) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float s = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Where part i of n begins among `total` things.  In 32 bits: a division in 64 is a hundred instructions, ahead of a workgroup's first load.
__device__ __forceinline__ int part_of(int i, int total, int n) { return (int)((unsigned)i * (unsigned)total / (unsigned)n); }

// sum of ss[c][m] over c = start, start + stride, ... < nch, in that order; the loads are issued
// eight at a time so that their latencies overlap
__device__ __forceinline__ float sum_ss(const float *__restrict__ ss, int nch, int m_pad, int m, int start, int stride) {
    float s = 0.f;
    for (int c0 = start; c0 < nch; c0 += 8 * stride) {
        float t[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = (c0 + j * stride < nch) ? ss[(size_t)(c0 + j * stride) * m_pad + m] : 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) s += t[j];
    }
    return s;
}

// the same sum in two parts: the first eight loads now, the rest and the additions when they are needed
struct SsLoads {
    float t[8];
    __device__ __forceinline__ void load(const float *__restrict__ ss, int nch, int m_pad, int m, int start, int stride) {
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = (start + j * stride < nch) ? ss[(size_t)(start + j * stride) * m_pad + m] : 0.f;
    }
    __device__ __forceinline__ float sum(const float *__restrict__ ss, int nch, int m_pad, int m, int start, int stride) const {
        float s = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) s += t[j];
        for (int c = start + 8 * stride; c < nch; c += stride) s += ss[(size_t)c * m_pad + m];
        return s;
    }
};

// 1 / sqrt(mean(x^2) + eps) of every token from its `nch` partial sums of squares, written to `rs`: the partials stay as they
// are (one preparation serves every emulated rank's MLP).  A consumer told nch = 0 takes the factor as it is.  A projection's epilogue that adds 256 partials per
// token by itself waits for eight dependent rounds of loads per m-tile: 28 of 150 us in the gate/up projection of 1000
// tokens of the 70B shard, 42 of 440 at 4096 (with 8 partials: one round, the launch then costs more than it saves).
// One workgroup per m-tile.
constexpr int ROW_SCALE_MIN_NCH = 65;
__global__ void __launch_bounds__(512) k_row_scale(const float *__restrict__ ss, int nch, int m_pad, int h, float eps,
                                                   float *__restrict__ rs) {
    __shared__ float red[32][16];
    const int r = threadIdx.x & 15, part = threadIdx.x >> 4, m = blockIdx.x * 16 + r;
    red[part][r] = sum_ss(ss, nch, m_pad, m, part, 32);
    __syncthreads();
    if (threadIdx.x < 16) {
        float t = 0.f;
#pragma unroll
        for (int q = 0; q < 32; ++q) t += red[q][threadIdx.x];
        rs[m] = 1.0f / sqrtf(t / (float)h + eps);
    }
}

constexpr int PREP_BY_WAVE = 16;
// ------------------------------------------------------------------------------------------
// prep: out = base + (slot0 + slot1 + ...), xhat = fp16(out * gain) in packed layout (plus its
// lo plane), and the partial sums of squares of `out` per (workgroup, token), up to PREP_BY_WAVE tokens per (wave, token).  One wave per
// (m-tile, chunk of `tpw` k-tiles); lane l handles token l%16 and 8 consecutive features.  (With a partial per wave the QKV projection of 48
// sequences read 256 of them per token in four rounds, 3.7 us of its 13.  Up to 16 tokens its 64 threads per token read them in one, and as
// many partials as the fused epilogues leave are added in the same order.)
// ------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_prep(const float *__restrict__ base, const float *__restrict__ slots,
                                              int n_slots, size_t slot_stride, float *__restrict__ out,
                                              const float *__restrict__ gain, __bf16 *__restrict__ xhat,
                                              __bf16 *__restrict__ xlo, float *__restrict__ ss, int M, int h, int tpw,
                                              int m_pad, const float *__restrict__ bias) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int KT = h >> 5;
    const int chunk = blockIdx.x * 4 + wave;
    const int mt = blockIdx.y;
    const int m = mt * 16 + (lane & 15), g = lane >> 4;
    const bool valid = m < M;
    float ssum = 0.f;
    for (int t = 0; t < tpw; ++t) {
        const int kt = chunk * tpw + t;
        if (kt >= KT) break;
        const int col = kt * 32 + g * 8;
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = 0.f;
        if (valid) {
            const size_t o = (size_t)m * h + col;
            // partials in ascending slot order; the loads of a group of 8 slots are issued together
            for (int s0 = 0; s0 < n_slots; s0 += 8) {
                float4 p0[8], p1[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    if (s0 + j < n_slots) {
                        p0[j] = *(const float4 *)(slots + (size_t)(s0 + j) * slot_stride + o);
                        p1[j] = *(const float4 *)(slots + (size_t)(s0 + j) * slot_stride + o + 4);
                    }
                }
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    if (s0 + j < n_slots) {
                        if (s0 + j == 0) {
                            v[0] = p0[j].x; v[1] = p0[j].y; v[2] = p0[j].z; v[3] = p0[j].w;
                            v[4] = p1[j].x; v[5] = p1[j].y; v[6] = p1[j].z; v[7] = p1[j].w;
                        } else {
                            v[0] += p0[j].x; v[1] += p0[j].y; v[2] += p0[j].z; v[3] += p0[j].w;
                            v[4] += p1[j].x; v[5] += p1[j].y; v[6] += p1[j].z; v[7] += p1[j].w;
                        }
                    }
                }
            }
            if (base) {
                const float4 b0 = *(const float4 *)(base + o), b1 = *(const float4 *)(base + o + 4);
                v[0] = b0.x + v[0]; v[1] = b0.y + v[1]; v[2] = b0.z + v[2]; v[3] = b0.w + v[3];
                v[4] = b1.x + v[4]; v[5] = b1.y + v[5]; v[6] = b1.z + v[6]; v[7] = b1.w + v[7];
            }
            if (bias) {      // the output projection's bias, once, after the sum (Sec. 4.1.2)
                const float4 c0 = *(const float4 *)(bias + col), c1 = *(const float4 *)(bias + col + 4);
                v[0] += c0.x; v[1] += c0.y; v[2] += c0.z; v[3] += c0.w;
                v[4] += c1.x; v[5] += c1.y; v[6] += c1.z; v[7] += c1.w;
            }
            if (out) {
                *(float4 *)(out + o) = make_float4(v[0], v[1], v[2], v[3]);
                *(float4 *)(out + o + 4) = make_float4(v[4], v[5], v[6], v[7]);
            }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) ssum += v[i] * v[i];
        if (xhat) {
            bf16x8 x, xl;
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = xl[i] = (__bf16)0.f;
            if (valid) {
                const float4 g0 = *(const float4 *)(gain + col), g1 = *(const float4 *)(gain + col + 4);
                const float gg[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float p = v[i] * gg[i];
                    x[i] = act_one(p);
                    xl[i] = act_one(p - act_back(x[i]));
                }
            }
            const size_t fo = spd_act_index(mt, kt, KT, (M + 15) >> 4) + lane * 8;
            *(bf16x8 *)(xhat + fo) = x;
            if (xlo) *(bf16x8 *)(xlo + fo) = xl;
        }
    }
    ssum += shfl_xor_f(ssum, 16);
    ssum += shfl_xor_f(ssum, 32);
    if (!ss) return;
    if (M <= PREP_BY_WAVE) {
        if (g == 0 && chunk * tpw < KT) ss[(size_t)chunk * m_pad + m] = ssum;
        return;
    }
    __shared__ float part[4][16];
    if (g == 0) part[wave][lane] = ssum;
    __syncthreads();
    if (threadIdx.x < 16)
        ss[(size_t)blockIdx.x * m_pad + m] = (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]);
}

// prep for long calls (more than 512 tokens, hidden size a multiple of 256): the same sums in the
// same order, but every load and store of fp32 data covers 1 KiB of one token's row (a wave per
// token, lane l at features 4l .. 4l+3 of a chunk of 256) instead of 128-byte pieces of 16 rows, which
// the HBM serves at a higher rate.  One workgroup per (NP chunks of 256 features, m-tile); wave w takes
// tokens w, w+4, w+8, w+12.  The normalised bf16 values are turned into fragments through LDS.
// Sums of squares: one partial per (chunk, token), as k_prep with 8 k-tiles per wave.
// streaming 16-byte load (data that is read once)
__device__ __forceinline__ float4 ldnt4(const float *p) {
    const f32x4 v = __builtin_nontemporal_load((const f32x4 *)p);
    return make_float4(v[0], v[1], v[2], v[3]);
}

// The launch is a fixed number of workgroups (two per compute unit) that walk the (chunk, m-tile) items with a stride.
// SLOTS = false (the first norm of a call: nothing to sum) needs few registers, so that four workgroups share a compute unit
// and hide each other's latency: 1000 tokens of the 70B shard 22 -> 15 us.
template <int NP, bool SLOTS>     // NP pieces of 256 features per workgroup and token (1 or 2): NP KiB contiguous per token row
__global__ void __launch_bounds__(256) k_prep_rows(const float *__restrict__ base, const float *__restrict__ slots, int n_slots,
                                                   size_t slot_stride, float *__restrict__ out,
                                                   const float *__restrict__ gain, __bf16 *__restrict__ xhat,
                                                   __bf16 *__restrict__ xlo, float *__restrict__ ss, int M, int h,
                                                   int m_pad, const float *__restrict__ bias, int n_chunks, int n_items) {
    constexpr int PITCH = NP * 256;          // bf16 elements (no pad: 16 KiB for both planes)
    __shared__ __attribute__((aligned(16))) __bf16 tile[2][16][PITCH];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int KT = h >> 5;
  for (int item = blockIdx.x; item < n_items; item += gridDim.x) {
    const int chunk0 = (item % n_chunks) * NP, mt = item / n_chunks;
    const int col = chunk0 * 256 + lane * 4;           // piece q: + 256 q
    float4 gn[NP], bs[NP];
#pragma unroll
    for (int q = 0; q < NP; ++q) {
        gn[q] = bs[q] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (xhat) gn[q] = *(const float4 *)(gain + col + 256 * q);
        if (bias) bs[q] = *(const float4 *)(bias + col + 256 * q);
    }
    constexpr int TB = NP == 1 ? 4 : 1;      // tokens whose loads are in flight together
#pragma unroll
    for (int it = 0; it < 4 / TB; ++it) {
        float4 p[SLOTS ? TB : 1][NP][8], b[TB][NP], v[TB][NP];
        bool valid[TB];
        size_t off[TB];
#pragma unroll
        for (int t = 0; t < TB; ++t) {
            const int m = mt * 16 + wave + 4 * (TB * it + t);
            valid[t] = m < M;
            off[t] = (size_t)(valid[t] ? m : M - 1) * h + col;
#pragma unroll
            for (int q = 0; q < NP; ++q) v[t][q] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        if constexpr (SLOTS)
        for (int s0 = 0; s0 < n_slots; s0 += 8) {
#pragma unroll
            for (int t = 0; t < TB; ++t)
#pragma unroll
                for (int j = 0; j < 8; ++j)
#pragma unroll
                    for (int q = 0; q < NP; ++q)
                        if (s0 + j < n_slots) p[t][q][j] = ldnt4(slots + (size_t)(s0 + j) * slot_stride + off[t] + 256 * q);
#pragma unroll
            for (int t = 0; t < TB; ++t)
#pragma unroll
                for (int q = 0; q < NP; ++q)
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        if (s0 + j < n_slots) {
                            const float4 a = p[t][q][j];
                            if (s0 + j == 0) v[t][q] = a;
                            else { v[t][q].x += a.x; v[t][q].y += a.y; v[t][q].z += a.z; v[t][q].w += a.w; }
                        }
        }
        if (base) {
#pragma unroll
            for (int t = 0; t < TB; ++t)
#pragma unroll
                for (int q = 0; q < NP; ++q) b[t][q] = ldnt4(base + off[t] + 256 * q);
#pragma unroll
            for (int t = 0; t < TB; ++t)
#pragma unroll
                for (int q = 0; q < NP; ++q) {
                    v[t][q].x = b[t][q].x + v[t][q].x; v[t][q].y = b[t][q].y + v[t][q].y;
                    v[t][q].z = b[t][q].z + v[t][q].z; v[t][q].w = b[t][q].w + v[t][q].w;
                }
        }
#pragma unroll
        for (int t = 0; t < TB; ++t) {
            const int r = wave + 4 * (TB * it + t);
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                float4 u = v[t][q];
                if (bias) { u.x += bs[q].x; u.y += bs[q].y; u.z += bs[q].z; u.w += bs[q].w; }
                if (!valid[t]) u = make_float4(0.f, 0.f, 0.f, 0.f);
                if (out && valid[t]) *(float4 *)(out + off[t] + 256 * q) = u;
                float sq = u.x * u.x + u.y * u.y + u.z * u.z + u.w * u.w;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) sq += shfl_xor_f(sq, o);
                if (ss && lane == 0) ss[(size_t)(chunk0 + q) * m_pad + mt * 16 + r] = sq;
                if (xhat) {
                    const float q0 = u.x * gn[q].x, q1 = u.y * gn[q].y, q2 = u.z * gn[q].z, q3 = u.w * gn[q].w;
                    const bf16x4 hi = cvt4h(q0, q1, q2, q3);
                    *(bf16x4 *)&tile[0][r][256 * q + lane * 4] = hi;
                    if (xlo) *(bf16x4 *)&tile[1][r][256 * q + lane * 4] = cvt4h_lo(q0, q1, q2, q3, hi);
                }
            }
        }
    }
    if (!xhat) continue;
    __syncthreads();
    // wave w writes fragments 2 NP w .. 2 NP w + 2 NP - 1 of the workgroup's 8 NP k-tiles
#pragma unroll
    for (int f = 0; f < 2 * NP; ++f) {
        const int kt = 2 * NP * wave + f, r = lane & 15, g = lane >> 4;
        const size_t fo = spd_act_index(mt, chunk0 * 8 + kt, KT, (M + 15) >> 4) + lane * 8;
        *(bf16x8 *)(xhat + fo) = *(const bf16x8 *)&tile[0][r][kt * 32 + g * 8];
        if (xlo) *(bf16x8 *)(xlo + fo) = *(const bf16x8 *)&tile[1][r][kt * 32 + g * 8];
    }
    __syncthreads();      // the tile is free for the next item
  }
}

// The same preparation for a chain of a two-chain prefill, where it shares the chip with the other chain's GEMM:
// a few workgroups that each fill a whole compute unit (16 waves) and keep the next item's loads in flight
// while the current item is summed, stored and turned into fragments, so that a fraction of the compute units
// draws the HBM's full rate and the rest stay with the GEMM.  An item is (chunk of 256 features, m-tile); wave w
// takes token w of the m-tile, lane l features 4l .. 4l+3 of the chunk (1 KiB per wave, slot and row).  Sums in
// the order of k_prep_rows (slots ascending, then the base, then the bias).  At most 8 slots.
template <int NS, bool XH, bool BIAS>     // slots; fragments of the normalised values wanted; bias joins the sum
__global__ void __launch_bounds__(1024) k_prep_cu(const float *__restrict__ base, const float *__restrict__ slots,
                                                  size_t slot_stride, float *__restrict__ out,
                                                  const float *__restrict__ gain, __bf16 *__restrict__ xhat,
                                                  __bf16 *__restrict__ xlo, float *__restrict__ ss, int M, int h,
                                                  int m_pad, const float *__restrict__ bias, int n_chunks, int n_items) {
    __shared__ __attribute__((aligned(16))) __bf16 tile[2][2][16][256];      // [buffer][plane][token][feature]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int KT = h >> 5;
    int item = blockIdx.x;
    if (item >= n_items) return;
    // everything an item reads, issued as one group without branches (the wait for the current group can then
    // leave the next group's loads in flight)
    struct Loads {
        float4 p[NS], b, gn, bs;
        size_t off;
        bool valid;
    };
    auto issue = [&](int it, Loads &L) {
        const int chunk = it % n_chunks, mt = it / n_chunks;
        const int m = mt * 16 + wave;
        const int col = chunk * 256 + lane * 4;
        L.valid = m < M;
        L.off = (size_t)(L.valid ? m : M - 1) * h + col;
#pragma unroll
        for (int j = 0; j < NS; ++j) L.p[j] = ldnt4(slots + (size_t)j * slot_stride + L.off);
        L.b = ldnt4(base + L.off);
        if constexpr (XH) L.gn = *(const float4 *)(gain + col);
        if constexpr (BIAS) L.bs = *(const float4 *)(bias + col);
    };
    int buf = 0;
    // one item: the next item's loads go out first, into the other register set (the two sets swap roles from item
    // to item, so that nothing is copied and nothing waits for loads it does not use yet)
    auto step = [&](Loads &cur, Loads &nxt, int it) {
        const int ni = it + gridDim.x;
        // (past the end: the last item's addresses once more, so that the group stays branch-free; never used)
        issue(ni < n_items ? ni : it, nxt);
        const int chunk = it % n_chunks, mt = it / n_chunks;
        float4 v = cur.p[0];
#pragma unroll
        for (int j = 1; j < NS; ++j) { v.x += cur.p[j].x; v.y += cur.p[j].y; v.z += cur.p[j].z; v.w += cur.p[j].w; }
        v.x = cur.b.x + v.x; v.y = cur.b.y + v.y; v.z = cur.b.z + v.z; v.w = cur.b.w + v.w;
        if constexpr (BIAS) { v.x += cur.bs.x; v.y += cur.bs.y; v.z += cur.bs.z; v.w += cur.bs.w; }
        if (!cur.valid) v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (cur.valid) *(float4 *)(out + cur.off) = v;
        float sq = v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) sq += shfl_xor_f(sq, o);
        if constexpr (XH) {
            if (lane == 0) ss[(size_t)chunk * m_pad + mt * 16 + wave] = sq;
            const float q0 = v.x * cur.gn.x, q1 = v.y * cur.gn.y, q2 = v.z * cur.gn.z, q3 = v.w * cur.gn.w;
            const bf16x4 hi = cvt4h(q0, q1, q2, q3);
            *(bf16x4 *)&tile[buf][0][wave][lane * 4] = hi;
            if (xlo) *(bf16x4 *)&tile[buf][1][wave][lane * 4] = cvt4h_lo(q0, q1, q2, q3, hi);
            // the barrier orders LDS traffic only: the loads of the next item stay in flight across it.  One
            // barrier per item is enough with two tile buffers: whoever writes buffer b for item i + 2 has passed
            // the barrier of item i + 1, which every wave reaches after its reads of item i
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
            // wave w writes k-tile w % 8 of plane w / 8: 1 KiB, lane = (row, group of 8 features)
            const int plane = wave >> 3, kt = wave & 7, r = lane & 15, g = lane >> 4;
            const size_t fo = spd_act_index(mt, chunk * 8 + kt, KT, (M + 15) >> 4) + lane * 8;
            const bf16x8 f = *(const bf16x8 *)&tile[buf][plane][r][kt * 32 + g * 8];
            if (plane == 0) *(bf16x8 *)(xhat + fo) = f;
            else if (xlo) *(bf16x8 *)(xlo + fo) = f;
            buf ^= 1;
        }
    };
    Loads A, B;
    issue(item, A);
    for (;;) {
        step(A, B, item);
        item += gridDim.x;
        if (item >= n_items) break;
        step(B, A, item);
        item += gridDim.x;
        if (item >= n_items) break;
    }
}

template <int NS>
hipError_t launch_prep_cu(hipStream_t s, int n_wgs, const float *base, const float *slots, size_t slot_stride, float *out,
                          const float *gain, __bf16 *xhat, __bf16 *xlo, float *ss, int M, int h, int m_pad, const float *bias) {
    const int n_chunks = h / 256, n_items = n_chunks * ((M + 15) / 16);
    const dim3 grid(n_items < n_wgs ? n_items : n_wgs), block(1024);
#define SPD_PREP_CU_GO(XH, BIAS)                                                                                         \
    hipLaunchKernelGGL((k_prep_cu<NS, XH, BIAS>), grid, block, 0, s, base, slots, slot_stride, out, gain, xhat, xlo, ss, M, h, \
                       m_pad, bias, n_chunks, n_items)
    if (xhat) { if (bias) SPD_PREP_CU_GO(true, true); else SPD_PREP_CU_GO(true, false); }
    else { if (bias) SPD_PREP_CU_GO(false, true); else SPD_PREP_CU_GO(false, false); }
#undef SPD_PREP_CU_GO
    return hipGetLastError();
}

// The sum over the ranks at a sync point, for one rank whose own partial is still in registers:
// out = base + (slot_0 + ... + slot_tp-1) [+ bias], the own partial standing in for slot `rank`.
// both halves of a tile at once, eight slots at a time: all 16 loads of a round (and the two base
// loads) are issued together (indices clamped, named registers: nothing here may end up in
// scratch memory); additions in ascending slot order, the base last, then the bias
__device__ __forceinline__ void rank_sum_pair(const float *__restrict__ slots, size_t slot_stride, int tp, int rank,
                                          const float *__restrict__ base, size_t oa, float4 own_a, float4 own_b, float4 &ra, float4 &rb) {
    const size_t ob = oa + 16;
    float4 acc_a = make_float4(0.f, 0.f, 0.f, 0.f), acc_b = acc_a;
    // (past the end: the last slot again; the own slot is in registers: a neighbour's line, which is on its way anyway)
    const int last = tp - 1, other = rank > 0 ? rank - 1 : (tp > 1 ? 1 : 0);
    auto at = [&](int s) { return s == rank ? other : min(s, last); };
    const float4 bs_a = *(const float4 *)(base + oa), bs_b = *(const float4 *)(base + ob);
    for (int s0 = 0; s0 < tp; s0 += 8) {
#define SPD_LD(j)                                                                                         \
const float4 ta##j = *(const float4 *)(slots + (size_t)at(s0 + j) * slot_stride + oa);                \
const float4 tb##j = *(const float4 *)(slots + (size_t)at(s0 + j) * slot_stride + ob);
        SPD_LD(0) SPD_LD(1) SPD_LD(2) SPD_LD(3) SPD_LD(4) SPD_LD(5) SPD_LD(6) SPD_LD(7)
#undef SPD_LD
        auto add = [&](int s, const float4 &ta, const float4 &tb) {
            if (s >= tp) return;
            const float4 va = (s == rank) ? own_a : ta, vb = (s == rank) ? own_b : tb;
            if (s == 0) {
                acc_a = va;
                acc_b = vb;
            } else {
                acc_a.x += va.x; acc_a.y += va.y; acc_a.z += va.z; acc_a.w += va.w;
                acc_b.x += vb.x; acc_b.y += vb.y; acc_b.z += vb.z; acc_b.w += vb.w;
            }
        };
        add(s0, ta0, tb0); add(s0 + 1, ta1, tb1); add(s0 + 2, ta2, tb2); add(s0 + 3, ta3, tb3);
        add(s0 + 4, ta4, tb4); add(s0 + 5, ta5, tb5); add(s0 + 6, ta6, tb6); add(s0 + 7, ta7, tb7);
    }
    ra = make_float4(bs_a.x + acc_a.x, bs_a.y + acc_a.y, bs_a.z + acc_a.z, bs_a.w + acc_a.w);
    rb = make_float4(bs_b.x + acc_b.x, bs_b.y + acc_b.y, bs_b.z + acc_b.z, bs_b.w + acc_b.w);
}

// What such a sum reads, requested ahead of the contraction: the first slots and the base of one (pair of n-tiles, m-tile).  Asked
// for in the epilogue, which all workgroups of a launch reach together, it was a trip to the memory of its own after the weights.
constexpr int SYNC_EARLY = 8;
struct SyncRegs {          // ... in registers
    float4 s[SYNC_EARLY][2], base[2];      // (the own slot's place is not used)
    __device__ __forceinline__ float4 slot(int i, int half) const { return s[i][half]; }
    __device__ __forceinline__ float4 at_base(int half) const { return base[half]; }
};
struct SyncLds {           // ... in LDS, [slot][half][lane]; the base in the own slot's place or, with a rank beyond them, behind the slots
    const f32x4 *p;
    int rank;
    __device__ __forceinline__ float4 slot(int i, int half) const { return __builtin_bit_cast(float4, p[(i * 2 + half) * 64]); }
    __device__ __forceinline__ float4 at_base(int half) const { return slot(rank < SYNC_EARLY ? rank : SYNC_EARLY, half); }
};
struct SyncNone {};        // nothing requested yet
struct SyncDone {          // the sum is there: the own partial and the result in LDS, [half][lane] each
    const f32x4 *own, *x;
};
struct SyncSum {           // the sync point an epilogue performs
    const float *slots, *base, *bias;
    size_t slot_stride;
    int tp, rank, M, h;
    // offset of a lane's first feature (rows past the call: its last one)
    __device__ __forceinline__ size_t at(int pair, int mt, int lane) const {
        const int m = mt * 16 + (lane & 15);
        return (size_t)(m < M ? m : M - 1) * h + pair * 32 + 4 * (lane >> 4);
    }
    __device__ __forceinline__ void load(SyncRegs &t, size_t o) const {
        t.base[0] = *(const float4 *)(base + o);
        t.base[1] = *(const float4 *)(base + o + 16);
#pragma unroll
        for (int s = 0; s < SYNC_EARLY; ++s) {
            const float *p = (s == rank ? base : slots + (size_t)(s < tp ? s : tp - 1) * slot_stride) + o;
            t.s[s][0] = *(const float4 *)p;
            t.s[s][1] = *(const float4 *)(p + 16);
        }
    }
    // the sum of rank_sum_pair(), in the same order; o: offset of the first half's features, na: its column
    template <class T>
    __device__ __forceinline__ void sum(const T &t, size_t o, int na, float4 own_a, float4 own_b, float4 &ra, float4 &rb) const {
        float4 acc_a = own_a, acc_b = own_b;
        auto add = [&](int s, float4 va, float4 vb) {
            if (s == rank) { va = own_a; vb = own_b; }
            if (s == 0) {
                acc_a = va;
                acc_b = vb;
            } else {
                acc_a.x += va.x; acc_a.y += va.y; acc_a.z += va.z; acc_a.w += va.w;
                acc_b.x += vb.x; acc_b.y += vb.y; acc_b.z += vb.z; acc_b.w += vb.w;
            }
        };
#pragma unroll
        for (int s = 0; s < SYNC_EARLY; ++s)
            if (s < tp) add(s, t.slot(s, 0), t.slot(s, 1));
        for (int s = SYNC_EARLY; s < tp; ++s) {
            const float *p = (s == rank ? base : slots + (size_t)s * slot_stride) + o;
            add(s, *(const float4 *)p, *(const float4 *)(p + 16));
        }
        const float4 ba = t.at_base(0), bb = t.at_base(1);
        ra = make_float4(ba.x + acc_a.x, ba.y + acc_a.y, ba.z + acc_a.z, ba.w + acc_a.w);
        rb = make_float4(bb.x + acc_b.x, bb.y + acc_b.y, bb.z + acc_b.z, bb.w + acc_b.w);
        add_bias(na, ra, rb);
    }
    __device__ __forceinline__ void sum(const SyncNone &, size_t o, int na, float4 own_a, float4 own_b, float4 &ra, float4 &rb) const {
        rank_sum_pair(slots, slot_stride, tp, rank, base, o, own_a, own_b, ra, rb);
        add_bias(na, ra, rb);
    }
    __device__ __forceinline__ void sum(const SyncDone &t, size_t, int, float4, float4, float4 &ra, float4 &rb) const {
        ra = __builtin_bit_cast(float4, t.x[0]);
        rb = __builtin_bit_cast(float4, t.x[64]);
    }
    // element e = 256 half + 4 lane + i of the tile pair's sum, in the same order; slots and base as SyncLds holds them.  Up to SYNC_EARLY ranks.
    __device__ __forceinline__ float element(const float *peers, int e, float own, float bs) const {
        float acc = own;
#pragma unroll
        for (int s = 0; s < SYNC_EARLY; ++s) {
            if (s >= tp) break;
            const float v = s == rank ? own : peers[s * 512 + e];
            acc = s == 0 ? v : acc + v;
        }
        const float r = peers[(rank < SYNC_EARLY ? rank : SYNC_EARLY) * 512 + e] + acc;
        return bias ? r + bs : r;
    }
    // where element e lies in a [tokens][h] buffer (rows past the call: its last one), and its column
    __device__ __forceinline__ int col(int pair, int e) const { return pair * 32 + (e >> 8) * 16 + 4 * ((e & 255) >> 6) + (e & 3); }
    __device__ __forceinline__ size_t at_element(int pair, int e) const {
        const int m = (e >> 2) & 15;
        return (size_t)(m < M ? m : M - 1) * h + col(pair, e);
    }
    __device__ __forceinline__ void add_bias(int na, float4 &ra, float4 &rb) const {
        if (!bias) return;
        const float4 ba = *(const float4 *)(bias + na), bb = *(const float4 *)(bias + na + 16);
        ra.x += ba.x; ra.y += ba.y; ra.z += ba.z; ra.w += ba.w;
        rb.x += bb.x; rb.y += bb.y; rb.z += bb.z; rb.w += bb.w;
    }
};

// ------------------------------------------------------------------------------------------
// Epilogues.  Each receives the accumulators of one (pair of n-tiles, m-tile): a = tile
// 2*pair, b = tile 2*pair+1; lane l: token m = mt*16 + l%16, features 4*(l/16) + i.
// ------------------------------------------------------------------------------------------
// Every epilogue has two parts: pre() issues the loads that do not depend on the accumulators
// (so that they can be started before the weights are streamed), operator() finishes the tile.
// (The matrix's factor among them: read where it is used, it was a trip to the memory of 1.2 us at the end of every launch of a decode step.)
// kNeedsRs: the tile must be scaled by 1/sqrt(mean(x^2)+eps) of the token, which the caller
// computes from the partial sums of squares ss[nch][m_pad].
struct EpiQKV {
    static constexpr bool kByElement = false;
    static constexpr bool kSync = false;
    static constexpr bool kLong = true;        // used by calls of any length
    static constexpr bool kWideSum = true;     // K slices are added in 64 bits
    static constexpr bool kNeedsRs = true;
    static constexpr bool kSliced = false;
    int M, q_len, q, kv, d, h, max_ctx, nch, m_pad;
    float eps;
    const float *ss, *cosT, *sinT;
    const float *wsc;                 // the factor 2^-k that undoes the power of two in the packed weights
    __bf16 *qbuf, *qlo, *kc, *vc;     // queries are kept as hi + lo pairs
    spd_positions P;
    struct Pre {
        float4 c, s;
        float sc;
    };

    __device__ __forceinline__ Pre pre(int pair, int mt, int lane) const {
        Pre p;
        p.c = p.s = make_float4(0.f, 0.f, 0.f, 0.f);
        p.sc = *wsc;
        const int m = mt * 16 + (lane & 15), g = lane >> 4;
        const int tph = d >> 4, half = d >> 1;
        const int head = (2 * pair) / tph;
        if (m < M && head < q + kv) {
            const int pos = P.pos[m / q_len] + (m % q_len);
            const int ca = spd_qkv_tile_col0(2 * pair, q, kv, d) - head * d + 4 * g;
            p.c = *(const float4 *)(cosT + (size_t)pos * half + ca);
            p.s = *(const float4 *)(sinT + (size_t)pos * half + ca);
        }
        return p;
    }

    __device__ __forceinline__ void operator()(int pair, int mt, f32x4 a, f32x4 b, int lane, float rs, const Pre &p) const {
        const int m = mt * 16 + (lane & 15), g = lane >> 4;
        if (m >= M) return;
        const int tph = d >> 4;
        const int head = (2 * pair) / tph;
        const int bseq = m / q_len, pos = P.pos[bseq] + (m % q_len);
        const int ca = spd_qkv_tile_col0(2 * pair, q, kv, d) - head * d + 4 * g;       // column inside the head
        const int cb = spd_qkv_tile_col0(2 * pair + 1, q, kv, d) - head * d + 4 * g;
        rs *= p.sc;
        a *= rs;
        b *= rs;
        if (head < q + kv) {
            // rotary partners: a holds j = ca .. ca+3 (< d/2), b holds j + d/2
            const float4 c = p.c, s = p.s;
            const float l0 = a[0] * c.x - b[0] * s.x, l1 = a[1] * c.y - b[1] * s.y, l2 = a[2] * c.z - b[2] * s.z,
                        l3 = a[3] * c.w - b[3] * s.w;
            const float h0 = b[0] * c.x + a[0] * s.x, h1 = b[1] * c.y + a[1] * s.y, h2 = b[2] * c.z + a[2] * s.z,
                        h3 = b[3] * c.w + a[3] * s.w;
            const bf16x4 lo = cvt4(l0, l1, l2, l3), hi = cvt4(h0, h1, h2, h3);
            if (head < q) {
                const size_t o = (size_t)m * (q * d) + head * d;
                *(bf16x4 *)(qbuf + o + ca) = lo;
                *(bf16x4 *)(qbuf + o + cb) = hi;
                *(bf16x4 *)(qlo + o + ca) = cvt4_lo(l0, l1, l2, l3, lo);
                *(bf16x4 *)(qlo + o + cb) = cvt4_lo(h0, h1, h2, h3, hi);
            } else {
                __bf16 *dst = kc + ((size_t)bseq * kv + (head - q)) * (size_t)max_ctx * d;
                *(bf16x4 *)(dst + spd_kcache_off(pos, ca, d)) = lo;
                *(bf16x4 *)(dst + spd_kcache_off(pos, cb, d)) = hi;
            }
        } else {
            __bf16 *dst = vc + ((size_t)bseq * kv + (head - q - kv)) * (size_t)max_ctx * d;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                dst[spd_vcache_off(pos, ca + i, d)] = (__bf16)a[i];
                dst[spd_vcache_off(pos, cb + i, d)] = (__bf16)b[i];
            }
        }
    }
};

// QKV projection of a decode step whose K is cut into slices: norm scale and rotation are linear,
// so every slice applies them to its own partial sums and parks the result, fp32, in
// part[slice][token][column] (columns in natural order: head * d + j).  The attention kernel adds
// the slices in ascending order, rounds, and appends the new key and value to the cache.
struct EpiQKVPart {
    static constexpr bool kByElement = false;
    static constexpr bool kSync = false;
    static constexpr bool kNeedsRs = true;
    int M, q_len, q, kv, d, h, nqkv, nch, m_pad;
    int part_rows;             // token rows per slice of `part`
    float eps;
    const float *ss, *cosT, *sinT;
    const float *wsc;
    float *part;
    spd_positions P;
    struct Pre {
        float4 c, s;
        float sc;
        int ca, cb;            // the lane's first column of either tile
        bool rot;
    };

    __device__ __forceinline__ Pre pre(int pair, int mt, int lane) const {
        Pre p;
        p.c = p.s = make_float4(0.f, 0.f, 0.f, 0.f);
        p.sc = *wsc;
        const int m = mt * 16 + (lane & 15), g = lane >> 4;
        const int tph = d >> 4, half = d >> 1;
        const int head = (int)((unsigned)(2 * pair) / (unsigned)tph), w = 2 * pair - head * tph;      // (as spd_qkv_tile_col0(); tph is even)
        p.rot = head < q + kv;
        p.ca = head * d + (p.rot ? (w >> 1) << 4 : w << 4) + 4 * g;
        p.cb = p.ca + (p.rot ? half : 16);
        if (m < M && p.rot) {
            const int pos = q_len == 1 ? P.pos[m] : P.pos[m / q_len] + (m % q_len);
            const size_t o = (size_t)pos * half + p.ca - head * d;
            p.c = *(const float4 *)(cosT + o);
            p.s = *(const float4 *)(sinT + o);
        }
        return p;
    }

    __device__ __forceinline__ void slice(int, int ks, int mt, f32x4 a, f32x4 b, int lane, float rs, const Pre &p) const {
        const int m = mt * 16 + (lane & 15);
        if (m >= M) return;
        rs *= p.sc;
        a *= rs;
        b *= rs;
        float4 lo = make_float4(a[0], a[1], a[2], a[3]), hi = make_float4(b[0], b[1], b[2], b[3]);
        if (p.rot) {
            const float4 c = p.c, s = p.s;
            lo = make_float4(a[0] * c.x - b[0] * s.x, a[1] * c.y - b[1] * s.y, a[2] * c.z - b[2] * s.z, a[3] * c.w - b[3] * s.w);
            hi = make_float4(b[0] * c.x + a[0] * s.x, b[1] * c.y + a[1] * s.y, b[2] * c.z + a[2] * s.z, b[3] * c.w + a[3] * s.w);
        }
        float *dst = part + ((size_t)ks * part_rows + m) * nqkv;
        *(float4 *)(dst + p.ca) = lo;
        *(float4 *)(dst + p.cb) = hi;
    }
};

template <bool MID>      // MID: the epilogue can also perform the kept attention sync point (spd = 2)
struct EpiOT {
    static constexpr bool kByElement = false;
    static constexpr bool kSync = MID;         // can perform a sync point (one rank, the peers' partial sums are inputs)
    static constexpr bool kWideSum = false;
    static constexpr bool kNeedsRs = false;
    static constexpr bool kSliced = false;
    int M, h, spd, m_pad;
    const float *x, *g2;
    const float *bo = nullptr; // bias of the output projection or NULL: part of the SPD block's MLP input (Sec. 4.1.2)
    const float *wsc;
    float *ybuf, *slot, *ss2;
    __bf16 *xhat2, *xlo2;      // xlo2 may be NULL
    // spd = 2: TP block whose kept attention sync point is performed here (one rank, the peers' partial
    // sums already in `slots`): R = X + sum of the slots (+ bias) goes to rbuf and on to the second norm
    const float *slots = nullptr;
    size_t slot_stride = 0;
    int tp = 0, rank = 0;
    float *rbuf = nullptr;
    __device__ __forceinline__ SyncSum sync() const { return SyncSum{slots, x, bo, slot_stride, tp, rank, M, h}; }
    __device__ __forceinline__ const float *joins_own() const { return nullptr; }      // what is added to the own partial before the sum
    struct Pre {
        float4 x0, x1, ga, gb;
        float sc;
    };

    __device__ __forceinline__ Pre pre(int pair, int mt, int lane) const {
        Pre p;
        p.x0 = p.x1 = p.ga = p.gb = make_float4(0.f, 0.f, 0.f, 0.f);
        p.sc = *wsc;
        const int m = mt * 16 + (lane & 15), g = lane >> 4;
        const int na = pair * 32 + 4 * g, nb = na + 16;
        if (MID && spd == 2 && m < M) {      // the sum loads X itself
            p.ga = *(const float4 *)(g2 + na);
            p.gb = *(const float4 *)(g2 + nb);
        } else if (spd && m < M) {
            const size_t o = (size_t)m * h;
            p.x0 = *(const float4 *)(x + o + na);
            p.x1 = *(const float4 *)(x + o + nb);
            if (bo) {        // X + b now, P_r when the accumulators are there
                const float4 ba = *(const float4 *)(bo + na), bb = *(const float4 *)(bo + nb);
                p.x0.x += ba.x; p.x0.y += ba.y; p.x0.z += ba.z; p.x0.w += ba.w;
                p.x1.x += bb.x; p.x1.y += bb.y; p.x1.z += bb.z; p.x1.w += bb.w;
            }
            p.ga = *(const float4 *)(g2 + na);
            p.gb = *(const float4 *)(g2 + nb);
        }
        return p;
    }

    template <class Peers = SyncNone>
    __device__ __forceinline__ void operator()(int pair, int mt, f32x4 a, f32x4 b, int lane, float, const Pre &p,
                                               const Peers &peers = Peers()) const {
        const int r = lane & 15, m = mt * 16 + r, g = lane >> 4;
        const int na = pair * 32 + 4 * g, nb = na + 16;
        const bool valid = m < M;
        if constexpr (std::is_same<Peers, SyncDone>::value) {
            a = peers.own[0];
            b = peers.own[64];
        } else {
            a *= p.sc;
            b *= p.sc;
        }
        if (!spd) {
            if (valid) {
                *(float4 *)(slot + (size_t)m * h + na) = make_float4(a[0], a[1], a[2], a[3]);
                *(float4 *)(slot + (size_t)m * h + nb) = make_float4(b[0], b[1], b[2], b[3]);
            }
            return;
        }
        float ra[4] = {0.f, 0.f, 0.f, 0.f}, rb[4] = {0.f, 0.f, 0.f, 0.f};
        float pa[4] = {0.f, 0.f, 0.f, 0.f}, pb[4] = {0.f, 0.f, 0.f, 0.f};
        if (MID && valid && spd == 2) {
            const size_t o = (size_t)m * h;
            const float4 own_a = make_float4(a[0], a[1], a[2], a[3]), own_b = make_float4(b[0], b[1], b[2], b[3]);
            *(float4 *)(slot + o + na) = own_a;
            *(float4 *)(slot + o + nb) = own_b;
            float4 qa, qb;
            sync().sum(peers, o + na, na, own_a, own_b, qa, qb);
            *(float4 *)(rbuf + o + na) = qa;
            *(float4 *)(rbuf + o + nb) = qb;
            ra[0] = qa.x; ra[1] = qa.y; ra[2] = qa.z; ra[3] = qa.w;
            rb[0] = qb.x; rb[1] = qb.y; rb[2] = qb.z; rb[3] = qb.w;
            pa[0] = ra[0] * p.ga.x; pa[1] = ra[1] * p.ga.y; pa[2] = ra[2] * p.ga.z; pa[3] = ra[3] * p.ga.w;
            pb[0] = rb[0] * p.gb.x; pb[1] = rb[1] * p.gb.y; pb[2] = rb[2] * p.gb.z; pb[3] = rb[3] * p.gb.w;
        } else if (valid) {
            const size_t o = (size_t)m * h;
            *(float4 *)(ybuf + o + na) = make_float4(a[0], a[1], a[2], a[3]);
            *(float4 *)(ybuf + o + nb) = make_float4(b[0], b[1], b[2], b[3]);
            ra[0] = p.x0.x + a[0]; ra[1] = p.x0.y + a[1]; ra[2] = p.x0.z + a[2]; ra[3] = p.x0.w + a[3];
            rb[0] = p.x1.x + b[0]; rb[1] = p.x1.y + b[1]; rb[2] = p.x1.z + b[2]; rb[3] = p.x1.w + b[3];
            pa[0] = ra[0] * p.ga.x; pa[1] = ra[1] * p.ga.y; pa[2] = ra[2] * p.ga.z; pa[3] = ra[3] * p.ga.w;
            pb[0] = rb[0] * p.gb.x; pb[1] = rb[1] * p.gb.y; pb[2] = rb[2] * p.gb.z; pb[3] = rb[3] * p.gb.w;
        }
        const bf16x4 xa = cvt4h(pa[0], pa[1], pa[2], pa[3]), xb = cvt4h(pb[0], pb[1], pb[2], pb[3]);
        // the pair's 32 features are k-tile `pair` of the next contraction
        const size_t fo = spd_act_index(mt, pair, h >> 5, (M + 15) >> 4);
        const int ea = spd_frag_elem(r, 4 * g), eb = spd_frag_elem(r, 16 + 4 * g);
        *(bf16x4 *)(xhat2 + fo + ea) = xa;
        *(bf16x4 *)(xhat2 + fo + eb) = xb;
        if (xlo2) {
            *(bf16x4 *)(xlo2 + fo + ea) = cvt4h_lo(pa[0], pa[1], pa[2], pa[3], xa);
            *(bf16x4 *)(xlo2 + fo + eb) = cvt4h_lo(pb[0], pb[1], pb[2], pb[3], xb);
        }
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) s += ra[i] * ra[i] + rb[i] * rb[i];
        s += shfl_xor_f(s, 16);
        s += shfl_xor_f(s, 32);
        if (g == 0) ss2[(size_t)pair * m_pad + m] = s;
    }
};

struct EpiGU {
    static constexpr bool kByElement = true;
    static constexpr bool kSync = false;
    static constexpr bool kLong = true;
    static constexpr bool kWideSum = false;
    static constexpr bool kNeedsRs = true;
    static constexpr bool kSliced = false;
    int M, h, f_pad, nch, m_pad;
    int cols = 16;             // FFN columns per group: 16, or fewer for the decode-only narrow groups
    float eps;
    const float *ss;
    const float *wsc;
    __bf16 *uhat, *ulo;        // ulo may be NULL
    struct Pre {
        float sc;
    };

    __device__ __forceinline__ Pre pre(int, int, int) const { return Pre{*wsc}; }

    // narrow groups: feature i of a lane is FFN column cols * pair + 4 g + i, stored by itself (operator() is for 16 columns; see launch_gemv())
    __device__ __forceinline__ bool by_element() const { return cols != 16; }
    __device__ __forceinline__ void element(int pair, int i, float a, float b, int lane, float rs, const Pre &p) const {
        const int r = lane & 15, row = 4 * (lane >> 4) + i, col = pair * cols + row;
        if (row >= cols || col >= f_pad) return;
        rs *= p.sc;
        const float gt = a * rs, up = b * rs;
        const float o = r < M ? gt / (1.0f + __expf(-gt)) * up : 0.f;
        const __bf16 u = act_one(o);
        const size_t fo = spd_act_index(0, col >> 5, f_pad >> 5, 1) + spd_frag_elem(r, col & 31);
        uhat[fo] = u;
        if (ulo) ulo[fo] = act_one(o - act_back(u));
    }

    __device__ __forceinline__ void operator()(int pair, int mt, f32x4 a, f32x4 b, int lane, float rs, const Pre &p) const {
        const int r = lane & 15, m = mt * 16 + r, g = lane >> 4;
        float o[4] = {0.f, 0.f, 0.f, 0.f};
        rs *= p.sc;
        if (m < M) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float gt = a[i] * rs, up = b[i] * rs;
                o[i] = gt / (1.0f + __expf(-gt)) * up;
            }
        }
        const bf16x4 u = cvt4h(o[0], o[1], o[2], o[3]);
        // gate/up pair p covers FFN columns [16p, 16p+16): half of k-tile p/2 of the down projection
        const size_t fo = spd_act_index(mt, pair >> 1, f_pad >> 5, (M + 15) >> 4) + spd_frag_elem(r, 16 * (pair & 1) + 4 * g);
        *(bf16x4 *)(uhat + fo) = u;
        if (ulo) *(bf16x4 *)(ulo + fo) = cvt4h_lo(o[0], o[1], o[2], o[3], u);
    }
};

template <bool FUSED>
struct EpiDownT {
    static constexpr bool kByElement = false;
    static constexpr bool kSync = FUSED;
    static constexpr bool kLong = !FUSED;
    static constexpr bool kWideSum = false;
    static constexpr bool kNeedsRs = false;
    static constexpr bool kSliced = false;
    int M, h, spd;
    const float *ybuf;
    float *slot;
    // optional: the sync point that ends the block, fused (one rank; the peers' partial sums are
    // inputs).  base == NULL: not fused.
    const float *base, *slots, *g1;
    const float *bias;         // [h] added once after the sum (SPD block with bias) or NULL
    const float *wsc;
    size_t slot_stride;
    int tp, rank, m_pad;
    float *x_out, *ss1;
    __bf16 *xhat, *xlo;        // next block's first-norm activations (xhat NULL: last block)
    __device__ __forceinline__ SyncSum sync() const { return SyncSum{slots, base, bias, slot_stride, tp, rank, M, h}; }
    __device__ __forceinline__ const float *joins_own() const { return spd ? ybuf : nullptr; }
    struct Pre {
        float4 ya, yb, ga, gb;
        float sc;
    };

    __device__ __forceinline__ Pre pre(int pair, int mt, int lane) const {
        Pre p;
        p.ya = p.yb = p.ga = p.gb = make_float4(0.f, 0.f, 0.f, 0.f);
        p.sc = *wsc;
        const int m = mt * 16 + (lane & 15), g = lane >> 4;
        if (FUSED && xhat) {
            p.ga = *(const float4 *)(g1 + pair * 32 + 4 * g);
            p.gb = *(const float4 *)(g1 + pair * 32 + 16 + 4 * g);
        }
        if (spd && m < M) {
            const size_t oa = (size_t)m * h + pair * 32 + 4 * g;
            p.ya = *(const float4 *)(ybuf + oa);
            p.yb = *(const float4 *)(ybuf + oa + 16);
        }
        return p;
    }

    template <class Peers = SyncNone>
    __device__ __forceinline__ void operator()(int pair, int mt, f32x4 a, f32x4 b, int lane, float, const Pre &p,
                                               const Peers &peers = Peers()) const {
        const int r = lane & 15, m = mt * 16 + r, g = lane >> 4;
        const bool valid = m < M;
        const size_t oa = (size_t)m * h + pair * 32 + 4 * g, ob = oa + 16;
        // SPD block: Y_r joins the partial sum before the sync point (Sec. 4.1.1); p.y* are zero otherwise
        float4 pa, pb;
        if constexpr (std::is_same<Peers, SyncDone>::value) {
            pa = __builtin_bit_cast(float4, peers.own[0]);
            pb = __builtin_bit_cast(float4, peers.own[64]);
        } else {
            a *= p.sc;
            b *= p.sc;
            pa = make_float4(a[0] + p.ya.x, a[1] + p.ya.y, a[2] + p.ya.z, a[3] + p.ya.w);
            pb = make_float4(b[0] + p.yb.x, b[1] + p.yb.y, b[2] + p.yb.z, b[3] + p.yb.w);
        }
        if (valid) {
            *(float4 *)(slot + oa) = pa;
            *(float4 *)(slot + ob) = pb;
        }
        if (!FUSED) return;
        float4 xa = make_float4(0.f, 0.f, 0.f, 0.f), xb = xa;
        if (valid) {
            // out = base + (slot_0 + slot_1 + ...), own partial standing in for slot `rank`: the same
            // order of additions as the stand-alone rank-sum
            sync().sum(peers, oa, pair * 32 + 4 * g, pa, pb, xa, xb);
            *(float4 *)(x_out + oa) = xa;
            *(float4 *)(x_out + ob) = xb;
        }
        if (!xhat) return;
        float qa[4] = {0.f, 0.f, 0.f, 0.f}, qb[4] = {0.f, 0.f, 0.f, 0.f};
        if (valid) {
            qa[0] = xa.x * p.ga.x; qa[1] = xa.y * p.ga.y; qa[2] = xa.z * p.ga.z; qa[3] = xa.w * p.ga.w;
            qb[0] = xb.x * p.gb.x; qb[1] = xb.y * p.gb.y; qb[2] = xb.z * p.gb.z; qb[3] = xb.w * p.gb.w;
        }
        const bf16x4 ha = cvt4h(qa[0], qa[1], qa[2], qa[3]), hb = cvt4h(qb[0], qb[1], qb[2], qb[3]);
        const size_t fo = spd_act_index(mt, pair, h >> 5, (M + 15) >> 4);
        const int ea = spd_frag_elem(r, 4 * g), eb = spd_frag_elem(r, 16 + 4 * g);
        *(bf16x4 *)(xhat + fo + ea) = ha;
        *(bf16x4 *)(xhat + fo + eb) = hb;
        if (xlo) {
            *(bf16x4 *)(xlo + fo + ea) = cvt4h_lo(qa[0], qa[1], qa[2], qa[3], ha);
            *(bf16x4 *)(xlo + fo + eb) = cvt4h_lo(qb[0], qb[1], qb[2], qb[3], hb);
        }
        float sq = xa.x * xa.x + xa.y * xa.y + xa.z * xa.z + xa.w * xa.w + xb.x * xb.x + xb.y * xb.y + xb.z * xb.z + xb.w * xb.w;
        sq += shfl_xor_f(sq, 16);
        sq += shfl_xor_f(sq, 32);
        if (g == 0) ss1[(size_t)pair * m_pad + m] = sq;
    }
};

// Epilogue of a K-sliced launch whose real epilogue is not linear: parks the tile pair's partial sums in
// kpart[pair][slice][m-tile] for k_mid_finish.
struct EpiPark {
    static constexpr bool kNeedsRs = false;
    static constexpr bool kSliced = true;
    int KS, n_mtiles;
    f32x4 *kpart;
    const float *ss = nullptr;
    int nch = 0, m_pad = 0, h = 0;
    float eps = 0.f;
    struct Pre {};
    __device__ __forceinline__ Pre pre(int, int, int) const { return Pre(); }
    __device__ __forceinline__ void slice(int pair, int ks, int mt, f32x4 a, f32x4 b, int lane, float, const Pre &) const {
        f32x4 *dst = kpart + ((((size_t)pair * KS + ks) * n_mtiles + mt) * 2) * 64 + lane;
        dst[0] = a;
        dst[64] = b;
    }
};

// ------------------------------------------------------------------------------------------
// Partial softmax states of a decode step's attention, one per (sequence, KV head = "unit"; split of the context; query head c of the
// group): d unnormalised sums, maximum and sum of the exponentials.  [unit][split][c][d] first, then [unit][split][2][c]: only the
// group's real heads (1 of an MFMA's 16 columns in multi-head attention), a head's features side by side.  (Whole tiles of 16 columns
// before: us per layer 70B 16 sequences of 4096 63.8 -> 62.6, 13B 8 of 4096 56.3 -> 54.8, 7B 1 of 2048 40.4 -> 38.8.)
// ------------------------------------------------------------------------------------------
struct AttnParts {
    float *o;
    int units, n_splits, group, d;
    Divider by_quads, by_heads, by_group;      // quads of features of a head; query heads of the rank; of a KV head
    __device__ __forceinline__ float *sums(int u, int split, int c) const { return o + (((size_t)u * n_splits + split) * group + c) * d; }
    __device__ __forceinline__ float *max_sum(int u, int split, int c) const {       // maximum; `group` floats further the sum
        return o + (size_t)units * n_splits * group * d + ((size_t)u * n_splits + split) * 2 * group + c;
    }
};
// CH splits of four features, requested together
template <int CH>
struct MergeLoads {
    float m[CH], l[CH];
    float4 o[CH];
    __device__ __forceinline__ void load(const AttnParts &P, int u, int c, int quad, int s0) {
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            const int sp = s0 + j < P.n_splits ? s0 + j : P.n_splits - 1;
            const float *ml = P.max_sum(u, sp, c);
            m[j] = ml[0];
            l[j] = ml[P.group];
            o[j] = *(const float4 *)(P.sums(u, sp, c) + 4 * quad);
        }
    }
};
// The merge of the splits in ascending order, CH at a time: the normalised output of four features.  `first` holds the first CH.
template <int CH>
__device__ __forceinline__ float4 merge_splits(const AttnParts &P, int u, int c, int quad, MergeLoads<CH> first) {
    float M = -INFINITY, den = 0.f;
    float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s0 = 0; s0 < P.n_splits; s0 += CH) {
        if (s0) first.load(P, u, c, quad, s0);
        float mc = M;
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            if (s0 + j >= P.n_splits) {
                first.m[j] = -INFINITY;
                first.l[j] = 0.f;
            }
            mc = fmaxf(mc, first.m[j]);
        }
        const float keep = (M == -INFINITY) ? 0.f : __expf(M - mc);
        num.x *= keep; num.y *= keep; num.z *= keep; num.w *= keep;
        den *= keep;
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            // (a split without keys; one whose keys all have no score, NaN, has this maximum too, and its sums are NaN)
            if (first.m[j] == -INFINITY && first.l[j] == 0.f) continue;
            const float sc = __expf(first.m[j] - mc);
            num.x += first.o[j].x * sc; num.y += first.o[j].y * sc; num.z += first.o[j].z * sc; num.w += first.o[j].w * sc;
            den += first.l[j] * sc;
        }
        M = mc;
    }
    return make_float4(num.x / den, num.y / den, num.z / den, num.w / den);
}

// ------------------------------------------------------------------------------------------
// GEMV-like projection for at most 16 tokens (one m-tile): bound by streaming the weights.
//   out^T[n][m] = sum_k W[k][n] x[m][k]
// grid = (pairs of n-tiles, KS).  A workgroup owns one pair and one of KS slices of K; its W
// waves split that slice, each wave streaming its weight fragments straight from HBM into
// registers, four k-tiles in flight while a fifth feeds the MFMAs (70B shard, 16 tokens, us, the ring against two sets of two k-tiles
// that the compiler had put back into one: gate/up 22.4 / 21.3, down 13.7 / 13.0, QKV 7.6 / 7.2; 3, 4, 6 and 8 sets: gate/up 22.0,
// 21.9, 21.6, 21.7; four more with no memory access past the end instead of a branch: 23.0, every load of zeros
// takes its turn).  What the epilogue reads besides, the peers' partial sums above all, is requested in the same breath
// (down 13.0 -> 12.5).  The rest of a small launch is latency: 2 us to start, one trip to the memory, the
// sum over the waves.  The waves' partial tiles are added through LDS in wave order.  With KS = 1 the first
// wave then runs the epilogue; with KS > 1 and MODE 1 the workgroup parks its tile in `kpart`
// and k_gemv_finish adds the KS tiles in slice order: sums never depend on timing.  MODE 2 is
// for epilogues that are linear in the accumulators: every slice runs Epi::slice() on its own
// partial sums and the consumer of the result adds the slices.
// ------------------------------------------------------------------------------------------
// A wave's walk over its n k-tiles with a ring of NB register sets: the loads of NB - 1 k-tiles are in flight while one is
// multiplied.  The scheduling barriers are what makes it so: without them the compiler puts a set's loads after the
// MFMAs of the one before and directly in front of their own.  The steady state has no branch between the loads and their use,
// otherwise the compiler's counts of what is in flight assume the worst (it may, for the last few).  `between` runs once, after the first loads.
#define SPD_SCHED_BARRIER() __builtin_amdgcn_sched_barrier(0)
template <int NB, class Set, class Load, class Use, class Between>
__device__ __forceinline__ void stream_tiles(int n, const Load &load, const Use &use, const Between &between) {
    Set R[NB];
    if (n < NB) {                            // everything is requested at once
#pragma unroll
        for (int j = 0; j < NB - 1; ++j)
            if (j < n) load(R[j], j);
        SPD_SCHED_BARRIER();
        between();
        SPD_SCHED_BARRIER();
#pragma unroll
        for (int j = 0; j < NB - 1; ++j)
            if (j < n) use(R[j]);
        return;
    }
#pragma unroll
    for (int j = 0; j < NB - 1; ++j) load(R[j], j);
    SPD_SCHED_BARRIER();
    between();
    SPD_SCHED_BARRIER();
    int i = 0;
    for (; i + 2 * NB - 1 <= n; i += NB) {
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            load(R[(j + NB - 1) % NB], i + j + NB - 1);
            SPD_SCHED_BARRIER();
            use(R[j]);
            SPD_SCHED_BARRIER();
        }
    }
    const int left = n - i;                  // NB - 1 of them are on their way: NB - 1 <= left < 2 NB - 1
#pragma unroll
    for (int j = 0; j < NB - 1; ++j) {
        if (j + NB - 1 < left) load(R[(j + NB - 1) % NB], i + j + NB - 1);
        SPD_SCHED_BARRIER();
        use(R[j]);
        SPD_SCHED_BARRIER();
    }
#pragma unroll
    for (int j = NB - 1; j < 2 * NB - 2; ++j)
        if (j < left) use(R[j % NB]);
}
// 16 bytes per lane at p + off of the `bytes` bytes from the wave-uniform address p on (zeros past them).  A buffer load: the
// address stays in scalar registers.  STREAM: data that is read once.
template <bool STREAM>
__device__ __forceinline__ bf16x8 frag(const char *p, unsigned bytes, unsigned off) {
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, (int)bytes, 0x00020000);
    return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, STREAM ? 2 : 0));
}

template <bool SPLIT>
struct GemvSet {
    bf16x8 fa, fb, fh, fl;      // fl: SPLIT only
    static constexpr int kRing = SPLIT ? 3 : 5;      // (16 waves: 128 registers each)
};

// SRC_MERGE: the input is the attention's output, merged here from the splits' states: every workgroup merges all of it, a thread
// four features of a (token, head), into fragments in LDS while its weights are on their way.  SRC_MERGE3: up to three such quads per thread and
// 8 splits; the splits' factors of a (token, head) and their sum are computed once, by one thread, and go through LDS.  The arithmetic is
// k_attn_combine's for as many splits, operation for operation.
// SRC_X: the input is the residual stream itself, the first norm's elementwise part done on the way; every slice leaves its sums of squares
// in ss[slice][16], and whoever adds the slices applies the factor.
struct NoParts {};
struct RawX {
    const float *x, *gain;
    float *ss;
};
struct GemvSetX {
    bf16x8 fa, fb;
    float4 x0, x1, g0, g1;
};
constexpr int GEMV_MERGE_TILES = 5;      // k-tiles per wave
enum { SRC_PACKED, SRC_MERGE, SRC_X, SRC_MERGE3 };
template <int SRC> struct GemvSrc { typedef NoParts type; };
template <> struct GemvSrc<SRC_MERGE> { typedef AttnParts type; };
template <> struct GemvSrc<SRC_MERGE3> { typedef AttnParts type; };
template <> struct GemvSrc<SRC_X> { typedef RawX type; };
template <int W, bool SPLIT, int MODE, class Epi, int SRC = SRC_PACKED>     // MODE 0: whole K, 1: slices -> kpart, 2: slices -> Epi::slice
__global__ void __launch_bounds__(W * 64) k_gemv(const __bf16 *__restrict__ Wp, const __bf16 *__restrict__ Xhi,
                                                  const __bf16 *__restrict__ Xlo, int KT, int KS,
                                                  float *__restrict__ kpart, int rows, Epi epi,
                                                  typename GemvSrc<SRC>::type parts) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int pair = blockIdx.x, ks = blockIdx.y;
    const int kb0 = MODE == 0 ? 0 : part_of(ks, KT, KS), kb1 = MODE == 0 ? KT : part_of(ks + 1, KT, KS);
    const int nk = kb1 - kb0;
    const int k0 = kb0 + (int)((unsigned)(wave * nk) / W), k1 = kb0 + (int)((unsigned)((wave + 1) * nk) / W);
    f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = {0.f, 0.f, 0.f, 0.f};
    // rows == 16: two n-tiles of 1 KiB fragments.  rows < 16 (narrow groups of the decode-only
    // gate/up copy): per k-tile `rows` rows of the first tile then `rows` rows of the second, 16
    // bytes per row and quarter of the k-tile; the lanes of the missing rows repeat the last row
    // (same cache lines; the epilogue does not store them).
    // (wave-uniform addresses plus a lane's offset: the loads need no vector registers for addresses)
    const char *wa, *wb;
    unsigned wlane, kstr;        // a lane's offset, distance between k-tiles, in bytes
    if (rows == 16) {
        wa = (const char *)(Wp + spd_frag_index(2 * pair, 0, KT));
        wb = (const char *)(Wp + spd_frag_index(2 * pair + 1, 0, KT));
        wlane = lane * 16;
        kstr = 1024;
    } else {
        const int rr = (lane & 15) < rows ? (lane & 15) : rows - 1;
        wa = (const char *)Wp + (size_t)pair * KT * 128 * rows;
        wb = wa + 64 * rows;
        wlane = ((lane >> 4) * rows + rr) * 16;
        kstr = 128 * rows;
    }
    const char *xh = (const char *)Xhi, *xl = (const char *)Xlo;
    const unsigned xlane = lane * 16;

    auto load = [&](GemvSet<SPLIT> &B, int i) {
        const size_t kt = k0 + i;
        const unsigned wn = 64 * rows, xn = 1024;
        B.fa = frag<true>(wa + kt * kstr, wn, wlane);
        B.fb = frag<true>(wb + kt * kstr, wn, wlane);
        B.fh = frag<false>(xh + kt * 1024, xn, xlane);
        if (SPLIT) B.fl = frag<false>(xl + kt * 1024, xn, xlane);
    };
    auto consume = [&](const GemvSet<SPLIT> &B) {
        a = MFMA16(B.fa, B.fh, a);
        b = MFMA16(B.fb, B.fh, b);
        if (SPLIT) {
            a = MFMA16(B.fa, B.fl, a);
            b = MFMA16(B.fb, B.fl, b);
        }
    };

    // every wave walks its share of K front to back (measured: any other order, e.g. one rotated
    // per workgroup to spread the activation reads, costs a fifth of the streaming rate)
    typename Epi::Pre pre;
    SsLoads ssl;
    constexpr bool PARTIAL = MODE == 1, EARLY = Epi::kSync && MODE == 0;
    f32x4 sla = {0.f, 0.f, 0.f, 0.f}, slb = sla, bsa = sla, bsb = sla;
    float el_y = 0.f, el_b = 0.f, el_sc = 1.f;
    auto between = [&]() {
        // loads that do not depend on the stream: the epilogue's inputs (first wave) and this wave's
        // share of the sum-of-squares partials, issued while the first weights are on their way
        if (!PARTIAL) {
            if (wave == 0 || (Epi::kByElement && wave < 4)) pre = epi.pre(pair, 0, lane);
            if constexpr (EARLY) {
                // wave s takes slot s, the own slot's wave the base
                const SyncSum sy = epi.sync();
                if (wave < SYNC_EARLY) {
                    const int sl = wave < sy.tp ? wave : sy.tp - 1;
                    const float *p = (sl == sy.rank ? sy.base : sy.slots + (size_t)sl * sy.slot_stride) + sy.at(pair, 0, lane);
                    sla = *(const f32x4 *)p;
                    slb = *(const f32x4 *)(p + 16);
                }
                if (sy.rank >= SYNC_EARLY && wave == 0) {
                    const float *p = sy.base + sy.at(pair, 0, lane);
                    bsa = *(const f32x4 *)p;
                    bsb = *(const f32x4 *)(p + 16);
                }
                if (threadIdx.x < 512 && sy.tp <= SYNC_EARLY) {
                    if (epi.joins_own()) el_y = epi.joins_own()[sy.at_element(pair, threadIdx.x)];
                    if (sy.bias) el_b = sy.bias[sy.col(pair, threadIdx.x)];
                    el_sc = *epi.wsc;
                }
            }
            if constexpr (Epi::kNeedsRs && SRC != SRC_X) {
                ssl.load(epi.ss, epi.nch, epi.m_pad, lane & 15, wave * 4 + (lane >> 4), W * 4);
            }
        }
    };
    float xsq = 0.f;
    if constexpr (SRC == SRC_PACKED) {
        stream_tiles<GemvSet<SPLIT>::kRing, GemvSet<SPLIT>>(k1 - k0, load, consume, between);
    } else if constexpr (SRC == SRC_X) {
        static_assert(!SPLIT && MODE == 2, "raw input: one plane, K slices");
        const int m = (lane & 15) < epi.M ? (lane & 15) : epi.M - 1;           // (rows past the call: its last one)
        const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc((void *)parts.x, 0, epi.M * epi.h * 4, 0x00020000),
                                     gbuf = __builtin_amdgcn_make_buffer_rsrc((void *)parts.gain, 0, epi.h * 4, 0x00020000);
        const int grow = (lane >> 4) * 32, xrow = m * epi.h * 4 + grow;
        auto at = [](__amdgpu_buffer_rsrc_t r, int off, int soff) {
            return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, 0));
        };
        auto loadx = [&](GemvSetX &B, int i) {
            const int kt = k0 + i;
            B.fa = frag<true>(wa + (size_t)kt * kstr, 64 * rows, wlane);
            B.fb = frag<true>(wb + (size_t)kt * kstr, 64 * rows, wlane);
            B.x0 = at(xbuf, xrow, kt * 128);
            B.x1 = at(xbuf, xrow + 16, kt * 128);
            B.g0 = at(gbuf, grow, kt * 128);
            B.g1 = at(gbuf, grow + 16, kt * 128);
        };
        auto usex = [&](const GemvSetX &B) {
            const bf16x4 lo = mul4h(B.x0, B.g0), hi = mul4h(B.x1, B.g1);      // (as k_prep rounds them)
            const bf16x8 f = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            a = MFMA16(B.fa, f, a);
            b = MFMA16(B.fb, f, b);
            xsq += B.x0.x * B.x0.x + B.x0.y * B.x0.y + B.x0.z * B.x0.z + B.x0.w * B.x0.w;
            xsq += B.x1.x * B.x1.x + B.x1.y * B.x1.y + B.x1.z * B.x1.z + B.x1.w * B.x1.w;
        };
        // (two or three k-tiles per wave, mostly: everything at once; a ring of this much per k-tile spills)
        constexpr int NB = 3;
        GemvSetX R[NB];
        const int n = k1 - k0;
        for (int i = 0; i < n || i == 0; i += NB) {
#pragma unroll
            for (int j = 0; j < NB; ++j)
                if (i + j < n) loadx(R[j], i + j);
            SPD_SCHED_BARRIER();
            if (i == 0) between();
            SPD_SCHED_BARRIER();
#pragma unroll
            for (int j = 0; j < NB; ++j)
                if (i + j < n) usex(R[j]);
        }
    } else {
        static_assert(!SPLIT && MODE == 0, "merged input: one plane, whole K");
        extern __shared__ __attribute__((aligned(16))) char merged[];          // [KT] fragments (rows past the call: anything)
        constexpr bool ONE = SRC == SRC_MERGE;
        constexpr int CH = ONE ? 16 : 8, NI = ONE ? 1 : 3;
        // (states first: what returns in order behind them may take its time)
        const int per_tok = KT * 8, n_items = epi.M * per_tok, heads = parts.by_heads.d;
        auto unit = [&](int th) { return parts.by_group.div(th); };                // of (token, head) th: KV heads have whole groups
        auto column = [&](int th) { return parts.by_group.mod(th); };
        auto th_of = [&](int item) { return parts.by_quads.div(item); };           // an item: four features of a (token, head)
        MergeLoads<CH> L;
        float4 o[ONE ? 1 : NI][CH];
        const int e = min((int)threadIdx.x, n_items - 1), n_th = epi.M * heads;
        __shared__ __attribute__((aligned(16))) float fac[ONE ? 1 : W * 64][CH];
        __shared__ float2 dens[ONE ? 1 : W * 64];
        if constexpr (ONE) {
            L.load(parts, unit(th_of(e)), column(th_of(e)), parts.by_quads.mod(e), 0);
        } else {
            const int th = min((int)threadIdx.x, n_th - 1);
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                const float *ml = parts.max_sum(unit(th), min(j, parts.n_splits - 1), column(th));
                L.m[j] = ml[0];
                L.l[j] = ml[parts.group];
            }
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int ei = min(e + i * W * 64, n_items - 1);
#pragma unroll
                for (int j = 0; j < CH; ++j)
                    o[i][j] = *(const float4 *)(parts.sums(unit(th_of(ei)), min(j, parts.n_splits - 1), column(th_of(ei))) + 4 * parts.by_quads.mod(ei));
            }
        }
        SPD_SCHED_BARRIER();
        GemvSet<false> R[GEMV_MERGE_TILES];
        const int n = k1 - k0;
#pragma unroll
        for (int j = 0; j < GEMV_MERGE_TILES; ++j) {
            const size_t kt = k0 + (j < n ? j : 0);                            // (a wave's first k-tile again, not used)
            R[j].fa = frag<true>(wa + (n > 0 ? kt : 0) * kstr, 64 * rows, wlane);
            R[j].fb = frag<true>(wb + (n > 0 ? kt : 0) * kstr, 64 * rows, wlane);
        }
        SPD_SCHED_BARRIER();
        between();
        SPD_SCHED_BARRIER();
        auto put = [&](int item, float4 v) {
            const int tok = parts.by_heads.div(th_of(item)), k = 4 * (item - tok * per_tok);
            *(bf16x4 *)(merged + (k >> 5) * 1024 + 2 * spd_frag_elem(tok, k & 31)) = cvt4h(v.x, v.y, v.z, v.w);
        };
        if constexpr (ONE) {
            if ((int)threadIdx.x < n_items) put(e, merge_splits<CH>(parts, unit(th_of(e)), column(th_of(e)), parts.by_quads.mod(e), L));
        } else {
            float mc = -INFINITY, den = 0.f;
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                if (j >= parts.n_splits) L.m[j] = -INFINITY;
                mc = fmaxf(mc, L.m[j]);
            }
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                L.m[j] = L.m[j] == -INFINITY ? 0.f : __expf(L.m[j] - mc);
                den += L.l[j] * L.m[j];
            }
            if ((int)threadIdx.x < n_th) {
#pragma unroll
                for (int j = 0; j < CH; ++j) fac[threadIdx.x][j] = L.m[j];
                dens[threadIdx.x] = make_float2(den, 1.0f / den);
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int ei = (int)threadIdx.x + i * W * 64;
                if (ei >= n_items) break;
                float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (int j = 0; j < CH; ++j) {
                    const float f = fac[th_of(ei)][j];
                    v.x += o[i][j].x * f; v.y += o[i][j].y * f; v.z += o[i][j].z * f; v.w += o[i][j].w * f;
                }
                // v / den as a division rounds it: the quotient by the reciprocal, corrected by its remainder
                const float2 dn = dens[th_of(ei)];
                auto quotient = [&](float n) {
                    const float q = n * dn.y, r = __builtin_fmaf(-dn.x, q, n);
                    return __builtin_isfinite(q) ? __builtin_fmaf(r, dn.y, q) : q;
                };
                put(ei, make_float4(quotient(v.x), quotient(v.y), quotient(v.z), quotient(v.w)));
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < GEMV_MERGE_TILES; ++j)
            if (j < n) {
                R[j].fh = *(const bf16x8 *)(merged + (k0 + j) * 1024 + lane * 16);
                consume(R[j]);
            }
    }
    __shared__ f32x4 red[W][2][64];
    __shared__ float red_ss[W][64];
    __shared__ f32x4 peers[EARLY ? SYNC_EARLY + 1 : 1][2][64], xsum[EARLY ? 2 : 1][64];
    red[wave][0][lane] = a;
    red[wave][1][lane] = b;
    if constexpr (SRC == SRC_X) red_ss[wave][lane] = xsq;
    else if constexpr (Epi::kNeedsRs && !PARTIAL) red_ss[wave][lane] = ssl.sum(epi.ss, epi.nch, epi.m_pad, lane & 15, wave * 4 + (lane >> 4), W * 4);
    if constexpr (EARLY) {
        if (wave < SYNC_EARLY) {
            peers[wave][0][lane] = sla;
            peers[wave][1][lane] = slb;
        }
        if (wave == 0) {
            peers[SYNC_EARLY][0][lane] = bsa;
            peers[SYNC_EARLY][1][lane] = bsb;
        }
    }
    __syncthreads();
    // Eight waves add an element a thread over the waves (in place: nobody else reads that column), and one the sums of squares; by the first
    // wave alone these were half of the 400 instructions behind the last weights.
    static_assert(W >= 8, "an element a thread");
    {
        float *sum = (float *)&red[0][0][0] + threadIdx.x;
        if (threadIdx.x < 512) {
            float v = sum[0];
#pragma unroll
            for (int w = 1; w < W; ++w) v += sum[w * 512];
            if (PARTIAL) {
                kpart[((size_t)pair * KS + ks) * 512 + threadIdx.x] = v;
                return;
            }
            if constexpr (EARLY) {
                const SyncSum sy = epi.sync();
                if (sy.tp <= SYNC_EARLY) {
                    v = epi.joins_own() ? v * el_sc + el_y : v * el_sc;
                    ((float *)xsum)[threadIdx.x] = sy.element((const float *)peers, threadIdx.x, v, el_b);
                }
            }
            sum[0] = v;
        }
        if (PARTIAL) return;
    }
    if constexpr (Epi::kNeedsRs) {
        if (wave == W - 1) {
            float sq = red_ss[0][lane];
#pragma unroll
            for (int w = 1; w < W; ++w) sq += red_ss[w][lane];
            sq += shfl_xor_f(sq, 16);
            sq += shfl_xor_f(sq, 32);
            if constexpr (SRC == SRC_X) {
                if (pair == 0 && lane < 16) parts.ss[ks * 16 + lane] = sq;
            } else {
                red_ss[0][lane] = 1.0f / sqrtf(sq / (float)epi.h + epi.eps);
            }
        }
    }
    __syncthreads();
    const float rs = Epi::kNeedsRs && SRC != SRC_X ? red_ss[0][lane] : 1.f;
    if constexpr (Epi::kByElement) {
        if (epi.by_element()) {          // a wave takes one of the four features of every lane
            const float *sum = (const float *)&red[0][0][0] + lane * 4 + wave;
            if (wave < 4) epi.element(pair, wave, sum[0], sum[256], lane, rs, pre);
            return;
        }
    }
    if (wave != 0) return;
    a = red[0][0][lane];
    b = red[0][1][lane];
    if constexpr (MODE == 2) {
        epi.slice(pair, ks, 0, a, b, lane, rs, pre);
    } else if constexpr (EARLY) {
        if (epi.sync().tp <= SYNC_EARLY) epi(pair, 0, a, b, lane, rs, pre, SyncDone{&red[0][0][lane], &xsum[0][lane]});
        else epi(pair, 0, a, b, lane, rs, pre, SyncLds{&peers[0][0][lane], epi.sync().rank});
    } else {
        epi(pair, 0, a, b, lane, rs, pre);
    }
}

// Adds the KS partial tiles of a pair in slice order and runs the epilogue.  grid = pairs,
// 4 waves: wave w adds the slices s = w, w+4, ...; the four sums are then added in wave order.
template <class Epi>
__global__ void __launch_bounds__(256) k_gemv_finish(const float *__restrict__ kpart, int KS, Epi epi) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int pair = blockIdx.x;
    typename Epi::Pre pre;
    if (wave == 0) pre = epi.pre(pair, 0, lane);
    f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = wave; s0 < KS; s0 += 16) {
        f32x4 ta[4], tb[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int sl = s0 + 4 * j;
            if (sl < KS) {
                const float *src = kpart + ((size_t)pair * KS + sl) * 512 + lane * 4;
                ta[j] = *(const f32x4 *)src;
                tb[j] = *(const f32x4 *)(src + 256);
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (s0 + 4 * j < KS) {
                a += ta[j];
                b += tb[j];
            }
    }
    float ssp = 0.f;
    if constexpr (Epi::kNeedsRs) {
        ssp = sum_ss(epi.ss, epi.nch, epi.m_pad, lane & 15, wave * 4 + (lane >> 4), 16);
    }
    __shared__ f32x4 red[4][2][64];
    __shared__ float red_ss[4][64];
    red[wave][0][lane] = a;
    red[wave][1][lane] = b;
    red_ss[wave][lane] = ssp;
    __syncthreads();
    if (wave != 0) return;
#pragma unroll
    for (int w = 1; w < 4; ++w) {
        a += red[w][0][lane];
        b += red[w][1][lane];
    }
    float rs = 1.f;
    if constexpr (Epi::kNeedsRs) {
        float sq = red_ss[0][lane];
#pragma unroll
        for (int w = 1; w < 4; ++w) sq += red_ss[w][lane];
        sq += shfl_xor_f(sq, 16);
        sq += shfl_xor_f(sq, 32);
        rs = 1.0f / sqrtf(sq / (float)epi.h + epi.eps);
    }
    epi(pair, 0, a, b, lane, rs, pre);
}

// ------------------------------------------------------------------------------------------
// Projection for 17 .. 16*MT tokens per workgroup ("skinny": still bound by streaming the weights); fp16 operands.
// Like k_gemv, one workgroup per pair of n-tiles and slice of K, the W waves
// splitting K; every wave multiplies each weight fragment it streams with MT m-tiles of
// activations (read through the L2, where they stay resident).  grid = (pairs, KS, groups of MT
// m-tiles).  The W x MT partial tile pairs meet in LDS; wave w finishes m-tiles w, w + W, ...
//   MODE 0: whole K (KS = 1), Epi::operator();  MODE 2: K slices, Epi::slice (linear epilogues)
// ------------------------------------------------------------------------------------------
template <int MT, bool SPLIT, int NP>
struct SkinnySet {
    bf16x8 fa[NP], fb[NP], fh[MT], fl[SPLIT ? MT : 1];
    static constexpr int kRing = MT == 2 ? (SPLIT ? 3 : 4) : 2;      // (three or four sets of 8 m-tiles: 70B 128 tokens 103 -> 124, 136 us)
};

// NP pairs of n-tiles per workgroup: 1, or 2 with 4 m-tiles (see launch_skinny()).  KEEP: the weights stay in the L2 for the other groups of m-tiles
template <int W, int MT, bool SPLIT, int MODE, class Epi, int NP = 1, bool KEEP = false>
__global__ void __launch_bounds__(W * 64) k_skinny(const __bf16 *__restrict__ Wp, const __bf16 *__restrict__ Xhi,
                                                    const __bf16 *__restrict__ Xlo, int KT, int KS, int n_mtiles, unsigned rot_step, Epi epi) {
    extern __shared__ __attribute__((aligned(16))) char sk_lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int pair0 = blockIdx.x * NP, ks = blockIdx.y, mt0 = blockIdx.z * MT;
    const int kb0 = MODE == 0 ? 0 : part_of(ks, KT, KS), kb1 = MODE == 0 ? KT : part_of(ks + 1, KT, KS);
    const int nk = kb1 - kb0;
    const int k0 = kb0 + (int)((unsigned)(wave * nk) / W), k1 = kb0 + (int)((unsigned)((wave + 1) * nk) / W);
    f32x4 acc[NP][MT][2];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int i = 0; i < MT; ++i) acc[p][i][0] = acc[p][i][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const char *wa = (const char *)(Wp + spd_frag_index(2 * pair0, 0, KT));
    const size_t wrow = (size_t)KT * 1024;             // bytes between two n-tiles
    // (MT divides a group's 8 m-tiles; m-tiles past the call's last one are zeros)
    const char *xh = (const char *)(Xhi + spd_act_index(mt0, 0, KT, n_mtiles)), *xl = (const char *)(Xlo + spd_act_index(mt0, 0, KT, n_mtiles));
    const unsigned xstr = 1024u * spd_act_width(mt0, n_mtiles), xlen = spd_act_bytes(mt0, n_mtiles), l16 = lane * 16;
    const int n = k1 - k0;
    // Each workgroup starts at its own k-tile (rot_step, see launch_skinny_mt()), so that an XCD's compute units don't all ask
    // one L2 channel for the same activations.
    const int rot = n > 0 ? (int)(blockIdx.x * rot_step % (unsigned)n) : 0;
    auto load = [&](SkinnySet<MT, SPLIT, NP> &B, int q) {
        const unsigned wn = 1024, xn = xlen;
        q += rot;
        const size_t kt = k0 + (q >= n ? q - n : q);
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            B.fa[p] = frag<!KEEP>(wa + 2 * p * wrow + kt * 1024, wn, l16);
            B.fb[p] = frag<!KEEP>(wa + (2 * p + 1) * wrow + kt * 1024, wn, l16);
        }
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            B.fh[i] = frag<false>(xh + kt * xstr, xn, l16 + i * 1024);
            if (SPLIT) B.fl[i] = frag<false>(xl + kt * xstr, xn, l16 + i * 1024);
        }
    };
    auto consume = [&](const SkinnySet<MT, SPLIT, NP> &B) {
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                acc[p][i][0] = MFMA16(B.fa[p], B.fh[i], acc[p][i][0]);
                acc[p][i][1] = MFMA16(B.fb[p], B.fh[i], acc[p][i][1]);
                if (SPLIT) {
                    acc[p][i][0] = MFMA16(B.fa[p], B.fl[i], acc[p][i][0]);
                    acc[p][i][1] = MFMA16(B.fb[p], B.fl[i], acc[p][i][1]);
                }
            }
    };
    // the norm statistics by all threads while the first weights are on their way: at the end, a wave per m-tile, they were
    // eight dependent rounds of loads for 256 partials per token
    __shared__ float early_ss[Epi::kNeedsRs ? W * 64 : 1];
    constexpr int RS_PARTS = W * 4 / MT;               // threads per token
    // wave w finishes m-tile w % MT of pair w / MT: what its epilogue reads is requested now
    static_assert(NP * MT <= W, "a wave per m-tile and pair");
    const int pair = pair0 + wave / MT, wmt = mt0 + wave % MT;
    const bool fin = wave < NP * MT && wmt < n_mtiles;
    typename Epi::Pre pre;
    constexpr bool EARLY = Epi::kSync && !(SPLIT && MT == 8);      // (the registers for 8 m-tiles of pairs are all taken)
    SyncRegs peers;
    stream_tiles<SkinnySet<MT, SPLIT, NP>::kRing, SkinnySet<MT, SPLIT, NP>>(n, load, consume, [&]() {
        if (fin) pre = epi.pre(pair, wmt, lane);
        if constexpr (EARLY) {
            const SyncSum sy = epi.sync();
            if (fin) sy.load(peers, sy.at(pair, wmt, lane));
        }
        if constexpr (Epi::kNeedsRs) {
            int m = mt0 * 16 + (int)threadIdx.x % (MT * 16);
            m = m < n_mtiles * 16 ? m : n_mtiles * 16 - 1;
            early_ss[threadIdx.x] = sum_ss(epi.ss, epi.nch, epi.m_pad, m, (int)threadIdx.x / (MT * 16), RS_PARTS);
        }
    });
    f32x4 *red = (f32x4 *)sk_lds;        // [W][NP * MT][2][64]
    constexpr int NT = NP * MT;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        red[((wave * NT + t) * 2 + 0) * 64 + lane] = acc[t / MT][t % MT][0];
        red[((wave * NT + t) * 2 + 1) * 64 + lane] = acc[t / MT][t % MT][1];
    }
    __syncthreads();
    if (!fin) return;
    const int t = wave, mt = wmt;
    f32x4 a = red[((0 * NT + t) * 2 + 0) * 64 + lane], b = red[((0 * NT + t) * 2 + 1) * 64 + lane];
#pragma unroll
    for (int w = 1; w < W; ++w) {
        a += red[((w * NT + t) * 2 + 0) * 64 + lane];
        b += red[((w * NT + t) * 2 + 1) * 64 + lane];
    }
    float rs = 1.f;
    if constexpr (Epi::kNeedsRs) {
        float q = 0.f;
#pragma unroll
        for (int part = 0; part < RS_PARTS; ++part) q += early_ss[part * MT * 16 + t % MT * 16 + (lane & 15)];
        rs = 1.0f / sqrtf(q / (float)epi.h + epi.eps);
    }
    if constexpr (MODE == 2) epi.slice(pair, ks, mt, a, b, lane, rs, pre);
    else if constexpr (EARLY) epi(pair, mt, a, b, lane, rs, pre, peers);
    else epi(pair, mt, a, b, lane, rs, pre);
}

// ------------------------------------------------------------------------------------------
// Projection with many n-tiles for 17 .. 128 tokens ("mid").  In k_skinny every workgroup pulls all
// activations of its slice of K through the L2 for only two n-tiles, and from about 64 tokens on
// that traffic (K x M x 2 B per workgroup), not the weight stream, sets the time.  Here a
// workgroup owns 8 pairs of n-tiles (wave w: pair 8 * group + w) and one of KS slices of K; all
// waves walk the same k-tiles, so the activation fragments of a stage (MID_KB k-tiles x MT
// m-tiles) are fetched once per workgroup, by one wave each, and shared through LDS, while each
// wave streams its own weight fragments HBM -> registers.  Loads run three stages ahead of the
// MFMAs in a ring of four register sets; the steady-state loop has no branch (stages past the
// slice's end repeat its last one and are never consumed).  Workgroups start their slice at
// different stages (a rotation), otherwise all of them hit the same memory channels together.
// K is cut into slices because 8 pairs per workgroup leave too few workgroups: the partial tiles go
// to `kpart` [pair][slice][m-tile] and k_mid_finish adds them in slice order and runs the epilogue.
// ------------------------------------------------------------------------------------------
constexpr int MID_KB = 2;        // k-tiles per stage
constexpr int MID_PAIRS = 8;     // pairs of n-tiles per workgroup (one per wave)
template <int MT>
struct MidSet {
    bf16x8 wa[MID_KB], wb[MID_KB], x[MT >= 4 ? MT / 4 : 1];
};

template <int MT>
__global__ void __launch_bounds__(MID_PAIRS * 64) k_mid(const __bf16 *__restrict__ Wp, const __bf16 *__restrict__ Xp, int KT, int KS, int n_pairs,
                                                        int n_mtiles, f32x4 *__restrict__ kpart) {
    // activation fragments of a stage fetched by one wave (with 2 m-tiles there are only 4 fragments: waves
    // 4 .. 7 fetch and store the same ones again, which keeps the loop free of branches)
    constexpr int XPW = MT >= 4 ? MT / 4 : 1, NFRAG = MT * MID_KB;
    __shared__ __attribute__((aligned(1024))) char lds[2 * NFRAG * 1024];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int pair = blockIdx.x * MID_PAIRS + wave;
    const bool live = pair < n_pairs;
    if (!live) pair = n_pairs - 1;        // a spare wave repeats the last pair and drops the result
    const int ks = blockIdx.y;
    const int nst = (KT + MID_KB - 1) / MID_KB;                  // stages in all of K
    const int sb0 = part_of(ks, nst, KS), sb1 = part_of(ks + 1, nst, KS);
    const int ns = sb1 - sb0;                                    // >= 1: the launcher keeps KS <= nst
    const int rot = (int)((blockIdx.x * 5u + blockIdx.y * 3u) % (unsigned)ns);
    auto stage_of = [&](int st) {
        st = st < ns ? st : ns - 1;
        st += rot;
        return sb0 + (st >= ns ? st - ns : st);
    };
    const bf16x8 *wa = (const bf16x8 *)(Wp + spd_frag_index(2 * pair, 0, KT)) + lane;
    const bf16x8 *wb = (const bf16x8 *)(Wp + spd_frag_index(2 * pair + 1, 0, KT)) + lane;
    size_t xoff[XPW];
#pragma unroll
    for (int i = 0; i < XPW; ++i) {
        const int mt = ((wave * XPW + i) % NFRAG) / MID_KB;
        xoff[i] = spd_act_index(mt < n_mtiles ? mt : n_mtiles - 1, 0, KT, n_mtiles) + (size_t)lane * 8;
    }
    f32x4 acc[MT][2];
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[m][0] = acc[m][1] = (f32x4){0.f, 0.f, 0.f, 0.f};

    auto load = [&](MidSet<MT> &S, int st) {
        const int kt0 = stage_of(st) * MID_KB;
#pragma unroll
        for (int i = 0; i < XPW; ++i) {
            const int kt = kt0 + ((wave * XPW + i) % NFRAG) % MID_KB;
            const size_t o = xoff[i] + (size_t)(kt < KT ? kt : KT - 1) * n_mtiles * SPD_FRAG_ELEMS;      // (one group)
            S.x[i] = *(const bf16x8 *)(Xp + o);
        }
#pragma unroll
        for (int kb = 0; kb < MID_KB; ++kb) {
            const int kt = kt0 + kb < KT ? kt0 + kb : KT - 1;
            S.wa[kb] = __builtin_nontemporal_load(wa + (size_t)kt * 64);
            S.wb[kb] = __builtin_nontemporal_load(wb + (size_t)kt * 64);
        }
    };
    auto put = [&](const MidSet<MT> &S, int buf) {
#pragma unroll
        for (int i = 0; i < XPW; ++i) {
            char *dst = lds + (buf * NFRAG + (wave * XPW + i) % NFRAG) * 1024 + lane * 16;
            *(bf16x8 *)dst = S.x[i];
        }
    };
    auto compute = [&](const MidSet<MT> &S, int buf, int st) {
        const int kt0 = stage_of(st) * MID_KB;
#pragma unroll
        for (int kb = 0; kb < MID_KB; ++kb) {
            if (kb > 0 && kt0 + kb >= KT) break;                 // odd number of k-tiles: the last stage holds one
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                const char *src = lds + (buf * NFRAG + m * MID_KB + kb) * 1024 + lane * 16;
                const bf16x8 x = *(const bf16x8 *)src;
                acc[m][0] = MFMA16(S.wa[kb], x, acc[m][0]);
                acc[m][1] = MFMA16(S.wb[kb], x, acc[m][1]);
            }
        }
    };
    // stage t lives in set t % 4, its activations in LDS buffer t % 2
    MidSet<MT> st[4];
    load(st[0], 0);
    load(st[1], 1);
    load(st[2], 2);
    put(st[0], 0);
    __syncthreads();
    int s0 = 0;
    for (; s0 + 4 <= ns; s0 += 4) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            load(st[(j + 3) & 3], s0 + j + 3);
            compute(st[j], j & 1, s0 + j);
            put(st[(j + 1) & 3], (j + 1) & 1);
            __syncthreads();       // everybody is done with buffer j % 2, buffer (j + 1) % 2 is complete
        }
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        if (s0 + j < ns) {
            compute(st[j], j & 1, s0 + j);
            put(st[(j + 1) & 3], (j + 1) & 1);
        }
        __syncthreads();
    }
    if (!live) return;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        if (m >= n_mtiles) break;
        f32x4 *dst = kpart + ((((size_t)pair * KS + ks) * n_mtiles + m) * 2) * 64 + lane;
        dst[0] = acc[m][0];
        dst[64] = acc[m][1];
    }
}

// Adds the KS partial tiles of (pair, m-tile) and runs the epilogue.  A workgroup of 8 waves takes PP pairs, 8 / PP waves each: wave q of
// a pair adds the slices q, q + 8 / PP, ... and the pair's first wave the waves' sums, in that order.  grid = (groups of PP pairs, m-tiles).
// The norm scale of the m-tile's 16 tokens is computed once per workgroup: thread t adds the
// partial sums of squares t/16, t/16 + 32, ... of token t%16, then 16 threads add the 32 results
// in order.
constexpr int FIN_WAVES = 8;
template <int PP, class Epi>
__global__ void __launch_bounds__(FIN_WAVES * 64) k_mid_finish(const f32x4 *__restrict__ kpart, int KS, int n_pairs, int n_mtiles, Epi epi) {
    // the QKV projection's slices are added in 64 bits: its keys and values are rounded to bf16 next, and the sums over up to
    // 16 slices are the larger part of what decides the last place of a near tie
    typedef typename std::conditional<Epi::kWideSum, double, float>::type Sum;
    constexpr int NQ = FIN_WAVES / PP;                   // waves per pair
    constexpr int NL = NQ <= 2 ? 8 : 4;                   // slices a wave requests at once
    __shared__ float red[32][16];
    __shared__ float rs_row[16];
    __shared__ Sum sums[NQ > 1 ? NQ - 1 : 1][NQ > 1 ? PP : 1][8][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), q = wave % NQ;
    const int pair = blockIdx.x * PP + wave / NQ, mt = blockIdx.y;
    const bool live = pair < n_pairs;
    typename Epi::Pre pre;
    if (live && q == 0) pre = epi.pre(pair, mt, lane);
    const f32x4 *src = kpart + (((size_t)(live ? pair : n_pairs - 1) * KS * n_mtiles + mt) * 2) * 64 + lane;
    const size_t sstr = (size_t)n_mtiles * 128;
    f32x4 ta[NL], tb[NL];
    auto load = [&](int s0) {
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            const int sl = s0 + NQ * j < KS ? s0 + NQ * j : KS - 1;
            ta[j] = src[(size_t)sl * sstr];
            tb[j] = src[(size_t)sl * sstr + 64];
        }
    };
    SsLoads ssl;                             // (ahead of the slices: loads return in order)
    if constexpr (Epi::kNeedsRs)
        if (epi.nch != 0) ssl.load(epi.ss, epi.nch, epi.m_pad, mt * 16 + (threadIdx.x & 15), threadIdx.x >> 4, 32);
    load(q);
    float rs = 1.f;
    if constexpr (Epi::kNeedsRs) {
        if (epi.nch == 0) {                  // the factor itself (k_row_scale)
            rs = epi.ss[mt * 16 + (lane & 15)];
        } else {
            const int r = threadIdx.x & 15, part = threadIdx.x >> 4;       // 32 parts
            red[part][r] = ssl.sum(epi.ss, epi.nch, epi.m_pad, mt * 16 + r, part, 32);
            __syncthreads();
            if (threadIdx.x < 16) {
                float t = 0.f;
#pragma unroll
                for (int i = 0; i < 32; ++i) t += red[i][threadIdx.x];
                rs_row[threadIdx.x] = 1.0f / sqrtf(t / (float)epi.h + epi.eps);
            }
            __syncthreads();
            rs = rs_row[lane & 15];
        }
    }
    if (NQ == 1 && !live) return;
    Sum s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int s0 = q; s0 < KS; s0 += NL * NQ) {
        if (s0 != q) load(s0);
#pragma unroll
        for (int j = 0; j < NL; ++j)
            if (s0 + NQ * j < KS) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    s[e] += (Sum)ta[j][e];
                    s[4 + e] += (Sum)tb[j][e];
                }
            }
    }
    if constexpr (NQ > 1) {
        const int p = wave / NQ;
        if (q > 0) {
#pragma unroll
            for (int e = 0; e < 8; ++e) sums[q - 1][p][e][lane] = s[e];
        }
        __syncthreads();
        if (!live || q > 0) return;
#pragma unroll
        for (int i = 0; i < NQ - 1; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) s[e] += sums[i][p][e][lane];
    }
    const f32x4 a = {(float)s[0], (float)s[1], (float)s[2], (float)s[3]}, b = {(float)s[4], (float)s[5], (float)s[6], (float)s[7]};
    epi(pair, mt, a, b, lane, rs, pre);
}
// Pairs per workgroup: 8 from 128 workgroups on, fewer below, so that a narrow projection's sums are not left to a few compute units, one
// wave's loads after the other.  us per call, always 8 / 4 from 64 and 2 below: 7B 24 tokens (12 and 22 workgroups of 8 pairs) 44.9 / 41.6, 64
// (24, 44) 51.8 / 46.8; 70B 40 tokens (15, 84) 76.5 / 72.6, 128 (40, 224) 101.6 / 98.8; 13B 100 (105, 189) 66.5 / 64.3.  The lines at 160 and
// 80 and at 257 and 128: 13B 180 tokens (180, 324) 89.2 / 90.8 against 89.1, 7B 200 (78, 143) 73.4 both against 72.6; with 4 or 2 pairs at
// any size 512 tokens of 70B (160, 896 and 1024) 244 -> 252 and 254, the norm's statistics being summed once per workgroup.
template <class Epi>
hipError_t launch_mid_finish(hipStream_t s, const f32x4 *kpart, int KS, int n_pairs, int n_mtiles, const Epi &epi) {
    const int n8 = (n_pairs + 7) / 8 * n_mtiles;
#define SPD_FIN(PP) \
    hipLaunchKernelGGL((k_mid_finish<PP, Epi>), dim3((n_pairs + PP - 1) / PP, n_mtiles), dim3(FIN_WAVES * 64), 0, s, kpart, KS, n_pairs, n_mtiles, epi)
    if (n8 >= 128) SPD_FIN(8);
    else if (n8 >= 64) SPD_FIN(4);
    else SPD_FIN(2);
#undef SPD_FIN
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// GEMM for prefill-sized calls: a workgroup computes a tile of 256 (output features) x 256 (tokens), or one of the
// shapes below, with 8 waves; both operands are staged through LDS.  The operands already are sequences of 1 KiB
// MFMA fragments in global memory, so a stage is filled with gfx950's direct loads into LDS (one instruction per
// fragment, no staging registers) and read back with conflict-free 16-byte LDS reads.
//
// A stage holds two fragments per m-tile: k-tiles 2s and 2s + 1 (with the weights of both), or, for activations kept
// as a hi + lo pair (XS), the two planes of k-tile s (with its weights once: the second pass re-uses them from
// registers).  A step is two sub-steps, one per fragment: while the MFMAs of one run, the fragment reads of the next
// are dealt between them (so that neither the LDS nor the load unit is asked for a burst while the matrix cores
// wait), and in the second one the copies of the stage NST steps ahead.  The one barrier of a step sits between its
// sub-steps: passing it means that everybody has read both fragments of the current stage (whose place the copies
// take) and that the next stage has landed; the copies of the stages after that stay in flight across it.
// What bounds it: the matrix cores at the clock they hold under load (gate/up of 4096 tokens of the 70B shard runs at 1.3 PFLOP/s, spd_mfma_probe(), the
// same MFMAs on register-resident random data and nothing else, at 1.63 .. 1.76; matrix cores busy 70 % of the cycles), and
// in calls of one or two rounds what a compute unit draws through its load path.  Loads return in order, and a unit with a panel of its own gets 46 to 55 GB/s
// from the HBM while at most half of the units read, 27 when all do (7 TB/s in all), 92 and 23 from the last-level cache, 104 to 116 from the L2, however many loads are
// on their way; panels from the HBM that 2, 8, 32 units of an XCD read together 44, 61, 68, but panels shared across XCDs 27: an XCD's L2 takes in 0.9 TB/s.  Gate/up of
// 1000 tokens (256 x 128 tiles, 224 of them) by itself, us: the copies alone 112 with the weights from the HBM and 73 from the cache, the MFMAs alone 71, MFMAs and
// LDS reads 95, all of it 118 and 104 (in a call, traced: 131 to 133).  (The LDS is not it: a kernel of
// nothing but such reads draws 212 bytes per clock and compute unit, and MFMAs with 12 reads per 32 and this barrier run as fast as MFMAs alone.
// 32 x 32 x 16 MFMAs: 1.63 against 1.78 PFLOP/s on random data.  One of the workgroups that share a panel touching it some stages ahead: copies
// alone 110 -> 80 us, the kernel 118 -> 115, from the cache 102 -> 106.)
// ------------------------------------------------------------------------------------------
// Tile shapes.  WN x WM waves, each TI n-tiles x TJ m-tiles; stages of the plain and of the split (XS) kind.
struct GemmBig {      // 256 x 256: two stages of 64 KiB (split: three of 48 KiB)
    static constexpr int WN = 4, WM = 2, TI = 4, TJ = 8, NST = 2, NSTX = 3;
};
struct GemmHalf {     // 256 x 128: three stages of 48 KiB, four of 32 KiB (a step is too short for a copy to arrive within it)
    static constexpr int WN = 4, WM = 2, TI = 4, TJ = 4, NST = 3, NSTX = 4;
};
struct GemmTall {     // 128 x 384: for few n-tiles, where 256 x 256 tiles leave compute units idle
    static constexpr int WN = 2, WM = 4, TI = 4, TJ = 6, NST = 2, NSTX = 2;
};
struct GemmThird {    // 128 x 192, three stages of 40 KiB (split: four of 32 KiB): where 256 x 128 tiles leave compute units idle (see launch_gemm_lds())
    static constexpr int WN = 2, WM = 4, TI = 4, TJ = 3, NST = 3, NSTX = 4;
};
struct GemmWide {     // 160 x 256, every wave all 10 n-tiles of 2 m-tiles: for split activations and few n-tiles
    static constexpr int WN = 1, WM = 8, TI = 10, TJ = 2, NST = 2, NSTX = 3;      // (80 n-tiles x 512 m-tiles = exactly 256 tiles)
};
struct GemmSquare {   // 128 x 128, four stages of 32 KiB (split: five of 24 KiB): calls of 65 .. 256 tokens and few n-tiles, in K slices
    static constexpr int WN = 4, WM = 2, TI = 2, TJ = 4, NST = 4, NSTX = 5;
};
struct GemmSmall {    // 128 x 64: calls of at most 64 tokens, in K slices
    static constexpr int WN = 4, WM = 2, TI = 2, TJ = 2, NST = 6, NSTX = 6;
};
// operand of s_waitcnt: at most vm vector loads and lgkm LDS / scalar operations still in flight (63 / 15: any number)
constexpr int waitcnt_imm(int vm, int lgkm) { return (vm & 15) | ((vm >> 4) << 14) | (7 << 4) | (lgkm << 8); }
// descriptor of `bytes` bytes at p (raw access)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t panel(const char *p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, (int)bytes, 0x00020000);
}

template <class Epi, class G, bool XS>
__global__ void __launch_bounds__(G::WN *G::WM * 64, 1)
    k_gemm_lds(const __bf16 *Wp, const __bf16 *Xp, const __bf16 *Xlo, int KT, int n_ntiles, int n_mtiles, spd_tile_order ord,
               int tile0, int n_tiles, int msub, int kslices, Epi epi) {
    constexpr int TI = G::TI, TJ = G::TJ, NST = XS ? G::NSTX : G::NST;
    constexpr int NW = G::WN * G::WM, BN = G::WN * TI, BM = G::WM * TJ;
    constexpr int KW = XS ? 1 : 2;                                       // k-tiles per stage
    constexpr int W_BYTES = BN * KW * 1024, STAGE = W_BYTES + BM * 2048;
    constexpr int CW = (BN * KW + NW - 1) / NW, CX = BM * 2 / NW, NCP = CW + CX;      // fragments copied per wave and stage
    static_assert(TI % 2 == 0 && (BM * 2) % NW == 0 && (NST - 1) * NCP < 64, "tile shape");
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wn = wave % G::WN, wm = wave / G::WN;
    // A launch covers `n_tiles` tiles of the order from `tile0` on, each cut into `msub` workgroup tiles along M
    // (1, or 2 for the launch that finishes a ragged last round with half tiles; `ord` counts the uncut tiles).
    // kslices > 1 (sliced epilogues only): the launch covers the tiles once per slice of K, slice after slice, workgroups
    // of slice s contracting the s-th part of K and handing s to the epilogue.  The XCDs take equal shares of all
    // (slice, tile) items together: dealt slice by slice, 3 slices of 84 tiles gave most XCDs 33 workgroups for
    // their 32 compute units, a second round for one of them.
    int tn, tm, sub = 0, kslice = 0;
    {
        int idx;
        if (msub == 1) {
            idx = spd_tile_deal((int)blockIdx.x, n_tiles * kslices);
            if (idx < 0) return;                 // spare workgroup of a ragged share (whole workgroup, before any barrier)
            kslice = idx / n_tiles;
            idx -= kslice * n_tiles;
        } else {
            idx = (int)blockIdx.x / msub;
            sub = (int)blockIdx.x % msub;
        }
        spd_tile_at(ord, tile0 + idx, tn, tm);
    }
    const int kt_first = part_of(kslice, KT, kslices), nk = part_of(kslice + 1, KT, kslices) - kt_first;
    const int nt0 = tn * BN, mt0 = (tm * msub + sub) * BM;
    if (mt0 >= n_mtiles) return;                 // second half of a tile whose first half holds all the rows (whole workgroup)
    // Copies go through buffer descriptors of the tile's panels: a lane's offset plus one wave-uniform offset per
    // fragment.  (The global_load_lds form counts as an access to both memories at once, which makes the compiler wait for
    // every pending LDS read instead of the one it needs.)  Rows past the matrix repeat its last tile, spare copies
    // the last fragment.
    const int l16 = lane * 16;
    const unsigned pitch = (unsigned)KT * 1024;  // bytes between two tiles of a panel
    const int n_rows = n_ntiles - nt0 < BN ? n_ntiles - nt0 : BN, m_rows = n_mtiles - mt0 < BM ? n_mtiles - mt0 : BM;
    // (the activations' panels begin and end with a group of m-tiles)
    const int mg0 = mt0 & ~(SPD_ACT_GROUP - 1), mlast = mt0 + m_rows - 1,
              mg_rows = (mlast & ~(SPD_ACT_GROUP - 1)) + spd_act_width(mlast, n_mtiles) - mg0;
    const __amdgpu_buffer_rsrc_t wbuf = panel((const char *)Wp + (size_t)nt0 * pitch, n_rows * pitch),
                                 xbuf = panel((const char *)Xp + (size_t)mg0 * pitch, mg_rows * pitch),
                                 lbuf = panel((const char *)(XS ? Xlo : Xp) + (size_t)mg0 * pitch, mg_rows * pitch);
    unsigned wsrc[CW], xsrc[CX], xstr[CX];       // (wave-uniform)
    int wdst[CW];
#pragma unroll
    for (int n = 0; n < CW; ++n) {
        int f = wave * CW + n;
        f = f < BN * KW ? f : BN * KW - 1;
        const int t = f / KW;
        wsrc[n] = (unsigned)(t < n_rows ? t : n_rows - 1) * pitch + kt_first * 1024;
        wdst[n] = f;
    }
#pragma unroll
    for (int n = 0; n < CX; ++n) {
        const int t = (wave * CX + n) >> 1;
        const int mt = mt0 + (t < m_rows ? t : m_rows - 1), mg = mt & ~(SPD_ACT_GROUP - 1);
        xstr[n] = (unsigned)spd_act_width(mt, n_mtiles) * 1024;
        xsrc[n] = (unsigned)(mg - mg0) * pitch + (unsigned)(mt - mg) * 1024 + kt_first * xstr[n];
    }
    // Where the registers allow, the lo plane's products are summed on their own: half as many roundings of the large sums.
    constexpr bool LO_ACC = XS && TI * TJ <= 16;
    f32x4 acc[TI][TJ], acc_lo[LO_ACC ? TI : 1][LO_ACC ? TJ : 1];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
            acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
            if constexpr (LO_ACC) acc_lo[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
        }
    // copy n of stage st into the place `slot` (a k-tile past the end, the odd one's partner, repeats the last)
    auto copy1 = [&](int st, int slot, int n) __attribute__((always_inline)) {
        if (n < CW) {
            int kt = KW * st + (XS ? 0 : wdst[n] & 1);
            kt = kt < nk ? kt : nk - 1;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wbuf, (__attribute__((address_space(3))) void *)(lds + slot * STAGE + wdst[n] * 1024),
                                                     16, l16, (int)(wsrc[n] + kt * 1024), 0, 0);
        } else {
            const int c = wave * CX + (n - CW);
            int kt = XS ? st : 2 * st + (c & 1);
            kt = kt < nk ? kt : nk - 1;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(XS && (c & 1) ? lbuf : xbuf,
                                                     (__attribute__((address_space(3))) void *)(lds + slot * STAGE + W_BYTES + c * 1024),
                                                     16, l16, (int)(xsrc[n - CW] + kt * xstr[n - CW]), 0, 0);
        }
    };
    const char *a_base = lds + wn * TI * KW * 1024 + l16, *b_base = lds + W_BYTES + wm * TJ * 2048 + l16;
    // fragment r of sub-step p of the stage in `slot`: the wave's TJ activation fragments, then its TI weight fragments
    auto read1 = [&](int slot, int p, int r, bf16x8(&a)[TI], bf16x8(&b)[TJ]) __attribute__((always_inline)) {
        if (r < TJ) b[r] = *(const bf16x8 *)(b_base + slot * STAGE + (2 * r + p) * 1024);
        else a[r - TJ] = *(const bf16x8 *)(a_base + slot * STAGE + ((r - TJ) * KW + (XS ? 0 : p)) * 1024);
    };
    const int n_stages = (nk + KW - 1) / KW, nsteps = nk / KW;
#pragma unroll
    for (int st = 0; st < NST; ++st)
        if (st < n_stages) {
#pragma unroll
            for (int n = 0; n < NCP; ++n) copy1(st, st, n);
        }
    __builtin_amdgcn_sched_barrier(0);
    // (the builtin, unlike a wait in asm, is one the compiler's own count of pending operations knows of)
    if (n_stages >= NST) __builtin_amdgcn_s_waitcnt(waitcnt_imm((NST - 1) * NCP, 0));
    else __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 a0[TI], a1[TI], b0[TJ], b1[TJ];
#pragma unroll
    for (int r = 0; r < TI + TJ; ++r) read1(0, 0, r, a0, b0);

    // the MFMAs of a sub-step on (a, b); meanwhile NR fragments of the next one are read into (an, bn) and, with COPY, the
    // copies of stage cst go out
    auto substep = [&](auto nr_, auto copy_, auto lo_, const bf16x8(&a)[TI], const bf16x8(&b)[TJ], bf16x8(&an)[TI], bf16x8(&bn)[TJ], int rslot,
                       int rp, int cst, int cslot) __attribute__((always_inline)) {
        constexpr int NR = decltype(nr_)::value, NM = TI * TJ;
        constexpr bool COPY = decltype(copy_)::value;
        int r = 0, cp = 0;
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                const int n = i * TJ + j;
                if constexpr (LO_ACC && decltype(lo_)::value) acc_lo[i][j] = MFMA16(a[i], b[j], acc_lo[i][j]);
                else acc[i][j] = MFMA16(a[i], b[j], acc[i][j]);
                __builtin_amdgcn_sched_barrier(0);
                if (r < NR && n >= (2 * NR <= NM ? 2 * r : r * NM / NR)) read1(rslot, rp, r++, an, bn);
                if (COPY && cp < NCP && n >= cp * (NM / NCP) + 1) copy1(cst, cslot, cp++);
                __builtin_amdgcn_sched_barrier(0);
            }
    };
    int slot = 0;                                      // of the current stage
    auto step = [&](auto copy_, auto odd_, int s) __attribute__((always_inline)) {
        constexpr bool COPY = decltype(copy_)::value, ODD = decltype(odd_)::value;
        using All = std::integral_constant<int, TI + TJ>;
        const int next = slot + 1 == NST ? 0 : slot + 1;
        if constexpr (XS) substep(std::integral_constant<int, TJ>(), std::false_type(), std::false_type(), ODD ? a1 : a0, b0, ODD ? a0 : a1, b1, slot, 1, 0, 0);
        else substep(All(), std::false_type(), std::false_type(), a0, b0, a1, b1, slot, 1, 0, 0);
        // the next stage's copies of this wave have landed, those of the NST - 2 stages after it may be in flight; every
        // read of the current stage is done
        __builtin_amdgcn_s_waitcnt(waitcnt_imm(COPY ? (NST - 2) * NCP : 0, 0));
        asm volatile("s_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        // (in the last step: fragments read and never used)
        if constexpr (XS) substep(All(), copy_, std::true_type(), ODD ? a1 : a0, b1, ODD ? a0 : a1, b0, next, 0, s + NST, slot);
        else substep(All(), copy_, std::false_type(), a1, b1, a0, b0, next, 0, s + NST, slot);
        slot = next;
    };
    int s = 0;
    if constexpr (XS) {                                // (the weight registers of a pair of steps take turns)
        for (; s + 1 + NST < n_stages; s += 2) {
            step(std::true_type(), std::false_type(), s);
            step(std::true_type(), std::true_type(), s + 1);
        }
        // at most one stage is left to copy
        if (s + NST < n_stages) {
            step(std::true_type(), std::false_type(), s++);
            if (s < nsteps) step(std::false_type(), std::true_type(), s++);
        }
        for (; s + 1 < nsteps; s += 2) {
            step(std::false_type(), std::false_type(), s);
            step(std::false_type(), std::true_type(), s + 1);
        }
        if (s < nsteps) step(std::false_type(), std::false_type(), s);
    } else {
        for (; s + NST < n_stages; ++s) step(std::true_type(), std::false_type(), s);
        for (; s < nsteps; ++s) step(std::false_type(), std::false_type(), s);
        if (nk & 1) {                                  // odd number of k-tiles: the last one on its own (its fragments are read already)
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int j = 0; j < TJ; ++j) acc[i][j] = MFMA16(a0[i], b0[j], acc[i][j]);
        }
    }
    if constexpr (LO_ACC) {
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j) acc[i][j] += acc_lo[i][j];
    }
    // norm factors of all the wave's m-tiles first, so that their loads are in flight together
    float rs[TJ];
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
        rs[j] = 1.f;
        if constexpr (Epi::kNeedsRs) {
            int mt = mt0 + wm * TJ + j;
            if (mt >= n_mtiles) mt = n_mtiles - 1;
            rs[j] = epi.nch == 0 ? epi.ss[mt * 16 + (lane & 15)]
                                 : sum_ss(epi.ss, epi.nch, epi.m_pad, mt * 16 + (lane & 15), lane >> 4, 4);
        }
    }
    if constexpr (Epi::kNeedsRs) {
        if (epi.nch != 0) {
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                float q = rs[j];
                q += shfl_xor_f(q, 16);
                q += shfl_xor_f(q, 32);
                rs[j] = 1.0f / sqrtf(q / (float)epi.h + epi.eps);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
        const int mt = mt0 + wm * TJ + j;
        if (mt >= n_mtiles) continue;
        typename Epi::Pre pre[TI / 2];
#pragma unroll
        for (int i = 0; i < TI; i += 2) {
            int nt = nt0 + wn * TI + i;
            if (nt >= n_ntiles) nt = n_ntiles - 2;
            pre[i / 2] = epi.pre(nt >> 1, mt, lane);
        }
#pragma unroll
        for (int i = 0; i < TI; i += 2) {
            const int nt = nt0 + wn * TI + i;
            if (nt >= n_ntiles) continue;
            if constexpr (Epi::kSliced) epi.slice(nt >> 1, kslice, mt, acc[i][j], acc[i + 1][j], lane, rs[j], pre[i / 2]);
            else epi(nt >> 1, mt, acc[i][j], acc[i + 1][j], lane, rs[j], pre[i / 2]);
        }
    }
}

template <class G, bool XS, class Epi>
hipError_t launch_gemm_lds_cfg(const spd_call &c, const __bf16 *Wp, const __bf16 *Xp, const __bf16 *Xlo, int n_pairs, int KT,
                               const Epi &epi, int tile0 = 0, int msub = 1, int n_tiles = -1, int kslices = 1) {
    // with msub = 2 the tiles are counted in the shape of twice G's height (GemmHalf finishing a GemmBig launch)
    constexpr int BN = G::WN * G::TI;
    constexpr int LDS = (XS ? G::NSTX : G::NST) * (BN * (XS ? 1 : 2) + G::WM * G::TJ * 2) * 1024;
    static_assert(LDS <= 160 * 1024, "the stages must fit the LDS of a compute unit");
    static_assert(BN <= SPD_GEMM_MAX_ROWS && G::WM * G::TJ <= SPD_GEMM_MAX_ROWS, "panel rows, see spd_gemm_fits()");
    if (!spd_gemm_fits(KT)) return hipErrorInvalidValue;         // (the callers take another kernel)
    const int BM = G::WM * G::TJ * msub;
    // the attribute is per kernel instantiation: set once, whichever thread comes first
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [] {
        attr_err = hipFuncSetAttribute((const void *)k_gemm_lds<Epi, G, XS>, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
    });
    if (attr_err != hipSuccess) return attr_err;
    const int n_ntiles = 2 * n_pairs, n_mtiles = (c.M + 15) / 16;
    spd_tile_order ord;
    ord.TN = (n_ntiles + BN - 1) / BN;
    ord.TM = (n_mtiles + BM - 1) / BM;
    spd_pick_block(ord.TN, ord.TM, BN * 16, BM * 16, ord.bn, ord.bm);
    if (n_tiles < 0) n_tiles = ord.TN * ord.TM - tile0;
    // msub = 1: whole rounds of 256, then eight equal shares (the spare workgroups of a ragged share exit at once)
    // (msub = 2 comes with one slice only)
    const int n_wgs = msub == 1 ? spd_tile_launch_size(n_tiles * kslices) : n_tiles * msub;
    hipLaunchKernelGGL((k_gemm_lds<Epi, G, XS>), dim3(n_wgs), dim3(G::WN * G::WM * 64), LDS, c.s, Wp, Xp, Xlo, KT, n_ntiles,
                       n_mtiles, ord, tile0, n_tiles, msub, kslices, epi);
    return hipGetLastError();
}

template <bool XS, class Epi>
hipError_t launch_gemm_lds(const spd_call &c, const __bf16 *Wp, const __bf16 *Xp, const __bf16 *Xlo, int n_pairs, int KT,
                           const Epi &epi) {
    // fewer 256 x 256 tiles than compute units (the QKV projection of a shard): 128 x 384 tiles when they
    // fill one round better
    const int n_mtiles = (c.M + 15) / 16;
    const int big = ((2 * n_pairs + 15) / 16) * ((n_mtiles + 15) / 16), tall = ((2 * n_pairs + 7) / 8) * ((n_mtiles + 23) / 24);
    if constexpr (XS) {
        // split activations, few n-tiles: 160 x 256 tiles when they come to one full round of the chip with less work
        // per tile than the other shapes (the QKV projection of the 70B shard: 8 x 32 = 256 tiles)
        // (a call that is not one of two chains: only when the 256 x 128 tiles below would need a second round; 4096
        // tokens: 128 wide tiles 176 us, 160 half tiles 155)
        const int wide = ((2 * n_pairs + 9) / 10) * ((n_mtiles + 15) / 16), halves = ((2 * n_pairs + 15) / 16) * ((n_mtiles + 7) / 8);
        if (big < 224 && wide <= 256 && wide > tall && (c.chained || halves > 256))
            return launch_gemm_lds_cfg<GemmWide, XS>(c, Wp, Xp, Xlo, n_pairs, KT, epi);
    }
    {
        // at most half a round of 256 x 256 tiles: 256 x 128 half tiles when they occupy more compute units than
        // the other shapes
        const int halves = ((2 * n_pairs + 15) / 16) * ((n_mtiles + 7) / 8);
        const int other = (big < 224 && tall <= 256 && tall > big) ? tall : big;
        // 128 x 192 tiles, three quarters of a half tile's work, where they still come to one round: us per call, half / these: 7B 1100
        // tokens 192.5 / 183.3, 1500: 237.5 / 218.6, 2048 (gate/up 176 / 242 tiles) 335.5 / 325.0; 13B 800 195.7 / 184.2, 1400 285.3 / 269.0; 70B
        // 550 293.7 / 256.4, 760 (gate/up 168 / 224) 325.4 / 280.1; calls of two chains equal (70B) to - 4 % (13B 2 x 1500)
        const int thirds = ((2 * n_pairs + 7) / 8) * ((n_mtiles + 11) / 12);
        if (big <= 128 && halves <= 256 && thirds <= 256 && thirds > halves)
            return launch_gemm_lds_cfg<GemmThird, XS>(c, Wp, Xp, Xlo, n_pairs, KT, epi);
        if (big <= 128 && halves <= 256 && halves > other)
            return launch_gemm_lds_cfg<GemmHalf, XS>(c, Wp, Xp, Xlo, n_pairs, KT, epi, 0, 2, big);
    }
    if (big < 224 && tall <= 256 && tall > big) return launch_gemm_lds_cfg<GemmTall, XS>(c, Wp, Xp, Xlo, n_pairs, KT, epi);
    // a last round that would occupy at most half of the compute units runs as twice as many half tiles
    // in a second launch (gate/up of the 70B shard: 896 tiles = 3.5 rounds of 256)
    const int rem = big % 256;
    if (big > 256 && rem > 0 && rem <= 128) {
        const hipError_t e = launch_gemm_lds_cfg<GemmBig, XS>(c, Wp, Xp, Xlo, n_pairs, KT, epi, 0, 1, big - rem);
        if (e != hipSuccess) return e;
        return launch_gemm_lds_cfg<GemmHalf, XS>(c, Wp, Xp, Xlo, n_pairs, KT, epi, big - rem, 2, rem);
    }
    return launch_gemm_lds_cfg<GemmBig, XS>(c, Wp, Xp, Xlo, n_pairs, KT, epi);
}

// ------------------------------------------------------------------------------------------
// Attention.  Scores are computed transposed, S^T[key][col] = K q, so that the probabilities
// leave the MFMA already in the operand layout of the second contraction O^T = V^T P^T.
// A "column" is a (token, query head of the KV group) pair: col = t * group + c.
// ------------------------------------------------------------------------------------------
template <int DT>   // DT = head_dim / 16
struct AttnState {
    f32x4 o[DT];    // O^T[d = dt*16 + 4g + i][col = lane%16], unnormalised
    float m, l;     // running max (of scaled scores) and sum for col = lane%16
};

template <int DT>
struct KVFrags {
    bf16x8 k0[DT / 2], k1[DT / 2], v[DT];
};

// all fragments of one 32-key block: 2 x 16 keys x d for K, d x 32 keys for V.  STREAM: not to be kept in the caches
template <int DT, bool STREAM = false>
__device__ __forceinline__ void load_kv(KVFrags<DT> &f, const __bf16 *__restrict__ kbase, const __bf16 *__restrict__ vbase,
                                        int vb, int d, int lane) {
    const bf16x8 *k0 = (const bf16x8 *)(kbase + (size_t)(2 * vb) * 16 * d) + lane;
    const bf16x8 *k1 = (const bf16x8 *)(kbase + (size_t)(2 * vb + 1) * 16 * d) + lane;
    const bf16x8 *vf = (const bf16x8 *)(vbase + (size_t)vb * 32 * d) + lane;
#pragma unroll
    for (int t = 0; t < DT / 2; ++t) {
        f.k0[t] = STREAM ? __builtin_nontemporal_load(k0 + t * 64) : k0[t * 64];
        f.k1[t] = STREAM ? __builtin_nontemporal_load(k1 + t * 64) : k1[t * 64];
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) f.v[dt] = STREAM ? __builtin_nontemporal_load(vf + dt * 64) : vf[dt * 64];
}

// one 32-key block: keys [vb*32, vb*32+32) of one (sequence, KV head); n_keys_col = number of
// keys column lane%16 may attend (causal), 0 for a padding column
template <int DT, bool LAZY = false>      // LAZY (prefill): the running output is rescaled only when some column's maximum moved; probabilities on one plane
__device__ __forceinline__ void attn_block(AttnState<DT> &st, const bf16x8 *__restrict__ qf, const KVFrags<DT> &f, int vb,
                                           int n_keys_col, float scale, int lane) {
    // qf[0 .. DT/2) are the hi halves of the query fragments, qf[DT/2 .. DT) the lo halves
    const int g = lane >> 4;
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < DT / 2; ++t) {
        s0 = MFMA(f.k0[t], qf[t], s0);
        s1 = MFMA(f.k1[t], qf[t], s1);
        s0 = MFMA(f.k0[t], qf[DT / 2 + t], s0);
        s1 = MFMA(f.k1[t], qf[DT / 2 + t], s1);
    }
    const int key0 = vb * 32 + 4 * g;
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        s0[i] = (key0 + i < n_keys_col) ? s0[i] * scale : -INFINITY;
        s1[i] = (key0 + 16 + i < n_keys_col) ? s1[i] * scale : -INFINITY;
        mx = fmaxf(mx, fmaxf(s0[i], s1[i]));
    }
    mx = quad_max(mx);
    const float m_new = fmaxf(st.m, mx);
    // every key of this block masked for this column and nothing seen before: keep the state
    const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
    const float alpha = __expf(st.m - m_use);          // exp(-inf) = 0 on the first block
    float p0[4], p1[4], ps = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        p0[i] = __expf(s0[i] - m_use);
        p1[i] = __expf(s1[i] - m_use);
        ps += p0[i] + p1[i];
    }
    ps = quad_sum(ps);
    st.l = st.l * alpha + ps;
    st.m = m_new;
    // probabilities: hi + lo pairs in a decode step (bound by the cache stream, the second pass is free); one bf16
    // plane in a prefill, which is bound by this vector work: a probability's rounding error (2^-9 relative) reaches
    // the block output through a sum over keys and the O projection, and measured 7.0e-3 -> 7.6e-3 there
    constexpr bool PLO = !LAZY;
    bf16x8 pb, pl;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        pb[i] = (__bf16)p0[i];
        pb[4 + i] = (__bf16)p1[i];
        if (PLO) {
            pl[i] = (__bf16)(p0[i] - (float)pb[i]);
            pl[4 + i] = (__bf16)(p1[i] - (float)pb[4 + i]);
        }
    }
    // (a factor of exactly 1 changes nothing: skipping the multiplication when no column of the wave needs it
    // gives the same bits; in a causal prefill the maxima settle after the first blocks)
    if (!LAZY || __builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) st.o[dt] *= alpha;
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
        st.o[dt] = MFMA(f.v[dt], pb, st.o[dt]);
        if (PLO) st.o[dt] = MFMA(f.v[dt], pl, st.o[dt]);
    }
}

// query fragments of one column tile: col -> (token t, head c); zero for padding columns
template <int DT>
__device__ __forceinline__ void load_q(bf16x8 *qf, const __bf16 *__restrict__ qbuf, const __bf16 *__restrict__ qlo, int m,
                                       int head, int qd, int d, bool valid, int lane) {
    const int g = lane >> 4;
#pragma unroll
    for (int t = 0; t < DT / 2; ++t) {
        if (valid) {
            const size_t o = (size_t)m * qd + head * d + t * 32 + g * 8;
            qf[t] = *(const bf16x8 *)(qbuf + o);
            qf[DT / 2 + t] = *(const bf16x8 *)(qlo + o);
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) qf[t][i] = qf[DT / 2 + t][i] = (__bf16)0.f;
        }
    }
}

// Decode (q_len = 1): grid (splits, kv heads, sequences), 4 waves.  The waves of a workgroup
// take the 32-key blocks of their split round-robin, the next block's fragments being loaded
// while the current one is processed; the workgroup writes one partial (unnormalised O^T,
// running max, running sum) per split.
//
// FUSED: the QKV projection ran in K slices and left fp32 partial rows qkvp[slice][token][nqkv]
// (EpiQKVPart).  Every workgroup adds the slices of its queries (ascending order), keeps them as
// hi + lo bf16 pairs; the cache then holds the P.pos[b] earlier positions only, and the
// workgroup of the last split adds the new token: it sums its key and value, rounds them to the
// cache's bf16, appends them to the cache and attends to them as one more (single-key) block.
//
// STREAM: caches that do not fit beside the weights in what the chip keeps from one step to the next (256 MB) are read past it.
template <int DT, bool FUSED, bool STREAM>
__global__ void __launch_bounds__(256) k_attn_decode(__bf16 *__restrict__ kc, __bf16 *__restrict__ vc, const float *__restrict__ qkvp, int q, int kv,
                                                     int max_ctx, int KS, int part_rows, int nqkv, const __bf16 *__restrict__ qbuf_in,
                                                     const __bf16 *__restrict__ qlo_in, const float *__restrict__ xss, float xh, float xeps,
                                                     __bf16 *__restrict__ qbuf_out, __bf16 *__restrict__ qlo_out, AttnParts parts,
                                                     spd_positions P) {
    constexpr int d = DT * 16;
    // the waves' states: a column's features side by side (padded, so that the 16 columns begin at different banks)
    __shared__ __attribute__((aligned(16))) float sm[4][16][DT * 16 + 4];
    __shared__ float sml[4][2][16];
    __shared__ __attribute__((aligned(16))) __bf16 sq[2][16 * d];      // hi / lo queries of the group's heads
    __shared__ __attribute__((aligned(16))) __bf16 snew[2][d];         // new key, new value
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int split = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z;
    const int group = parts.group, qd = q * d, n_splits = parts.n_splits;
    const int n_keys = FUSED ? P.pos[b] : P.pos[b] + 1;       // keys in the cache
    const int nblk = (n_keys + 31) >> 5;
    const int b0 = part_of(split, nblk, n_splits), b1 = part_of(split + 1, nblk, n_splits);
    const int col = lane & 15, g = lane >> 4;
    const bool cvalid = col < group;
    const bool newtok = FUSED && split == n_splits - 1;
    __bf16 *kbase = kc + ((size_t)b * kv + kvh) * (size_t)max_ctx * d;
    __bf16 *vbase = vc + ((size_t)b * kv + kvh) * (size_t)max_ctx * d;
    AttnState<DT> st;
#pragma unroll
    for (int i = 0; i < DT; ++i) st.o[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
    st.m = -INFINITY;
    st.l = 0.f;
    const float scale = 1.0f / sqrtf((float)d);
    const bool has_blocks = b0 + wave < b1;
    // FUSED: thread -> items of 4 consecutive columns of the group's queries (group * d / 4 items); in
    // the workgroup of the last split the first d / 2 threads also take the new key and the new value.
    // The slices of all items are requested first, then the first two key blocks; the sums are
    // formed while the key blocks are on their way.  All these loads are unconditional (indices are
    // clamped instead), so that nothing waits between them.
    constexpr int NQS = (16 * d / 4 + 255) / 256, MAXKS = SPD_MAX_QKV_SLICES;
    const int nq4 = group * d / 4, nk4 = d / 4;
    float4 qs[NQS][MAXKS], ns[MAXKS];
    if constexpr (FUSED) {
#pragma unroll
        for (int sl = 0; sl < NQS; ++sl) {
            if (256 * sl >= nq4) break;                                   // uniform
            const int e = min((int)threadIdx.x + 256 * sl, nq4 - 1);
            const float *src = qkvp + (size_t)b * nqkv + kvh * group * d + 4 * e;
#pragma unroll
            for (int j = 0; j < MAXKS; ++j) qs[sl][j] = *(const float4 *)(src + (size_t)min(j, KS - 1) * part_rows * nqkv);
        }
        if (newtok) {                                                     // uniform
            const int e = min((int)threadIdx.x, 2 * nk4 - 1);
            const int colq = e < nk4 ? qd + kvh * d + 4 * e : qd + kv * d + kvh * d + 4 * (e - nk4);
            const float *src = qkvp + (size_t)b * nqkv + colq;
#pragma unroll
            for (int j = 0; j < MAXKS; ++j) ns[j] = *(const float4 *)(src + (size_t)min(j, KS - 1) * part_rows * nqkv);
        }
    }
    // (a wave without blocks loads a block it will not use: one code path, no waiting at a join)
    // The first block only: a wave's second one ahead of the queries too held it at its requests until most of them had been served (4.5 of
    // 7.7 us at 16 sequences of 4096 of the 70B shard), and everything below came after that.
    KVFrags<DT> f0, f1;
    load_kv<DT, STREAM>(f0, kbase, vbase, min(b0 + wave, nblk > 0 ? nblk - 1 : 0), d, lane);      // (the cache holds at least one block)
    SPD_SCHED_BARRIER();
    bf16x8 qf[DT];
    if constexpr (FUSED) {
        float xrs = 1.f;
        if (xss) {
            float part[MAXKS];
#pragma unroll
            for (int j = 0; j < MAXKS; ++j) part[j] = xss[min(j, KS - 1) * 16 + b];
            float t = part[0];
#pragma unroll
            for (int j = 1; j < MAXKS; ++j) t += j < KS ? part[j] : 0.f;
            xrs = 1.0f / sqrtf(t / xh + xeps);
        }
        auto add_slices = [&](const float4 *v) {
            float4 acc = v[0];
#pragma unroll
            for (int j = 1; j < MAXKS; ++j) {
                const float on = j < KS ? 1.f : 0.f;      // a clamped repeat of the last slice counts for nothing
                acc.x += on * v[j].x; acc.y += on * v[j].y; acc.z += on * v[j].z; acc.w += on * v[j].w;
            }
            if (xss) { acc.x *= xrs; acc.y *= xrs; acc.z *= xrs; acc.w *= xrs; }
            return acc;
        };
#pragma unroll
        for (int sl = 0; sl < NQS; ++sl) {
            if (256 * sl >= nq4) break;
            const int e = threadIdx.x + 256 * sl;
            const float4 acc = add_slices(qs[sl]);
            const bf16x4 hi = cvt4(acc.x, acc.y, acc.z, acc.w);
            const bf16x4 lo = cvt4_lo(acc.x, acc.y, acc.z, acc.w, hi);
            if (e < nq4) {
                *(bf16x4 *)(&sq[0][4 * e]) = hi;
                *(bf16x4 *)(&sq[1][4 * e]) = lo;
                if (newtok) {        // the rotated queries stay readable in the workspace
                    *(bf16x4 *)(qbuf_out + (size_t)b * qd + kvh * group * d + 4 * e) = hi;
                    *(bf16x4 *)(qlo_out + (size_t)b * qd + kvh * group * d + 4 * e) = lo;
                }
            }
        }
        if (newtok) {
            const int e = threadIdx.x;
            const float4 acc = add_slices(ns);
            const bf16x4 hi = cvt4(acc.x, acc.y, acc.z, acc.w);
            if (e < nk4) {
                *(bf16x4 *)(&snew[0][4 * e]) = hi;
                *(bf16x4 *)(kbase + spd_kcache_off(P.pos[b], 4 * e, d)) = hi;
            } else if (e < 2 * nk4) {
                const int dc = 4 * (e - nk4);
                *(bf16x4 *)(&snew[1][dc]) = hi;
#pragma unroll
                for (int i = 0; i < 4; ++i) vbase[spd_vcache_off(P.pos[b], dc + i, d)] = hi[i];
            }
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < DT / 2; ++t) {
            if (cvalid) {
                qf[t] = *(const bf16x8 *)(&sq[0][col * d + t * 32 + g * 8]);
                qf[DT / 2 + t] = *(const bf16x8 *)(&sq[1][col * d + t * 32 + g * 8]);
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) qf[t][i] = qf[DT / 2 + t][i] = (__bf16)0.f;
            }
        }
    } else {
        load_q<DT>(qf, qbuf_in, qlo_in, b, kvh * group + col, qd, d, cvalid, lane);
    }
    // The wave's blocks are b0 + wave + 4 j, j < nw.  Two register buffers used alternately: while one block is processed the loads of the
    // next are in flight.  No branch between loads and use: an index past the wave's last block repeats that block.
    const int nw = has_blocks ? (b1 - b0 - wave + 3) >> 2 : 0;
    if (nw == 1) {
        attn_block<DT>(st, qf, f0, b0 + wave, cvalid ? n_keys : 0, scale, lane);
    } else if (nw > 1) {
        auto blk = [&](int j) { return b0 + wave + 4 * (j < nw ? j : nw - 1); };
        load_kv<DT, STREAM>(f1, kbase, vbase, blk(1), d, lane);
        SPD_SCHED_BARRIER();
        int j = 0;
        for (; j + 2 < nw; j += 2) {
            attn_block<DT>(st, qf, f0, blk(j), cvalid ? n_keys : 0, scale, lane);
            SPD_SCHED_BARRIER();
            load_kv<DT, STREAM>(f0, kbase, vbase, blk(j + 2), d, lane);
            SPD_SCHED_BARRIER();
            attn_block<DT>(st, qf, f1, blk(j + 1), cvalid ? n_keys : 0, scale, lane);
            SPD_SCHED_BARRIER();
            load_kv<DT, STREAM>(f1, kbase, vbase, blk(j + 3), d, lane);
            SPD_SCHED_BARRIER();
        }
        attn_block<DT>(st, qf, f0, blk(j), cvalid ? n_keys : 0, scale, lane);
        if (j + 1 < nw) attn_block<DT>(st, qf, f1, blk(j + 1), cvalid ? n_keys : 0, scale, lane);
    }
    if (newtok && wave == 0) {
        // the new token as a block whose only key is key 0: K row 0, V contraction slot 0
        KVFrags<DT> fn;
        const bf16x8 zero = {(__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f};
#pragma unroll
        for (int t = 0; t < DT / 2; ++t) {
            fn.k0[t] = col == 0 ? *(const bf16x8 *)(&snew[0][t * 32 + g * 8]) : zero;
            fn.k1[t] = zero;
        }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            fn.v[dt] = zero;
            if (g == 0) fn.v[dt][0] = snew[1][dt * 16 + col];
        }
        attn_block<DT>(st, qf, fn, 0, cvalid ? 1 : 0, scale, lane);
    }
    // merge the four waves: a thread takes four features of a head
    if (cvalid) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) *(f32x4 *)&sm[wave][col][dt * 16 + 4 * g] = st.o[dt];
        if (g == 0) {
            sml[wave][0][col] = st.m;
            sml[wave][1][col] = st.l;
        }
    }
    __syncthreads();
    const int u = b * kv + kvh;
    for (int e = threadIdx.x; e < group * (d / 4); e += 256) {
        const int c = e / (d / 4), f = 4 * (e % (d / 4));
        float mm = -INFINITY, l = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) mm = fmaxf(mm, sml[w][0][c]);
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float mw = sml[w][0][c];
            const float sc = (mw == -INFINITY) ? 0.f : __expf(mw - mm);
            v += *(const f32x4 *)&sm[w][c][f] * sc;
            l += sml[w][1][c] * sc;
        }
        *(f32x4 *)(parts.sums(u, split, c) + f) = v;
        if (f == 0) {
            float *ml = parts.max_sum(u, split, c);
            ml[0] = mm;
            ml[group] = l;
        }
    }
}

// merge the splits and write the normalised output as packed activations of the O projection: row = token, contraction index =
// head*d + dd.  grid (groups of 64 of a unit's group * d / 4 quads, KV heads, sequences); every thread reads the maximum and sum of its
// head itself (16 splits at a time, all loads issued together), so the kernel is one memory round trip per 16 splits.
__global__ void __launch_bounds__(64) k_attn_combine(float *po, int units, int n_splits, int group, int d, Divider by_quads,
                                                     __bf16 *__restrict__ ahat, __bf16 *__restrict__ alo) {
    AttnParts parts;
    parts.o = po; parts.units = units; parts.n_splits = n_splits; parts.group = group; parts.d = d;
    const int hq = parts.d >> 2, kvh = blockIdx.y, b = blockIdx.z, kv = gridDim.y, batch = gridDim.z, u = b * kv + kvh;
    const int e = blockIdx.x * 64 + threadIdx.x;
    if (e >= parts.group * hq) return;
    const int c = by_quads.div(e), quad = by_quads.mod(e), qd = kv * parts.group * parts.d;
    MergeLoads<16> L;
    L.load(parts, u, c, quad, 0);
    const float4 v = merge_splits<16>(parts, u, c, quad, L);
    const int kidx = (kvh * parts.group + c) * parts.d + 4 * quad;
    const size_t o = spd_act_index(b >> 4, kidx >> 5, qd >> 5, (batch + 15) >> 4) + spd_frag_elem(b & 15, kidx & 31);
    const bf16x4 hi = cvt4h(v.x, v.y, v.z, v.w);
    *(bf16x4 *)(ahat + o) = hi;
    if (alo) *(bf16x4 *)(alo + o) = cvt4h_lo(v.x, v.y, v.z, v.w, hi);
}

constexpr int PREFILL_ONE_WGS = 2;       // workgroups of one column tile that a compute unit holds
// Prefill (q_len > 1): grid (groups of CT column tiles x kv heads, 1, sequences), 4 waves.  (The heads side by side: workgroups go to the XCDs in turn, so
// that an XCD's L2 sees the keys of one or two of four heads; 2048 tokens of 7B, 4 heads, 25.0 -> 19.4 us.)  All four
// waves work on the same CT tiles of 16 (token, head) columns and deal the causal key range
// among themselves block by block (the latest tokens attend thousands of keys: one wave walking
// them alone would be the critical path of the launch); their partial states meet in LDS and
// every wave finishes a quarter of the (tile, 16-feature slice) outputs.
// With one tile two workgroups fit a compute unit, and the bound keeps it so: 128 features take exactly the 256 registers of two waves per
// SIMD, and a compiler that took 258 left one (us, two / one: 70B 2048 tokens behind 2500 85.9 / 108.2, 7B 4-way the same call 91 / 110).  Two tiles of
// 128 features do not fit twice.  The heads' number divides by its reciprocal: two divisions ahead of the first load cost 1 us of 20 (512 behind 1536).
template <int DT, int CT>
__global__ void __launch_bounds__(256, CT == 1 ? PREFILL_ONE_WGS : 1) k_attn_prefill(const __bf16 *__restrict__ qbuf, const __bf16 *__restrict__ qlo, const __bf16 *__restrict__ kc,
                                                      const __bf16 *__restrict__ vc, int q_len, int group, int max_ctx, int n_groups,
                                                      Divider by_kv, __bf16 *__restrict__ ahat, __bf16 *__restrict__ alo, spd_positions P) {
    constexpr int d = DT * 16;
    extern __shared__ __attribute__((aligned(16))) char ap_lds[];
    f32x4 *so = (f32x4 *)ap_lds;                                   // [4 waves][CT][DT][64 lanes]
    float *sml = (float *)(ap_lds + 4 * CT * DT * 64 * 16);        // [4 waves][CT][2][16]: running max, running sum
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int kv = (int)by_kv.d, b = blockIdx.z;
    int group0 = by_kv.div(blockIdx.x);
    group0 -= group0 * kv > (int)blockIdx.x;               // (from 2^32 / kv on it may be one too many)
    const int kvh = (int)blockIdx.x - group0 * kv, qd = kv * group * d;
    const int n_cols = q_len * group;
    // causal: the later a token, the more keys it attends; the long workgroups are launched first
    const int ct0 = (n_groups - 1 - group0) * CT;
    const int g = lane >> 4;
    const int pos0 = P.pos[b];
    bf16x8 qf[CT][DT];
    AttnState<DT> st[CT];
    int nk[CT], mrow[CT], hd[CT];
    int last_key = 0;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const int col = (ct0 + c) * 16 + (lane & 15);
        const bool valid = col < n_cols;
        const int t = col / group;
        hd[c] = kvh * group + col % group;
        mrow[c] = b * q_len + t;
        nk[c] = valid ? pos0 + t + 1 : 0;
        load_q<DT>(qf[c], qbuf, qlo, mrow[c], hd[c], qd, d, valid, lane);
#pragma unroll
        for (int i = 0; i < DT; ++i) st[c].o[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
        st[c].m = -INFINITY;
        st[c].l = 0.f;
        last_key = max(last_key, nk[c]);
    }
    // the block range must be uniform: take the maximum over the columns
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) last_key = max(last_key, __shfl_xor(last_key, o, 64));
    const __bf16 *kbase = kc + ((size_t)b * kv + kvh) * (size_t)max_ctx * d;
    const __bf16 *vbase = vc + ((size_t)b * kv + kvh) * (size_t)max_ctx * d;
    const float scale = 1.0f / sqrtf((float)d);
    const int nblk = (last_key + 31) >> 5;
    // The wave's blocks are wave + 4 j, j < nw.  Two register sets used alternately: the next block's keys and values are on
    // their way while one is worked on (few waves share a SIMD here, so nobody else hides that latency); an index past
    // the wave's last block repeats it and is not used.
    const int nw = nblk > wave ? (nblk - wave + 3) >> 2 : 0;
    auto blk = [&](int j) { return nw > 0 ? wave + 4 * (j < nw ? j : nw - 1) : 0; };
    KVFrags<DT> f0, f1;
    load_kv<DT>(f0, kbase, vbase, blk(0), d, lane);
    for (int j = 0; j < nw; j += 2) {
        load_kv<DT>(f1, kbase, vbase, blk(j + 1), d, lane);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < CT; ++c) attn_block<DT, true>(st[c], qf[c], f0, blk(j), nk[c], scale, lane);
        __builtin_amdgcn_sched_barrier(0);
        load_kv<DT>(f0, kbase, vbase, blk(j + 2), d, lane);
        __builtin_amdgcn_sched_barrier(0);
        if (j + 1 < nw) {
#pragma unroll
            for (int c = 0; c < CT; ++c) attn_block<DT, true>(st[c], qf[c], f1, blk(j + 1), nk[c], scale, lane);
        }
    }
    // partial states to LDS
#pragma unroll
    for (int c = 0; c < CT; ++c) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) so[((wave * CT + c) * DT + dt) * 64 + lane] = st[c].o[dt];
        if (g == 0) {
            sml[((wave * CT + c) * 2 + 0) * 16 + (lane & 15)] = st[c].m;
            sml[((wave * CT + c) * 2 + 1) * 16 + (lane & 15)] = st[c].l;
        }
    }
    __syncthreads();
    // wave w finishes the (tile, slice) pairs w, w + 4, ...: the four partial states are merged in wave order
    for (int pr = wave; pr < CT * DT; pr += 4) {
        const int c = pr / DT, dt = pr % DT;
        if (nk[c] == 0) continue;
        float mm = -INFINITY;
#pragma unroll
        for (int w = 0; w < 4; ++w) mm = fmaxf(mm, sml[((w * CT + c) * 2 + 0) * 16 + (lane & 15)]);
        float den = 0.f;
        f32x4 num = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float mw = sml[((w * CT + c) * 2 + 0) * 16 + (lane & 15)];
            const float sc = (mw == -INFINITY) ? 0.f : __expf(mw - mm);
            den += sml[((w * CT + c) * 2 + 1) * 16 + (lane & 15)] * sc;
            num += so[((w * CT + c) * DT + dt) * 64 + lane] * sc;
        }
        const float inv = 1.0f / den;
        const int mt = mrow[c] >> 4, r = mrow[c] & 15;
        const int kidx = hd[c] * d + dt * 16 + 4 * g;
        const float o0 = num[0] * inv, o1 = num[1] * inv, o2 = num[2] * inv, o3 = num[3] * inv;
        const bf16x4 v = cvt4h(o0, o1, o2, o3);
        const size_t o = spd_act_index(mt, kidx >> 5, qd >> 5, ((int)gridDim.z * q_len + 15) >> 4) + spd_frag_elem(r, kidx & 31);
        *(bf16x4 *)(ahat + o) = v;
        if (alo) *(bf16x4 *)(alo + o) = cvt4h_lo(o0, o1, o2, o3, v);
    }
}

// ------------------------------------------------------------------------------------------
// taps (tests only): packed bf16 (hi [+ lo]) -> natural fp32
// ------------------------------------------------------------------------------------------
__global__ void k_unpack_act(const __bf16 *__restrict__ src, const __bf16 *__restrict__ lo, float *__restrict__ dst, int M,
                             int K_packed, int K_out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)M * K_out) return;
    const int m = (int)(i / K_out), k = (int)(i % K_out);
    const size_t o = spd_act_index(m >> 4, k >> 5, K_packed >> 5, (M + 15) >> 4) + spd_frag_elem(m & 15, k & 31);
    dst[i] = act_back(src[o]) + (lo ? act_back(lo[o]) : 0.f);
}
__global__ void k_bf16_to_f32(const __bf16 *__restrict__ src, const __bf16 *__restrict__ lo, float *__restrict__ dst,
                              int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = (float)src[i] + (float)lo[i];
}

inline unsigned cdiv(int64_t a, int64_t b) { return (unsigned)((a + b - 1) / b); }


// Number of K slices of a weight-streaming launch: 1 when there are enough pairs of n-tiles to
// occupy the chip, or half of it with at most four k-tiles for each of 16 waves (everything is requested at once
// then, and the second kernel that adds slices takes 4 us: down projection of the 7B shard, 128 pairs x 43 k-tiles,
// 5.0 + 3.4 -> 6.4 us, of the 13B shard, 160 x 54, 5.9 + 4.3 -> 8.6); otherwise about two workgroups of 8 waves per compute unit.
constexpr int GEMV_SLICE_W = 8;
constexpr int GEMV_MANY_PAIRS = 192;
inline bool gemv_whole(int n_pairs, int KT) { return n_pairs >= GEMV_MANY_PAIRS || (n_pairs >= 96 && KT >= 32 && KT <= 64); }
inline int gemv_slices(int n_pairs, int KT) {
    if (gemv_whole(n_pairs, KT)) return 1;
    int KS = (512 + n_pairs - 1) / n_pairs;
    const int ks_max = KT / (2 * GEMV_SLICE_W) > 0 ? KT / (2 * GEMV_SLICE_W) : 1;         // at least two k-tiles per wave
    if (KS > ks_max) KS = ks_max;
    while ((size_t)n_pairs * KS > (size_t)SPD_MAX_KPART && KS > 1) --KS;
    return KS;
}

// Launch shape of a projection.  At most 16 tokens: the weight-streaming kernel, one workgroup
// per pair of n-tiles when there are enough pairs to occupy the chip, otherwise K is also cut
// into KS slices (about two workgroups per compute unit) and a second small kernel adds them.
template <bool SPLIT, class Epi>
hipError_t launch_gemv(const spd_call &c, const __bf16 *Wp, const __bf16 *Xhi, const __bf16 *Xlo, int n_pairs, int KT,
                       const Epi &epi, int rows = 16) {
    const spd_dims &D = *c.D;
    float *kpart = (float *)(c.ws + D.ws_kpart);
    // (narrow groups never in slices: only k_gemv stores them by element, k_gemv_finish takes a group for 16 columns)
    if (rows != 16 || gemv_whole(n_pairs, KT)) {
        // one workgroup per pair, no slices
        if (KT >= 32) {
            // 16 waves share 512 VGPRs per lane and SIMD.  With as few as
            // 2 k-tiles per wave everything is requested at once, which is what a short kernel wants.
            constexpr int W = 16;
            hipLaunchKernelGGL((k_gemv<W, SPLIT, 0, Epi>), dim3(n_pairs, 1), dim3(W * 64), 0, c.s, Wp, Xhi, Xlo, KT,
                               1, kpart, rows, epi, NoParts());
        } else {
            constexpr int W = 8;
            hipLaunchKernelGGL((k_gemv<W, SPLIT, 0, Epi>), dim3(n_pairs, 1), dim3(W * 64), 0, c.s, Wp, Xhi, Xlo, KT,
                               1, kpart, rows, epi, NoParts());
        }
        return hipGetLastError();
    }
    constexpr int W = GEMV_SLICE_W;
    const int KS = gemv_slices(n_pairs, KT);
    if (KS <= 1) {
        hipLaunchKernelGGL((k_gemv<W, SPLIT, 0, Epi>), dim3(n_pairs, 1), dim3(W * 64), 0, c.s, Wp, Xhi, Xlo, KT, 1,
                           kpart, rows, epi, NoParts());
        return hipGetLastError();
    }
    hipLaunchKernelGGL((k_gemv<W, SPLIT, 1, Epi>), dim3(n_pairs, KS), dim3(W * 64), 0, c.s, Wp, Xhi, Xlo, KT, KS,
                       kpart, rows, epi, NoParts());
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_gemv_finish<Epi>), dim3(n_pairs), dim3(256), 0, c.s, kpart, KS, epi);
    return hipGetLastError();
}

// K-sliced launch for an epilogue that is linear in the accumulators (Epi::slice); no second kernel.
// Workgroups of 16 waves, about one per compute unit: every wave requests its whole share at once.
constexpr int QKV_SLICE_W = 16;
template <class Epi>
hipError_t launch_gemv_sliced(const spd_call &c, bool split, const __bf16 *Wp, const __bf16 *Xhi, size_t plane, int n_pairs,
                              int KT, int KS, const Epi &epi, const RawX &raw) {
    constexpr int W = QKV_SLICE_W;
    const __bf16 *Xlo = Xhi + plane;
    if (raw.x)
        hipLaunchKernelGGL((k_gemv<W, false, 2, Epi, SRC_X>), dim3(n_pairs, KS), dim3(W * 64), 0, c.s, Wp, Xhi, Xlo, KT, KS,
                           (float *)nullptr, 16, epi, raw);
    else if (split)
        hipLaunchKernelGGL((k_gemv<W, true, 2, Epi>), dim3(n_pairs, KS), dim3(W * 64), 0, c.s, Wp, Xhi, Xlo, KT, KS,
                           (float *)nullptr, 16, epi, NoParts());
    else
        hipLaunchKernelGGL((k_gemv<W, false, 2, Epi>), dim3(n_pairs, KS), dim3(W * 64), 0, c.s, Wp, Xhi, Xlo, KT, KS,
                           (float *)nullptr, 16, epi, NoParts());
    return hipGetLastError();
}

// 17 .. 512 tokens, short contractions: the skinny kernel, groups of MT m-tiles in grid.z.  KS > 1 only with MODE 2.
constexpr int SKINNY_W = 8;
template <int MT, bool SPLIT, int MODE, int NP = 1, bool KEEP = false, class Epi>
hipError_t launch_skinny_mt(const spd_call &c, const __bf16 *Wp, const __bf16 *Xhi, const __bf16 *Xlo, int n_pairs, int KT,
                            int KS, int n_mtiles, const Epi &epi) {
    constexpr int lds = SKINNY_W * NP * MT * 2 * 1024;
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [] {
        attr_err = hipFuncSetAttribute((const void *)k_skinny<SKINNY_W, MT, SPLIT, MODE, Epi, NP, KEEP>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    });
    if (attr_err != hipSuccess) return attr_err;
    // k-tiles in a rotated order, but front to back when there are more pairs than compute units (from HBM, 32 sequences: down
    // of 7B, 128 pairs x 344 k-tiles, 34.6 us front to back / 31.0 rotated, 160 x 216 24.4 / 22.2; but QKV, 384 x 128, 31.4 / 39.6)
    const unsigned rot_step = n_pairs <= 256 ? 5 : 0;
    hipLaunchKernelGGL((k_skinny<SKINNY_W, MT, SPLIT, MODE, Epi, NP, KEEP>), dim3(n_pairs / NP, KS, (n_mtiles + MT - 1) / MT), dim3(SKINNY_W * 64),
                       lds, c.s, Wp, Xhi, Xlo, KT, KS, n_mtiles, rot_step, epi);
    return hipGetLastError();
}
inline bool skinny_two_pairs(int n_pairs, int n_mtiles) { return n_pairs % 16 == 0 && n_mtiles >= 8; }      // (single activation planes)
template <int MODE = 0, class Epi>
hipError_t launch_skinny(const spd_call &c, bool split, const __bf16 *Wp, const __bf16 *Xhi, size_t plane, int n_pairs, int KT,
                         const Epi &epi, int KS = 1) {
    const int n_mtiles = (c.M + 15) / 16;
    const __bf16 *Xlo = Xhi + plane;
    if (n_mtiles <= 2)
        return split ? launch_skinny_mt<2, true, MODE>(c, Wp, Xhi, Xlo, n_pairs, KT, KS, n_mtiles, epi)
                     : launch_skinny_mt<2, false, MODE>(c, Wp, Xhi, Xlo, n_pairs, KT, KS, n_mtiles, epi);
    if (n_mtiles <= 4)
        return split ? launch_skinny_mt<4, true, MODE>(c, Wp, Xhi, Xlo, n_pairs, KT, KS, n_mtiles, epi)
                     : launch_skinny_mt<4, false, MODE>(c, Wp, Xhi, Xlo, n_pairs, KT, KS, n_mtiles, epi);
    // Two pairs and four m-tiles per workgroup instead of one and eight: as many workgroups, but 64 + 64 rows of operands drawn through a compute
    // unit's load path instead of 32 + 128.  Loads return in order, so that a launch takes at least the sum of what a unit reads: down of 128 tokens of
    // 70B (27 to 30 us) 0.46 MB of weights that two units of an XCD share, at 44 GB/s, 0.46 MB of activations from the L2 at 104 and 0.15 MB of slots at 27, 20 us.
    // The weights are asked for by two or more workgroups, on one XCD as long as their number per group of m-tiles is a multiple of 8.  us per call, one pair / two: 13B 333 tokens with the
    // kept sync point 125.1 / 121.3, 7B 500 122.2 / 115.8, 270 89.4 / 86.3, 70B 160 141.5 / 139.9.  Eight m-tiles, read by two workgroups at the same time, as
    // data that is read once: 70B 128 tokens 104.8 / 103.2 (kept sync point 107.6 / 105.1), 13B 74.4 / 71.1, 4-way 98.4 / 93.9, 7B 58.6 / 58.0.
    // (Seven m-tiles: 70B 97.7 / 98.7, 13B 70.8 / 70.2; fewer draw more than with one pair.)
    if constexpr (MODE == 0)
        if (!split && skinny_two_pairs(n_pairs, n_mtiles))
            return n_mtiles > 8 ? launch_skinny_mt<4, false, MODE, 2, true>(c, Wp, Xhi, Xlo, n_pairs, KT, KS, n_mtiles, epi)
                                : launch_skinny_mt<4, false, MODE, 2, false>(c, Wp, Xhi, Xlo, n_pairs, KT, KS, n_mtiles, epi);
    return split ? launch_skinny_mt<8, true, MODE>(c, Wp, Xhi, Xlo, n_pairs, KT, KS, n_mtiles, epi)
                 : launch_skinny_mt<8, false, MODE>(c, Wp, Xhi, Xlo, n_pairs, KT, KS, n_mtiles, epi);
}
// 17 .. 128 tokens, activations not split, large gate/up projections: the mid kernel and its finishing kernel.  It draws
// the HBM's rate better than the sliced GEMM; on what is small enough to stay in a cache the two are level or the GEMM is
// ahead.  Weights from HBM, us per layer, mid against slices: 88 MB (344 pairs x 128 k-tiles) 17 tokens 73.6 / 80.6,
// 64: 87.7 / 93.2, 128: 120 / 124; beyond 64 tokens also 71 MB (216 x 160) 86.5 / 88.3 at 65, 99.6 / 101.8 at 128, 45 MB
// (172 x 128) 74.9 / 75.8, 84.8 / 85.0; but 35 MB (108 x 160) 69.3 / 65.5, and 45 MB at 33 sequences 73.5 / 72.0.
// Returns false in *done when the shape is not its kind.
constexpr int SKINNY_MAX_MTILES = 32;      // beyond 512 tokens one launch of the LDS-tiled GEMM does without K slices
constexpr int MID_MAX_MTILES = 8;
constexpr int MID_MIN_TILES = 40 * 1024;         // (pairs of n-tiles) x (k-tiles): 2 KiB each
constexpr int MID_LONG_MIN_TILES = 20 * 1024;    // ... of calls of more than 64 tokens, with at least 128 pairs
// K slices the mid kernel would use for this shape, 0 when the shape is not its kind
inline int mid_slices(const spd_call &c, int n_pairs, int KT) {
    const spd_dims &D = *c.D;
    const int n_mtiles = (c.M + 15) / 16;
    const long tiles = (long)n_pairs * KT;
    if (n_mtiles <= 1 || n_mtiles > MID_MAX_MTILES) return 0;
    if (tiles < MID_MIN_TILES && !(n_mtiles > 4 && n_pairs >= 128 && tiles >= MID_LONG_MIN_TILES)) return 0;
    const int groups = (n_pairs + MID_PAIRS - 1) / MID_PAIRS, nst = (KT + MID_KB - 1) / MID_KB;
    // one round of workgroups (one fits a compute unit), at least four stages per slice
    int KS = 256 / groups;
    if (KS > nst / 4) KS = nst / 4;
    while (KS > 1 && (size_t)n_pairs * KS * n_mtiles > D.kpart_tiles) --KS;
    return KS < 2 ? 0 : KS;
}
template <class Epi>
hipError_t launch_mid(const spd_call &c, const __bf16 *Wp, const __bf16 *X, int n_pairs, int KT, const Epi &epi, bool *done) {
    const spd_dims &D = *c.D;
    const int n_mtiles = (c.M + 15) / 16;
    *done = false;
    const int KS = mid_slices(c, n_pairs, KT);
    if (KS == 0) return hipSuccess;
    const int groups = (n_pairs + MID_PAIRS - 1) / MID_PAIRS;
    f32x4 *kpart = (f32x4 *)(c.ws + D.ws_kpart);
    const dim3 grid(groups, KS), wg(MID_PAIRS * 64);
    if (n_mtiles <= 2) hipLaunchKernelGGL((k_mid<2>), grid, wg, 0, c.s, Wp, X, KT, KS, n_pairs, n_mtiles, kpart);
    else if (n_mtiles <= 4) hipLaunchKernelGGL((k_mid<4>), grid, wg, 0, c.s, Wp, X, KT, KS, n_pairs, n_mtiles, kpart);
    else hipLaunchKernelGGL((k_mid<8>), grid, wg, 0, c.s, Wp, X, KT, KS, n_pairs, n_mtiles, kpart);
    SPD_TRY(hipGetLastError());
    *done = true;
    return launch_mid_finish(c.s, kpart, KS, n_pairs, n_mtiles, epi);
}

// K slices of launch_sliced() (1: none) and the tiles they are made of.
inline int sliced_count(const spd_dims &D, int n_pairs, int KT, int n_mtiles, int *kind) {
    const int halves = ((2 * n_pairs + 15) / 16) * ((n_mtiles + 7) / 8);
    *kind = n_mtiles <= 4 ? 0 : (n_mtiles > 8 && (n_pairs >= 64 || halves >= 32) ? 2 : 1);      // 128 x 64, 128 x 128, 256 x 128
    const int bn = *kind == 2 ? 16 : 8, bm = *kind == 0 ? 4 : 8;
    const int tiles = ((2 * n_pairs + bn - 1) / bn) * ((n_mtiles + bm - 1) / bm);
    int KS = 256 / tiles;
    if (KS > 16) KS = 16;
    if (KS > KT / 8) KS = KT / 8;
    while (KS > 1 && (size_t)n_pairs * KS * n_mtiles > D.kpart_tiles) --KS;
    return KS;
}

// Projection in K slices: the LDS-tiled GEMM in one launch of (tiles x slices) workgroups, at most one per compute unit,
// that park their partial sums, and a finishing kernel that adds them in slice order and runs the epilogue.  For
// calls whose tiles alone leave most compute units idle.  Tile shape: 128 x 64 up to 64 tokens, 256 x 128 beyond 128
// tokens where there are 64 pairs of n-tiles or 32 such tiles, 128 x 128 otherwise (main kernel, us, 128 x 128 against 256 x 128: gate/up of
// the 70B shard 256 tokens 48.7 / 44.5, 512: 84 / 72; its QKV projection on pairs 128 tokens 10.8 / 17, 256: 15 / 22.5,
// 512: 23.3 / 24.6).  Slices: as many as fit the round of 256 with 8 k-tiles each (beyond 16 the partial sums cost more
// than the idle compute units: gate/up of the 13B shard, 128 tokens, 18 / 13 slices: 13.8 + 9.3 / 12.6 + 5.1 us).
// Returns false in *done when fewer than two slices come of it or they do not fit the workspace.
template <class Epi>
hipError_t launch_sliced(const spd_call &c, bool split, const __bf16 *Wp, const __bf16 *Xhi, size_t plane, int n_pairs, int KT,
                         const Epi &epi, bool *done) {
    const spd_dims &D = *c.D;
    const int n_mtiles = (c.M + 15) / 16;
    int kind;
    const int KS = sliced_count(D, n_pairs, KT, n_mtiles, &kind);
    *done = KS > 1;
    if (!*done) return hipSuccess;
    EpiPark park;
    park.KS = KS; park.n_mtiles = n_mtiles; park.kpart = (f32x4 *)(c.ws + D.ws_kpart);
    const __bf16 *Xlo = Xhi + plane;
#define SPD_SLICED(G)                                                                                              \
    SPD_TRY((split ? launch_gemm_lds_cfg<G, true>(c, Wp, Xhi, Xlo, n_pairs, KT, park, 0, 1, -1, KS)                \
                   : launch_gemm_lds_cfg<G, false>(c, Wp, Xhi, Xlo, n_pairs, KT, park, 0, 1, -1, KS)))
    if (kind == 0) SPD_SLICED(GemmSmall);
    else if (kind == 1) SPD_SLICED(GemmSquare);
    else SPD_SLICED(GemmHalf);
#undef SPD_SLICED
    return launch_mid_finish(c.s, (const f32x4 *)park.kpart, KS, n_pairs, n_mtiles, epi);
}

// 17 .. 512 tokens, short contractions: the skinny kernel with the whole epilogue is done before K slices and the launch that
// adds them are.  Beyond 128 tokens (one workgroup per compute unit: 128 KiB of LDS each) its workgroups should fill half a
// round of the chip and not begin a second one, unless the contraction is very short.  Skinny against slices, weights
// from HBM, us per layer:
//   gate/up, 24 tokens: 44 x 32 (pairs x k-tiles) 33 / 37, 86 x 64 38 / 40, 128 x 96 48.5 / 50, 216 x 160 62 / 66; but 108 x 160 53.5 / 52.4;
//     64 tokens: 88 x 32 41 / 43, 172 x 64 52 / 56; but 44 x 64 and 64 x 96 equal / + 1 %; 128 tokens: 44 .. 176 x 32 - 4 .. - 6 %, x 64 + 1 .. + 4 %
//   QKV on pairs of planes (twice the k-tiles): 24 tokens x 32 - 10 %, x 64 - 3 .. - 9 %, x 128 + 3 %
//   decode QKV of 17 .. 32 sequences that fill the chip: 192 x 64 - 10 %, 240 x 160 - 6 %; 320 x 256 + 1 %
//   down, 200 tokens: 128 x 43 - 8 %, 96 x 64 - 11 %, 128 x 86 - 5 %, 96 x 128 equal, 160 x 108 + 12 %; 384: 128 x 43 - 3 %, 128 x 86 + 6 %
inline bool skinny_first(int n_pairs, int KT, bool split, int n_mtiles) {
    const int kp = split ? 2 * KT : KT, wgs = n_pairs * ((n_mtiles + 7) / 8);
    if (n_mtiles <= 2) return kp <= 128 || (!split && KT <= 160 && n_pairs >= 128);
    if (n_mtiles <= 4) return kp <= 32 || (kp <= 64 && n_pairs >= 48);
    if (n_mtiles <= 8) return kp <= 32;
    return (kp <= 48 && wgs <= 512) || (kp <= 96 && wgs >= 128 && wgs <= 256);
}

inline int square_tiles(int n_pairs, int n_mtiles) { return (2 * n_pairs + 7) / 8 * ((n_mtiles + 7) / 8); }      // of 128 x 128

// The down projection of 257 to 512 tokens, where it is not the skinny kernel's: 128 x 128 tiles over the whole of K, and the closing sync point a launch
// of its own, instead of slices and a sync point in the launch that adds them: a slice's rows are written and read once more.  At most one
// round of the chip and at least a third of one.  A tile takes 0.3 us per k-tile whatever the number of tiles, slices a part of that and a time that goes with
// the rows there are: the more slices, the longer K and the fuller the groups of 8 m-tiles, the better for them.  us per call, slices / this: 4 or 5 slices, groups full:
// 96 pairs x 64 k-tiles 102.7 / 102.0, x 96 128.2 / 131.9, x 128 134.0 / 146.0, x 256 189.8 / 225.6, 128 x 86 140.5 / 143.1, 160 x 108 148.4 / 154.2; 272 tokens (5.7 m-tiles a
// group) 128 x 86 116.4 / 113.7, 160 x 108 136.4 / 136.5, 128 x 172 180.3 / 186.6; 3 slices, full: 144 x 96 148.0 / 146.8, 160 x 108 179.6 / 180.0, x 216 278.9 / 293.8; 400
// tokens 161.1 / 159.0, x 216 256.6 / 260.0; 2 slices: 256 x 112 400 tokens 196.8 / 188.7, 512 218.5 / 216.6, x 224 334.1 / 332.2, but 384 tokens 184.0 / 186.3, 304.4 / 309.4.
// Pairs of planes count twice (128 x 86, 272 to 512 tokens 0.7 .. 4.6 % slower in tiles, 160 x 108 -1.5 .. + 5.4, 256 x 112 -2 .. + 1.7 as above).
// (200 tokens of 70B 156.4 / 161.4; instead of the skinny kernel, 7B 300 and 500: 87.1 / 89.6, 121.1 / 124.0.)
inline bool down_whole(const spd_dims &D, int n_pairs, int KT, bool split, int n_mtiles) {
    const int tiles = square_tiles(n_pairs, n_mtiles), groups = (n_mtiles + 7) / 8;
    if (n_mtiles <= 16 || n_mtiles > SKINNY_MAX_MTILES || tiles < 96 || tiles > 256 || !spd_gemm_fits(KT) ||
        skinny_first(n_pairs, KT, split, n_mtiles))
        return false;
    int kind;
    const int KS = sliced_count(D, n_pairs, KT, n_mtiles, &kind);
    if (KS <= 1) return true;
    if (KS == 2) return groups != 3 || n_mtiles < 23;
    return (split ? 2 * KT : KT) <= (KS == 3 ? 104 : 64) + 20 * (8 * groups - n_mtiles) / groups;
}

// Projection of a call of any size: the weight-streaming kernel up to 16 tokens; up to 512 tokens the skinny kernel for short
// contractions and K slices of the LDS-tiled GEMM for the others; slices beyond for a call of one chain whose tiles leave half of the compute units idle (the QKV projection of the
// 70B shard, 1000 tokens: 6 slices 37 us, 160 x 256 tiles in 8 slices 58); one launch of the GEMM otherwise.  The skinny
// kernel also takes what is left with a single slice.
template <class Epi>
hipError_t launch_proj(const spd_call &c, bool split, const __bf16 *Wp, const __bf16 *Xhi, size_t plane, int n_pairs, int KT,
                       const Epi &epi) {
    const int n_mtiles = (c.M + 15) / 16;
    const __bf16 *Xlo = Xhi + plane;
    if (n_mtiles == 1)
        return split ? launch_gemv<true>(c, Wp, Xhi, Xlo, n_pairs, KT, epi) : launch_gemv<false>(c, Wp, Xhi, Xlo, n_pairs, KT, epi);
    if ((n_mtiles <= SKINNY_MAX_MTILES && skinny_first(n_pairs, KT, split, n_mtiles)) || !spd_gemm_fits(KT))
        return launch_skinny(c, split, Wp, Xhi, plane, n_pairs, KT, epi);
    if (!c.chained) {
        bool done = false;
        SPD_TRY(launch_sliced(c, split, Wp, Xhi, plane, n_pairs, KT, epi, &done));
        if (done) return hipSuccess;
    }
    if (n_mtiles <= SKINNY_MAX_MTILES) {
        // no slices: half a round of 256 x 128 tiles by themselves, the skinny kernel below that
        const int halves = ((2 * n_pairs + 15) / 16) * ((n_mtiles + 7) / 8);
        if (n_mtiles > 8 && halves >= 128)
            return split ? launch_gemm_lds_cfg<GemmHalf, true>(c, Wp, Xhi, Xlo, n_pairs, KT, epi)
                         : launch_gemm_lds_cfg<GemmHalf, false>(c, Wp, Xhi, Xlo, n_pairs, KT, epi);
        return launch_skinny(c, split, Wp, Xhi, plane, n_pairs, KT, epi);
    }
    if constexpr (Epi::kLong) return split ? launch_gemm_lds<true>(c, Wp, Xhi, Xlo, n_pairs, KT, epi) : launch_gemm_lds<false>(c, Wp, Xhi, Xlo, n_pairs, KT, epi);
    else return hipErrorInvalidValue;         // epilogues that carry a sync point: calls of up to 512 tokens
}

// Does the O projection's epilogue perform a kept attention sync point (one rank, TP block)?  In the skinny kernel, as long
// as its workgroups (128 KiB of LDS each, one per compute unit) come to two rounds of the chip at most; a rank-sum of its
// own beyond.  Whole layer, weights from HBM, us, in the epilogue / kernel of its own: 70B 129 tokens 135.6 / 143.1, 256 (512
// workgroups) 165.4 / 172.3, 384 (768) 211.8 / 210.0, 512 263.2 / 252.7; 13B 129 tokens 88.0 / 93.5, 384 (480) 129.7 / 132.2, 512
// (640) 157.4 / 157.4; 7B 129 tokens 76.5 / 80.2, 512 (512) 126.4 / 132.8; up to 128 tokens 2 .. 4 us less on every shard.  With fewer slots the
// kernel of its own has less to read: 7B 4-way (32 k-tiles) 256 tokens 104.0 / 111.4, 384 139.7 / 139.1, 512 156.6 / 162.3, but 13B
// 4-way (40) 256 142.5 / 141.6, 333 155.8 / 155.3.
inline bool sync_in_o(int n_pairs, int KT, int tp, int n_mtiles) {
    return n_mtiles <= 8 || (n_mtiles <= SKINNY_MAX_MTILES && n_pairs * ((n_mtiles + 7) / 8) <= 512 && KT <= 8 * tp);
}

// Does a decode step's O projection merge the attention's splits itself, instead of a kernel in between?  Every workgroup then reads
// all states, so only where that is 200 KB at most: a quad of features per thread, or up to three of up to 8 splits.  us per call, kernel of its
// own / in the projection: 7B 1 sequence of 2000 positions 38.8 / 37.5, 2: 39.3 / 37.9, 4 (512 quads, 131 KB): 41.4 / 40.5, 1 of 16000 47.3 / 45.6; 70B 1 of
// 4096 (32 splits, 131 KB) 60.8 / 59.8; three quads: 13B 8 of 4096, 4 layers 216.0 / 213.5, 7B 6 of 3000 42.7 / 42.0, 70B 4 of 1000 57.5 / 56.6 (every
// thread with the factors of its own quads: 219.1 / 225.7, 8 sequences of 7B 40.5 / 41.4).
constexpr int GEMV_MERGE_W = 8;
inline bool merge_in_o(const spd_call &c, int n_pairs, int KT, int n_splits) {
    const int quads = c.M * KT * 8;
    if (c.M > 16 || c.sp_a) return false;
    if (KT > GEMV_MERGE_W * GEMV_MERGE_TILES || n_pairs < 96) return false;
    if (quads > GEMV_MERGE_W * 64 && (quads > 3 * GEMV_MERGE_W * 64 || n_splits > 8)) return false;
    return (int64_t)quads * n_splits * 16 <= 200 * 1024;
}

// The output projection's contraction is short (a rank's heads): up to 128 tokens the skinny kernel with the whole epilogue
// beats slices and their finishing kernel, and beyond it beats tiles as long as it has two pairs and four m-tiles per workgroup and these come to two and a half
// rounds of the chip (us per call, skinny / 128 x 128 tiles, by workgroups: 512: 70B 129 tokens 124.2 / 128.6, 256 149.3 / 153.6, 7B 400 97.4 / 101.4, 4-way 512
// 145.2 / 149.7; 640: 13B 400 124.2 / 125.6, 512 140.2 / 141.6; but 768: 70B 300 171.4 / 170.7, 384 behind 500 positions 193.0 / 191.3; 1024: 512 behind
// 1536 235.4 / 230.6); with one pair and eight m-tiles, below two rounds (tiles of 256 x 128, main kernel, us, skinny / tiles: 70B 192 tokens 15.8 / 14.7, 512: 30.9 / 17.2).
// Tiles of 128 x 128 as long as these come to one round, 256 x 128 beyond (such a launch is its reads of X and its writes, and a part of the compute units draws a
// part of what the chip does; us per call, 256 x 128 / 128 x 128: 70B 256 tokens 161.7 / 153.6, 300 185.6 / 176.2, 512 behind 1536 245.0 / 237.4).
// With a kept sync point in its epilogue (MID) always the skinny kernel.
// `merge`: the splits' states of a decode step whose O projection merges them itself (see merge_in_o()).
template <bool MID>
hipError_t launch_o(const spd_call &c, bool split, const __bf16 *Wp, const __bf16 *Xhi, size_t plane, int n_pairs, int KT,
                    const EpiOT<MID> &epi, const AttnParts &merge) {
    const int n_mtiles = (c.M + 15) / 16, wgs = n_pairs * ((n_mtiles + 7) / 8);
    const __bf16 *Xlo = Xhi + plane;
    if (n_mtiles == 1 && merge.o) {
        constexpr int W = GEMV_MERGE_W;
        static std::once_flag once;
        static hipError_t attr_err = hipSuccess;
        std::call_once(once, [] {
            for (const void *k : {(const void *)k_gemv<W, false, 0, EpiOT<MID>, SRC_MERGE>, (const void *)k_gemv<W, false, 0, EpiOT<MID>, SRC_MERGE3>})
                if (attr_err == hipSuccess)
                    attr_err = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, W * GEMV_MERGE_TILES * 1024);
        });
        if (attr_err != hipSuccess) return attr_err;
        if (c.M * KT * 8 <= W * 64)
            hipLaunchKernelGGL((k_gemv<W, false, 0, EpiOT<MID>, SRC_MERGE>), dim3(n_pairs, 1), dim3(W * 64), KT * 1024, c.s, Wp, Xhi, Xlo, KT, 1,
                               (float *)nullptr, 16, epi, merge);
        else
            hipLaunchKernelGGL((k_gemv<W, false, 0, EpiOT<MID>, SRC_MERGE3>), dim3(n_pairs, 1), dim3(W * 64), KT * 1024, c.s, Wp, Xhi, Xlo, KT, 1,
                               (float *)nullptr, 16, epi, merge);
        return hipGetLastError();
    }
    if (n_mtiles == 1)
        return split ? launch_gemv<true>(c, Wp, Xhi, Xlo, n_pairs, KT, epi) : launch_gemv<false>(c, Wp, Xhi, Xlo, n_pairs, KT, epi);
    if (n_mtiles <= 8 || (n_mtiles <= SKINNY_MAX_MTILES && (MID || wgs < (!split && skinny_two_pairs(n_pairs, n_mtiles) ? 641 : 512))) || !spd_gemm_fits(KT))
        return launch_skinny(c, split, Wp, Xhi, plane, n_pairs, KT, epi);
    if constexpr (MID) {
        return hipErrorInvalidValue;         // (see sync_in_o())
    } else {
        if (n_mtiles <= SKINNY_MAX_MTILES && square_tiles(n_pairs, n_mtiles) <= 256)
            return split ? launch_gemm_lds_cfg<GemmSquare, true>(c, Wp, Xhi, Xlo, n_pairs, KT, epi)
                         : launch_gemm_lds_cfg<GemmSquare, false>(c, Wp, Xhi, Xlo, n_pairs, KT, epi);
        if (n_mtiles <= SKINNY_MAX_MTILES)
            return split ? launch_gemm_lds_cfg<GemmHalf, true>(c, Wp, Xhi, Xlo, n_pairs, KT, epi)
                         : launch_gemm_lds_cfg<GemmHalf, false>(c, Wp, Xhi, Xlo, n_pairs, KT, epi);
        return split ? launch_gemm_lds<true>(c, Wp, Xhi, Xlo, n_pairs, KT, epi) : launch_gemm_lds<false>(c, Wp, Xhi, Xlo, n_pairs, KT, epi);
    }
}

constexpr int PREP_ROWS_WGS = 512;       // workgroups of the row-wise preparation kernel (two per compute unit)
// workgroups (one compute unit each) of a chain's rank-sum in a two-chain prefill.  70B shard, 4 x 2048 tokens, us per
// layer with all sync points dropped / all kept: 64: 2459 / 2790, 96: 2408 / 2702, 112: 2374 / 2699, 128: 2367 / 2552,
// 144: 2442 / 2712, 192: 2426 / 2718; k_prep_rows: 2454 / 2690
constexpr int PREP_CU_WGS = 128;
// chunking of the sum-of-squares partials written by prep(): k-tiles per wave of k_prep (one partial for its four waves), enough
// waves to occupy the chip at every call size; 256 features in the row-wise kernels
inline int prep_tpw(int M) { return M <= 64 ? 1 : (M <= 512 ? 2 : 8); }
inline int prep_nch(int h, int M) {
    if (M <= PREP_BY_WAVE) return (int)cdiv(h / 32, prep_tpw(M));
    return prep_tpw(M) == 8 && h % 256 == 0 ? h / 256 : (int)cdiv(h / 32, 4 * prep_tpw(M));
}

}  // namespace

namespace spd_bf16 {

hipError_t prep(const spd_call &c, const float *base, const float *slots, int n_slots, float *out, const float *gain,
                bool want_xhat, int which, const float *bias) {
    const spd_dims &D = *c.D;
    const int tpw = prep_tpw(c.M), nch = prep_nch(D.h, c.M);
    __bf16 *xhat = want_xhat ? (__bf16 *)(c.ws + (which ? D.ws_xhat2 : D.ws_xhat)) : nullptr;
    __bf16 *xlo = (want_xhat && (which ? c.sp_m : c.sp_x)) ? xhat + D.pl_x : nullptr;
    float *ss = want_xhat ? (float *)(c.ws + (which ? D.ws_ss2 : D.ws_ss1)) : nullptr;
    if (n_slots == 0 && out == base && !bias) out = nullptr;   // nothing to rewrite
    if (!c.on(SPD_STAGE_PREP)) return hipSuccess;
    spd_stage_scope prof(c, SPD_STAGE_PREP);
    // (two adjacent chunks per workgroup, 2 KiB per row, measured slower: 547 against 505 us on the 70B prefill shape)
    // a chain of a two-chain prefill summing the slots of a sync point: few workgroups, a compute unit each
    if (tpw == 8 && D.h % 256 == 0 && c.chained && base && out && (n_slots == 8 || n_slots == 4)) {
        return n_slots == 8 ? launch_prep_cu<8>(c.s, PREP_CU_WGS, base, slots, c.slot_stride, out, gain, xhat, xlo, ss, c.M, D.h,
                                                D.m_pad, bias)
                            : launch_prep_cu<4>(c.s, PREP_CU_WGS, base, slots, c.slot_stride, out, gain, xhat, xlo, ss, c.M, D.h,
                                                D.m_pad, bias);
    }
    if (tpw == 8 && D.h % 256 == 0)
    {
        const int n_chunks = D.h / 256, n_items = n_chunks * (int)cdiv(c.M, 16);
        if (n_slots > 0)
            hipLaunchKernelGGL((k_prep_rows<1, true>), dim3(n_items < PREP_ROWS_WGS ? n_items : PREP_ROWS_WGS), dim3(256), 0, c.s, base,
                               slots, n_slots, c.slot_stride, out, gain, xhat, xlo, ss, c.M, D.h, D.m_pad, bias, n_chunks, n_items);
        else
            hipLaunchKernelGGL((k_prep_rows<1, false>), dim3(n_items < 4 * PREP_ROWS_WGS ? n_items : 4 * PREP_ROWS_WGS), dim3(256), 0, c.s,
                               base, slots, 0, c.slot_stride, out, gain, xhat, xlo, ss, c.M, D.h, D.m_pad, bias, n_chunks, n_items);
    }
    else
        hipLaunchKernelGGL(k_prep, dim3(c.M <= PREP_BY_WAVE ? cdiv(nch, 4) : nch, cdiv(c.M, 16)), dim3(256), 0, c.s, base, slots, n_slots,
                           c.slot_stride, out, gain, xhat, xlo, ss, c.M, D.h, tpw, D.m_pad, bias);
    return hipGetLastError();
}

int prep_chunks(const spd_call &c) { return prep_nch(c.D->h, c.M); }

namespace {
// weights of projection `i` (0 QKV, 1 O, 2 gate/up, 3 down) and the factor 2^-k that undoes their power of two
struct ProjW {
    const __bf16 *w;
    const float *wsc;
};
inline ProjW proj_weights(const spd_call &c, const char *w, int i) {
    const spd_dims &D = *c.D;
    const size_t off[4] = {D.w_qkv, D.w_o, D.w_g, D.w_d};
    ProjW p;
    p.w = (const __bf16 *)(w + off[i]);
    p.wsc = (const float *)(w + D.w_scale) + i;
    return p;
}
// K slices of the QKV projection that the attention kernel adds up itself, 1: none.
// A decode step whose QKV projection has too few column tiles to occupy the chip: K slices with the linear epilogue (at
// most SPD_MAX_QKV_SLICES), whose partial rows the attention kernel adds itself.  Up to 16 sequences about 240
// workgroups of 16 waves, at least two k-tiles per wave; more of them, workgroups of the skinny kernel's 8 waves (two fit a compute unit): as many
// slices as fill their rounds of the chip best, up to two of them, the fewer among equals.  us per call of 24 / 48 sequences: 70B (40 pairs) 8 slices
// (1.25 rounds) 71.1 / 76.4, 6 (0.94) 70.0 / 75.1; 7B 4-way (96) 2 (0.75) 80.3 / 85.5, 5 (1.88) 80.2 / 85.3, at 17 and 32 53.8 / 57.9 and 53.4 / 57.2;
// 132 pairs 2 (1.03) 69.7 / 81.6, 3 (1.55) 66.2 / 77.7; 160 2 (1.25) 64.3 / 78.2, 3 (1.88) 61.3 / 74.8; level: 7B (48) 8 (1.5) / 5 (0.94), 13B (60)
// 8 (1.88) / 4 (0.94), 4-way (120) 4 / 2, 72 pairs 3 (0.84) / 7 (1.97).
// (Also where gemv_whole() would contract K in one launch: the slices cost no second kernel here.  hidden 2048, 96 pairs,
// slices / whole, us per layer: 4 sequences of 4000 positions 52 / 53.6, 8: 67.5 / 70, 16: 102 / 104.5.)
int qkv_slices_wanted(int pairs) {
    int best = 2;
    auto fill = [&](int KS) { return KS * pairs / (double)((KS * pairs + 255) / 256); };        // workgroups per round
    for (int KS = 3; KS <= SPD_MAX_QKV_SLICES && KS * pairs <= 512; ++KS)
        if (fill(KS) > fill(best)) best = KS;
    return best;
}
}  // namespace

bool down_in_tiles(const spd_dims &D, int tokens, bool split) { return down_whole(D, D.h / 32, D.f_pad / 32, split, (tokens + 15) / 16); }

constexpr int prefill_lds(int DT, int CT) { return 4 * CT * DT * 64 * 16 + 4 * CT * 2 * 16 * 4; }

hipError_t prefill_workgroups(int head_dim, int *n) {
    const void *f;
    switch (head_dim) {
        case 32: f = (const void *)k_attn_prefill<2, 1>; break;
        case 64: f = (const void *)k_attn_prefill<4, 1>; break;
        case 96: f = (const void *)k_attn_prefill<6, 1>; break;
        case 128: f = (const void *)k_attn_prefill<8, 1>; break;
        default: return hipErrorInvalidValue;
    }
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(n, f, 256, prefill_lds(head_dim / 16, 1));
}

// A step goes through the caches of all of the context's layers before it comes to a layer's again, whether its program calls the model or walks the
// blocks (the weights are read past the chip's caches, 256 MB, anyway).  From 256 MB on nothing is found again; us per layer, block calls walking that
// many layers, kept / past the caches: 70B 16 of 4096, 12 layers (403 MB) 61.5 / 60.4, 7B 8 of 4000, 8 (524 MB) 43.3 / 41.8, 4 of 2048, 32 (537 MB)
// 34.8 / 34.1, 13B 1 of 4096, 40 (419 MB) 36.9 / 35.9, 16 of 4000, 6 (983 MB) 69.4 / 66.0; level from 295 to 335 MB.  Of a context of few layers below
// that, repeated, they are: 70B 16 of 4096, 4 (134 MB) level, 16 of 1000, 16 (131 MB) 58.9 / 59.0, 7B 1 of 2048, 32 (134 MB) 31.9 / 32.0, 32 of 500, 8 (262
// MB) 46.2 / 47.0, 13B 8 of 4096, 3 (252 MB) 49.2 / 52.0.  But such a context stands for a slice of a model, whose caches are cold: with three such in
// turn one layer of 70B 48 of 3000 (74 MB) 90.5 / 88.0, 13B 16 of 4000 (164 MB) 68.9 / 64.8, 7B 64 of 1000 (131 MB) 74.3 / 66.8, four of 70B 16 of 4096
// (134 MB) 234.4 / 232.6 a call, and below 64 MB level or worse (one of 7B 8 of 4000 42.4 / 43.4, 13B 8 of 2000 44.4 / 44.9): the line lies at 64 MB.
bool decode_past_caches(const spd_dims &D, const int32_t *positions, int sequences) {
    int64_t keys = 0;
    for (int i = 0; i < sequences; ++i) keys += positions[i];
    return 4.0 * D.kv * D.d * D.n_layers * (double)keys >= 64.0 * (1 << 20);
}

int decode_qkv_slices(const spd_dims &D, int sequences) {
    const int n_mtiles = (sequences + 15) / 16, qkv_pairs = D.nqkv / 32;
    int qkv_slices = 1;
    if (n_mtiles <= 4 && qkv_pairs < GEMV_MANY_PAIRS) {
        const int want = n_mtiles == 1 ? (240 + qkv_pairs - 1) / qkv_pairs : qkv_slices_wanted(qkv_pairs);
        qkv_slices = want < 2 ? 2 : (want > SPD_MAX_QKV_SLICES ? SPD_MAX_QKV_SLICES : want);
        const int most = D.h / 32 / (2 * (n_mtiles == 1 ? QKV_SLICE_W : SKINNY_W));
        if (qkv_slices > most) qkv_slices = most > 1 ? most : 1;
        while (qkv_slices > 1 && (size_t)qkv_slices * 16 * n_mtiles * D.nqkv > (size_t)SPD_MAX_KPART * 512) --qkv_slices;
    }
    return qkv_slices;
}
static int decode_qkv_slices(const spd_call &c) { return c.q_len == 1 ? decode_qkv_slices(*c.D, c.M) : 1; }

// A block call of a decode step of up to 8 sequences whose QKV projection runs in slices takes the residual stream itself: no launch for
// the first norm's elementwise part, for twice the activation bytes.  us per call, launch / this: 7B 1 sequence 37.6 / 35.5, 4: 40.5 / 38.1; 13B 8: 44.4 /
// 42.9, 4-way 65.5 / 64.1; 70B 1: 57.6 / 55.7, 4-way 91.8 / 89.6.
// Not beyond 8 sequences (with weights from HBM 16 of 70B, 4 layers, 252.1 / 253.8), nor beyond one round of the chip (7B 4-way, 288
// workgroups, 4: 51.6 / 52.1, 8: 55.3 / 57.0).
// Not in a model call, whose other blocks get their first norm from the block before: 2 us once, and the norm's factor, applied to the slices'
// sum instead of every slice, is another order of 32-bit operations, which through the fp16 activations of the blocks that follow
// changes the call's output by as much as its rounding (13B, 8 sequences, four layers, slots: 6.5e-4 of an error of 7.4e-4
// on either side).
bool qkv_reads_x(const spd_call &c) {
    if (c.q_len != 1 || c.M > 8 || c.sp_x) return false;
    const int KS = decode_qkv_slices(c);
    return KS > 1 && KS * (c.D->nqkv / 32) <= 256;
}

hipError_t attention_half(const spd_call &c, const char *w, char *kvc, const float *x, int spd, float *slot,
                          const spd_mid_sync *mid, bool *mid_done) {
    const spd_dims &D = *c.D;
    const int M = c.M, qd = D.q * D.d;
    const __bf16 *xhat = (const __bf16 *)(c.ws + D.ws_xhat);
    __bf16 *qbuf = (__bf16 *)(c.ws + D.ws_q), *ahat = (__bf16 *)(c.ws + D.ws_ahat);
    __bf16 *alo = c.sp_a ? ahat + D.pl_a : nullptr;
    __bf16 *qlo = qbuf + D.pl_a;
    __bf16 *kc = (__bf16 *)kvc, *vc = (__bf16 *)(kvc + D.kv_v);
    float *ybuf = (float *)(c.ws + D.ws_y);
    const ProjW wqkv = proj_weights(c, w, 0), wo = proj_weights(c, w, 1);

    const int n_mtiles = (M + 15) / 16, qkv_pairs = D.nqkv / 32, qkv_slices = decode_qkv_slices(c);
    const bool fused_q = qkv_slices > 1;
    float *qkvp = (float *)(c.ws + D.ws_kpart);
    RawX raw = {};
    if (fused_q) {
        if (c.raw_x) {
            raw.x = c.raw_x; raw.gain = (const float *)(w + D.w_g1);
            raw.ss = (float *)(c.ws + D.ws_ss1);           // (h / 32 rows of at least 16 tokens: room for the slices)
        }
        EpiQKVPart e1;
        e1.M = M; e1.q_len = c.q_len; e1.q = D.q; e1.kv = D.kv; e1.d = D.d; e1.h = D.h; e1.nqkv = D.nqkv;
        e1.nch = c.nch1; e1.m_pad = D.m_pad; e1.part_rows = 16 * n_mtiles; e1.eps = D.eps;
        e1.ss = (const float *)(c.ws + D.ws_ss1);
        e1.cosT = (const float *)(c.ws + D.ws_cos); e1.sinT = (const float *)(c.ws + D.ws_sin);
        e1.wsc = wqkv.wsc;
        e1.part = qkvp; e1.P = c.pos;
        if (c.on(SPD_STAGE_QKV)) {
            spd_stage_scope prof(c, SPD_STAGE_QKV);
            if (n_mtiles == 1)
                SPD_TRY(launch_gemv_sliced(c, c.sp_x, wqkv.w, xhat, D.pl_x, qkv_pairs, D.h / 32, qkv_slices, e1, raw));
            else
                SPD_TRY(launch_skinny<2>(c, c.sp_x, wqkv.w, xhat, D.pl_x, qkv_pairs, D.h / 32, e1, qkv_slices));
        }
    } else {
        EpiQKV e1;
        e1.M = M; e1.q_len = c.q_len; e1.q = D.q; e1.kv = D.kv; e1.d = D.d; e1.h = D.h; e1.max_ctx = D.max_ctx;
        e1.nch = c.nch1; e1.m_pad = D.m_pad; e1.eps = D.eps;
        e1.ss = (const float *)(c.ws + D.ws_ss1);
        e1.cosT = (const float *)(c.ws + D.ws_cos); e1.sinT = (const float *)(c.ws + D.ws_sin);
        e1.wsc = wqkv.wsc;
        e1.qbuf = qbuf; e1.qlo = qlo; e1.kc = kc; e1.vc = vc; e1.P = c.pos;
        if (c.on(SPD_STAGE_QKV)) {
            spd_stage_scope prof(c, SPD_STAGE_QKV);
            // decode of 17 .. 64 sequences that fills the chip: one launch of the skinny kernel. After slices and their finishing
            // kernel the attention kernel waits longer for the appended keys too (192 pairs x 128 k-tiles, 64 sequences:
            // 13.4 + 15.0 and attention 21.4 us; skinny 26.0 and 16.7; 240 x 160, us per layer, 33 sequences 131 / 125.5, 64: 159 / 150; 320 x
            // 256 the other way, 393 / 404)
            if (c.q_len == 1 && n_mtiles > 1 && n_mtiles <= 4 && !c.sp_x && D.h / 32 <= 160)
                SPD_TRY(launch_skinny(c, false, wqkv.w, xhat, D.pl_x, qkv_pairs, D.h / 32, e1));
            else
                SPD_TRY(launch_proj(c, c.sp_x, wqkv.w, xhat, D.pl_x, qkv_pairs, D.h / 32, e1));
        }
    }

    spd_stage_begin(c, SPD_STAGE_EMPTY);      // (timers only) an empty bracket between two kernels of the block
    spd_stage_end(c, SPD_STAGE_EMPTY);
    const int DT = D.d / 16;
    AttnParts parts = {};
    bool merge_o = false;
    if (c.q_len == 1) {
        // key blocks per workgroup (4 waves, so multiples of 4): the number of rounds the launch takes
        // on 256 compute units times the length of a round, a round costing about 5 blocks' worth of
        // start-up besides its blocks
        const int nblk = (c.max_pos_end + 31) / 32, units = D.kv * c.batch;
        int splits = 1;
        long best = -1;
        for (int per = 4; per <= 64; per += 4) {
            int sp = (nblk + per - 1) / per;
            if (sp < 1) sp = 1;
            if (sp > SPD_MAX_SPLITS) continue;
            const long rounds = ((long)sp * units + 255) / 256, cost = rounds * (per + 5);
            if (best < 0 || cost < best) {
                best = cost;
                splits = sp;
            }
        }
        parts.o = (float *)(c.ws + D.ws_apart);
        parts.units = units; parts.n_splits = splits; parts.group = D.group; parts.d = D.d;
        parts.by_quads = Divider::by(D.d / 4); parts.by_heads = Divider::by(D.q); parts.by_group = Divider::by(D.group);
        merge_o = merge_in_o(c, D.h / 32, qd / 32, splits);
    }
    spd_stage_begin(c, SPD_STAGE_ATTN);
    if (!c.on(SPD_STAGE_ATTN)) {
        // skipped
    } else if (c.q_len == 1) {
        const dim3 grid(parts.n_splits, D.kv, c.batch);
        const bool stream = decode_past_caches(D, c.pos.pos, c.batch);
#define SPD_DECODE_AS(DTV, FUSED_, STREAM_)                                                                                                    \
    hipLaunchKernelGGL((k_attn_decode<DTV, FUSED_, STREAM_>), grid, dim3(256), 0, c.s, kc, vc, fused_q ? qkvp : nullptr, D.q, D.kv, D.max_ctx,  \
                       qkv_slices, 16 * n_mtiles, D.nqkv, qbuf, qlo, raw.ss, (float)D.h, D.eps, qbuf, qlo, parts, c.pos)
#define SPD_DECODE(DTV)                                   \
    if (fused_q && stream) SPD_DECODE_AS(DTV, true, true);  \
    else if (fused_q) SPD_DECODE_AS(DTV, true, false);      \
    else if (stream) SPD_DECODE_AS(DTV, false, true);       \
    else SPD_DECODE_AS(DTV, false, false)
        switch (DT) {
            case 2: SPD_DECODE(2); break;
            case 4: SPD_DECODE(4); break;
            case 6: SPD_DECODE(6); break;
            case 8: SPD_DECODE(8); break;
            default: return hipErrorInvalidValue;
        }
#undef SPD_DECODE
#undef SPD_DECODE_AS
        SPD_TRY(hipGetLastError());
        if (!merge_o || c.taps) {      // (a tapped call also wants what the O projection would keep to itself)
            hipLaunchKernelGGL(k_attn_combine, dim3(cdiv(D.group * D.d / 4, 64), D.kv, c.batch), dim3(64), 0, c.s, parts.o, parts.units, parts.n_splits,
                               parts.group, parts.d, parts.by_quads, ahat, alo);
            SPD_TRY(hipGetLastError());
        }
    } else {
        const int n_ct = (c.q_len * D.group + 15) / 16;
        // Two column tiles per workgroup read each key and value once for both; up to two rounds of such workgroups, one
        // tile each gives twice the waves instead (70B shard, us: 128 tokens 6.4 -> 4.5, 512 behind 1536 positions 29 -> 26
        // and 19 with the next block prefetched, 1000: 18 -> 16; 4 x 2048 tokens stay with two).
        const bool one = (int64_t)cdiv(n_ct, 2) * D.kv * c.batch <= 512;
#define SPD_PREFILL_CT(DTV, CT)                                                                                            \
    {                                                                                                                      \
        const dim3 grid(D.kv * cdiv(n_ct, CT), 1, c.batch);                                                                  \
        constexpr int lds = prefill_lds(DTV, CT);                                                                            \
        static std::once_flag once;                                                                                        \
        static hipError_t attr_err = hipSuccess;                                                                           \
        std::call_once(once, [] {                                                                                          \
            attr_err = hipFuncSetAttribute((const void *)k_attn_prefill<DTV, CT>, hipFuncAttributeMaxDynamicSharedMemorySize, lds); \
        });                                                                                                                \
        SPD_TRY(attr_err);                                                                                                 \
        hipLaunchKernelGGL((k_attn_prefill<DTV, CT>), grid, dim3(256), lds, c.s, qbuf, qlo, kc, vc, c.q_len, D.group,    \
                           D.max_ctx, (int)cdiv(n_ct, CT), Divider::by(D.kv), ahat, alo, c.pos);                            \
    }
#define SPD_PREFILL(DTV)           \
    if (one) SPD_PREFILL_CT(DTV, 1) \
    else SPD_PREFILL_CT(DTV, 2)
        switch (DT) {
            case 2: SPD_PREFILL(2); break;
            case 4: SPD_PREFILL(4); break;
            case 6: SPD_PREFILL(6); break;
            case 8: SPD_PREFILL(8); break;
            default: return hipErrorInvalidValue;
        }
#undef SPD_PREFILL
#undef SPD_PREFILL_CT
        SPD_TRY(hipGetLastError());
    }
    spd_stage_end(c, SPD_STAGE_ATTN);

    const bool fuse_mid = mid && !spd && sync_in_o(D.h / 32, qd / 32, D.tp, n_mtiles);
    if (mid_done) *mid_done = fuse_mid;
    auto fill_o = [&](auto &e2) {
        e2.M = M; e2.h = D.h; e2.spd = spd; e2.m_pad = D.m_pad;
        e2.x = x; e2.g2 = (const float *)(w + D.w_g2);
        e2.bo = D.o_bias ? (const float *)(w + D.w_bo) : nullptr;
        e2.wsc = wo.wsc;
        e2.ybuf = ybuf; e2.slot = slot; e2.ss2 = (float *)(c.ws + D.ws_ss2);
        e2.xhat2 = (__bf16 *)(c.ws + D.ws_xhat2);
        e2.xlo2 = c.sp_m ? e2.xhat2 + D.pl_x : nullptr;
    };
    if (c.on(SPD_STAGE_O)) {
        spd_stage_scope prof(c, SPD_STAGE_O);
        if (fuse_mid) {
            // k_gemv and k_skinny only
            EpiOT<true> e2;
            fill_o(e2);
            e2.spd = 2;
            e2.slots = mid->slots; e2.slot_stride = c.slot_stride; e2.tp = mid->tp; e2.rank = mid->rank; e2.rbuf = mid->rbuf;
            SPD_TRY(launch_o(c, c.sp_a, wo.w, ahat, D.pl_a, D.h / 32, qd / 32, e2, merge_o ? parts : AttnParts()));
        } else {
            EpiOT<false> e2;
            fill_o(e2);
            SPD_TRY(launch_o(c, c.sp_a, wo.w, ahat, D.pl_a, D.h / 32, qd / 32, e2, merge_o ? parts : AttnParts()));
        }
    }

    if (c.taps) {
        if (c.taps->q) {
            hipLaunchKernelGGL(k_bf16_to_f32, dim3(cdiv((int64_t)M * qd, 256)), dim3(256), 0, c.s, qbuf, qlo, c.taps->q,
                               (int64_t)M * qd);
            SPD_TRY(hipGetLastError());
        }
        if (c.taps->attn) {
            hipLaunchKernelGGL(k_unpack_act, dim3(cdiv((int64_t)M * qd, 256)), dim3(256), 0, c.s, ahat, alo, c.taps->attn, M,
                               qd, qd);
            SPD_TRY(hipGetLastError());
        }
        if (c.taps->y) SPD_TRY(spd_common::copy2d(spd ? ybuf : slot, D.h, c.taps->y, D.h, M, D.h, c.s));
    }
    return hipSuccess;
}

hipError_t mlp_half(const spd_call &c, const char *w, int spd, float *slot, const spd_end_sync *fuse, bool *fused,
                    bool ss_per_pair) {
    const spd_dims &D = *c.D;
    const int M = c.M;
    const __bf16 *xhat = (const __bf16 *)(c.ws + D.ws_xhat2);
    __bf16 *uhat = (__bf16 *)(c.ws + D.ws_uhat);
    __bf16 *ulo = c.sp_m ? uhat + D.pl_u : nullptr;
    const ProjW wgu = proj_weights(c, w, 2), wdn = proj_weights(c, w, 3);

    EpiGU e1;
    e1.M = M; e1.h = D.h; e1.f_pad = D.f_pad; e1.m_pad = D.m_pad; e1.eps = D.eps;
    // SPD block: the O-projection epilogue wrote one partial per pair of n-tiles (h/32 of them);
    // TP block: prep() wrote them after the kept sync point
    e1.nch = ss_per_pair ? D.h / 32 : prep_nch(D.h, M);
    e1.ss = (const float *)(c.ws + D.ws_ss2);
    e1.wsc = wgu.wsc;
    e1.uhat = uhat; e1.ulo = ulo;
    if (c.on(SPD_STAGE_GATEUP)) {
        spd_stage_scope prof(c, SPD_STAGE_GATEUP);
        // (the skinny kernel, which takes what the GEMM cannot, adds the partials itself)
        if (M > 16 * SKINNY_MAX_MTILES && e1.nch >= ROW_SCALE_MIN_NCH && spd_gemm_fits(D.h / 32)) {
            // the factors (4 bytes per token) go where this rank's queries were (64 bytes per token and more): attention is done with them
            float *rs = (float *)(c.ws + D.ws_q);
            hipLaunchKernelGGL(k_row_scale, dim3(cdiv(M, 16)), dim3(512), 0, c.s, e1.ss, e1.nch, D.m_pad, D.h, D.eps, rs);
            SPD_TRY(hipGetLastError());
            e1.ss = rs;
            e1.nch = 0;
        }
        if (M <= 16) {
            if (D.gud_cols) {
                // decode: the copy with narrow column groups, one workgroup per group
                e1.cols = D.gud_cols;
                const __bf16 *wd = (const __bf16 *)(w + D.w_gud), *xlo = xhat + D.pl_x;
                SPD_TRY(c.sp_m ? launch_gemv<true>(c, wd, xhat, xlo, D.gud_groups, D.h / 32, e1, D.gud_cols)
                               : launch_gemv<false>(c, wd, xhat, xlo, D.gud_groups, D.h / 32, e1, D.gud_cols));
            } else {
                SPD_TRY(launch_proj(c, c.sp_m, wgu.w, xhat, D.pl_x, D.f_pad / 16, D.h / 32, e1));
            }
        } else {
            bool mid = false;
            if (!c.sp_m) SPD_TRY(launch_mid(c, wgu.w, xhat, D.f_pad / 16, D.h / 32, e1, &mid));
            if (!mid) SPD_TRY(launch_proj(c, c.sp_m, wgu.w, xhat, D.pl_x, D.f_pad / 16, D.h / 32, e1));
        }
    }

    // the closing sync point rides in the down projection's epilogue up to 512 tokens (but see down_whole()): that of the
    // weight-streaming kernels, of the kernel that adds K slices, or of one launch of 256 x 128 tiles.  In a long call's GEMM it gains nothing: measured on the 70B prefill shape, the
    // workgroups of a compute unit reach their epilogues together, so the slot reads do not overlap with
    // anybody's contraction and the fused kernel takes exactly as long as GEMM + rank-sum kernel.
    const bool whole = down_whole(D, D.h / 32, D.f_pad / 32, c.sp_m, (M + 15) / 16);
    const bool do_fuse = fuse && M <= 16 * SKINNY_MAX_MTILES && !whole;
    if (fused) *fused = do_fuse;
    auto fill = [&](auto &e2) {
        e2.M = M; e2.h = D.h; e2.spd = spd;
        e2.ybuf = (const float *)(c.ws + D.ws_y); e2.slot = slot;
        e2.base = nullptr; e2.slots = nullptr; e2.g1 = nullptr; e2.bias = nullptr; e2.slot_stride = 0; e2.tp = 0; e2.rank = 0; e2.m_pad = D.m_pad;
        e2.x_out = nullptr; e2.ss1 = nullptr; e2.xhat = nullptr; e2.xlo = nullptr;
        e2.wsc = wdn.wsc;
        if (do_fuse) {
            e2.base = fuse->base; e2.slots = fuse->slots; e2.slot_stride = c.slot_stride; e2.tp = fuse->tp;
            e2.rank = fuse->rank; e2.x_out = fuse->x_out; e2.g1 = fuse->next_g1; e2.bias = fuse->bias; e2.ss1 = (float *)(c.ws + D.ws_ss1);
            if (fuse->next_g1) {
                e2.xhat = (__bf16 *)(c.ws + D.ws_xhat);
                e2.xlo = c.sp_x ? e2.xhat + D.pl_x : nullptr;
            }
        }
    };
    if (c.on(SPD_STAGE_DOWN)) {
        spd_stage_scope prof(c, SPD_STAGE_DOWN);
        if (do_fuse) {
            EpiDownT<true> e2;
            fill(e2);
            // (up to 128 tokens the finishing kernel of the slices, which then carries the closing sync point, costs more than
            // the better contraction saves: 70B shard, 48 tokens 15.7 + 8.3 us against 20.2, 128: 19.5 + 13.1 against 30)
            if (M > 16 && M <= 128) SPD_TRY(launch_skinny(c, c.sp_m, wdn.w, uhat, D.pl_u, D.h / 32, D.f_pad / 32, e2));
            else SPD_TRY(launch_proj(c, c.sp_m, wdn.w, uhat, D.pl_u, D.h / 32, D.f_pad / 32, e2));
        } else {
            EpiDownT<false> e2;
            fill(e2);
            const __bf16 *lo = uhat + D.pl_u;
            if (whole)
                SPD_TRY((c.sp_m ? launch_gemm_lds_cfg<GemmSquare, true>(c, wdn.w, uhat, lo, D.h / 32, D.f_pad / 32, e2)
                                : launch_gemm_lds_cfg<GemmSquare, false>(c, wdn.w, uhat, lo, D.h / 32, D.f_pad / 32, e2)));
            else SPD_TRY(launch_proj(c, c.sp_m, wdn.w, uhat, D.pl_u, D.h / 32, D.f_pad / 32, e2));
        }
    }

    if (c.taps && c.taps->u) {
        hipLaunchKernelGGL(k_unpack_act, dim3(cdiv((int64_t)M * D.f, 256)), dim3(256), 0, c.s, uhat, ulo, c.taps->u, M,
                           D.f_pad, D.f);
        SPD_TRY(hipGetLastError());
    }
    return hipSuccess;
}

}  // namespace spd_bf16

// ------------------------------------------------------------------------------------------
// Benchmark aid: the rate of the matrix cores on register-resident operands (see spd_testing.h)
// ------------------------------------------------------------------------------------------
namespace {
__global__ void __launch_bounds__(512) k_mfma_probe(int iters, int random_data, float *__restrict__ out,
                                                    unsigned long long *__restrict__ clk) {
    // operands: a counter-based hash of (thread, fragment, element) mapped to fp16 values in (-2, 2), or ones
    bf16x8 a[4], b[8];
    auto fill = [&](int f) {
        bf16x8 v;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            unsigned h = (threadIdx.x * 12u + f) * 8u + e;
            h ^= h >> 16; h *= 0x7feb352du; h ^= h >> 15; h *= 0x846ca68bu; h ^= h >> 16;
            const float x = random_data ? ((float)(h & 0xffffu) - 32767.5f) * (2.0f / 32768.0f) : 1.0f;
            const _Float16 hf = (_Float16)x;
            v[e] = __builtin_bit_cast(__bf16, hf);
        }
        return v;
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = fill(i);
#pragma unroll
    for (int j = 0; j < 8; ++j) b[j] = fill(4 + j);
    f32x4 acc[4][8];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const bool stamp = blockIdx.x == gridDim.x / 2 && threadIdx.x == 0;
    unsigned long long c0 = 0, w0 = 0;
    if (stamp) {
        c0 = clock64();
        w0 = wall_clock64();
    }
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[i][j] = MFMA16(a[i], b[j], acc[i][j]);
    }
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) s += acc[i][j];
    if (stamp) {
        clk[0] = clock64() - c0;
        clk[1] = wall_clock64() - w0;
    }
    out[blockIdx.x * 512 + threadIdx.x] = s[0] + s[1] + s[2] + s[3];
}
}  // namespace

namespace {
// benchmark aid: every wave reads a contiguous share of `per_wave` KiB, four 1 KiB non-temporal loads in flight
__global__ void __launch_bounds__(1024) k_read_probe(const f32x4 *__restrict__ p, size_t per_wave, float *__restrict__ sink) {
    const int lane = threadIdx.x & 63;
    const size_t wave = (size_t)blockIdx.x * 16 + (threadIdx.x >> 6);
    const f32x4 *q = p + wave * per_wave * 64 + lane;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (size_t i = 0; i + 4 <= per_wave; i += 4) {
        f32x4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = __builtin_nontemporal_load(q + (i + u) * 64);
#pragma unroll
        for (int u = 0; u < 4; ++u) acc += v[u];
    }
    if (acc[0] == 1234.5f && acc[1] == -77.25f) sink[0] = acc[2];      // keeps the loads alive
}
}  // namespace

namespace spd_bf16 {
hipError_t read_probe(const void *buf, size_t chunk_bytes, int n_chunks, int reps, void *sink, hipStream_t s, double *us) {
    const size_t per_wave = chunk_bytes / (256 * 16 * 1024);        // KiB per wave (chunk_bytes is a multiple of 4 MiB)
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipError_t e = hipEventCreate(&e0);
    if (e == hipSuccess) e = hipEventCreate(&e1);
    auto launch = [&](int i) {
        const char *src = (const char *)buf + (size_t)(i % n_chunks) * chunk_bytes;
        hipLaunchKernelGGL(k_read_probe, dim3(256), dim3(1024), 0, s, (const f32x4 *)src, per_wave, (float *)sink);
    };
    if (e == hipSuccess) {
        for (int i = 0; i < 3; ++i) launch(i);                         // warm-up
        e = hipEventRecord(e0, s);
    }
    if (e == hipSuccess) {
        for (int i = 0; i < reps; ++i) launch(3 + i);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipEventRecord(e1, s);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    float ms = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (e != hipSuccess) return e;
    *us = (double)ms * 1000.0 / reps;
    return hipSuccess;
}
}  // namespace spd_bf16

namespace spd_bf16 {
hipError_t mfma_probe(int iters, int random_data, void *scratch, hipStream_t s, double *tflops, double *mhz) {
    constexpr int kGrid = 256;
    float *out = (float *)scratch;
    unsigned long long *clk = (unsigned long long *)((char *)scratch + (size_t)kGrid * 512 * 4);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipError_t e = hipEventCreate(&e0);
    if (e == hipSuccess) e = hipEventCreate(&e1);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_mfma_probe, dim3(kGrid), dim3(512), 0, s, 16, random_data, out, clk);      // warm-up
        e = hipEventRecord(e0, s);
    }
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_mfma_probe, dim3(kGrid), dim3(512), 0, s, iters, random_data, out, clk);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipEventRecord(e1, s);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    float ms = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    unsigned long long hc[2] = {0, 0};
    if (e == hipSuccess) e = hipMemcpy(hc, clk, sizeof(hc), hipMemcpyDeviceToHost);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (e != hipSuccess) return e;
    const double flops = (double)kGrid * 8 * (double)iters * 32 * 2.0 * 16 * 16 * 32;
    *tflops = flops / ((double)ms * 1e-3) / 1e12;
    *mhz = hc[1] ? 100.0 * (double)hc[0] / (double)hc[1] : 0.0;      // the real-time counter runs at 100 MHz
    return hipSuccess;
}
}  // namespace spd_bf16
