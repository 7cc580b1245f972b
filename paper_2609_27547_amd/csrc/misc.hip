// Row-wise kernels of the policy forward: RMSNorm, embedding gathers, patch extraction, the 256-bin action
// head with its argmax, and the flow-matching expert's input and Euler
// update.  All reductions run in a fixed order (deterministic results).
#include <math.h>

#include <type_traits>

#include "kernels.h"

namespace ebrl {

template <typename T> EBRL_DEV void load8v(const T* p, float* o);
template <> EBRL_DEV void load8v<bf16_t>(const bf16_t* p, float* o) {
    const uint4 u = *reinterpret_cast<const uint4*>(p);
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        o[2 * i] = __uint_as_float(w[i] << 16);
        o[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
    }
}
template <> EBRL_DEV void load8v<float>(const float* p, float* o) {
    const float4 a = *reinterpret_cast<const float4*>(p);
    const float4 b = *reinterpret_cast<const float4*>(p + 4);
    o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w;
    o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
}

template <typename TW, int VEC> EBRL_DEV void load_vec(const TW* p, float (&o)[VEC]) {
    if constexpr (VEC == 8) {
        load8v<TW>(p, o);
    } else if constexpr (sizeof(TW) == 4) {
        const float4 v = *reinterpret_cast<const float4*>(p);
        o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
    } else {
        const uint2 v = *reinterpret_cast<const uint2*>(p);
        o[0] = __uint_as_float(v.x << 16); o[1] = __uint_as_float(v.x & 0xFFFF0000u);
        o[2] = __uint_as_float(v.y << 16); o[3] = __uint_as_float(v.y & 0xFFFF0000u);
    }
}

// four squares, the order that row sums of squares are fixed to
EBRL_DEV float sq4(float4 v) { return fmaf(v.w, v.w, fmaf(v.z, v.z, fmaf(v.x, v.x, v.y * v.y))); }

// sum of squares of a row (fixed order), then 1/sqrt(mean + eps)
EBRL_DEV float row_rstd(const float* x, int d, float eps, float* red) {
    float ss = 0.f;
    for (int j = threadIdx.x * 4; j < d; j += blockDim.x * 4) {
        const float4 v = *reinterpret_cast<const float4*>(x + j);
        ss += sq4(v);
    }
    ss = block_sum(ss, red);
    return 1.0f / sqrtf(ss / (float)d + eps);
}

// ------------------------------------------------------------- RMSNorm --
template <typename TO>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const float* X, int ldx, const int* rows, TO* Y,
                                                      int ldy, int d, float eps)
{
    __shared__ float red[16];
    const int i = blockIdx.x;
    const int src = rows ? rows[i] : i;
    const float* x = X + (size_t)src * ldx;
    const float rs = row_rstd(x, d, eps, red);
    TO* y = Y + (size_t)i * ldy;
    for (int j = threadIdx.x * 4; j < d; j += blockDim.x * 4) {
        const float4 v = *reinterpret_cast<const float4*>(x + j);
        st4<TO>(y + j, v.x * rs, v.y * rs, v.z * rs, v.w * rs);
    }
}

// One wave per row for d % 256 == 0: the row stays in registers (NV float4
// per lane, lane-interleaved so each load instruction reads 1 KB of the row),
// the sum of squares is a wave reduction, no workgroup barrier.
template <typename TO, int NV>
__global__ __launch_bounds__(256) void rmsnorm_wave_kernel(const float* X, int ldx, const int* rows, TO* Y,
                                                           int ldy, int n_rows, int d, float eps)
{
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= n_rows) return;
    const int lane = threadIdx.x & 63;
    const int src = rows ? rows[i] : i;
    const float* x = X + (size_t)src * ldx;
    float4 v[NV];
    float ss = 0.f;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        v[k] = *reinterpret_cast<const float4*>(x + (k * 64 + lane) * 4);
        ss += v[k].x * v[k].x + v[k].y * v[k].y + v[k].z * v[k].z + v[k].w * v[k].w;
    }
    ss = wave_sum(ss);
    const float rs = 1.0f / sqrtf(ss / (float)d + eps);
    TO* y = Y + (size_t)i * ldy;
#pragma unroll
    for (int k = 0; k < NV; ++k)
        st4<TO>(y + (k * 64 + lane) * 4, v[k].x * rs, v[k].y * rs, v[k].z * rs, v[k].w * rs);
}

template <typename TO>
static bool rmsnorm_wave(const float* X, int ldx, const int* rows, TO* Y, int ldy, int n_rows, int d,
                         float eps, hipStream_t s) {
    if (d % 256) return false;
    const dim3 grid((n_rows + 3) / 4), block(256);
    switch (d / 256) {
    case 1: hipLaunchKernelGGL((rmsnorm_wave_kernel<TO, 1>), grid, block, 0, s, X, ldx, rows, Y, ldy, n_rows, d, eps); return true;
    case 2: hipLaunchKernelGGL((rmsnorm_wave_kernel<TO, 2>), grid, block, 0, s, X, ldx, rows, Y, ldy, n_rows, d, eps); return true;
    case 4: hipLaunchKernelGGL((rmsnorm_wave_kernel<TO, 4>), grid, block, 0, s, X, ldx, rows, Y, ldy, n_rows, d, eps); return true;
    case 8: hipLaunchKernelGGL((rmsnorm_wave_kernel<TO, 8>), grid, block, 0, s, X, ldx, rows, Y, ldy, n_rows, d, eps); return true;
    case 16: hipLaunchKernelGGL((rmsnorm_wave_kernel<TO, 16>), grid, block, 0, s, X, ldx, rows, Y, ldy, n_rows, d, eps); return true;
    default: return false;
    }
}

void rmsnorm_rows(bool bf16_out, const float* X, int ldx, const int* rows, void* Y, int ldy,
                  int n_rows, int d, float eps, hipStream_t s) {
    if (n_rows <= 0) return;
    if (bf16_out ? rmsnorm_wave<bf16_t>(X, ldx, rows, (bf16_t*)Y, ldy, n_rows, d, eps, s)
                 : rmsnorm_wave<float>(X, ldx, rows, (float*)Y, ldy, n_rows, d, eps, s))
        return;
    if (bf16_out)
        hipLaunchKernelGGL(rmsnorm_kernel<bf16_t>, dim3(n_rows), dim3(256), 0, s, X, ldx, rows,
                           (bf16_t*)Y, ldy, d, eps);
    else
        hipLaunchKernelGGL(rmsnorm_kernel<float>, dim3(n_rows), dim3(256), 0, s, X, ldx, rows,
                           (float*)Y, ldy, d, eps);
}

// ------------------------------------------------------------ embedding --
template <typename T>
__global__ __launch_bounds__(256) void embed_kernel(const T* E, int n_rows_e, int d, const int* ids,
                                                    const int* src, const int* dst_rows, float* X, int ldx)
{
    const int i = blockIdx.x;
    const int id = ids[src[i]];
    float* x = X + (size_t)dst_rows[i] * ldx;
    // four elements a thread and access (d % 4 == 0), 16-byte stores: 7959 rows of
    // 4096 55 -> 35 us against one element each
    const bool ok = id >= 0 && id < n_rows_e;   // out-of-range ids embed as zero rows
    const T* e = E + (size_t)(ok ? id : 0) * d;
    for (int j = threadIdx.x * 4; j < d; j += blockDim.x * 4) {
        float v[4] = {0.f, 0.f, 0.f, 0.f};
        if (ok) load_vec<T, 4>(e + j, v);
        st4<float>(x + j, v[0], v[1], v[2], v[3]);
    }
}

void embed_rows(bool bf16, const void* E, int n_rows_e, int d, const int* ids, const int* src, const int* dst_rows,
                float* X, int ldx, int n, hipStream_t s) {
    if (n <= 0) return;
    if (bf16)
        hipLaunchKernelGGL(embed_kernel<bf16_t>, dim3(n), dim3(256), 0, s, (const bf16_t*)E, n_rows_e, d, ids, src,
                           dst_rows, X, ldx);
    else
        hipLaunchKernelGGL(embed_kernel<float>, dim3(n), dim3(256), 0, s, (const float*)E, n_rows_e, d, ids, src,
                           dst_rows, X, ldx);
}

// ----------------------------------------------------------- patchify --
// One thread per 8 consecutive K elements of a patch row (a 16-byte bf16
// store); 32-bit index arithmetic.  kpad % 8 == 0; K elements past P*P*3 are
// the zero padding.
template <typename T>
__global__ __launch_bounds__(256) void im2col_kernel(const float* img, int rows, int cams, int H, int W, int P,
                                                     T* out, int kpad)
{
    const int gw = W / P, np = (H / P) * gw;
    const int kreal = P * P * 3, kc = kpad / 8;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= rows * kc) return;
    const int row = e / kc, k0 = (e - row * kc) * 8;
    const int env = row / (cams * np), p = row - env * cams * np;
    const int cam = p / np, pp = p - cam * np;
    const int py = pp / gw, px = pp - py * gw;
    const float* base = img + ((size_t)(env * cams + cam) * H + py * P) * W * 3 + (size_t)px * P * 3;
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int k = k0 + j;
        v[j] = 0.f;
        if (k < kreal) {
            const int dy = k / (3 * P), rem = k - dy * 3 * P;
            v[j] = base[(size_t)dy * W * 3 + rem];
        }
    }
    st4<T>(out + (size_t)e * 8, v[0], v[1], v[2], v[3]);
    st4<T>(out + (size_t)e * 8 + 4, v[4], v[5], v[6], v[7]);
}

void im2col(bool bf16, const float* img, int n, int cams, int H, int W, int P, void* out, int kpad,
            hipStream_t s) {
    const long rows = (long)n * cams * (H / P) * (W / P);
    if (rows <= 0) return;
    const long threads = rows * (kpad / 8);
    const int blocks = (int)((threads + 255) / 256);
    if (bf16)
        hipLaunchKernelGGL(im2col_kernel<bf16_t>, dim3(blocks), dim3(256), 0, s, img, (int)rows, cams, H, W, P,
                           (bf16_t*)out, kpad);
    else
        hipLaunchKernelGGL(im2col_kernel<float>, dim3(blocks), dim3(256), 0, s, img, (int)rows, cams, H, W, P,
                           (float*)out, kpad);
}

// --------------------------------------------------------- action head --
// Grid (groups of RG rows, groups of 16 bins).  The four waves deal the
// columns out in pieces of 64 VEC; a wave loads its piece of 16 weight rows and
// RG input rows (every weight serves RG rows, every input 16 bins) with all
// loads in flight, and its 16 RG sums are reduced across the lanes by halving
// (lane swaps that leave every lane a quarter of the sums), then across the
// waves in wave order.  The rows' sums of squares come from the same loads and
// scale the logits at the end, so nothing waits for a normalised copy of the
// row.  The logits go to a scratch row, and the last of the row group's
// workgroups (device-scope counter) takes each row's argmax (ties to the
// lowest bin) and top-2 margin, one wave per row, and writes the token's
// embedding as the next step's input row, all its loads issued together.
// Latency bounds it (the weights come from HBM once a step): 32 rows of 4096
// 20.0 -> 13.0 us and one row of 1024 9.4 -> 7.9 us against waves that walked all
// columns for four bins each and read the embedding 256 columns at a time.  An
// element's summation order depends on d alone.
EBRL_DEV float sum_xor32(float a, float b) {   // lanes < 32: a's pair sums, others: b's
    const auto s = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b),
                                                    false, false);
    return __builtin_bit_cast(float, (unsigned)s[0]) + __builtin_bit_cast(float, (unsigned)s[1]);
}
EBRL_DEV float sum_xor16(float a, float b) {   // even rows of 16 lanes: a's pair sums, odd rows: b's
    const auto s = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b),
                                                    false, false);
    return __builtin_bit_cast(float, (unsigned)s[0]) + __builtin_bit_cast(float, (unsigned)s[1]);
}

constexpr int LOGIT_BINS = 16;   // bins per workgroup
template <typename TW, int VEC, int RG>
__global__ __launch_bounds__(256, 2) void logits_kernel(LogitsArgs a)
{
    constexpr int NB = LOGIT_BINS, NA = NB * RG;
    __shared__ float s_acc[4][NA], s_ssq[4][RG];
    __shared__ int s_last, s_tok[RG];
    const int i0 = blockIdx.x * RG, b0 = blockIdx.y * NB;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const TW* w[NB];   // bins past the last repeat it
#pragma unroll
    for (int b = 0; b < NB; ++b) w[b] = (const TW*)a.W + (size_t)min(b0 + b, a.n_bins - 1) * a.d;
    const float* x[RG];
#pragma unroll
    for (int q = 0; q < RG; ++q) {
        const int i = min(i0 + q, a.n - 1);
        x[q] = a.X + (size_t)(a.rows ? a.rows[i] : i) * a.ldx;
    }
    float acc[NA], ssq[RG];
#pragma unroll
    for (int q = 0; q < RG; ++q) ssq[q] = 0.f;
#pragma unroll
    for (int k = 0; k < NA; ++k) acc[k] = 0.f;
    for (int c = wave * 64 * VEC; c < a.d; c += 4 * 64 * VEC) {
        const int col = c + lane * VEC, at = min(col, a.d - VEC);   // d % VEC == 0
        float wf[NB][VEC], h[RG][VEC];
#pragma unroll
        for (int b = 0; b < NB; ++b) load_vec<TW, VEC>(w[b] + at, wf[b]);
#pragma unroll
        for (int q = 0; q < RG; ++q) load_vec<float, VEC>(x[q] + at, h[q]);
        if (col >= a.d) {
#pragma unroll
            for (int u = 0; u < VEC; ++u) {
#pragma unroll
                for (int b = 0; b < NB; ++b) wf[b][u] = 0.f;
#pragma unroll
                for (int q = 0; q < RG; ++q) h[q][u] = 0.f;
            }
        }
#pragma unroll
        for (int q = 0; q < RG; ++q)
#pragma unroll
            for (int u = 0; u < VEC; ++u) {
                ssq[q] = fmaf(h[q][u], h[q][u], ssq[q]);
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[b * RG + q] = fmaf(wf[b][u], h[q][u], acc[b * RG + q]);
            }
    }
    // Row g of 16 lanes ends with the sums NA / 2 (g >> 1) + NA / 4 (g & 1) + i;
    // its lane i writes the i-th.
    {
        float t[NA / 2];
#pragma unroll
        for (int k = 0; k < NA / 2; ++k) t[k] = sum_xor32(acc[k], acc[k + NA / 2]);
        const int r = lane & 15, g = lane >> 4;
        float mine = 0.f;
#pragma unroll
        for (int k = 0; k < NA / 4; ++k) {
            const float v = sum_lanes16(sum_xor16(t[k], t[k + NA / 4]));
            if (r == k) mine = v;
        }
        if (r < NA / 4) s_acc[wave][NA / 2 * (g >> 1) + NA / 4 * (g & 1) + r] = mine;
#pragma unroll
        for (int q = 0; q < RG; ++q) {
            const float v = wave_sum(ssq[q]);
            if (lane == 0) s_ssq[wave][q] = v;
        }
    }
    __syncthreads();
    const __amdgpu_buffer_rsrc_t lgr = coherent_rsrc(a.lg + (size_t)i0 * a.n_bins);
    if (tid < NA) {
        const int q = tid % RG, b = b0 + tid / RG;
        const float ss = ((s_ssq[0][q] + s_ssq[1][q]) + s_ssq[2][q]) + s_ssq[3][q];
        const float rs = 1.0f / sqrtf(ss / (float)a.d + a.eps);
        const float v = ((s_acc[0][tid] + s_acc[1][tid]) + s_acc[2][tid]) + s_acc[3][tid];
        if (b < a.n_bins && i0 + q < a.n) st_coherent1(lgr, (q * a.n_bins + b) * 4, v * rs);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0)
        s_last = __hip_atomic_fetch_add(a.counters + blockIdx.x, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                 (unsigned)(gridDim.y - 1);
    __syncthreads();
    if (!s_last) return;
    if (tid == 0) __hip_atomic_store(a.counters + blockIdx.x, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (wave < RG && i0 + wave < a.n) {
        const int i = i0 + wave;
        // per lane: its largest logit (lowest bin of equals) and the largest of its others
        float bv = -INFINITY, sv = -INFINITY;
        int bi = 0x7fffffff;
#pragma unroll 4
        for (int b = lane; b < a.n_bins; b += 64) {
            const float v = ld_coherent1(lgr, (wave * a.n_bins + b) * 4);
            if (v > bv || (v == bv && b < bi)) { sv = bv; bv = v; bi = b; }
            else sv = fmaxf(sv, v);
        }
        const float own = bv;
        const int own_i = bi;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const float ov = __shfl_xor(bv, off, 64);
            const int oi = __shfl_xor(bi, off, 64);
            if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
        }
        sv = wave_max(own_i == bi ? sv : own);
        if (lane == 0) {
            const int o = i * a.ntok + a.col;
            a.tokens[o] = bi;
            if (a.actions) a.actions[o] = -1.0f + (2.0f * (float)bi + 1.0f) / (float)a.n_bins;
            if (a.margins) a.margins[o] = bv - sv;
            s_tok[wave] = bi;
        }
    }
    if (!a.emb) return;
    __syncthreads();
    for (int j = tid * 8; j < a.d; j += 2048) {   // d % 8 == 0
        float v[RG][8];
#pragma unroll
        for (int q = 0; q < RG; ++q) {
            const int bi = s_tok[min(q, a.n - 1 - i0)];
            // NaN logits leave no maximum: a zero row, as for any id past the bins
            const bool ok = (unsigned)bi < (unsigned)a.n_bins;
            load8v<TW>((const TW*)a.emb + (size_t)(ok ? bi : 0) * a.d + j, v[q]);
            if (!ok) {
#pragma unroll
                for (int u = 0; u < 8; ++u) v[q][u] = 0.f;
            }
        }
#pragma unroll
        for (int q = 0; q < RG; ++q) {
            if (i0 + q >= a.n) break;
            float* const o = a.nx + (size_t)(i0 + q) * a.ldnx + j;
            st4<float>(o, v[q][0], v[q][1], v[q][2], v[q][3]);
            st4<float>(o + 4, v[q][4], v[q][5], v[q][6], v[q][7]);
            if (a.nxb) {
                bf16_t* const ob = (bf16_t*)a.nxb + (size_t)(i0 + q) * a.ldnxb + j;
                st4<bf16_t>(ob, v[q][0], v[q][1], v[q][2], v[q][3]);
                st4<bf16_t>(ob + 4, v[q][4], v[q][5], v[q][6], v[q][7]);
            }
        }
    }
}

void action_logits(const LogitsArgs& a, hipStream_t s) {
    if (a.n <= 0) return;
    // Rows per workgroup: one up to 64 rows (each has n_bins / 16 workgroups of
    // its own), four above (a weight read serves four rows); one against four, 256
    // bins: d 4096, 24 rows 11.6 and 14.6 us, 32 13.0 and 15.5, 64 16.2 and 17.4, 80 19.9
    // and 19.6, 128 26.1 and 20.6; d 1024, 32 rows 9.6 and 9.9, 64 11.7 and 11.5, 128 12.6
    // and 11.6.  16-byte weight loads once a row gives all four waves
    // such a piece, 8-byte ones below; d alone decides, as it orders the sums.
    auto go = [&](auto kern, int rg) {
        hipLaunchKernelGGL(kern, dim3((a.n + rg - 1) / rg, (a.n_bins + LOGIT_BINS - 1) / LOGIT_BINS), dim3(256), 0, s,
                           a);
    };
    auto rows = [&](auto kern1, auto kern4) {
        if (a.n <= 64) go(kern1, 1);
        else go(kern4, 4);
    };
    if (!a.bf16) rows(logits_kernel<float, 4, 1>, logits_kernel<float, 4, 4>);
    else if (a.d >= 2048) rows(logits_kernel<bf16_t, 8, 1>, logits_kernel<bf16_t, 8, 4>);
    else rows(logits_kernel<bf16_t, 4, 1>, logits_kernel<bf16_t, 4, 4>);
}

// ---------------------------------------------------- last prefix row --
__global__ __launch_bounds__(256) void gather_last_kernel(const float* X, int ldx, const int* seq_env,
                                                          const int* last_row, int d, float eps,
                                                          float* h_pre, float* h_norm)
{
    __shared__ float red[16];
    const int i = blockIdx.x;
    const float* x = X + (size_t)last_row[i] * ldx;
    const int env = seq_env[i];
    const float rs = row_rstd(x, d, eps, red);
    for (int j = threadIdx.x; j < d; j += blockDim.x) {
        h_pre[(size_t)env * d + j] = x[j];
        h_norm[(size_t)env * d + j] = x[j] * rs;
    }
}

void gather_last(const float* X, int ldx, const int* seq_env, const int* last_row, int n, int d,
                 float eps, float* h_pre, float* h_norm, hipStream_t s) {
    if (n <= 0) return;
    hipLaunchKernelGGL(gather_last_kernel, dim3(n), dim3(256), 0, s, X, ldx, seq_env, last_row, d,
                       eps, h_pre, h_norm);
}

// ------------------------------------------------------- small linear --
// One wave per output column n and SL_ROWS input rows (grid: columns x row
// groups): lane l sums columns l + 64 i of W's row n and of the input rows, every
// weight used for all the rows, then the lanes are summed (wave_sum): that order
// is fixed, as for the step ends below.  One row after the other behind its own
// loads took 60 us for the ten time embeddings of a 1024-wide expert (now 11).
constexpr int SL_ROWS = 4;
template <typename T>
__global__ __launch_bounds__(256) void small_linear_kernel(const float* in, int R, int K, const T* W, int N,
                                                           float* out, int silu_input)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int n = blockIdx.x * 4 + wave, r0 = blockIdx.y * SL_ROWS;
    if (n >= N) return;
    const T* w = W + (size_t)n * K;
    float acc[SL_ROWS];
#pragma unroll
    for (int r = 0; r < SL_ROWS; ++r) acc[r] = 0.f;
#pragma unroll 8
    for (int k = lane; k < K; k += 64) {
        const float wv = ld_elem<T>(w + k);
        float xv[SL_ROWS];
#pragma unroll
        for (int r = 0; r < SL_ROWS; ++r) xv[r] = in[(size_t)min(r0 + r, R - 1) * K + k];
#pragma unroll
        for (int r = 0; r < SL_ROWS; ++r) {
            const float v = xv[r];
            acc[r] = fmaf(silu_input ? v / (1.0f + expf(-v)) : v, wv, acc[r]);
        }
    }
#pragma unroll
    for (int r = 0; r < SL_ROWS; ++r) {
        const float v = wave_sum(acc[r]);
        if (lane == 0 && r0 + r < R) out[(size_t)(r0 + r) * N + n] = v;
    }
}

void small_linear(bool bf16, const float* in, int R, int K, const void* W, int N, float* out,
                  bool silu_input, hipStream_t s) {
    if (R <= 0 || N <= 0) return;
    const dim3 grid((N + 3) / 4, (R + SL_ROWS - 1) / SL_ROWS);
    if (bf16)
        hipLaunchKernelGGL(small_linear_kernel<bf16_t>, grid, dim3(256), 0, s, in, R, K, (const bf16_t*)W, N,
                           out, (int)silu_input);
    else
        hipLaunchKernelGGL(small_linear_kernel<float>, grid, dim3(256), 0, s, in, R, K, (const float*)W, N, out,
                           (int)silu_input);
}

// ------------------------------------------------------------- flow --
// The denoised tokens of one env sit in `per_out` consecutive rows of H; a
// modality's token r (its rows numbered env by env, `per_in` per env) is
// H row (r / per_in) * per_out + off + r % per_in.  Actions alone: per_in =
// per_out = chunk, off = 0; the world-action model puts an env's future-frame
// latents first and its action tokens after them.
EBRL_DEV size_t flow_row(int r, int per_in, int per_out, int off) {
    return (size_t)(r / per_in) * per_out + off + r % per_in;
}

// The expert's ends of a denoising step, FLOW_ROWS tokens of one modality per
// workgroup: output head and Euler update of the step that ends (`last`), then
// input projection plus time vector of the step that begins (`first`).  A token
// needs only itself for both, so a step costs one launch for all modalities,
// where a launch per modality and end (a scalar weight load per channel, a wave
// reduction per output) took 78 us on the world action model at 37 envs and this
// takes 28 (rows from and to memory: 45 MB, 8 us); 64 envs of the flow policy 18.
//
// These sums have one fixed order: a change of it passes through every bf16
// layer that follows and ends as 4e-4 of the actions after ten steps.  (The
// order that fits 16-byte loads and 16x16x4 MFMAs best, with the row factor
// applied to the sums, took 25 us on the world action model.)  Both products run
// on v_mfma_f32_16x16x1_4b_f32, whose four blocks each take one fma per element:
// an accumulator is an fma chain.
//  * Head: a normalised row h * rs has 64 partial sums: chains over columns
//    256 i + 4 l + e (i, then e; l = 0 .. 63) where the width is 1, 2, 3, 4, 6 or 8
//    times 256 (16-byte loads), over columns l + 64 i for other widths.  They are
//    added as a balanced tree, neighbours first.  Block g of an MFMA is partial
//    sum 4 u + g; a wave has eight of them (two u), so that it adds its own subtree
//    of eight, and the waves' sums are the last three levels.  A row's sum of
//    squares takes the same tree (other widths: row_rstd's with 256 threads).
//    The row is read again after it, from the caches: kept in registers it would
//    leave one workgroup a CU.
//  * Input: chains over the channels; block g is output columns 16 g .. of 64,
//    the updated tokens come from LDS.
constexpr int FLOW_ROWS = 16, FLOW_WAVES = 8;

// row_rstd's sum of squares (256 threads) by one wave
EBRL_DEV float row_ssq_wave(const float* x, int d, int lane) {
    float t = 0.f;
    for (int v = 0; v < 4; ++v) {
        float ss = 0.f;
        for (int j = (v * 64 + lane) * 4; j < d; j += 1024) ss += sq4(*reinterpret_cast<const float4*>(x + j));
        t += wave_sum(ss);
    }
    return t;
}

template <typename T, int NT>   // NT: 16-channel tiles that cover adim
EBRL_DEV void flow_step_body(const FlowStepArgs& a, const FlowMod& m, int r0, float* s_red, float (*s_ssq)[FLOW_ROWS],
                             float* s_x)
{
    constexpr int XLD = 16 * NT + 4;             // LDS row of the tokens
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int d = a.d, adim = m.adim, row = min(r0 + r, m.rows - 1);
    float* const hrow = a.H + flow_row(row, m.per_in, a.per_out, m.off) * a.ldh;
    f32x16 zero;
#pragma unroll
    for (int i = 0; i < 16; ++i) zero[i] = 0.f;

    if (a.last) {
        const T* pw[NT];   // channels past the last repeat it
#pragma unroll
        for (int j = 0; j < NT; ++j) pw[j] = (const T*)m.w_out + (size_t)min(j * 16 + r, adim - 1) * d;
        // the wave's sums: lane (r, g) of tile j holds row r, channels 16 j + 4 g ..
        f32x4* const red = reinterpret_cast<f32x4*>(s_red);
        auto add_sums = [&](const f32x16 (&acc)[NT], int u) {
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                // register 4 b + i of an accumulator: block b, channel 4 g + i, row r
                f32x4 t;
#pragma unroll
                for (int i = 0; i < 4; ++i) t[i] = (acc[j][i] + acc[j][4 + i]) + (acc[j][8 + i] + acc[j][12 + i]);
                f32x4& at = red[(wave * NT + j) * 64 + lane];
                at = u ? at + t : t;
            }
        };
        auto rstd = [&](float ss) { return 1.0f / sqrtf(ss / (float)d + a.eps); };
        const int d4 = d >> 8;
        if ((d & 255) == 0 && (d4 <= 4 || d4 == 6 || d4 == 8)) {
            const int c0 = 32 * wave + 4 * g;   // columns of partial sum 8 wave + 4 u + g: c0 + 16 u ..
            float ss[2] = {0.f, 0.f};
#pragma unroll 4
            for (int i = 0; i < d4; ++i)
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    float h[4];
                    load_vec<float, 4>(hrow + 256 * i + c0 + 16 * u, h);
#pragma unroll
                    for (int e = 0; e < 4; ++e) ss[u] = fmaf(h[e], h[e], ss[u]);
                }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                ss[u] += __shfl_xor(ss[u], 16, 64);
                ss[u] += __shfl_xor(ss[u], 32, 64);
            }
            if (g == 0) s_ssq[wave][r] = ss[0] + ss[1];
            __syncthreads();
            const float rs = rstd(((s_ssq[0][r] + s_ssq[1][r]) + (s_ssq[2][r] + s_ssq[3][r])) +
                                  ((s_ssq[4][r] + s_ssq[5][r]) + (s_ssq[6][r] + s_ssq[7][r])));
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                f32x16 acc[NT];
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[j] = zero;
#pragma unroll 2
                for (int i = 0; i < d4; ++i) {
                    float h[4], w[NT][4];
                    load_vec<float, 4>(hrow + 256 * i + c0 + 16 * u, h);
#pragma unroll
                    for (int j = 0; j < NT; ++j) load_vec<T, 4>(pw[j] + 256 * i + c0 + 16 * u, w[j]);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int j = 0; j < NT; ++j)
                            acc[j] = __builtin_amdgcn_mfma_f32_16x16x1f32(w[j][e], h[e] * rs, acc[j], 0, 0, 0);
                }
                add_sums(acc, u);
            }
        } else {
            for (int q = wave; q < FLOW_ROWS; q += FLOW_WAVES) {
                const int qr = min(r0 + q, m.rows - 1);
                const float ss = row_ssq_wave(a.H + flow_row(qr, m.per_in, a.per_out, m.off) * a.ldh, d, lane);
                if (lane == 0) s_ssq[0][q] = ss;
            }
            __syncthreads();
            const float rs = rstd(s_ssq[0][r]);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                f32x16 acc[NT];
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[j] = zero;
#pragma unroll 2
                for (int col = 8 * wave + 4 * u + g; col < d; col += 64) {   // d % 64 == 0
                    const float x = hrow[col] * rs;
#pragma unroll
                    for (int j = 0; j < NT; ++j)
                        acc[j] = __builtin_amdgcn_mfma_f32_16x16x1f32(ld_elem<T>(pw[j] + col), x, acc[j], 0, 0, 0);
                }
                add_sums(acc, u);
            }
        }
        __syncthreads();
        if (tid < NT * 64) {
            const int j = tid >> 6;
            auto of = [&](int w) { return red[(w * NT + j) * 64 + lane]; };
            const f32x4 vel = ((of(0) + of(1)) + (of(2) + of(3))) + ((of(4) + of(5)) + (of(6) + of(7)));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int c = j * 16 + 4 * g + e;
                float xn = 0.f;
                if (c < adim) {
                    const size_t at = (size_t)row * adim + c;
                    xn = m.x[at] - vel[e] / a.n_steps;
                    if (r0 + r < m.rows) {
                        m.x_out[at] = xn;
                        if (m.v_out) m.v_out[at] = vel[e];
                    }
                }
                s_x[r * XLD + c] = xn;
            }
        }
    } else {
        for (int u = tid; u < FLOW_ROWS * 16 * NT; u += 64 * FLOW_WAVES) {
            const int q = u / (16 * NT), c = u % (16 * NT);
            s_x[q * XLD + c] = c < adim ? m.x[(size_t)min(r0 + q, m.rows - 1) * adim + c] : 0.f;
        }
    }
    if (!a.first) return;
    __syncthreads();
    const bool vec = (adim & 3) == 0;
    for (int t = wave; t < d >> 6; t += FLOW_WAVES) {
        const T* const pw_in = (const T*)m.w_in + (size_t)(t * 64 + lane) * adim;   // block g, column r of it
        float w[4 * NT][4];   // channels past the last: zeros, which leave a sum as it is
        if (vec) {
#pragma unroll
            for (int c = 0; c < 4 * NT; ++c) load_vec<T, 4>(pw_in + min(4 * c, adim - 4), w[c]);
        } else {
#pragma unroll
            for (int c = 0; c < 4 * NT; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    w[c][e] = ld_elem<T>(pw_in + min(4 * c + e, adim - 1));
                    if (4 * c + e >= adim) w[c][e] = 0.f;
                }
        }
        f32x16 acc = zero;
#pragma unroll
        for (int c = 0; c < 4 * NT; ++c) {
            const f32x4 x = *reinterpret_cast<const f32x4*>(s_x + r * XLD + 4 * c);   // zeros past adim
            if (4 * c < adim) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    acc = __builtin_amdgcn_mfma_f32_16x16x1f32(w[c][e], x[e], acc, 0, 0, 0);
            }
        }
        if (r0 + r < m.rows)
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const int col = t * 64 + 16 * b + 4 * g;
                const float4 tv = *reinterpret_cast<const float4*>(a.tvec + col);
                st4<float>(hrow + col, acc[4 * b] + tv.x, acc[4 * b + 1] + tv.y, acc[4 * b + 2] + tv.z,
                           acc[4 * b + 3] + tv.w);
            }
    }
}

// MAX_NT: tiles of the widest modality; up to 32 channels two workgroups fit a
// CU's registers.
template <typename T, int MAX_NT>
__global__ __launch_bounds__(64 * FLOW_WAVES, MAX_NT <= 2 && sizeof(T) == 2 ? 4 : 2) void flow_step_kernel(FlowStepArgs a)
{
    __shared__ __attribute__((aligned(16))) float s_red[FLOW_WAVES * MAX_NT * 256];
    __shared__ float s_ssq[FLOW_WAVES][FLOW_ROWS];
    __shared__ __attribute__((aligned(16))) float s_x[FLOW_ROWS * (16 * MAX_NT + 4)];
    const int blocks0 = (a.mod[0].rows + FLOW_ROWS - 1) / FLOW_ROWS;
    const bool second = (int)blockIdx.x >= blocks0;
    const FlowMod& m = a.mod[second ? 1 : 0];
    const int r0 = ((int)blockIdx.x - (second ? blocks0 : 0)) * FLOW_ROWS;
    if (MAX_NT == 1 || m.adim <= 16) flow_step_body<T, 1>(a, m, r0, s_red, s_ssq, s_x);
    else if (MAX_NT == 2 || m.adim <= 32) flow_step_body<T, 2>(a, m, r0, s_red, s_ssq, s_x);
    else flow_step_body<T, MAX_NT>(a, m, r0, s_red, s_ssq, s_x);
}

void flow_step(const FlowStepArgs& a, hipStream_t s) {
    const int blocks = (a.mod[0].rows + FLOW_ROWS - 1) / FLOW_ROWS + (a.mod[1].rows + FLOW_ROWS - 1) / FLOW_ROWS;
    if (blocks <= 0) return;
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(blocks), dim3(64 * FLOW_WAVES), 0, s, a); };
    const int wide = std::max(a.mod[0].adim, a.mod[1].adim);   // <= 64 (checked at policy creation)
    if (wide <= 16) a.bf16 ? go(flow_step_kernel<bf16_t, 1>) : go(flow_step_kernel<float, 1>);
    else if (wide <= 32) a.bf16 ? go(flow_step_kernel<bf16_t, 2>) : go(flow_step_kernel<float, 2>);
    else a.bf16 ? go(flow_step_kernel<bf16_t, 4>) : go(flow_step_kernel<float, 4>);
}

__global__ void copy_f32_kernel(const float* src, float* dst, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        dst[i] = src[i];
}

void copy_f32(const float* src, float* dst, size_t n, hipStream_t s) {
    if (n == 0) return;
    const int blocks = (int)std::min<size_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(copy_f32_kernel, dim3(blocks), dim3(256), 0, s, src, dst, n);
}

__global__ void copy_decode_out_kernel(const int* tok, const float* act, const float* mar, int count, int* out_tok,
                                       float* out_act, float* out_mar) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += gridDim.x * blockDim.x) {
        out_tok[i] = tok[i];
        if (out_act) out_act[i] = act[i];
        if (out_mar) out_mar[i] = mar[i];
    }
}

void copy_decode_out(const int* tok, const float* act, const float* mar, int count, int* out_tok, float* out_act,
                     float* out_mar, hipStream_t s) {
    if (count <= 0) return;
    const int blocks = std::min((count + 255) / 256, 1024);
    hipLaunchKernelGGL(copy_decode_out_kernel, dim3(blocks), dim3(256), 0, s, tok, act, mar, count, out_tok, out_act,
                       out_mar);
}


// ---------------------------------------------------------- seeded noise --
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11), ten rounds of
//   (c0, c1, c2, c3) <- (mulhi(B, c2) ^ c1 ^ k0, mullo(B, c2),
//                        mulhi(A, c0) ^ c3 ^ k1, mullo(A, c0)),
// A = 0xD2511F53, B = 0xCD9E8D57, key bumped by (0x9E3779B9, 0xBB67AE85)
// before every round but the first; then Box-Muller (1958) on the first two
// words, u = (x + 1/2) 2^-32, in double, rounded to float.  Row i's pair j
// takes counter (j, calls[i], env[i], stream) under key (lo, hi of seed).
__device__ __forceinline__ void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        const uint32_t hb = __umulhi(0xCD9E8D57u, c[2]), lb = 0xCD9E8D57u * c[2];
        const uint32_t ha = __umulhi(0xD2511F53u, c[0]), la = 0xD2511F53u * c[0];
        const uint32_t n0 = hb ^ c[1] ^ k0, n2 = ha ^ c[3] ^ k1;
        c[0] = n0;
        c[1] = lb;
        c[2] = n2;
        c[3] = la;
    }
}

__global__ __launch_bounds__(256) void normal_noise_kernel(float* __restrict__ out, int per_row,
                                                           const int* __restrict__ env,
                                                           const int* __restrict__ calls, uint32_t k0,
                                                           uint32_t k1, uint32_t stream) {
    const int i = blockIdx.y;
    const int pairs = (per_row + 1) / 2;
    const uint32_t e = (uint32_t)env[i], call = (uint32_t)calls[i];
    for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < pairs; j += gridDim.x * blockDim.x) {
        uint32_t c[4] = {(uint32_t)j, call, e, stream};
        philox4x32_10(c, k0, k1);
        const double u1 = ((double)c[0] + 0.5) * (1.0 / 4294967296.0);
        const double u2 = ((double)c[1] + 0.5) * (1.0 / 4294967296.0);
        const double rad = sqrt(-2.0 * log(u1));
        const double ang = 6.283185307179586 * u2;
        float* o = out + (size_t)i * per_row + 2 * j;
        o[0] = (float)(rad * cos(ang));
        if (2 * j + 1 < per_row) o[1] = (float)(rad * sin(ang));
    }
}

void normal_noise(float* out, int rows, int per_row, const int* env, const int* calls, uint64_t seed,
                  uint32_t stream, hipStream_t s) {
    if (rows <= 0 || per_row <= 0) return;
    const int pairs = (per_row + 1) / 2;
    dim3 grid((unsigned)std::min((pairs + 255) / 256, 64), (unsigned)rows);
    hipLaunchKernelGGL(normal_noise_kernel, grid, dim3(256), 0, s, out, per_row, env, calls,
                       (uint32_t)(seed & 0xFFFFFFFFu), (uint32_t)(seed >> 32), stream);
}


// ------------------------------------------------------- streaming read --
// Workgroup b reads 16-byte words [b * per, (b + 1) * per) with eight
// non-temporal loads in flight per lane.  A lane writes *out only if the XOR
// of its words equals a fixed constant, so every load's value is used.
__global__ __launch_bounds__(256) void stream_read_kernel(const u32x4* __restrict__ p, size_t n16, size_t per,
                                                          unsigned* out)
{
    constexpr int U = 8;
    u32x4 acc = {0u, 0u, 0u, 0u};
    const size_t b0 = blockIdx.x * per, b1 = min(n16, b0 + per);
    for (size_t i = b0 + threadIdx.x; i < b1; i += 256 * U) {
        u32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const size_t j = i + (size_t)u * 256;
            v[u] = j < b1 ? __builtin_nontemporal_load(p + j) : u32x4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int u = 0; u < U; ++u) acc ^= v[u];
    }
    const unsigned x = acc[0] ^ acc[1] ^ acc[2] ^ acc[3];
    if (x == 0x9E3779B9u) *out = x;
}

void stream_read(const void* buf, size_t bytes, unsigned* out, hipStream_t s) {
    const size_t n16 = bytes / 16;
    const int grid = 4096;
    const size_t per = (n16 + grid - 1) / grid;
    hipLaunchKernelGGL(stream_read_kernel, dim3(grid), dim3(256), 0, s, (const u32x4*)buf, n16, per, out);
}

}  // namespace ebrl
