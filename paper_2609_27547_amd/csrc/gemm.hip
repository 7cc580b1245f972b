// Projections y = x W^T of every linear layer (W stored [out, in]).
//
// bf16 path, four kernels, all on v_mfma_f32_16x16x32_bf16 with fp32
// accumulation.  The weight tile feeds the MFMA "A" operand and the
// activation tile the "B" operand, so a lane ends up owning four consecutive
// output columns of one row: a SwiGLU gate/up pair lands in the same lane
// (weights packed in 32-row groups: 16 gate rows, then the 16 matching up
// rows), and so does a rotary pair of the fused QKV projection.
//  * gemm_bf16_big_kernel (prefill, ViT, experts): 256 x 256 tiles on two
//    groups of four waves, operands DMA'd global -> LDS, epilogue staged
//    through LDS for whole-row stores.
//  * gemm_bf16_ring_kernel (the same, outputs with few such tiles): 64 x 128,
//    64 x 64 or 32 x 64 tiles, K tiles in an LDS ring.
//  * gemm_bf16_decode_kernel (decode, M <= 256): 32-, 64- or 96-column slices, per-wave
//    LDS pipelines fed by whole-line DMA; K split across workgroups only for
//    narrow outputs, the partials summed in split order inside the kernel by
//    the last workgroup of each tile.
//  * gemm_bf16_kernel: register-staged LDS tiles for the remaining shapes
//    (K not a multiple of 64), with split-K partials reduced in split order
//    by splitk_reduce_kernel.
// fp32 path (fp32 policies): fp32 MFMA on fragments from global memory, one
// launch per product, with the same epilogues.
// Every choice that orders a sum -- the K split count -- is a function of
// (N, K) alone; tile shapes, slice
// widths and block order, which may follow M and the stream's CU count,
// never change an element's summation order.  Results therefore do not
// depend on timing, on the number of compute units or on how many rows a
// decode call holds.
#include <type_traits>

#include "kernels.h"

namespace ebrl {

// ------------------------------------------------------------ epilogues --

struct EpiF32 {
    float* C; int ldc;
    EBRL_DEV void operator()(int m, int n, float a, float b, float c, float d) const {
        st4<float>(C + (size_t)m * ldc + n, a, b, c, d);
    }
};
template <typename T> struct EpiStore {
    T* C; int ldc;
    EBRL_DEV void operator()(int m, int n, float a, float b, float c, float d) const {
        st4<T>(C + (size_t)m * ldc + n, a, b, c, d);
    }
};
// Residual add; with xb set it also stores the updated rows in bf16 (the
// operand of a following projection that folds in the RMSNorm).
struct EpiResid {
    float* C; int ldc; bf16_t* xb; int ldxb;
    EBRL_DEV void operator()(int m, int n, float a, float b, float c, float d) const {
        float4* p = reinterpret_cast<float4*>(C + (size_t)m * ldc + n);
        float4 r = *p;
        r.x += a; r.y += b; r.z += c; r.w += d;
        *p = r;
        if (xb) st4<bf16_t>(xb + (size_t)m * ldxb + n, r.x, r.y, r.z, r.w);
    }
};
// Output row m goes to row_base[m / group] + m % group; optionally adds a
// per-(m % group) row of `add` (position embedding).
template <typename TA> struct EpiRemap {
    float* C; int ldc; const int* row_base; int group; const TA* add; int add_ld;
    EBRL_DEV void operator()(int m, int n, float a, float b, float c, float d) const {
        int g = m / group, r = m - g * group;
        size_t dst = (size_t)(row_base ? row_base[g] + r : m);
        if (add) {
            const TA* ap = add + (size_t)r * add_ld + n;
            a += ld_elem<TA>(ap); b += ld_elem<TA>(ap + 1);
            c += ld_elem<TA>(ap + 2); d += ld_elem<TA>(ap + 3);
        }
        st4<float>(C + dst * ldc + n, a, b, c, d);
    }
};
EBRL_DEV float silu_f(float g) { return g / (1.0f + __expf(-g)); }
// Paired epilogue: gate at packed column n (n % 32 < 16), up at n + 16.
template <typename T> struct EpiSwiGLU {
    T* H; int ldh;
    EBRL_DEV void pair(int m, int n, const float* g, const float* u) const {
        int col = (n >> 5) * 16 + (n & 15);
        st4<T>(H + (size_t)m * ldh + col, silu_f(g[0]) * u[0], silu_f(g[1]) * u[1],
               silu_f(g[2]) * u[2], silu_f(g[3]) * u[3]);
    }
};

// Paired epilogue of the fused QKV projection: columns n (first half of a
// head-local 32-row group) and n + 16 hold rotation partners e and e + hd/2.
template <typename T> struct EpiQKV {
    T* Q; int ldq; T* kv; int hq, hkv, hd;
    const int2* row_dst;
    const float* cos_tab; const float* sin_tab; int use_rope;
    // Per-row part of the destination: the row's position and its cache block.
    EBRL_DEV int2 row_info(int m) const { return row_dst[m]; }
    EBRL_DEV void pair_at(int2 ri, int m, int n, const float* x1, const float* x2) const {
        const int qn = hq * hd, kn = hkv * hd;
        const int region = n < qn ? 0 : (n < qn + kn ? 1 : 2);
        const int local = n - (region == 0 ? 0 : (region == 1 ? qn : qn + kn));
        const int h = local / hd, pc = local - h * hd;
        const int e = (pc >> 5) * 16 + (pc & 15);
        const int half = hd >> 1;
        const int pos = ri.x;
        float a[4], b[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) { a[t] = x1[t]; b[t] = x2[t]; }
        if (region < 2 && use_rope) {
            const float4 c = *reinterpret_cast<const float4*>(cos_tab + (size_t)pos * half + e);
            const float4 sn = *reinterpret_cast<const float4*>(sin_tab + (size_t)pos * half + e);
            const float cc[4] = {c.x, c.y, c.z, c.w}, ss[4] = {sn.x, sn.y, sn.z, sn.w};
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                a[t] = x1[t] * cc[t] - x2[t] * ss[t];
                b[t] = x2[t] * cc[t] + x1[t] * ss[t];
            }
        }
        T* dst;
        if (region == 0) {
            dst = Q + (size_t)m * ldq + h * hd;
        } else {
            // token row pos % 16 of head h's K (or V) rows in the block
            const size_t row = ((size_t)ri.y * 2 * hkv + (region == 2 ? hkv : 0) + h) * KV_BLOCK + (pos & (KV_BLOCK - 1));
            dst = kv + row * hd;
        }
        st4<T>(dst + e, a[0], a[1], a[2], a[3]);
        st4<T>(dst + e + half, b[0], b[1], b[2], b[3]);
    }
    EBRL_DEV void pair(int m, int n, const float* x1, const float* x2) const {
        pair_at(row_info(m), m, n, x1, x2);
    }
};
// Epilogues whose per-row work the large-M kernel hoists out of the column loop.
template <class E> struct epi_row_info : std::false_type {};
template <typename T> struct epi_row_info<EpiQKV<T>> : std::true_type {};
template <typename T> EpiQKV<T> make_epi_qkv(const RopeKVArgs& r) {
    return EpiQKV<T>{(T*)r.Q, r.ldq, (T*)r.kv.base, r.q_heads, r.kv.kv_heads, r.kv.head_dim, r.row_dst,
                     r.cos_tab, r.sin_tab, (int)r.use_rope};
}

// ------------------------------------------------------- bf16 MFMA GEMM --

constexpr int BK = 64;
constexpr int LDSW = BK + 8;  // padded LDS row (bf16 elements)

template <int BM, int BN, int WM, int WN, bool PAIRED, bool SPLIT, class Epi>
__global__ __launch_bounds__(256) void gemm_bf16_kernel(
    const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ B, int ldb, int M, int N,
    int K, int k_per_split, float* __restrict__ ws, Epi epi)
{
    static_assert(WM * WN == 4, "4 waves");
    constexpr int WTM = BM / WM, WTN = BN / WN;
    constexpr int TM = WTM / 16, TN = WTN / 16;
    static_assert(TM >= 1 && TN >= 1, "wave tile");
    static_assert(!PAIRED || (TN % 2 == 0), "paired epilogue needs tile pairs");
    constexpr int A_CHUNKS = BM * (BK / 8), B_CHUNKS = BN * (BK / 8);
    constexpr int A_ITERS = (A_CHUNKS + 255) / 256, B_ITERS = (B_CHUNKS + 255) / 256;

    __shared__ __attribute__((aligned(16))) bf16_t sA[2][BM * LDSW];
    __shared__ __attribute__((aligned(16))) bf16_t sB[2][BN * LDSW];

    const int tid = threadIdx.x;
    const int tiles_n = (N + BN - 1) / BN;
    const int tm_idx = blockIdx.x / tiles_n, tn_idx = blockIdx.x - tm_idx * tiles_n;
    const int m0 = tm_idx * BM, n0 = tn_idx * BN;
    const int k_begin = blockIdx.y * k_per_split;
    const int k_end = min(K, k_begin + k_per_split);
    const int nk = (k_end - k_begin + BK - 1) / BK;

    uint4 ra[A_ITERS], rb[B_ITERS];
    auto load_tiles = [&](int k0) {
#pragma unroll
        for (int i = 0; i < A_ITERS; ++i) {
            int c = tid + 256 * i;
            uint4 v = make_uint4(0, 0, 0, 0);
            if (c < A_CHUNKS) {
                int row = c >> 3, kc = (c & 7) * 8;
                int gr = min(m0 + row, M - 1), gk = k0 + kc;
                if (gk < k_end) v = *reinterpret_cast<const uint4*>(A + (size_t)gr * lda + gk);
            }
            ra[i] = v;
        }
#pragma unroll
        for (int i = 0; i < B_ITERS; ++i) {
            int c = tid + 256 * i;
            uint4 v = make_uint4(0, 0, 0, 0);
            if (c < B_CHUNKS) {
                int row = c >> 3, kc = (c & 7) * 8;
                int gr = min(n0 + row, N - 1), gk = k0 + kc;
                if (gk < k_end) v = *reinterpret_cast<const uint4*>(B + (size_t)gr * ldb + gk);
            }
            rb[i] = v;
        }
    };
    auto store_tiles = [&](int buf) {
#pragma unroll
        for (int i = 0; i < A_ITERS; ++i) {
            int c = tid + 256 * i;
            if (c < A_CHUNKS) {
                int row = c >> 3, kc = (c & 7) * 8;
                *reinterpret_cast<uint4*>(&sA[buf][row * LDSW + kc]) = ra[i];
            }
        }
#pragma unroll
        for (int i = 0; i < B_ITERS; ++i) {
            int c = tid + 256 * i;
            if (c < B_CHUNKS) {
                int row = c >> 3, kc = (c & 7) * 8;
                *reinterpret_cast<uint4*>(&sB[buf][row * LDSW + kc]) = rb[i];
            }
        }
    };

    const int wave = tid >> 6, lane = tid & 63;
    const int wm = wave / WN, wn = wave - wm * WN;
    const int r = lane & 15, g = lane >> 4;

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    if (nk > 0) {
        load_tiles(k_begin);
        store_tiles(0);
        __syncthreads();
        for (int kt = 0; kt < nk; ++kt) {
            const int buf = kt & 1;
            if (kt + 1 < nk) load_tiles(k_begin + (kt + 1) * BK);
#pragma unroll
            for (int ks = 0; ks < BK / 32; ++ks) {
                bf16x8 wa[TN], xb[TM];
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    wa[j] = *reinterpret_cast<const bf16x8*>(
                        &sB[buf][(wn * WTN + j * 16 + r) * LDSW + ks * 32 + g * 8]);
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    xb[i] = *reinterpret_cast<const bf16x8*>(
                        &sA[buf][(wm * WTM + i * 16 + r) * LDSW + ks * 32 + g * 8]);
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[j], xb[i], acc[i][j],
                                                                            0, 0, 0);
            }
            if (kt + 1 < nk) store_tiles(buf ^ 1);
            __syncthreads();
        }
    }

    // lane owns rows m = ... + r, columns n = ... + 4g .. 4g+3 of each tile
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int m = m0 + wm * WTM + i * 16 + r;
        if (m >= M) continue;
        if constexpr (SPLIT) {
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int n = n0 + wn * WTN + j * 16 + 4 * g;
                if (n < N)
                    st4<float>(ws + ((size_t)blockIdx.y * M + m) * N + n, acc[i][j][0],
                               acc[i][j][1], acc[i][j][2], acc[i][j][3]);
            }
        } else if constexpr (PAIRED) {
#pragma unroll
            for (int j = 0; j < TN; j += 2) {
                const int n = n0 + wn * WTN + j * 16 + 4 * g;
                if (n < N) {
                    float gv[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
                    float uv[4] = {acc[i][j + 1][0], acc[i][j + 1][1], acc[i][j + 1][2],
                                   acc[i][j + 1][3]};
                    epi.pair(m, n, gv, uv);
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int n = n0 + wn * WTN + j * 16 + 4 * g;
                if (n < N) epi(m, n, acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
            }
        }
    }
}


// ------------------------------------------------ bf16 MFMA GEMM, large M --
// Operands go global -> LDS with global_load_lds_dwordx4 (no VGPR staging): a
// wave instruction writes 64 lanes x 16 bytes contiguously, i.e. 8 rows of a
// 64-wide K tile, stored as 16-byte chunks: chunk c of row q at q * 8 +
// (c ^ (q & 7)); the XOR makes the MFMA fragment reads of 8 consecutive rows
// hit 8 different bank groups.
typedef __attribute__((address_space(3))) void* lds_ptr_t;

// s_waitcnt on the vector-memory counter only (gfx9 encoding: expcnt and
// lgkmcnt fields at their maxima), and on the LDS counter only.
template <int N> EBRL_DEV void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | 0x70 | 0xF00 | ((N >> 4) << 14));
}
EBRL_DEV void wait_lds() { __builtin_amdgcn_s_waitcnt(0xC07F); }

// Waits until at most min(later, MAX) groups of PER loads each are in flight.
template <int MAX, int PER> EBRL_DEV void wait_tiles(int later) {
    if constexpr (MAX > 0) {
        if (later < MAX) { wait_tiles<MAX - 1, PER>(later); return; }
    }
    wait_vmcnt<MAX * PER>();
}

// Workgroup barrier without the waits of __syncthreads: the kernels below
// count their own loads.  Neither memory accesses nor MFMAs move across it.
EBRL_DEV void wg_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// global_load_lds_dwordx4 issued as inline assembly: the compiler neither
// counts these loads nor guards LDS reads against them, so its own waits
// stay partial; kernels that use it wait on vmcnt and synchronise
// themselves before reading what the DMA filled.
EBRL_DEV void dma16_to_lds(const void* g, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                 :: "v"(g), "s"(lds_addr) : "memory", "m0");
}
// The same with the non-temporal hint, for weights that no other workgroup of
// the launch reads again (streaming them keeps the activations cached).
EBRL_DEV void dma16_to_lds_nt(const void* g, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt"
                 :: "v"(g), "s"(lds_addr) : "memory", "m0");
}
// The same DMA in its scalar-base form: a wave-uniform 64-bit base in SGPRs
// plus a 32-bit per-lane byte offset, so a wave's row offsets stay fixed
// across K tiles (only the scalar base advances) and take one VGPR each.
EBRL_DEV void dma16_to_lds_s(const void* sbase, uint32_t voff, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(voff), "s"(sbase), "s"(lds_addr) : "memory", "m0");
}
// A wave-uniform address pinned to SGPRs (readfirstlane returns int: each half
// goes through uint32_t, so the low half is zero-extended).
EBRL_DEV const char* uniform_ptr(const void* p) {
    const uint64_t b = (uint64_t)(uintptr_t)p;
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    return (const char*)(uintptr_t)(((uint64_t)hi << 32) | (uint64_t)lo);
}

// Epilogue of one 16-row x COLS-column sub-tile that a wave has staged in LDS
// (`at(row, chunk)`: its 16-byte chunk `chunk` of row `row`): read back
// row-contiguous, so that each store (and the residual read) covers whole row
// segments instead of 16-byte pieces of 16 rows.  INSIDE: no bounds checks;
// a wave then issues exactly epi_stores<Epi> x COLS / 64 stores or more.
// ri(row): row_info of a row (epilogues that use it).
template <int COLS, bool PAIRED, bool INSIDE, class Epi, class At, class RowInfo>
EBRL_DEV void store_subtile(const Epi& epi, int mrow0, int ncol0, int M, int N, int lane, At at, RowInfo ri) {
    if constexpr (PAIRED) {
        // COLS / 8 lanes per row: gate columns c (c % 32 < 16) with up partner c + 16
        constexpr int LPR = COLS / 8;
#pragma unroll
        for (int pass = 0; pass < LPR / 4; ++pass) {
            const int row = pass * (64 / LPR) + lane / LPR;
            const int ch = ((lane % LPR) >> 2) * 8 + (lane & 3);
            const f32x4 gv4 = at(row, ch), uv4 = at(row, ch + 4);
            const int m = mrow0 + row, n = ncol0 + ch * 4;
            auto info = ri(row);
            if (INSIDE || (m < M && n < N)) {
                float gv[4] = {gv4[0], gv4[1], gv4[2], gv4[3]};
                float uv[4] = {uv4[0], uv4[1], uv4[2], uv4[3]};
                if constexpr (epi_row_info<Epi>::value) epi.pair_at(info, m, n, gv, uv);
                else epi.pair(m, n, gv, uv);
            }
        }
    } else {
        // COLS / 4 lanes per row, four columns each
        constexpr int LPR = COLS / 4;
#pragma unroll
        for (int pass = 0; pass < LPR / 4; ++pass) {
            const int row = pass * (64 / LPR) + lane / LPR;
            const int ch = lane % LPR;
            const f32x4 v = at(row, ch);
            const int m = mrow0 + row, n = ncol0 + ch * 4;
            if (INSIDE || (m < M && n < N)) epi(m, n, v[0], v[1], v[2], v[3]);
        }
    }
}
// Stores of a wave per 16 x 64 sub-tile inside the output.
template <class E> struct epi_stores { static constexpr int n = 4; };
template <typename T> struct epi_stores<EpiSwiGLU<T>> { static constexpr int n = 2; };

// Row-tile-major groups of four row tiles: consecutive tiles share weights
// (four at a time) and activations.
EBRL_DEV void tile_origin(int v, int tiles_m, int tiles_n, int bm, int bn, int& m0, int& n0) {
    constexpr int G = 4;
    const int group = G * tiles_n, gi = v / group, first_m = gi * G;
    const int gsz = min(tiles_m - first_m, G), within = v - gi * group;
    m0 = (first_m + within % gsz) * bm;
    n0 = (within / gsz) * bn;
}

// 256 x 256 macro tiles, 8 waves of 128 x 64 in two groups of four (one wave
// of each group per SIMD) that run half a phase apart: while one group
// multiplies 32 MFMAs per wave from registers, the other reads its next
// fragments from LDS and issues DMA, so the MFMA pipes change hands at every
// barrier instead of idling through LDS latency.  A K tile of 64 is two
// phases: all of the wave's B columns with its first 64 A rows, then its last
// 64 rows.  Two LDS stages of 64 KB; a stage's four half-operands are refilled
// as soon as both groups have read them, so up to 14 KB per wave are in flight
// and no wait is for the loads just issued.
//  * What bounds it: a K tile is 0.86 us of MFMAs at 2.4 GHz.  It takes 0.75 to
//    0.9 us of a launch with few tiles and 1.24 to 1.39 us with one on every CU,
//    where the clock falls to 2.1 GHz (0.98 us) and 256 CUs share the caches: each
//    then streams 47-53 GB/s of operands, where a bare loop of such DMAs over
//    panels in L2 reaches 130 and one over panels beyond it 27.  1.55 PFLOP/s at
//    8192 x 8192 x 8192 (fp32 output) against 1.33 for the 16-wave kernel that read,
//    waited and multiplied in step, and 1.59 for hipBLASLt.
//  * Registers: 256 of 256.  The instances for plain stores, row remap and
//    residual spill 9, 3 and 1 of them once a tile, outside the K loop; the gate/up
//    and QKV ones none.
//  * Workgroups are persistent (one per CU): the next tile's first DMAs are
//    issued before the epilogue of the current one, whose stores then drain
//    behind the next tile's first K tile (7B-class gate/up, 8329 x 22016 x
//    4096: 1127 -> 1076 us).
//  * `full` tiles (a multiple of the grid) are dealt evenly; the tiles of the
//    last, partly filled round are cut in `split` = 2 (128 x 256) or 4 (128 x
//    128) where that still fits one round, so that more CUs work on them:
//    7B-class down projection (576 tiles on 256 CUs) 656 -> 587 us, 9600 x
//    2048 x 8192 291 -> 235 us.
// Every element is summed over K in order, 32 at a time, whatever its tile.
template <bool PAIRED, class Epi>
__global__ __launch_bounds__(512, 2) void gemm_bf16_big_kernel(
    const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ B, int ldb, int M, int N, int K,
    int full, int split, Epi epi)
{
    constexpr int STAGES = 2 * 65536;   // operand stages; 4 KB of epilogue staging per wave follow
    __shared__ __attribute__((aligned(1024))) char smem[STAGES + 8 * 4096];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave >> 2, wc = wave & 3;   // group (row half of the tile) and column quarter
    const int r = lane & 15, g = lane >> 4;
    const int tiles_m = (M + 255) >> 8, tiles_n = (N + 255) >> 8;
    const int nk = K >> 6;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr_t)smem);

    // Runs tiles of (64 FA) x (128 FB) until next(m0, n0) says there are no
    // more.  A half-operand h holds the rows (columns) that phase h (the
    // wave's h-th fragment set) multiplies: LDS row q of A half h is tile row
    // (q / HA) 2 HA + h HA + q % HA, i.e. each wave's rows are contiguous in
    // the output.
    auto run = [&](auto FAC, auto FBC, int m0, int n0, auto next) {
        constexpr int FA = decltype(FAC)::value, FB = decltype(FBC)::value;
        constexpr int HA = 16 * FA, HB = 16 * FB;        // a wave's rows / columns per half
        constexpr int NA = FA / 2, NB = FB;              // DMA instructions per wave and half
        constexpr int AHALF = 2 * HA * 128, BHALF = 4 * HB * 128, SB = 2 * (AHALF + BHALF);
        constexpr int W = 2 * NA + 2 * NB;               // DMA instructions per wave and K tile
        static_assert(2 * SB <= STAGES, "stages");
        // stores of an interior tile's epilogue that may still be in flight
        // behind the next tile's first loads
        constexpr int EST = 2 * FA * epi_stores<Epi>::n * FB / 2;
        static_assert(W + EST < 64, "vmcnt range");
        uint32_t va[2][NA], vb[2][NB];
        const char *pA, *pB;
        auto dmaA = [&](int t, int h) {
            const char* p = pA + (size_t)t * 128;
            const uint32_t l = lds0 + (t & 1) * SB + h * AHALF + wave * NA * 1024;
#pragma unroll
            for (int j = 0; j < NA; ++j) dma16_to_lds_s(p, va[h][j], l + j * 1024);
        };
        auto dmaB = [&](int t, int h) {
            const char* p = pB + (size_t)t * 128;
            const uint32_t l = lds0 + (t & 1) * SB + 2 * AHALF + h * BHALF + wave * NB * 1024;
#pragma unroll
            for (int j = 0; j < NB; ++j) dma16_to_lds_s(p, vb[h][j], l + j * 1024);
        };
        // K tiles 0 and 1 but for the second half of A's tile 1; rows past
        // the operand repeat its last one
        auto prologue = [&]() {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int j = 0; j < NA; ++j) {
                    const int q = (wave * NA + j) * 8 + (lane >> 3);
                    const int row = (q / HA) * 2 * HA + h * HA + q % HA;
                    va[h][j] = (uint32_t)(min(row, M - 1 - m0) * lda + ((lane & 7) ^ (q & 7)) * 8) * 2u;
                }
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    const int q = (wave * NB + j) * 8 + (lane >> 3);
                    const int row = (q / HB) * 2 * HB + h * HB + q % HB;
                    vb[h][j] = (uint32_t)(min(row, N - 1 - n0) * ldb + ((lane & 7) ^ (q & 7)) * 8) * 2u;
                }
            }
            pA = uniform_ptr(A + (size_t)m0 * lda);
            pB = uniform_ptr(B + (size_t)n0 * ldb);
            dmaB(0, 0); dmaA(0, 0); dmaB(0, 1); dmaA(0, 1);
            if (nk > 1) { dmaB(1, 0); dmaA(1, 0); dmaB(1, 1); }
        };
        uint32_t a_off[2], b_off[2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            a_off[ks] = (uint32_t)((wr * HA + r) * 128 + (((ks * 4 + g) ^ (r & 7)) << 4));
            b_off[ks] = (uint32_t)(2 * AHALF + (wc * HB + r) * 128 + (((ks * 4 + g) ^ (r & 7)) << 4));
        }
        f32x4 acc[2][2][FA][FB];
        bf16x8 fa[2][FA], fb0[2][FB], fb1[2][FB];
        auto readA = [&](int st, int h) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int i = 0; i < FA; ++i)
                    fa[ks][i] = *reinterpret_cast<const bf16x8*>(smem + st + a_off[ks] + h * AHALF + i * 2048);
        };
        auto readB = [&](int st, int h, bf16x8 (&f)[2][FB]) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int j = 0; j < FB; ++j)
                    f[ks][j] = *reinterpret_cast<const bf16x8*>(smem + st + b_off[ks] + h * BHALF + j * 2048);
        };
        auto mma = [&](f32x4 (&c)[FA][FB], const bf16x8 (&f)[2][FB]) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int i = 0; i < FA; ++i)
#pragma unroll
                    for (int j = 0; j < FB; ++j)
                        c[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[ks][j], fa[ks][i], c[i][j], 0, 0, 0);
        };
        // Phase p of a group: read fragments, issue DMA, wait for the DMA that
        // phase p + 1 reads (`wait`), barrier, multiply, barrier.  A group's
        // reads are complete before its first barrier, so what phase p reads
        // may be refilled from phase p + 1 on, by either group.
        // One K tile with L further ones (0, 1, 2 = two or more); ov: the
        // previous output tile's stores sit between this tile's DMAs.
        auto ktile = [&](int t, bool ov, auto LC) {
            constexpr int L = decltype(LC)::value;
            const int st = (t & 1) * SB;
            readB(st, 0, fb0); readA(st, 0); readB(st, 1, fb1);
            if constexpr (L >= 1) dmaA(t + 1, 1);
            if constexpr (L >= 2) { if (ov) wait_vmcnt<W + EST>(); else wait_vmcnt<W>(); }
            else if constexpr (L == 1) wait_vmcnt<W>();
            else wait_vmcnt<0>();
            wait_lds();
            wg_barrier();
            mma(acc[0][0], fb0); mma(acc[0][1], fb1);
            wg_barrier();
            readA(st, 1);
            if constexpr (L >= 2) {
                dmaB(t + 2, 0); dmaA(t + 2, 0); dmaB(t + 2, 1);
                if (ov) wait_vmcnt<W + EST>(); else wait_vmcnt<W>();
            } else if constexpr (L == 1) wait_vmcnt<NA>();
            wait_lds();
            wg_barrier();
            mma(acc[1][0], fb0); mma(acc[1][1], fb1);
            wg_barrier();
        };
        prologue();
        bool over = false;   // an interior tile's stores were issued behind the prologue
        for (;;) {
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int i = 0; i < FA; ++i)
#pragma unroll
                        for (int j = 0; j < FB; ++j) acc[a][b][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            // first B halves and first A half of K tile 0
            if (nk > 1) { if (over) wait_vmcnt<W + EST>(); else wait_vmcnt<W>(); }
            else wait_vmcnt<NA>();
            wg_barrier();
            if (wr == 1) wg_barrier();   // the second group runs half a phase behind
            int t = 0;
            for (; t + 2 < nk; ++t) ktile(t, over && t == 0, std::integral_constant<int, 2>{});
            if (t + 1 < nk) { ktile(t, false, std::integral_constant<int, 1>{}); ++t; }
            ktile(t, false, std::integral_constant<int, 0>{});
            if (wr == 0) wg_barrier();   // both groups are done with the stages
            const int mw = m0 + wr * 2 * HA, nw = n0 + wc * 2 * HB;
            const bool inside = m0 + 4 * HA <= M && n0 + 8 * HB <= N;
            // per-row epilogue data: lane l holds the wave's rows l and 64 + l
            constexpr bool ROWS = epi_row_info<Epi>::value;
            constexpr int RV = ROWS ? FA / 2 : 1;
            int2 info[RV];
            if constexpr (ROWS) {
#pragma unroll
                for (int v = 0; v < RV; ++v) info[v] = epi.row_info(min(mw + v * 64 + lane, M - 1));
            }
            const bool more = next(m0, n0);
            if (more) prologue();
            // Through the wave's own staging LDS, 16 rows at a time; chunks
            // swizzled by row so that the fragment-layout writes and the
            // row-contiguous reads (gate/up pairs: 8 lanes on each of two
            // rows) spread over all banks.
            char* const stage = smem + STAGES + wave * 4096;
            auto swz = [](int row) { return ((row & 1) << 2) | ((row >> 1) & 3) | (row & 8); };
            auto at = [&](int row, int ch) {
                return *reinterpret_cast<const f32x4*>(stage + row * 256 + ((ch ^ swz(row)) << 4));
            };
            auto epilogue = [&](auto IN) {
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int i = 0; i < FA; ++i) {
#pragma unroll
                        for (int b = 0; b < 2; ++b)
#pragma unroll
                            for (int j = 0; j < FB; ++j)
                                *reinterpret_cast<f32x4*>(stage + r * 256 + ((((b * FB + j) * 4 + g) ^ swz(r)) << 4)) =
                                    acc[a][b][i][j];
                        const int row0 = a * HA + i * 16;
                        store_subtile<2 * HB, PAIRED, decltype(IN)::value>(
                            epi, mw + row0, nw, M, N, lane, at, [&](int row) {
                                const int2 v = info[ROWS ? row0 / 64 : 0];
                                if constexpr (!ROWS) return v;
                                else return make_int2(__shfl(v.x, row0 % 64 + row, 64), __shfl(v.y, row0 % 64 + row, 64));
                            });
                    }
            };
            if (inside) epilogue(std::true_type{});
            else epilogue(std::false_type{});
            if (!more) break;
            over = inside;
        }
    };

    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I4 = std::integral_constant<int, 4>;
    // Full tiles: full / grid per workgroup.  The dispatcher deals workgroup
    // ids round-robin over the 8 XCDs: XCD x's workgroups walk a contiguous
    // range of tiles together, so that they share operands in its L2.
    const int P = gridDim.x, bid = blockIdx.x;
    if (full > 0) {
        const int rounds = full / P;
        int i = 0;
        auto origin = [&](int k, int& m, int& n) {
            const int v = (P & 7) == 0 ? (bid & 7) * (full >> 3) + k * (P >> 3) + (bid >> 3) : k * P + bid;
            tile_origin(v, tiles_m, tiles_n, 256, 256, m, n);
        };
        int m0, n0;
        origin(0, m0, n0);
        run(I4{}, I2{}, m0, n0, [&](int& m, int& n) {
            if (++i >= rounds) return false;
            origin(i, m, n);
            return true;
        });
    }
    // The last round: at most one (part of a) tile per workgroup.
    const int items = (tiles_m * tiles_n - full) * split;
    if (bid >= items) return;
    const int x = bid & 7;
    const int s = x * (items >> 3) + min(x, items & 7) + (bid >> 3);
    int m0, n0;
    tile_origin(full + s / split, tiles_m, tiles_n, 256, 256, m0, n0);
    auto none = [](int&, int&) { return false; };
    const int part = s % split;
    m0 += (part & 1) * 128;
    n0 += (part >> 1) * 128;
    if (m0 >= M || n0 >= N) return;
    if (split == 1) run(I4{}, I2{}, m0, n0, none);
    else if (split == 2) run(I2{}, I2{}, m0, n0, none);
    else run(I2{}, I1{}, m0, n0, none);
}

// Small outputs (fewer 256 x 256 tiles than CUs): BM x BN tiles on four waves
// (2 x 2), a ring of ST K tiles in LDS with ST - 1 of them in flight, one
// barrier per K tile.  The two-stage kernel it replaces waited a full memory
// latency per K tile (0.6-0.9 us); here a K tile takes 0.18 (32 x 64), 0.23 (64 x
// 64) and 0.35 us (64 x 128) with one workgroup on a CU, 0.26, 0.36 and 0.61 with
// two, i.e. 70 and 80-94 GB/s of operands per CU whatever the tile and the depth
// of the ring; what holds it there is not isolated (a bare loop of such DMAs
// from L2 reaches 130).  424 x 1024 x 4096: 39 -> 15 us; 800 x 1024 x 4096: 39 -> 17
// us; 424 x 3072 x 1024: 9.9 -> 8.0 us.  Same K order as the kernel above.
template <int BM, int BN, int ST, bool PAIRED, class Epi>
__global__ __launch_bounds__(256, 2) void gemm_bf16_ring_kernel(
    const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ B, int ldb, int M, int N, int K, Epi epi)
{
    constexpr int WTM = BM / 2, WTN = BN / 2, TM = WTM / 16, TN = WTN / 16;
    static_assert(!PAIRED || TN % 2 == 0, "paired epilogue needs tile pairs");
    constexpr int SB = (BM + BN) * 128;                // bytes of a stage
    constexpr int PER = (BM + BN) / 32;                // DMA instructions per wave and K tile
    static_assert((BM + BN) % 32 == 0 && BM % 8 == 0 && ST >= 2 && ST <= 4, "ring");
    __shared__ __attribute__((aligned(1024))) char smem[ST * SB];
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    int bid = blockIdx.x;
    {
        // XCD x takes the x-th contiguous range of tiles
        const int nb = gridDim.x, x = bid & 7;
        bid = x * (nb >> 3) + min(x, nb & 7) + (bid >> 3);
    }
    int m0, n0;
    tile_origin(bid, tiles_m, tiles_n, BM, BN, m0, n0);
    const int nk = K >> 6;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int r = lane & 15, g = lane >> 4;

    // 8-row groups of a stage, A's first: PER per wave
    uint32_t vo[PER];
    const char* base[PER];
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr_t)smem + wave * PER * 1024);
    const char* const pA = uniform_ptr(A + (size_t)m0 * lda);
    const char* const pB = uniform_ptr(B + (size_t)n0 * ldb);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int q0 = (wave * PER + j) * 8;
        const int q = q0 + (lane >> 3), c = (lane & 7) ^ (q & 7);
        if (q0 < BM) {
            vo[j] = (uint32_t)(min(q, M - 1 - m0) * lda + c * 8) * 2u;
            base[j] = pA;
        } else {
            vo[j] = (uint32_t)(min(q - BM, N - 1 - n0) * ldb + c * 8) * 2u;
            base[j] = pB;
        }
    }
    auto dma = [&](int t, int st) {
#pragma unroll
        for (int j = 0; j < PER; ++j) dma16_to_lds_s(base[j] + (size_t)t * 128, vo[j], lds0 + st * SB + j * 1024);
    };
    // per-row epilogue data of the wave's rows, one row per lane
    constexpr bool ROWS = epi_row_info<Epi>::value;
    int2 info = make_int2(0, 0);
    if constexpr (ROWS) info = epi.row_info(min(m0 + wm * WTM + min(lane, WTM - 1), M - 1));
    uint32_t a_off[2], b_off[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        a_off[ks] = (uint32_t)((wm * WTM + r) * 128 + (((ks * 4 + g) ^ (r & 7)) << 4));
        b_off[ks] = (uint32_t)((BM + wn * WTN + r) * 128 + (((ks * 4 + g) ^ (r & 7)) << 4));
    }
    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int p = 0; p < ST - 1 && p < nk; ++p) dma(p, p);
    int st = 0, nst = ST - 1;
    for (int t = 0; t < nk; ++t) {
        // this wave's part of tile t has landed (the tiles issued after it may
        // stay in flight); after the barrier every wave's has, and all have
        // read tile t - 1, whose stage is refilled next
        const int later = min(ST - 2, nk - 1 - t);
        if (ST >= 4 && later >= 2) wait_vmcnt<2 * PER>();
        else if (ST >= 3 && later >= 1) wait_vmcnt<PER>();
        else wait_vmcnt<0>();
        wg_barrier();
        if (t + ST - 1 < nk) dma(t + ST - 1, nst);
        const char* const s = smem + st * SB;
        bf16x8 w[2][TN], x[2][TM];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
            for (int j = 0; j < TN; ++j) w[ks][j] = *reinterpret_cast<const bf16x8*>(s + b_off[ks] + j * 2048);
#pragma unroll
            for (int i = 0; i < TM; ++i) x[ks][i] = *reinterpret_cast<const bf16x8*>(s + a_off[ks] + i * 2048);
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks][j], x[ks][i], acc[i][j], 0, 0, 0);
        nst = st;
        st = st + 1 == ST ? 0 : st + 1;
    }
    wg_barrier();
    // epilogue staging in the stages: rows padded by one chunk
    constexpr int SROW = WTN + 4;
    static_assert(4 * 16 * SROW * 4 <= ST * SB, "staging space");
    float* const stage = reinterpret_cast<float*>(smem) + wave * 16 * SROW;
    auto at = [&](int row, int ch) { return *reinterpret_cast<const f32x4*>(stage + row * SROW + ch * 4); };
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int j = 0; j < TN; ++j) *reinterpret_cast<f32x4*>(stage + r * SROW + j * 16 + 4 * g) = acc[i][j];
        store_subtile<WTN, PAIRED, false>(epi, m0 + wm * WTM + i * 16, n0 + wn * WTN, M, N, lane, at, [&](int row) {
            if constexpr (!ROWS) return info;
            else return make_int2(__shfl(info.x, i * 16 + row, 64), __shfl(info.y, i * 16 + row, 64));
        });
    }
}

// ------------------------------------------- bf16 GEMM, decode-sized M --
// M <= 256 (one row per environment), K % 64 == 0.  A workgroup owns a
// 32-, 64- or 96-column slice of the output, at most 64 rows (further row tiles in more
// workgroups) and a contiguous range of 64-wide K groups; the range is the
// whole K unless the column slices alone are too few to occupy the chip.  The
// four waves split that range and run independent pipelines: each wave
// streams its weight and activation rows into its own LDS region with
// global_load_lds_dwordx4 (one instruction = 8 rows x 128 contiguous bytes,
// whole cache lines), two to four buffers deep, and multiplies from LDS.  Loading
// whole 128-byte row segments per instruction roughly doubles the rate a CU
// sustains compared with loading 16 rows x 64 bytes straight into MFMA
// register layout.  The waves' tiles are summed in wave order through LDS.
// With several K splits each workgroup stores its partial tile, and the
// workgroup that finishes a tile last (a device-scope counter per tile) sums
// the partials in split order, runs the epilogue and clears the counter for
// the next call.  An element's summation order depends only on (N, K).
constexpr int DEC_BN = 64;   // column slice of the split rule (the kernel also runs 32- and 96-wide slices)
constexpr int DEC_MAX_SPLITS = 16;
constexpr int DEC_TILE_FLOATS = 64 * 64;   // partial-tile stride in the workspace
constexpr int DEC_MAX_COUNTERS = 4096;

// One wave's DMA of ROWS rows x 64 bf16 (K group k0) into `lds`: row q of the
// group sits in instruction q / 8, lane (q % 8) * 8 + (c ^ (q % 8)) holds its
// 16-byte chunk c (the XOR spreads a fragment read over the banks).  Each
// wave reads only the region its own DMA fills.
template <int ROWS, bool NT = false>
EBRL_DEV void dec_dma(const bf16_t* __restrict__ G, int ld, int row0, int rows_valid, int k0, bf16_t* lds,
                      int lane) {
    const int q = lane >> 3, c = (lane & 7) ^ q;
    const uint32_t base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr_t)lds);
#pragma unroll
    for (int t = 0; t < ROWS / 8; ++t) {
        const int gr = min(row0 + t * 8 + q, rows_valid - 1);
        if constexpr (NT) dma16_to_lds_nt(G + (size_t)gr * ld + k0 + c * 8, base + t * 1024);
        else dma16_to_lds(G + (size_t)gr * ld + k0 + c * 8, base + t * 1024);
    }
}
EBRL_DEV bf16x8 dec_frag(const bf16_t* lds, int row, int c) {
    return *reinterpret_cast<const bf16x8*>(lds + (row >> 3) * 512 + ((row & 7) * 8 + (c ^ (row & 7))) * 8);
}

// K groups per wave in LDS, all but the one being multiplied in flight: three
// for 64-column slices where they fit (measured 1-13 % more bandwidth than two
// on the 7B-class decode shapes at 1-32 rows), two for 96-column slices (all of
// the LDS at 64 rows) and for 32-column ones, or four there where one workgroup
// has a CU to itself (plan_gemm).
constexpr int dec_stages(int tm, int bn, bool deep) {
    return bn == 96 ? 2 : bn == 32 ? (deep ? 4 : 2) : (3 * 4 * (bn + 16 * tm) * 128 <= 150 * 1024 ? 3 : 2);
}

template <int TM, int BN, bool NTW, bool DEEP, bool NORM, bool PAIRED, class Epi>
__global__ __launch_bounds__(256) void gemm_bf16_decode_kernel(
    const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ W, int ldw, int M, int N,
    int K, int groups_per_split, int splits, int m_tiles, float* __restrict__ ws,
    unsigned* __restrict__ counters, float norm_eps, Epi epi)
{
    constexpr int TN = BN / 16;
    static_assert(!PAIRED || TN % 2 == 0, "paired epilogue needs fragment pairs");
    constexpr int FR = TM * TN;            // output fragments per wave
    constexpr int WE = BN * 64;            // bf16 per wave per buffer: weights
    constexpr int XE = TM * 16 * 64;       //                             activations
    constexpr int NDMA = (BN + TM * 16) / 8;       // DMA instructions per K group
    constexpr int STAGE = (WE + XE) * 2;   // bytes per wave and group
    constexpr int STAGES = dec_stages(TM, BN, DEEP);
    __shared__ __attribute__((aligned(1024))) char smem[4 * STAGES * STAGE];
    // After the main loop (every DMA landed, a barrier passed) it holds the
    // waves' tiles for the reduction, the per-row sums of squares and the
    // last-workgroup flag.
    constexpr int RB = FR * 64 * 16;   // bytes of one wave's tile
    static_assert(4 * RB + (NORM ? 4 * TM * 16 * 4 : 0) + 4 <= (int)sizeof(smem), "reduction buffer");
    float (*const s_ssq)[TM * 16] = reinterpret_cast<float (*)[TM * 16]>(smem + 4 * RB);
    int* const s_last = reinterpret_cast<int*>(smem + 4 * RB) + (NORM ? 4 * TM * 16 : 0);
    // K-split partial tiles are DEC_TILE_FLOATS apart in the workspace: the
    // plan splits K only for kernels whose tile fits that stride.
    constexpr bool SPLITTABLE = FR * 64 * 4 <= DEC_TILE_FLOATS;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int tiles_n = (N + BN - 1) / BN;
    // XCD-aware order: the dispatcher deals workgroup ids round-robin over
    // the 8 XCDs; XCD x takes the x-th contiguous range of units (the first
    // nb % 8 ranges one longer), so the row tiles of one (column slice,
    // split) pair -- which read the same weights -- run on the same XCD.
    int bid = blockIdx.x;
    {
        const int nb = gridDim.x, x = bid & 7;
        bid = x * (nb >> 3) + min(x, nb & 7) + (bid >> 3);
    }
    const int mt = bid % m_tiles;
    const int unit = bid / m_tiles;
    const int split = unit % splits, nt = unit / splits;
    const int m0 = mt * 16 * TM, n0 = nt * BN;
    const int kgroups = K >> 6;
    const int s_begin = split * groups_per_split;
    const int s_end = min(kgroups, s_begin + groups_per_split);
    const int gpw = (groups_per_split + 3) >> 2;
    const int w_begin = min(s_end, s_begin + wave * gpw);
    const int w_end = min(s_end, w_begin + gpw);

    // this wave's buffers: BN weight rows, then 16 TM activation rows each
    auto buf = [&](int b) { return reinterpret_cast<bf16_t*>(smem + (wave * STAGES + b) * STAGE); };
    auto dma = [&](int grp, bf16_t* to) {
        dec_dma<BN, NTW>(W, ldw, n0, N, grp * 64, to, lane);
        dec_dma<TM * 16>(A, lda, m0, M, grp * 64, to + WE, lane);
    };

    // Output units: one fragment lane (or a gate/up fragment pair) each.
    constexpr int G = PAIRED ? 2 : 1;
    constexpr int UNITS = FR / G * 64;
    constexpr int PER = (UNITS + 255) / 256;
    // the units' destination rows, loaded here so that the epilogue does not
    // wait for them
    constexpr bool ROWS = epi_row_info<Epi>::value;
    int2 row_of[ROWS ? PER : 1];
    if constexpr (ROWS) {
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int u = min(tid + 256 * q, UNITS - 1);
            row_of[q] = epi.row_info(min(m0 + ((u >> 6) * G / TN) * 16 + (u & 15), M - 1));
        }
    }

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // NORM: per-lane sum of squares of the activation elements it reads
    // (row i * 16 + r, chunks g and 4 + g of every K group of the wave)
    float ssq[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) ssq[i] = 0.f;
    // both 32-wide steps of a K group: fragment reads first, then the MFMAs
    auto compute = [&](const bf16_t* wl) {
        const bf16_t* const xl = wl + WE;
        bf16x8 wa[2][TN], xb[2][TM];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int j = 0; j < TN; ++j) wa[u][j] = dec_frag(wl, j * 16 + r, u * 4 + g);
#pragma unroll
            for (int i = 0; i < TM; ++i) xb[u][i] = dec_frag(xl, i * 16 + r, u * 4 + g);
        }
        if constexpr (NORM) {
            typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    const uint4 w4 = __builtin_bit_cast(uint4, xb[u][i]);
                    const unsigned w[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const bf16x2_t pr = __builtin_bit_cast(bf16x2_t, w[e]);
                        ssq[i] = __builtin_amdgcn_fdot2_f32_bf16(pr, pr, ssq[i], false);
                    }
                }
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[u][j], xb[u][i], acc[i][j], 0, 0, 0);
    };

    // Group w_begin + i sits in buffer i % STAGES; multiplying it first puts
    // the group STAGES - 1 further on in flight, into the buffer that the
    // group before it has left (wait_lds: that one has been read).  Two and three
    // buffers as plain code: one loop over all depths costs the launches of
    // several row tiles 1-3 % (80 x 8192 x 1024: 9.14 -> 9.36 us).
    if constexpr (STAGES == 2) {
        bf16_t* const b0 = buf(0);
        bf16_t* const b1 = buf(1);
        auto step = [&](int gi, bf16_t* cur, bf16_t* nxt) {
            wait_lds();
            if (gi + 1 < w_end) {
                dma(gi + 1, nxt);
                wait_vmcnt<NDMA>();
            } else {
                wait_vmcnt<0>();
            }
            compute(cur);
        };
        if (w_begin < w_end) dma(w_begin, b0);
        for (int gi = w_begin; gi < w_end; gi += 2) {
            step(gi, b0, b1);
            if (gi + 1 >= w_end) break;
            step(gi + 1, b1, b0);
        }
    } else if constexpr (STAGES == 3) {
        bf16_t* const b0 = buf(0);
        bf16_t* const b1 = buf(1);
        bf16_t* const b2 = buf(2);
        auto step = [&](int gi, bf16_t* cur, bf16_t* nxt) {
            wait_lds();
            if (gi + 2 < w_end) {
                dma(gi + 2, nxt);
                wait_vmcnt<2 * NDMA>();
            } else if (gi + 1 < w_end) {
                wait_vmcnt<NDMA>();
            } else {
                wait_vmcnt<0>();
            }
            compute(cur);
        };
        if (w_begin < w_end) dma(w_begin, b0);
        if (w_begin + 1 < w_end) dma(w_begin + 1, b1);
        for (int gi = w_begin; gi < w_end; gi += 3) {
            step(gi, b0, b2);
            if (gi + 1 >= w_end) break;
            step(gi + 1, b1, b0);
            if (gi + 2 >= w_end) break;
            step(gi + 2, b2, b1);
        }
    } else {
#pragma unroll
        for (int i = 0; i < STAGES - 1; ++i)
            if (w_begin + i < w_end) dma(w_begin + i, buf(i));
        for (int gi = w_begin; gi < w_end; gi += STAGES) {
#pragma unroll
            for (int i = 0; i < STAGES; ++i) {
                if (gi + i >= w_end) break;
                wait_lds();
                if (gi + i + STAGES - 1 < w_end) dma(gi + i + STAGES - 1, buf((i + STAGES - 1) % STAGES));
                wait_tiles<STAGES - 1, NDMA>(w_end - 1 - gi - i);
                compute(buf(i));
            }
        }
    }

    // waves' tiles through LDS (the staging buffers, once every wave is done)
    __syncthreads();
    auto red_region = [&](int w) { return reinterpret_cast<f32x4*>(smem + w * RB); };
    f32x4* const red = red_region(wave);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) red[(i * TN + j) * 64 + lane] = acc[i][j];
    if constexpr (NORM) {
        // lanes r, r + 16, r + 32, r + 48 hold row r's four chunk columns
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            float t = ssq[i];
            t += __shfl_xor(t, 16, 64);
            t += __shfl_xor(t, 32, 64);
            if (g == 0) s_ssq[wave][i * 16 + r] = t;
        }
    }
    __syncthreads();
    auto red_at = [&](int w, int e) -> f32x4 { return red_region(w)[e]; };

    f32x4 v[PER][G];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int u = tid + 256 * q;
        if (u < UNITS) {
            const int f0 = (u >> 6) * G, l = u & 63;
#pragma unroll
            for (int h = 0; h < G; ++h) {
                const int e = (f0 + h) * 64 + l;
                v[q][h] = ((red_at(0, e) + red_at(1, e)) + red_at(2, e)) + red_at(3, e);
            }
        }
    }

    if (SPLITTABLE && splits > 1) {
        // A workgroup waits for its own partial stores to complete before it
        // bumps the counter; the last one reads the partials only after
        // seeing the final count.
        const int tile = nt * m_tiles + mt;
        const __amdgpu_buffer_rsrc_t part =
            coherent_rsrc(ws + (size_t)tile * splits * DEC_TILE_FLOATS);
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int u = tid + 256 * q;
            if (u < UNITS) {
                const int f0 = (u >> 6) * G, l = u & 63;
#pragma unroll
                for (int h = 0; h < G; ++h)
                    st_coherent4(part, (split * DEC_TILE_FLOATS + ((f0 + h) * 64 + l) * 4) * 4, v[q][h]);
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0)
            *s_last = __hip_atomic_fetch_add(counters + tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                      (unsigned)(splits - 1);
        __syncthreads();
        if (!*s_last) return;
        // all splits' loads in flight at once, then summed in split order
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int u = tid + 256 * q;
            if (u < UNITS) {
                const int f0 = (u >> 6) * G, l = u & 63;
#pragma unroll
                for (int h = 0; h < G; ++h) {
                    const int off = ((f0 + h) * 64 + l) * 16;
                    f32x4 t[DEC_MAX_SPLITS];
#pragma unroll
                    for (int sp = 0; sp < DEC_MAX_SPLITS; ++sp)
                        t[sp] = ld_coherent4(part, min(sp, splits - 1) * DEC_TILE_FLOATS * 4 + off);
                    f32x4 acc_t = t[0];
#pragma unroll
                    for (int sp = 1; sp < DEC_MAX_SPLITS; ++sp)
                        if (sp < splits) acc_t += t[sp];
                    v[q][h] = acc_t;
                }
            }
        }
        if (tid == 0) __hip_atomic_store(counters + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }

#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int u = tid + 256 * q;
        if (u < UNITS) {
            const int fg = u >> 6, l = u & 63;
            const int f0 = fg * G;
            const int i = f0 / TN, j = f0 - i * TN;
            const int m = m0 + i * 16 + (l & 15);
            const int n = n0 + j * 16 + 4 * (l >> 4);
            if constexpr (NORM) {
                // RMSNorm of the row, summed over the waves' K ranges in wave order
                const int row = i * 16 + (l & 15);
                const float ss = ((s_ssq[0][row] + s_ssq[1][row]) + s_ssq[2][row]) + s_ssq[3][row];
                const float rs = 1.0f / sqrtf(ss / (float)K + norm_eps);
#pragma unroll
                for (int h = 0; h < G; ++h) v[q][h] *= rs;
            }
            if (m < M && n < N) {
                if constexpr (PAIRED) {
                    float gv[4] = {v[q][0][0], v[q][0][1], v[q][0][2], v[q][0][3]};
                    float uv[4] = {v[q][1][0], v[q][1][1], v[q][1][2], v[q][1][3]};
                    if constexpr (ROWS) epi.pair_at(row_of[q], m, n, gv, uv);
                    else epi.pair(m, n, gv, uv);
                } else {
                    epi(m, n, v[q][0][0], v[q][0][1], v[q][0][2], v[q][0][3]);
                }
            }
        }
    }
}


// ------------------------------------------------------------ fp32 GEMM --
// (16 TM) x (16 TN) tiles on v_mfma_f32_16x16x4_f32 (fp32 products and sums),
// fragments loaded straight from global memory: lane (r, g) holds four
// consecutive K elements of row r, and MFMA step e takes element e of every
// lane, so one 16-byte load per fragment row feeds four steps.  The four waves
// take a quarter of K each and their tiles are summed in wave order through
// LDS: an element's order is a function of K alone.  The fp32 policies are
// small (launch latency, not bytes): splitting K inside the workgroup keeps
// the load chain short and a product is one launch -- the 64 x 64 LDS tiles
// it replaces took 24-91 us per prefill projection and 12.6 + 4.6 us (K split
// over workgroups, then a reduction launch) per decode projection of the tiny
// policy, where this takes 3-7.
// NORM: output rows scaled by the RMSNorm factor of the input rows.
// U: 16-wide K groups loaded at a time.
template <int TM, int TN, int U, bool NORM, bool PAIRED, class Epi>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ A, int lda,
                                                       const float* __restrict__ B, int ldb, int M, int N,
                                                       int K, float norm_eps, Epi epi)
{
    constexpr int FR = TM * TN, G = PAIRED ? 2 : 1;
    static_assert(!PAIRED || TN % 2 == 0, "paired epilogue needs fragment pairs");
    // operand rows need the alignment of a float only
    typedef f32x4 f32x4_u __attribute__((aligned(4)));
    __shared__ f32x4 red[4][FR * 64];
    __shared__ float s_ssq[4][NORM ? TM * 16 : 1];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int tiles_n = (N + 16 * TN - 1) / (16 * TN);
    const int tmi = blockIdx.x / tiles_n, tni = blockIdx.x - tmi * tiles_n;
    const int m0 = tmi * 16 * TM, n0 = tni * 16 * TN;
    const int groups = (K + 15) >> 4, gpw = (groups + 3) >> 2;
    const int g_begin = min(groups, wave * gpw), g_end = min(groups, g_begin + gpw);
    const float* pa[TM];
    const float* pb[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) pa[i] = A + (size_t)min(m0 + i * 16 + r, M - 1) * lda + 4 * g;
#pragma unroll
    for (int j = 0; j < TN; ++j) pb[j] = B + (size_t)min(n0 + j * 16 + r, N - 1) * ldb + 4 * g;
    f32x4 acc[TM][TN];
    float ssq[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        ssq[i] = 0.f;
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    for (int gi = g_begin; gi < g_end; gi += U) {
        f32x4 a[U][TM], b[U][TN];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = (gi + u) * 16;
            // past the wave's range (K % 4 == 0): loaded from inside the row
            // and zeroed, so that no load hangs on a branch
            const bool in = gi + u < g_end && k + 4 * g < K;
            const int off = min(k, K - 4 - 4 * g);
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                a[u][i] = *reinterpret_cast<const f32x4_u*>(pa[i] + off);
                if (!in) a[u][i] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                b[u][j] = *reinterpret_cast<const f32x4_u*>(pb[j] + off);
                if (!in) b[u][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    if constexpr (NORM) ssq[i] = fmaf(a[u][i][e], a[u][i][e], ssq[i]);
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[u][j][e], a[u][i][e], acc[i][j], 0, 0, 0);
                }
        }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int j = 0; j < TN; ++j) red[wave][(i * TN + j) * 64 + lane] = acc[i][j];
        if constexpr (NORM) {
            float t = ssq[i];
            t += __shfl_xor(t, 16, 64);
            t += __shfl_xor(t, 32, 64);
            if (g == 0) s_ssq[wave][i * 16 + r] = t;
        }
    }
    __syncthreads();
    for (int u = tid; u < FR / G * 64; u += 256) {
        const int f0 = (u >> 6) * G, l = u & 63;
        const int i = f0 / TN, j = f0 - i * TN;
        const int m = m0 + i * 16 + (l & 15), n = n0 + j * 16 + 4 * (l >> 4);
        f32x4 v[G];
#pragma unroll
        for (int h = 0; h < G; ++h) {
            const int e = (f0 + h) * 64 + l;
            v[h] = ((red[0][e] + red[1][e]) + red[2][e]) + red[3][e];
        }
        if constexpr (NORM) {
            const int row = i * 16 + (l & 15);
            const float ss = ((s_ssq[0][row] + s_ssq[1][row]) + s_ssq[2][row]) + s_ssq[3][row];
            const float rs = 1.0f / sqrtf(ss / (float)K + norm_eps);
#pragma unroll
            for (int h = 0; h < G; ++h) v[h] *= rs;
        }
        if (m < M && n < N) {
            if constexpr (PAIRED) {
                float gv[4] = {v[0][0], v[0][1], v[0][2], v[0][3]};
                float uv[4] = {v[1][0], v[1][1], v[1][2], v[1][3]};
                epi.pair(m, n, gv, uv);
            } else {
                epi(m, n, v[0][0], v[0][1], v[0][2], v[0][3]);
            }
        }
    }
}

// Sum split partials in split order, then apply the epilogue.  One thread
// per (row, 4 output columns); for paired epilogues the output columns are
// the gate columns (packed n % 32 < 16).
template <bool PAIRED, class Epi>
__global__ void splitk_reduce_kernel(const float* __restrict__ ws, int splits, int M, int N,
                                     Epi epi)
{
    const int groups = PAIRED ? N / 8 : N / 4;
    const long total = (long)M * groups;
    for (long idx = blockIdx.x * (long)blockDim.x + threadIdx.x; idx < total;
         idx += (long)gridDim.x * blockDim.x) {
        const int m = (int)(idx / groups);
        const int gq = (int)(idx - (long)m * groups);
        int n;
        if (PAIRED) n = (gq >> 2) * 32 + (gq & 3) * 4;
        else n = gq * 4;
        float v[4] = {0.f, 0.f, 0.f, 0.f}, u[4] = {0.f, 0.f, 0.f, 0.f};
        for (int s = 0; s < splits; ++s) {
            const float4 a = *reinterpret_cast<const float4*>(ws + ((size_t)s * M + m) * N + n);
            v[0] += a.x; v[1] += a.y; v[2] += a.z; v[3] += a.w;
            if (PAIRED) {
                const float4 b =
                    *reinterpret_cast<const float4*>(ws + ((size_t)s * M + m) * N + n + 16);
                u[0] += b.x; u[1] += b.y; u[2] += b.z; u[3] += b.w;
            }
        }
        if constexpr (PAIRED) epi.pair(m, n, v, u);
        else epi(m, n, v[0], v[1], v[2], v[3]);
    }
}

// ------------------------------------------------------------- dispatch --

// Tile and split choice depend only on (M, N, K), the stream's CU count and the
// epilogue; the split count, the only one that orders sums, on (N, K) alone.
struct GemmPlan {
    int bm; int splits; int k_per_split;
    bool seq;      // K in order: the large-M kernel (bm 256) or the ring kernel (bm x bn)
    int bn; int grid, full, split;   // large-M kernel: workgroups, evenly dealt tiles, cut of the last round's tiles
    bool dec; int steps_per_split; int tm; int m_tiles; int dbn; bool deep;   // decode kernel (steps: 64-wide K groups)
};

// Kernel and split choice.  The tile variant never changes an element's
// summation order; the split count (decode only) is a function of (N, K).
constexpr int SPLIT_MAX_M = DECODE_MAX_ROWS;

// Projections that sum K in order (prefill, ViT, experts): the kernel whose
// modelled time (us) is least.  The constants are a fit to all six variants on
// 184 products (fp32 output, M 257 to 8192, N 1024 to 22016, K 1024 to 11008, 256
// CUs; modelled times scatter by 5 %), and to the projections of 33 policy calls,
// each run with all six.  The variant it picks is on average 0.3 % (at worst 8 %)
// slower than the best one on the products, and costs the calls 0.1 % a projection;
// one constant per variant and no rounds cost 1.4 % and 0.3 % (640 x 4096 x 11008 104
// us instead of 79, 300 x 12288 x 4096 52 instead of 45).  No choice changes a sum's
// order.
// `extra`: how much longer a tile's epilogue takes the large kernel than the
// ring, whose other workgroup on the CU multiplies meanwhile (0 for plain stores
// and SwiGLU).
static void plan_in_order(GemmPlan& p, int M, int N, int K, int cus, double extra) {
    const double nk = K / 64;
    auto up = [](long a, long b) { return (a + b - 1) / b; };
    const long tiles = up(M, 256) * up(N, 256);
    const long rounds = tiles / cus, full = rounds * cus, rest = tiles - full;
    p.seq = true;
    p.bm = p.bn = 256;
    p.full = (int)full;
    double best = 0;
    // 256 x 256 tiles: whole rounds, then the remaining tiles whole or cut in
    // two or four where the pieces fit one round.  A K tile of a piece takes
    // `alone` with the chip nearly empty and `busy` with a piece on every CU.
    struct Cut { int split; double c, alone, busy; } cuts[] = {{1, 8.0, 0.75, 1.24}, {2, 5.6, 0.50, 0.78}, {4, 4.0, 0.38, 0.55}};
    for (const Cut& v : cuts) {
        if (v.split > 1 && (!rest || rest * v.split > cus)) continue;
        // (pieces past the last row or column have nothing to do)
        const long pieces = full || v.split == 1 ? rest * v.split : up(M, 128) * up(N, v.split == 2 ? 256 : 128);
        double t = v.c + extra + rounds * (8.7 + 1.39 * nk);
        if (rest) t += nk * (v.alone + (v.busy - v.alone) * pieces / cus);
        if (v.split == 1 || t < best) {
            best = t;
            p.split = v.split;
        }
    }
    p.grid = (int)(full ? cus : rest * p.split);
    // Ring tiles: two workgroups share a CU, so they take rounds of one (`one`
    // us a K tile) or two (`two`) a CU.  Each group of four row tiles streams the
    // weights once: the first at 5.5 TB/s, the others, on other XCDs, at 3.6; of
    // that and the K loop the shorter one shows by a tenth.
    struct Ring { int bm, bn; double c, epi, one, two; } rings[] = {{64, 128, 2.4, 1.7, 0.353, 0.610},
                                                                    {64, 64, 2.3, 1.0, 0.225, 0.355},
                                                                    {32, 64, 2.4, 0.7, 0.175, 0.262}};
    for (const Ring& v : rings) {
        const long wgs = up(M, v.bm) * up(N, v.bn), pairs = wgs / (2 * cus);
        const double left = (double)(wgs - pairs * 2 * cus) / cus;   // workgroups a CU in the last round
        double t = v.c + pairs * (v.epi + nk * v.two);
        if (left > 1) t += v.epi + nk * (v.one + (v.two - v.one) * (0.6 + 0.4 * (left - 1)));
        else if (left > 0) t += v.epi / 2 + nk * v.one;
        const double w = (double)N * K * 2e-6 * (1 / 5.5 + (up(up(M, v.bm), 4) - 1) / 3.6);
        t = std::max(t, w) + 0.1 * std::min(t, w);
        if (t < best) {
            best = t;
            p.bm = v.bm;
            p.bn = v.bn;
        }
    }
}

// bf16 products
static GemmPlan plan_gemm(int M, int N, int K, size_t ws_floats, bool split_ok, int cus = 256, double extra = 0) {
    GemmPlan p;
    p.seq = false;
    p.dec = false;
    p.splits = 1;
    p.k_per_split = K;
    if (split_ok && K % 64 == 0) {
        // K splits: about 64 (column slice, split) pairs, each split at least
        // 16 K groups (1024 wide) -- the cross-workgroup hand-off costs about
        // as much as streaming that much more.  Narrow outputs with a long K
        // (at least 8192, e.g. a down projection of an 11008-wide MLP) aim for
        // about 256 pairs with splits of at least 512: measured 19-45 % more
        // bandwidth there at 1-64 rows, while shorter K lost by splitting
        // further.  A function of (N, K) only.  The partial tiles (up to four
        // row tiles, 32- or 64-column slices: at most 8 x tiles_n tiles) must
        // fit the workspace and counters.
        p.dec = true;
        const int tiles_n = (N + DEC_BN - 1) / DEC_BN;
        const int kgroups = K / 64;
        const int want = (tiles_n < 128 && kgroups >= 128)
                             ? std::min({(256 + tiles_n - 1) / tiles_n, kgroups / 8, DEC_MAX_SPLITS})
                             : std::max(1, std::min({(64 + tiles_n - 1) / tiles_n, kgroups / 16, DEC_MAX_SPLITS}));
        int gps = (kgroups + want - 1) / want;
        for (;;) {
            const int sp = (kgroups + gps - 1) / gps;
            if (sp == 1) break;
            if (sp <= DEC_MAX_SPLITS && (size_t)sp * 8 * tiles_n * DEC_TILE_FLOATS <= ws_floats &&
                8 * tiles_n <= DEC_MAX_COUNTERS)
                break;
            ++gps;
        }
        p.steps_per_split = gps;
        p.splits = (kgroups + gps - 1) / gps;
        // Row tiles of 16, 32 or 64 rows (any choice leaves every sum's
        // order unchanged): up to four row tiles when the column slices x
        // splits alone fill under half the chip -- each workgroup then
        // streams a quarter of the activations; otherwise the fewest tiles.
        if ((long)tiles_n * p.splits >= 128) p.tm = M <= 16 ? 1 : (M <= 32 ? 2 : 4);
        else p.tm = M <= 64 ? 1 : (M <= 128 ? 2 : 4);
        p.m_tiles = (M + 16 * p.tm - 1) / (16 * p.tm);
        // 32-column slices when that still leaves under 3/4 of the CUs idle
        p.dbn = (long)tiles_n * p.splits * p.m_tiles < 3L * cus / 4 ? 32 : 64;
        // 96-column slices (fragment pairs stay whole; two LDS buffers) when
        // they take fewer rounds of one workgroup per CU: priced as rounds x
        // the bytes a workgroup streams per K element (weight plus
        // activation rows).  A CU's DMA stream runs at about the same rate
        // for either width, so the last, partly filled round is what the
        // wider slice saves: 7B-class gate/up (22016 outputs: 344 slices of
        // 64 = 1.34 rounds, 230 of 96 = one) measured 20-24 % faster at 1-32
        // rows; narrower outputs (one round either way) lose.  Row tiles of
        // 64 with 96 columns fill the LDS and leave no partial-tile stride
        // for K splits; smaller row tiles take 96 columns with one row tile
        // only.  The slice width never changes a sum's order.
        if (p.dbn == 64 && (p.tm == 4 ? p.splits == 1 : p.m_tiles == 1)) {
            auto cost = [&](int bn) {
                const long wgs = (long)((N + bn - 1) / bn) * p.splits * p.m_tiles;
                return ((wgs + cus - 1) / cus) * (bn + 16 * p.tm);
            };
            if (cost(96) < cost(64)) p.dbn = 96;
        }
        // 32-column slices of up to 32 rows keep four K groups in LDS where
        // every workgroup has a CU to itself: those launches are held by
        // latency (one row, weights from HBM as in a policy: 4096 x 4096 11.8 ->
        // 9.9 us, 3072 x 1024 4.40 -> 4.17; 17 rows of 4096 x 4096 11.8 -> 10.1;
        // weights left in L2 by the last call: 7.3 -> 6.9, 2.93 -> 3.11 and 7.5 ->
        // 8.4).  With more workgroups than CUs the 96 or 128 KB would leave one on a CU and the rest to a
        // second round, where two groups let two or three share it (3072
        // outputs, K 1024, 288 workgroups: 5.1 us with four, 3.8 with two at 40
        // rows, 6.3 and 4.7 at 80); 64 rows are slower with more than two as
        // well (7.5 -> 8.1 us).
        p.deep = p.dbn == 32 && p.tm <= 2 && (long)((N + 31) / 32) * p.splits * p.m_tiles <= cus;
        return p;
    }
    if (K % 64 == 0) {
        plan_in_order(p, M, N, K, cus, extra);
        return p;
    }
    if (M <= 16) p.bm = 16;
    else if (M <= 32) p.bm = 32;
    else if (M <= 64) p.bm = 64;
    else p.bm = 128;
    if (!split_ok) return p;
    // one row of 128-wide column tiles -> enough K splits for ~512 workgroups
    const long tiles = (N + 127) / 128;
    int splits = 1;
    if (tiles < 256) {
        const int kblocks = (K + BK - 1) / BK;
        splits = (int)std::min<long>((512 + tiles - 1) / tiles, (long)std::max(1, kblocks / 2));
        splits = std::max(1, std::min(splits, 16));
    }
    while (splits > 1 && (size_t)splits * SPLIT_MAX_M * N > ws_floats) --splits;
    int kps = (K + splits - 1) / splits;
    kps = (kps + BK - 1) / BK * BK;
    p.splits = (K + kps - 1) / kps;
    p.k_per_split = kps;
    return p;
}

template <bool PAIRED, class Epi>
static void launch_bf16(const GemmArgs& a, const GemmPlan& p, Epi epi, hipStream_t s) {
    const bool split = p.splits > 1;
    if (p.seq) {
        const bf16_t *A = (const bf16_t*)a.A, *B = (const bf16_t*)a.B;
        if (p.bm == 256) {
            hipLaunchKernelGGL((gemm_bf16_big_kernel<PAIRED, Epi>), dim3(p.grid), dim3(512), 0, s, A, a.lda, B, a.ldb,
                               a.M, a.N, a.K, p.full, p.split, epi);
            return;
        }
        const dim3 grid((unsigned)((long)((a.M + p.bm - 1) / p.bm) * ((a.N + p.bn - 1) / p.bn)));
        auto ring = [&](auto kern) {
            hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, A, a.lda, B, a.ldb, a.M, a.N, a.K, epi);
        };
        if (p.bn == 128) ring(gemm_bf16_ring_kernel<64, 128, 3, PAIRED, Epi>);
        else if (p.bm == 64) ring(gemm_bf16_ring_kernel<64, 64, 3, PAIRED, Epi>);
        else ring(gemm_bf16_ring_kernel<32, 64, 4, PAIRED, Epi>);
        return;
    }
    if (p.dec) {
        auto godec = [&](auto kern, int bn) {
            dim3 grid(((a.N + bn - 1) / bn) * p.splits * p.m_tiles);
            hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, (const bf16_t*)a.A, a.lda, (const bf16_t*)a.B,
                               a.ldb, a.M, a.N, a.K, p.steps_per_split, p.splits, p.m_tiles, a.ws,
                               a.counters, a.norm_eps, epi);
        };
        // Non-temporal weight loads where each weight slice is read by a
        // single workgroup (one row tile) of 64- or 96-column slices: measured 5-13 %
        // faster there, slower where row tiles or narrow slices re-read it.
        auto pick = [&](auto NORM) {
            constexpr bool NM = decltype(NORM)::value;
            if (p.dbn == 96) {   // row tiles of 16 or 32 rows: one tile (plan_gemm)
                if (p.tm == 1) godec(gemm_bf16_decode_kernel<1, 96, true, false, NM, PAIRED, Epi>, 96);
                else if (p.tm == 2) godec(gemm_bf16_decode_kernel<2, 96, true, false, NM, PAIRED, Epi>, 96);
                else if (p.m_tiles == 1) godec(gemm_bf16_decode_kernel<4, 96, true, false, NM, PAIRED, Epi>, 96);
                else godec(gemm_bf16_decode_kernel<4, 96, false, false, NM, PAIRED, Epi>, 96);
            } else if (p.dbn == 32) {
                if (p.tm == 4) godec(gemm_bf16_decode_kernel<4, 32, false, false, NM, PAIRED, Epi>, 32);
                else if (p.tm == 2 && p.deep) godec(gemm_bf16_decode_kernel<2, 32, false, true, NM, PAIRED, Epi>, 32);
                else if (p.tm == 2) godec(gemm_bf16_decode_kernel<2, 32, false, false, NM, PAIRED, Epi>, 32);
                else if (p.deep) godec(gemm_bf16_decode_kernel<1, 32, false, true, NM, PAIRED, Epi>, 32);
                else godec(gemm_bf16_decode_kernel<1, 32, false, false, NM, PAIRED, Epi>, 32);
            } else if (p.m_tiles == 1) {
                if (p.tm == 1) godec(gemm_bf16_decode_kernel<1, 64, true, false, NM, PAIRED, Epi>, 64);
                else if (p.tm == 2) godec(gemm_bf16_decode_kernel<2, 64, true, false, NM, PAIRED, Epi>, 64);
                else godec(gemm_bf16_decode_kernel<4, 64, true, false, NM, PAIRED, Epi>, 64);
            } else {
                if (p.tm == 1) godec(gemm_bf16_decode_kernel<1, 64, false, false, NM, PAIRED, Epi>, 64);
                else if (p.tm == 2) godec(gemm_bf16_decode_kernel<2, 64, false, false, NM, PAIRED, Epi>, 64);
                else godec(gemm_bf16_decode_kernel<4, 64, false, false, NM, PAIRED, Epi>, 64);
            }
        };
        // the folded RMSNorm exists for the projections that follow a norm
        // (fused QKV, gate/up) and needs the whole K in one workgroup
        if constexpr (PAIRED) {
            if (a.row_norm && p.splits == 1) { pick(std::true_type{}); return; }
        }
        pick(std::false_type{});
        return;
    }
    auto go = [&](auto kern, int bm, int bn) {
        dim3 grid(((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn), p.splits);
        hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, (const bf16_t*)a.A, a.lda,
                           (const bf16_t*)a.B, a.ldb, a.M, a.N, a.K, p.k_per_split, a.ws, epi);
    };
    switch (p.bm) {
    case 16:
        if (split) go(gemm_bf16_kernel<16, 256, 1, 4, PAIRED, true, Epi>, 16, 256);
        else go(gemm_bf16_kernel<16, 256, 1, 4, PAIRED, false, Epi>, 16, 256);
        break;
    case 32:
        if (split) go(gemm_bf16_kernel<32, 128, 1, 4, PAIRED, true, Epi>, 32, 128);
        else go(gemm_bf16_kernel<32, 128, 1, 4, PAIRED, false, Epi>, 32, 128);
        break;
    case 64:
        if (split) go(gemm_bf16_kernel<64, 128, 1, 4, PAIRED, true, Epi>, 64, 128);
        else go(gemm_bf16_kernel<64, 128, 1, 4, PAIRED, false, Epi>, 64, 128);
        break;
    default:
        if (split) go(gemm_bf16_kernel<128, 128, 2, 2, PAIRED, true, Epi>, 128, 128);
        else go(gemm_bf16_kernel<128, 128, 2, 2, PAIRED, false, Epi>, 128, 128);
        break;
    }
    if (split) {
        const int groups = PAIRED ? a.N / 8 : a.N / 4;
        long total = (long)a.M * groups;
        int blocks = (int)std::min<long>((total + 255) / 256, 4096);
        hipLaunchKernelGGL((splitk_reduce_kernel<PAIRED, Epi>), dim3(blocks), dim3(256), 0, s,
                           a.ws, p.splits, a.M, a.N, epi);
    }
}

template <bool PAIRED, class Epi>
static void launch_f32(const GemmArgs& a, Epi epi, hipStream_t s) {
    auto tiles = [&](int tm, int tn) {
        return (long)((a.M + 16 * tm - 1) / (16 * tm)) * ((a.N + 16 * tn - 1) / (16 * tn));
    };
    auto go = [&](auto kern, int tm, int tn) {
        hipLaunchKernelGGL(kern, dim3((unsigned)tiles(tm, tn)), dim3(256), 0, s, (const float*)a.A, a.lda,
                           (const float*)a.B, a.ldb, a.M, a.N, a.K, a.norm_eps, epi);
    };
    // The largest tile that still gives every CU two workgroups (64 x 64) or
    // one (32 x 32); below that, latency counts and the smallest fragments win.
    auto pick = [&](auto NORM) {
        constexpr bool NM = decltype(NORM)::value;
        if (a.M > 32 && tiles(4, 4) >= 512) go(gemm_f32_kernel<4, 4, 2, NM, PAIRED, Epi>, 4, 4);
        else if (a.M > 16 && tiles(2, 2) >= 256) go(gemm_f32_kernel<2, 2, 4, NM, PAIRED, Epi>, 2, 2);
        else if constexpr (PAIRED) go(gemm_f32_kernel<1, 2, 4, NM, PAIRED, Epi>, 1, 2);
        // Long K: a wave's quarter of it in rounds of 256 instead of 64 elements,
        // each a memory latency (8 rows, K 1024: 8.1 -> 6.9 us, the tiny policy's call
        // 438 -> 414 us); below, rounds of 256 would mostly load padding.
        else if (a.K >= 1024) go(gemm_f32_kernel<1, 1, 16, NM, PAIRED, Epi>, 1, 1);
        else go(gemm_f32_kernel<1, 1, 4, NM, PAIRED, Epi>, 1, 1);
    };
    if constexpr (PAIRED) {
        if (a.row_norm) { pick(std::true_type{}); return; }
    }
    pick(std::false_type{});
}

template <bool PAIRED, class Epi>
static int dispatch(const GemmArgs& a, Epi epi, hipStream_t s) {
    if (!a.bf16) {   // one launch, K split inside the workgroup
        launch_f32<PAIRED>(a, epi, s);
        return 1;
    }
    const GemmPlan p = plan_gemm(a.M, a.N, a.K, a.ws_floats, a.split_ok && a.M <= SPLIT_MAX_M && a.counters,
                                 std::max(1, std::min(a.cus, 256)),
                                 a.epi == EPI_QKV ? 6.0 : a.epi == EPI_RESID ? 1.5 : 0.0);
    launch_bf16<PAIRED>(a, p, epi, s);
    return p.splits;
}

int gemm(const GemmArgs& a, hipStream_t s) {
    if (a.M <= 0 || a.N <= 0) return 0;
    switch (a.epi) {
    case EPI_F32:
        return dispatch<false>(a, EpiF32{(float*)a.C, a.ldc}, s);
    case EPI_ACT:
        if (a.bf16) return dispatch<false>(a, EpiStore<bf16_t>{(bf16_t*)a.C, a.ldc}, s);
        return dispatch<false>(a, EpiStore<float>{(float*)a.C, a.ldc}, s);
    case EPI_RESID:
        return dispatch<false>(a, EpiResid{(float*)a.C, a.ldc, (bf16_t*)a.xb, a.ldxb}, s);
    case EPI_REMAP:
        if (a.bf16)
            return dispatch<false>(a, EpiRemap<bf16_t>{(float*)a.C, a.ldc, a.row_base, a.group,
                                                       (const bf16_t*)a.add, a.add_ld}, s);
        return dispatch<false>(a, EpiRemap<float>{(float*)a.C, a.ldc, a.row_base, a.group,
                                                  (const float*)a.add, a.add_ld}, s);
    case EPI_SWIGLU:
        if (a.bf16) return dispatch<true>(a, EpiSwiGLU<bf16_t>{(bf16_t*)a.C, a.ldc}, s);
        return dispatch<true>(a, EpiSwiGLU<float>{(float*)a.C, a.ldc}, s);
    case EPI_QKV:
        if (a.bf16) return dispatch<true>(a, make_epi_qkv<bf16_t>(*a.rope), s);
        return dispatch<true>(a, make_epi_qkv<float>(*a.rope), s);
    }
    return 0;
}

void gemm_plan_info(bool bf16, int M, int N, int K, size_t ws_floats, bool split_ok, int cus, int32_t* out) {
    std::fill(out, out + 8, 0);
    out[3] = 1;
    if (!bf16) { out[0] = GEMM_K_FP32; return; }
    const GemmPlan p = plan_gemm(M, N, K, ws_floats, split_ok && M <= SPLIT_MAX_M, cus);
    out[3] = p.splits;
    if (p.dec) {
        out[0] = GEMM_K_DECODE;
        out[1] = 16 * p.tm;
        out[2] = p.dbn;
        out[4] = ((N + p.dbn - 1) / p.dbn) * p.splits * p.m_tiles;
        out[5] = dec_stages(p.tm, p.dbn, p.deep);
    } else if (p.seq) {
        out[0] = p.bm == 256 ? GEMM_K_LARGE : GEMM_K_RING;
        out[1] = p.bm;
        out[2] = p.bn;
        out[4] = p.bm == 256 ? p.grid : ((M + p.bm - 1) / p.bm) * ((N + p.bn - 1) / p.bn);
        if (p.bm == 256) { out[6] = p.full; out[7] = p.split; }
    } else {
        out[0] = GEMM_K_TILES;
    }
}

bool gemm_row_norm_ok(bool bf16, int M, int N, int K, size_t ws_floats) {
    if (!bf16) return true;   // one workgroup always sees the whole K
    if (M > SPLIT_MAX_M || K % 64) return false;
    const GemmPlan p = plan_gemm(M, N, K, ws_floats, true);
    return p.dec && p.splits == 1;
}

size_t gemm_counter_words() {
    return DEC_MAX_COUNTERS;
}

size_t gemm_ws_floats_used(bool bf16, int M, int N, int K, size_t ws_floats, bool split_ok) {
    if (!bf16) return 0;
    const GemmPlan p = plan_gemm(M, N, K, ws_floats, split_ok && M <= SPLIT_MAX_M);
    if (p.splits <= 1) return 0;
    if (p.dec) return (size_t)((N + p.dbn - 1) / p.dbn) * p.m_tiles * p.splits * DEC_TILE_FLOATS;
    return (size_t)p.splits * M * N;
}

}  // namespace ebrl
