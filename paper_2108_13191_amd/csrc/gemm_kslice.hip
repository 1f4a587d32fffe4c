// The kernel for small results: eight wavefronts of a workgroup all work on the same small tile of C
// and take its k steps of 64 in turn; their sums are added through LDS at the end.
//
// Such problems are bound by latencies, not by any rate: with one tile per compute unit and the
// wavefronts side by side in the tile (gemm_tiled.hip) a k step costs 0.35 us -- a chain of LDS reads,
// MFMAs and a barrier with nothing else on the SIMD to run meanwhile -- whatever its size.  Here a
// wavefront owns whole k steps: it loads its chunks of A and B into registers (16 bytes a lane, 8
// consecutive lanes of A a row of 128 bytes), writes them to its own part of the LDS, requests its
// next step, reads the fragments back and multiplies.  No barrier in the loop, nothing shared, and
// eight independent chains to cover one another.  (Without the way through LDS a lane would load its own A
// fragment: consecutive lanes in different rows, which the memory pipeline takes one lane a
// clock, 38 GB/s a compute unit against 160.)
//
// Any alignment: a chunk is loaded at 2-byte alignment where the operands need it.  No access leaves
// the matrices and no chunk is taken apart: one that would reach past the end of its row is
// loaded as the row's last 8 elements.  For B that only changes which columns the results belong
// to (the store knows); for the k tail the same shift is applied to A and to the k rows of B, and what
// is then there twice is zeroed in both (in both: zero times infinity must not appear).  N, K >= 8.
#include "gemm_device.h"
#include "../../include/gemm_f16.h"

namespace {

using namespace gemm_dev;

constexpr int KW = 8;                                  // wavefronts: k groups

template <int BM, int BN> struct KsliceShape {
    static constexpr int A_BYTES = BM * BK * 2, B_BYTES = BK * BN * 2, STAGE = A_BYTES + B_BYTES;   // one wavefront's k step
    static constexpr int T_PITCH = BN * 4 + 16;                                       // sums: bytes per row
    static constexpr int LDS = KW * (STAGE > BM * T_PITCH ? STAGE : BM * T_PITCH);
};

typedef uintx4 chunk_any __attribute__((aligned(2)));

// Position of 16-byte chunk c of k row `row` within the row: 32-byte granules (what a transposing
// read takes of a row) are exchanged so that the 8 k rows that such a read touches at a time lie in 8
// different granules of the LDS's 256-byte lines.
template <int BN> __device__ __forceinline__ int b_place(int row, int c)
{
    const int gran = c >> 1, swz = BN >= 64 ? ((row >> 1) & 1) | ((row >> 2) & 2) : (row >> 3) & 1;
    return ((gran ^ swz) << 1) | (c & 1);
}

// U: k steps of a wavefront on their way in registers.
template <typename CT, int BM, int BN, int U, int WG_PER_CU>
__global__ __launch_bounds__(64 * KW, 2 * WG_PER_CU) void gemm_kslice_kernel(const TiledParams p)
{
    typedef KsliceShape<BM, BN> Shape;
    constexpr int MB = BM / 16, NB = BN / 16;
    constexpr int LA = BM / 8, LB = BN / 8;            // loads of a k step: 8 rows x 128 bytes of A, 1 KB of B
    constexpr int LPR = BN / 8, RPL = 64 / LPR;        // lanes (chunks) per k row of B, k rows per load
    __shared__ __attribute__((aligned(1024))) char smem[Shape::LDS];
    const uint32_t smem_base = (uint32_t)(uintptr_t)(lds_ptr_t)smem;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int tile_m, tile_n;
    tile_of_block(p, blockIdx.x, tile_m, tile_n);
    const int m0 = tile_m * BM, n0 = tile_n * BN;
    const bool edge = (m0 + BM > p.M) || (n0 + BN > p.N);

    // ---- global addresses and places in LDS of this lane's chunks -----------------------------
    // A: load t covers tile rows 8t .. 8t+7, lane i row 8t + i/8, chunk i%8 of 8 k, stored at chunk ^ ((row/2)%8)
    const int a_chunk = lane & 7;
    uint32_t a_off[LA];
#pragma unroll
    for (int t = 0; t < LA; t++) {
        int row = 8 * t + (lane >> 3);
        row = m0 + row < p.M ? row : p.M - 1 - m0;                    // loaded, never stored
        a_off[t] = ((uint32_t)row * (uint32_t)p.lda + 8 * a_chunk) * 2u;
    }
    const char* const a_tile = (const char*)(p.A + (int64_t)m0 * p.lda);
    const char* const b_mat = (const char*)p.B;
    const uint32_t stage = smem_base + (uint32_t)wave * Shape::STAGE;
    // row 8t + i/8: (row/2)%8 = (4t + i/16)%8
    const uint32_t a_wr[2] = {stage + (uint32_t)(lane >> 3) * 128u + (uint32_t)((a_chunk ^ (lane >> 4)) * 16),
                              stage + (uint32_t)(lane >> 3) * 128u + (uint32_t)((a_chunk ^ (4 + (lane >> 4))) * 16)};
    // B: load t covers k rows RPL t .., lane i k row RPL t + i/LPR, chunk i%LPR
    const int b_krow = lane / LPR;
    int b_col = n0 + 8 * (lane % LPR);
    if (b_col > p.N - 8) b_col = p.N - 8;
    const uint32_t b_off = ((uint32_t)b_krow * (uint32_t)p.ldb + (uint32_t)b_col) * 2u;
    uint32_t b_wr[2];                                  // loads t = 0 and 1; the k rows of load t + 2 are placed as those of load t
#pragma unroll
    for (int t = 0; t < 2; t++) b_wr[t] = stage + Shape::A_BYTES + (uint32_t)(b_krow * BN * 2 + b_place<BN>(RPL * t + b_krow, lane % LPR) * 16);
    // ---- fragment reads (as in gemm_w4a128.hip: 16x16x32 MFMA, lane l row / column l%16, k 8 (l/16) ..) --
    uint32_t a_rd[2], b_rd[NB];
#pragma unroll
    for (int s = 0; s < 2; s++) a_rd[s] = stage + (uint32_t)(lane & 15) * 128u + (uint32_t)(((4 * s + (lane >> 4)) ^ ((lane & 15) >> 1)) * 16);
    {
        const int j = lane & 15, krow = 8 * (lane >> 4) + (j >> 2);   // of the first read; the second is 4 rows on (placed alike)
#pragma unroll
        for (int fn = 0; fn < NB; fn++)
            b_rd[fn] = stage + Shape::A_BYTES + (uint32_t)(krow * BN * 2 + b_place<BN>(krow, 2 * fn + ((j & 3) >> 1)) * 16 + 8 * (j & 1));
    }

    // ---- k steps: this wavefront's step j is step wave + KW j ----------------------------------
    const int k_full = p.K / BK, KT = (p.K + BK - 1) / BK;
    const int n_whole = k_full > wave ? (k_full - wave + KW - 1) / KW : 0, n_all = KT > wave ? (KT - wave + KW - 1) / KW : 0;
    uintx4 ra[U][LA], rb[U][LB];
    floatx4 acc[MB][NB];
#pragma unroll
    for (int fm = 0; fm < MB; fm++)
#pragma unroll
        for (int fn = 0; fn < NB; fn++) acc[fm][fn] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};

    auto load_whole = [&](int j, uintx4 (&a)[LA], uintx4 (&b)[LB]) {
        const int64_t k0 = (int64_t)(wave + KW * j) * BK;
#pragma unroll
        for (int t = 0; t < LA; t++) a[t] = *reinterpret_cast<const chunk_any*>(a_tile + k0 * 2 + a_off[t]);
#pragma unroll
        for (int t = 0; t < LB; t++) b[t] = *reinterpret_cast<const chunk_any*>(b_mat + (k0 + RPL * t) * p.ldb * 2 + b_off);
    };
    // The step with the k tail: chunk c covers k = k0 + 8c .. + 7; past K - 8 it is loaded as the last 8
    // and its first (k - (K - 8)) elements, which belong to the chunk before it, are zeroed; the k
    // rows of B that sit in the same slots likewise.
    auto load_tail = [&](uintx4 (&a)[LA], uintx4 (&b)[LB]) {
        const int k0 = k_full * BK;
        {
            const int over = k0 + 8 * a_chunk - (p.K - 8), back = over > 0 ? over : 0;
            const char* const src = a_tile + ((int64_t)k0 - back) * 2;
#pragma unroll
            for (int t = 0; t < LA; t++) {
                uintx4 v = *reinterpret_cast<const chunk_any*>(src + a_off[t]);
#pragma unroll
                for (int e = 0; e < 4; e++) v[e] = (2 * e + 1 < back) ? 0u : (2 * e < back) ? (v[e] & 0xffff0000u) : v[e];
                a[t] = v;
            }
        }
#pragma unroll
        for (int t = 0; t < LB; t++) {
            const int slot = RPL * t + b_krow, over = k0 + (slot & ~7) - (p.K - 8), back = over > 0 ? over : 0;
            const uintx4 v = *reinterpret_cast<const chunk_any*>(b_mat + ((int64_t)(k0 + slot - back) * p.ldb + b_col) * 2);
            b[t] = (slot & 7) < back ? uintx4{0u, 0u, 0u, 0u} : v;
        }
    };
    auto load_any = [&](int j, uintx4 (&a)[LA], uintx4 (&b)[LB]) {
        if (j < n_whole) load_whole(j, a, b);
        else load_tail(a, b);
    };
    // The wavefront's LDS operations are carried out in order, so its one stage needs no waits of its own.
    auto put = [&](const uintx4 (&a)[LA], const uintx4 (&b)[LB]) {
#pragma unroll
        for (int t = 0; t < LA; t++) *(__attribute__((address_space(3))) uintx4*)(uintptr_t)(a_wr[t & 1] + 1024u * t) = a[t];
#pragma unroll
        for (int t = 0; t < LB; t++) *(__attribute__((address_space(3))) uintx4*)(uintptr_t)(b_wr[t & 1] + 1024u * t) = b[t];
        asm volatile("" ::: "memory");
    };
    auto mul = [&]() {
#pragma unroll
        for (int s = 0; s < 2; s++) {
            half8 fa[MB], fb[NB];
#pragma unroll
            for (int fn = 0; fn < NB; fn++)
                fb[fn] = __builtin_shufflevector(lds_read_tr16(b_rd[fn] + s * 32 * BN * 2), lds_read_tr16(b_rd[fn] + (s * 32 + 4) * BN * 2), 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
            for (int fm = 0; fm < MB; fm++) fa[fm] = lds_read_b128(a_rd[s] + fm * 16 * 128);
#pragma unroll
            for (int fm = 0; fm < MB; fm++)
#pragma unroll
                for (int fn = 0; fn < NB; fn++)
                    acc[fm][fn] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fb[fn], fa[fm], acc[fm][fn], 0, 0, 0);
        }
        asm volatile("" ::: "memory");
    };

#pragma unroll
    for (int u = 0; u < U; u++) if (u < n_all) load_any(u, ra[u], rb[u]);

    // ---- C and bias in: this thread's groups of 4 columns, on their way while the products are formed --
    typedef typename CVec4<CT>::type ctx4;
    constexpr int TPR = BN / 4, ROWS = 64 * KW / TPR, PASSES = BM > ROWS ? BM / ROWS : 1;
    const int c_row = threadIdx.x / TPR, x = 4 * (threadIdx.x % TPR), nominal = n0 + (x & ~7);
    const int first = (nominal < p.N - 8 ? nominal : p.N - 8) + (x & 7);   // where this thread's results belong: columns first .. first + 3, those >= nominal
    const bool active = BM >= ROWS || c_row < BM;
    CT* const cptr = (CT*)p.C + (int64_t)(m0 + c_row) * p.ldc + first;
    ctx4 cin[PASSES];
    float bias4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (p.bias) {
#pragma unroll
        for (int e = 0; e < 4; e++) bias4[e] = (float)reinterpret_cast<const CT*>(p.bias)[first + e];
    }
    // (reads stay in C: columns first .. first + 3 end by N, rows beyond M read the last one; columns before `nominal` belong to
    // another thread, maybe of another workgroup, which may be storing them: what is read of them is never used)
#pragma unroll
    for (int ps = 0; ps < PASSES; ps++) {
        const int row = m0 + c_row + ps * ROWS, down = (edge && row >= p.M) ? p.M - 1 - m0 - c_row : ps * ROWS;
        cin[ps] = active ? *reinterpret_cast<const ctx4*>(cptr + (int64_t)down * p.ldc) : ctx4{};
    }
    asm volatile("" ::: "memory");

    int j = 0;
    for (; j + 2 * U <= n_whole; j += U) {
#pragma unroll
        for (int u = 0; u < U; u++) { put(ra[u], rb[u]); load_whole(j + u + U, ra[u], rb[u]); mul(); }
    }
    for (; j < n_all; j += U) {
#pragma unroll
        for (int u = 0; u < U; u++)
            if (j + u < n_all) { put(ra[u], rb[u]); if (j + u + U < n_all) load_any(j + u + U, ra[u], rb[u]); mul(); }
    }

    // ---- the eight sums -> LDS -> + C, + bias, ReLU -> C -----------------------------------------
    __syncthreads();
    {
        const uint32_t t_w = smem_base + (uint32_t)wave * (BM * Shape::T_PITCH) + (uint32_t)(lane & 15) * Shape::T_PITCH + (uint32_t)(lane >> 4) * 16;
#pragma unroll
        for (int fm = 0; fm < MB; fm++)
#pragma unroll
            for (int fn = 0; fn < NB; fn++)
                *(__attribute__((address_space(3))) floatx4*)(uintptr_t)(t_w + fm * 16 * Shape::T_PITCH + fn * 64) = acc[fm][fn];
    }
    __syncthreads();
    if (!active) return;
    const uint32_t t_r = smem_base + (uint32_t)c_row * Shape::T_PITCH + (uint32_t)x * 4;
#pragma unroll
    for (int ps = 0; ps < PASSES; ps++) {
        floatx4 s4 = *(__attribute__((address_space(3))) const floatx4*)(uintptr_t)(t_r + ps * ROWS * Shape::T_PITCH);
#pragma unroll
        for (int w = 1; w < KW; w++) s4 += *(__attribute__((address_space(3))) const floatx4*)(uintptr_t)(t_r + w * (BM * Shape::T_PITCH) + ps * ROWS * Shape::T_PITCH);
        ctx4 o;
#pragma unroll
        for (int e = 0; e < 4; e++) o[e] = (CT)epilogue_value(s4[e] + (float)cin[ps][e], bias4[e], p.relu);     // f16: one rounding, to nearest even
        CT* const dst = cptr + (int64_t)(ps * ROWS) * p.ldc;
        const bool row_ok = !edge || m0 + c_row + ps * ROWS < p.M;
        if (row_ok && (!edge || first >= nominal)) *reinterpret_cast<ctx4*>(dst) = o;
        else if (row_ok) {
#pragma unroll
            for (int e = 0; e < 4; e++) if (first + e >= nominal) dst[e] = o[e];
        }
    }
}

template <int BM, int BN>
int64_t grid_kslice(int64_t M, int64_t N)
{
    const int64_t tm = (M + BM - 1) / BM, tn = (N + BN - 1) / BN;
    if (tm > 0 && tn > INT32_MAX / tm) return -1;
    return tm * tn;
}

template <int BM, int BN, int U, int WG_PER_CU>
int launch_kslice(const GemmArgs& a)
{
    const int64_t g = grid_kslice<BM, BN>(a.M, a.N);
    if (g < 0 || a.N < 8 || a.K < 8) return GEMM_F16_ERR_SIZE;
    const TiledParams p = make_tiled_params(a, BM, BN, 8);
    const dim3 grid((unsigned)g), block(64 * KW);
    if (a.c_is_f16) hipLaunchKernelGGL((gemm_kslice_kernel<half_t, BM, BN, U, WG_PER_CU>), grid, block, 0, a.stream, p);
    else            hipLaunchKernelGGL((gemm_kslice_kernel<float, BM, BN, U, WG_PER_CU>), grid, block, 0, a.stream, p);
    return hipGetLastError() == hipSuccess ? GEMM_F16_OK : GEMM_F16_ERR_LAUNCH;
}

#define KSLICE(NAME, BM, BN, U, WPC) { NAME, BM, BN, BK, 1, BM, BN, KsliceShape<BM, BN>::LDS, false, launch_kslice<BM, BN, U, WPC>, grid_kslice<BM, BN> }
#define KSLICE_ALL(PREFIX)                            \
    {KSLICE(PREFIX "ks16x32x64_k8", 16, 32, 2, 2),    \
     KSLICE(PREFIX "ks32x32x64_k8", 32, 32, 1, 2),    \
     KSLICE(PREFIX "ks16x64x64_k8", 16, 64, 1, 2),    \
     KSLICE(PREFIX "ks32x64x64_k8", 32, 64, 1, 1),    \
     KSLICE(PREFIX "ks64x64x64_k8", 64, 64, 1, 1)}
const GemmConfigDesc kKslice[] = KSLICE_ALL("");
const GemmConfigDesc kKsliceAny[] = KSLICE_ALL("generic_");      // the same kernels, as the any-shape family names them

}  // namespace

const GemmConfigDesc* kslice_config(int index, bool any_shape) { return any_shape ? &kKsliceAny[index] : &kKslice[index]; }
