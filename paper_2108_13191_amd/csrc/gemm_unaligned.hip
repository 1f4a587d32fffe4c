// The tiled kernel for operands without 16-byte alignment: any base address, any pitch, any N and
// K from 8 on.  The tuned kernels' global -> LDS copies need 16-byte aligned chunks; here a chunk
// of 8 elements is one 16-byte load at 2-byte alignment into registers and one ds_write_b128, and
// the LDS image, the fragment reads and the MFMAs are those of the 128 x 128 tuned forms
// (wavefront tile 64 x 64, k steps of 64, two LDS stages).
//
// No access leaves the matrices and no chunk is ever taken apart: a chunk that would reach past
// the end of its row is loaded as the row's last 8 elements.  For B that only changes which
// columns the chunk's results belong to (the store knows); for A and the k tail the same shift is
// applied to the k rows of B, and what is then there twice is zeroed in both operands (in both:
// zero times infinity must not appear).
//
// Bound by the loads: a 16-byte load at 2-byte alignment takes the CU's memory pipeline up to twice
// as long (256 workgroups streaming 128 x 64 and 64 x 128 blocks out of the L2s: 14.7 TB/s at 16- and
// at 4-byte alignment, 12.7 with an odd pitch, 9.0 with every row odd), so the tile is as large as
// leaves two workgroups a compute unit to cover each other, and two k steps are in flight in
// registers.  Before -> after, us: 2001 x 1999 x 2003 f32 264 -> 34, 4001 x 3999 x 4003 f32 2700 ->
// 206, (14159,1005,2990) f16 with bias and ReLU 1810 -> 160 (element-wise kernel before).
//
// KG = 2: two groups of four wavefronts take the k steps in turn, each on its own LDS stages, and
// their sums are added at the end -- for problems of at most one tile per compute unit, where
// otherwise one wavefront per SIMD would have nothing to hide its own waits.
#include "gemm_device.h"
#include "../../include/gemm_f16.h"
#include <type_traits>

namespace {

using namespace gemm_dev;

constexpr int UBM = 128, UBN = 128;
constexpr int UA_BUF = UBM * BK * 2, UB_BUF = BK * UBN * 2, USTAGE = UA_BUF + UB_BUF;    // 16 + 16 KB
constexpr int UB_ROW = UBN * 2;
constexpr int UT_PITCH = 64 * 4 + 16;                  // epilogue: bytes per row of 64 columns
constexpr int UT_HALF = 32 * UT_PITCH;                 // 32 rows of a wavefront's 64 x 64 block

template <int KG> constexpr int unaligned_lds() { return KG * 2 * USTAGE > KG * 8 * UT_HALF ? KG * 2 * USTAGE : KG * 8 * UT_HALF; }

typedef uintx4 uintx4_any __attribute__((aligned(2)));

template <typename CT, int KG>
__global__ __launch_bounds__(256 * KG, 2) void gemm_unaligned_kernel(const TiledParams p)
{
    __shared__ __attribute__((aligned(1024))) char smem[unaligned_lds<KG>()];
    const uint32_t smem_base = (uint32_t)(uintptr_t)(lds_ptr_t)smem;

    const int lane = threadIdx.x & 63;
    const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wave = wave_all & 3, kg = wave_all >> 2;
    const int wm_base = (wave >> 1) * 64, wn_base = (wave & 1) * 64;

    int tile_m, tile_n;
    tile_of_block(p, blockIdx.x, tile_m, tile_n);
    const int m0 = tile_m * UBM, n0 = tile_n * UBN;
    const bool edge = (m0 + UBM > p.M) || (n0 + UBN > p.N);

    // ---- copy plan: load t < 4 takes A rows 8 (wave + 4t) .. +7, 8 lanes a row; load 4 + t takes k rows 4 (wave + 4t) .. +3
    // of B, 16 lanes a row (columns clamped to the last 8).  Consecutive lanes fetch consecutive chunks, and
    // each chunk goes to the place that it has in the tuned 128 x 128 kernels (chunks fetched in the
    // order of those places: 2 to 8 % slower, (15552,2147,1467) f32 216 us against 202, (6750,7396,630) f16 142 against 130).
    const int a_chunk = lane & 7, b_chunk = lane & 15;
    uint32_t a_off[4];
#pragma unroll
    for (int t = 0; t < 4; t++) {
        int row = 8 * (wave + 4 * t) + (lane >> 3);
        row = (m0 + row < p.M) ? row : p.M - 1 - m0;
        a_off[t] = ((uint32_t)row * (uint32_t)p.lda + 8 * a_chunk) * 2;
    }
    const int b_krow0 = 4 * wave + (lane >> 4);                       // k row of load 4 + t: b_krow0 + 16t
    int b_col = n0 + 8 * b_chunk;                                     // first column of this lane's chunk
    if (b_col > p.N - 8) b_col = p.N - 8;
    const uint32_t b_off = ((uint32_t)b_krow0 * (uint32_t)p.ldb + (uint32_t)b_col) * 2u;
    const char* const a_tile = (const char*)(p.A + (int64_t)m0 * p.lda);
    const char* const b_mat = (const char*)p.B;
    const uint32_t lds_group = smem_base + (uint32_t)kg * (2 * USTAGE);
    const uint32_t a_wr = lds_group + 1024u * wave + 128u * (lane >> 3) + 16u * (a_chunk ^ (4 * (wave & 1) + (lane >> 4)));
    const uint32_t b_wr = lds_group + UA_BUF + 1024u * wave + 256u * (lane >> 4) + 16u * (b_chunk ^ (((lane >> 4) << 2) | (((wave >> 1) & 1) << 1)));

    // ---- fragment read addresses (as in gemm_w4a128.hip) ----------------------------------
    uint32_t a_rd[2], b_rd[4];
    {
        const uint32_t row_off = (uint32_t)(wm_base + (lane & 15)) * (BK * 2);
        const int sw = (lane & 15) >> 1;
#pragma unroll
        for (int s = 0; s < 2; s++) a_rd[s] = lds_group + row_off + (uint32_t)(((4 * s + (lane >> 4)) ^ sw) * 16);
        const int blk = lane >> 4, j = lane & 15;
        const uint32_t krow_off = (uint32_t)(8 * blk + (j >> 2)) * UB_ROW;
        const int swz = ((j >> 2) << 2) | ((blk & 1) << 1);
#pragma unroll
        for (int fn = 0; fn < 4; fn++) {
            const int chunk = 2 * ((wn_base >> 4) + fn) + ((j & 3) >> 1);
            b_rd[fn] = lds_group + UA_BUF + krow_off + (uint32_t)((chunk ^ swz) * 16 + 8 * (j & 1));
        }
    }

    // ---- k steps: this group's step j is step s = kg + KG j of the tile ------------------------
    const int k_full = p.K / BK, KT = (p.K + BK - 1) / BK;
    const int nj = (KT + KG - 1) / KG, jf = k_full / KG;               // steps per group; of them whole in every group
    uintx4 R[2][8];                                                   // two steps on their way: 4 chunks of A, 4 of B each

    auto load_whole = [&](int j, uintx4 (&r)[8], int t0, int t1) {    // chunks t0 .. t1 - 1 of a whole step
        const int64_t k0 = (int64_t)(kg + KG * j) * BK;
#pragma unroll
        for (int t = t0; t < t1; t++) {
            if (t < 4) r[t] = *reinterpret_cast<const uintx4_any*>(a_tile + k0 * 2 + a_off[t]);
            else       r[t] = *reinterpret_cast<const uintx4_any*>(b_mat + (k0 + 16 * (t - 4)) * p.ldb * 2 + b_off);
        }
    };
    // The step with the k tail (or beyond it: all zero).  Chunk c of the step covers k = k0 + 8c ..
    // + 7; past K - 8 it is loaded as the last 8 and its first (k - (K - 8)) elements, which belong
    // to the chunk before it, are zeroed; the k rows of B that sit in the same slots likewise.
    auto load_tail = [&](int j, uintx4 (&r)[8]) {
        const int k0 = (kg + KG * j) * BK;
        {
            const int k = k0 + 8 * a_chunk, over = k - (p.K - 8);      // > 0: elements 0 .. over - 1 are there twice (8: none left)
            const int back = over > 0 ? over : 0;
            const char* const src = a_tile + ((int64_t)k0 - back) * 2;
#pragma unroll
            for (int t = 0; t < 4; t++) {
                uintx4 v = *reinterpret_cast<const uintx4_any*>(src + a_off[t]);
#pragma unroll
                for (int e = 0; e < 4; e++) v[e] = (2 * e + 1 < back) ? 0u : (2 * e < back) ? (v[e] & 0xffff0000u) : v[e];
                r[t] = v;
            }
        }
#pragma unroll
        for (int t = 0; t < 4; t++) {
            const int slot = b_krow0 + 16 * t, c8 = k0 + (slot & ~7), over = c8 - (p.K - 8);
            const int back = over > 0 ? over : 0;
            const uintx4 v = *reinterpret_cast<const uintx4_any*>(b_mat + (((int64_t)(k0 + slot) - back) * p.ldb + b_col) * 2);
            r[4 + t] = (slot & 7) < back ? uintx4{0u, 0u, 0u, 0u} : v;
        }
    };
    auto load_any = [&](int j, uintx4 (&r)[8]) {
        if ((kg + KG * j) < k_full) load_whole(j, r, 0, 8);
        else load_tail(j, r);
    };
    auto put = [&](int stage, const uintx4 (&r)[8], int t0, int t1) {
#pragma unroll
        for (int t = t0; t < t1; t++)
            *(__attribute__((address_space(3))) uintx4*)(uintptr_t)((t < 4 ? a_wr + 4096u * t : b_wr + 4096u * (t - 4)) + (uint32_t)stage * USTAGE) = r[t];
    };

    floatx4 acc[4][4];
#pragma unroll
    for (int fm = 0; fm < 4; fm++)
#pragma unroll
        for (int fn = 0; fn < 4; fn++) acc[fm][fn] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    half8 fa[2][4], fb[2][4];
    half4 b_lo[4];
    auto read = [&](int stage, int s, int r) {                        // read r (0 .. 11) of slice s into fragment set s: 8 halves of B, 4 A
        if (r < 8) {
            const int fn = r >> 1;
            const uint32_t addr = b_rd[fn] + (uint32_t)stage * USTAGE + s * 32 * UB_ROW;
            if (!(r & 1)) b_lo[fn] = lds_read_tr16(addr);
            else fb[s][fn] = __builtin_shufflevector(b_lo[fn], lds_read_tr16(addr + 4 * UB_ROW), 0, 1, 2, 3, 4, 5, 6, 7);
        } else {
            fa[s][r - 8] = lds_read_b128(a_rd[s] + (uint32_t)stage * USTAGE + (r - 8) * 16 * (BK * 2));
        }
    };
    auto barrier = [&]() {
        __builtin_amdgcn_s_waitcnt(0xC07F);                           // lgkmcnt(0)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    // One k step.  Slice 0: multiply set 0 while slice 1 is read and the next step (loaded one and a
    // half steps ago) is written to the other stage; barrier; slice 1: multiply set 1 while slice
    // 0 of the next step is read and the step three ahead is requested.
    auto step = [&](int j, auto parity, auto loads) {
        constexpr int P = decltype(parity)::value, L = decltype(loads)::value;      // L: 0 none, 1 whole, 2 any
        const bool more = (L == 1) || j + 1 < nj;
#pragma unroll
        for (int c = 0; c < 4; c++) {
#pragma unroll
            for (int r = 3 * c; r < 3 * c + 3; r++) read(P, 1, r);
            if (more) put(P ^ 1, R[P ^ 1], 2 * c, 2 * c + 2);
#pragma unroll
            for (int i = 4 * c; i < 4 * c + 4; i++) {
                const int pr = i / 8, q = i % 8, gm = 2 * pr + ((q % 4 == 1 || q % 4 == 2) ? 1 : 0), gn = (pr & 1) ? 3 - q / 2 : q / 2;
                acc[gm][gn] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fb[0][gn], fa[0][gm], acc[gm][gn], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        barrier();
        if constexpr (L == 2) { if (j + 3 < nj) load_any(j + 3, R[P ^ 1]); }
#pragma unroll
        for (int c = 0; c < 4; c++) {
            if (more) {
#pragma unroll
                for (int r = 3 * c; r < 3 * c + 3; r++) read(P ^ 1, 0, r);
            }
            if constexpr (L == 1) load_whole(j + 3, R[P ^ 1], 2 * c, 2 * c + 2);
#pragma unroll
            for (int i = 4 * c; i < 4 * c + 4; i++) {
                const int pr = i / 8, q = i % 8, gm = 2 * pr + ((q % 4 == 1 || q % 4 == 2) ? 1 : 0), gn = (pr & 1) ? 3 - q / 2 : q / 2;
                acc[gm][gn] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fb[1][gn], fa[1][gm], acc[gm][gn], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    typedef std::integral_constant<int, 0> I0; typedef std::integral_constant<int, 1> I1; typedef std::integral_constant<int, 2> I2;

    load_any(0, R[0]);
    if (1 < nj) load_any(1, R[1]);
    put(0, R[0], 0, 8);
    if (2 < nj) load_any(2, R[0]);
    barrier();
#pragma unroll
    for (int r = 0; r < 12; r++) read(0, 0, r);
    int j = 0;
    for (; j + 4 < jf; j += 2) { step(j, I0{}, I1{}); step(j + 1, I1{}, I1{}); }
    for (; j < nj; j += 2) { step(j, I0{}, I2{}); if (j + 1 < nj) step(j + 1, I1{}, I2{}); }
    barrier();

    // ---- + C, + bias, ReLU, -> C ---------------------------------------------------------
    // The wavefront's 64 x 64 block goes through LDS in halves of 32 rows, so that C moves in rows
    // of 64 columns, 4 per lane.  With two k groups each stores one half and adds the other
    // group's sums to it there.
    typedef typename CVec4<CT>::type ctx4;
    const int x = wn_base + 4 * (lane & 15), nominal = n0 + (x & ~7);  // this lane's 4 columns within the tile; first column of their chunk
    const int first = (nominal < p.N - 8 ? nominal : p.N - 8) + (x & 7);   // ... and where those results belong
    float bias4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (p.bias) {
#pragma unroll
        for (int e = 0; e < 4; e++) bias4[e] = (float)reinterpret_cast<const CT*>(p.bias)[first + e];
    }
    const uint32_t t_w = smem_base + (uint32_t)(lane & 15) * UT_PITCH + (uint32_t)(lane >> 4) * 16;
    const uint32_t t_r = smem_base + (uint32_t)(lane >> 4) * UT_PITCH + (uint32_t)(lane & 15) * 16;
#pragma unroll
    for (int h = 0; h < 2; h++)
#pragma unroll
        for (int r = 0; r < 2; r++)
#pragma unroll
            for (int fn = 0; fn < 4; fn++)
                *(__attribute__((address_space(3))) floatx4*)(uintptr_t)(t_w + (uint32_t)((kg * 2 + h) * 4 + wave) * UT_HALF + r * 16 * UT_PITCH + fn * 64) = acc[2 * h + r][fn];
    if constexpr (KG > 1) barrier();
    CT* const Cbase = (CT*)p.C;
#pragma unroll
    for (int h = 0; h < 2; h++) {
        if (KG > 1 && h != kg) continue;
        const int row0 = m0 + wm_base + 32 * h + (lane >> 4);
        CT* const cptr = Cbase + (int64_t)row0 * p.ldc + first;
        // Reads stay in C whatever the tile: a lane's 4 columns end by N, rows beyond M read the last one; columns before `nominal` belong to
        // another lane, maybe of another workgroup, which may be storing them: what is read of them is never used.  (Element by
        // element under a test, as the stores at an edge are, each of the 32 reads waits for the one before:
        // (1000,1000,64) f32 13.6 us, 6.7 at 1024 x 1024.)
        ctx4 cin[8];
#pragma unroll
        for (int ps = 0; ps < 8; ps++) {
            const int down = (!edge || row0 + 4 * ps < p.M) ? 4 * ps : p.M - 1 - row0;
            cin[ps] = *reinterpret_cast<const ctx4*>(cptr + (int64_t)down * p.ldc);
        }
#pragma unroll
        for (int ps = 0; ps < 8; ps++) {
            floatx4 s4 = *(__attribute__((address_space(3))) const floatx4*)(uintptr_t)(t_r + (uint32_t)(h * 4 + wave) * UT_HALF + 4 * ps * UT_PITCH);
            if constexpr (KG > 1) s4 += *(__attribute__((address_space(3))) const floatx4*)(uintptr_t)(t_r + (uint32_t)(8 + h * 4 + wave) * UT_HALF + 4 * ps * UT_PITCH);
            ctx4 o;
#pragma unroll
            for (int e = 0; e < 4; e++) o[e] = (CT)epilogue_value(s4[e] + (float)cin[ps][e], bias4[e], p.relu);     // f16: one rounding, to nearest even
            CT* const dst = cptr + (int64_t)(4 * ps) * p.ldc;
            if (!edge || (first >= nominal && row0 + 4 * ps < p.M)) *reinterpret_cast<ctx4*>(dst) = o;
            else if (row0 + 4 * ps < p.M) {
#pragma unroll
                for (int e = 0; e < 4; e++) if (first + e >= nominal) dst[e] = o[e];
            }
        }
    }
}

int64_t grid_unaligned(int64_t M, int64_t N)
{
    const int64_t tm = (M + UBM - 1) / UBM, tn = (N + UBN - 1) / UBN;
    if (tm > 0 && tn > INT32_MAX / tm) return -1;
    return tm * tn;
}

template <int KG>
int launch_unaligned(const GemmArgs& a)
{
    const int64_t g = grid_unaligned(a.M, a.N);
    if (g < 0 || a.N < 8 || a.K < 8) return GEMM_F16_ERR_SIZE;
    const TiledParams p = make_tiled_params(a, UBM, UBN, 8);
    const dim3 grid((unsigned)g), block(256 * KG);
    if (a.c_is_f16) hipLaunchKernelGGL((gemm_unaligned_kernel<half_t, KG>), grid, block, 0, a.stream, p);
    else            hipLaunchKernelGGL((gemm_unaligned_kernel<float, KG>), grid, block, 0, a.stream, p);
    return hipGetLastError() == hipSuccess ? GEMM_F16_OK : GEMM_F16_ERR_LAUNCH;
}

const GemmConfigDesc kUnaligned128[2] = {
    {"generic128x128x64", UBM, UBN, BK, 4, 64, 64, unaligned_lds<1>(), false, launch_unaligned<1>, grid_unaligned},
    {"generic128x128x64_k2", UBM, UBN, BK, 4, 64, 64, unaligned_lds<2>(), false, launch_unaligned<2>, grid_unaligned}};

}  // namespace

const GemmConfigDesc* unaligned_config(int k_groups) { return &kUnaligned128[k_groups - 1]; }
