// Problems of about one 128 x 128 tile per compute unit: two groups of four wavefronts (64 x 64 each) that
// both hold the whole tile and take its k steps in turn, X the even ones, Y the odd ones, and alternate
// in phases like those of gemm_pingpong.hip: in a phase one group reads all fragments of its
// next step from LDS while the other multiplies (32 MFMAs a wavefront) and issues, between them, the copies of
// the step five ahead of the one it multiplies.  One barrier per k step.  The groups' sums are added
// through LDS at the end.
//
// A k step takes what its copies take: 32 KB in 0.33 us (100 GB/s a compute unit) on half a chip, 0.42 (78) on a full one -- the
// copies alone 0.33 and the same with MFMAs and LDS reads, those without copies 0.23.  That is no limit of the chip: other loops reach 150 GB/s a compute unit
// out of the L2s, and 128 KB in flight at 100 GB/s would be 1.3 us of latency; why the copies take so long was not found.  Neither the order
// in which a step is fetched (LDS image or rows) nor behind which MFMAs the copies stand changes it by more than 1 %.  The eight wavefronts of 64 x 32 in
// gemm_pingpong.hip read 96 KB of LDS a step where this split reads 64, and meet four barriers: 0.5 us.
// Outside the loop, start and C take about 8 us: an empty launch of this size 2.4, the stores and the sums' way through LDS 4.5 (17 MB; a kernel that
// only stores them 1.8 more than an empty one), the first operands; the read of C, requested during the last steps, 1.
// 2048^3 f32 25.1 -> 22.7 us when it was written, 24.2 -> 21.7 and 26.6 -> 23.4 in other sessions on other cards; C requested earlier, stored by whole rows and
// one barrier less, the three together 23.7 -> 23.0 (the barrier 0.2 of it: put back 22.4 -> 22.6), (2048,2048,4096) 37.5 -> 36.2, (2048,2048,1536) 20.2 -> 19.6, (1152,2432,2048) 19.4 -> 19.0.
//
// Automatic selection gives it f32 problems from K = 1472 to 6143 and f16 ones from 832 (on 64 to 128 tiles 704) to where the five-stage kernel begins (deep_ring_if_it_pays in gemm_api.hip has both sides).
#include "gemm_device.h"
#include "../../include/gemm_f16.h"
#include <type_traits>

namespace {

using namespace gemm_dev;

constexpr int QB = 128;                                 // tile rows and columns
constexpr int QA_BUF = QB * BK * 2, QSTAGE = 2 * QA_BUF, QSTAGES = 5;      // 16 KB of A and of B a stage; 160 KB
constexpr int QB_ROW = QB * 2;                          // bytes per k row of B
constexpr int QT_PITCH = 64 * 4 + 16, QT_HALF = 32 * QT_PITCH;             // epilogue: 32 rows of a wavefront's 64 x 64 block
constexpr int CQ = 2, C_STEPS = 8 / CQ;                 // loads of C a wavefront requests behind each of its last copying steps; such steps

// Phase P: the group of step P reads it, the other one multiplies step P - 1 and issues the copies of step P + 4,
// into the stage whose last reader was phase P - 1.  They have landed by the end of phase P + 3, where
// the issuing group, reading then, waits for them (only those it issued in phase P + 2 may be outstanding), and the barrier
// publishes them to the group that reads them in phase P + 4.
template <typename CT, bool TAIL>
__global__ __launch_bounds__(512) void gemm_pp128_kernel(const TiledParams p)
{
    __shared__ __attribute__((aligned(1024))) char smem[QSTAGES * QSTAGE];
    const uint32_t smem_base = (uint32_t)(uintptr_t)(lds_ptr_t)smem;

    const int lane = threadIdx.x & 63;
    const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wave = wave_all & 3, grp = wave_all >> 2;
    const int wm_base = (wave >> 1) * 64, wn_base = (wave & 1) * 64;

    int tile_m, tile_n;
    tile_of_block(p, blockIdx.x, tile_m, tile_n);
    const int m0 = tile_m * QB, n0 = tile_n * QB;
    const bool edge = (m0 + QB > p.M) || (n0 + QB > p.N);
    const int kt_full = p.K / BK, KT = (p.K + BK - 1) / BK;

    // ---- copy plan: copy t (of 4 + 4) brings rows 8 (wave + 4t) .. +7 of A, k rows 4 (wave + 4t) .. +3 of B; lane i
    // writes 16 bytes at 16 i and fetches the chunk that belongs there (positions as in gemm_w4a128.hip)
    const int a_chunk = (lane & 7) ^ (4 * (wave & 1) + (lane >> 4));
    uint32_t a_off[4], b_off;
#pragma unroll
    for (int t = 0; t < 4; t++) {
        int row = 8 * (wave + 4 * t) + (lane >> 3);
        row = (m0 + row < p.M) ? row : p.M - 1 - m0;                  // loaded, never stored
        a_off[t] = ((uint32_t)row * (uint32_t)p.lda + 8 * a_chunk) * 2;
    }
    const int b_krow = 4 * wave + (lane >> 4);                        // of copy t: b_krow + 16t
    {
        int col = 8 * ((lane & 15) ^ (((lane >> 4) << 2) | (((wave >> 1) & 1) << 1)));
        if (n0 + col + 8 > p.N) col = 0;                              // loaded, never stored
        b_off = ((uint32_t)b_krow * (uint32_t)p.ldb + (uint32_t)col) * 2;
    }
    const half_t* const a_tile = p.A + (int64_t)m0 * p.lda;
    const half_t* const b_tile = p.B + n0;
    const uint32_t dst_wave = smem_base + 1024u * wave;
    auto stage_at = [&](int s) -> uint32_t { return (uint32_t)(s % QSTAGES) * QSTAGE; };
    auto src_a = [&](int s) { return a_tile + (int64_t)s * BK; };
    auto src_b = [&](int s, int t) { return b_tile + ((int64_t)s * BK + 16 * t) * p.ldb; };
    // copy c of step s at once: 0 .. 3 A, 4 .. 7 B; whole steps go global -> LDS, the k tail through registers, zero beyond K
    auto copy_now = [&](int s, int c) {
        const uint32_t dst = dst_wave + stage_at(s) + (c < 4 ? 0 : QA_BUF) + 4096u * (c & 3);
        if (!TAIL || s < kt_full) {
            if (c < 4) async_copy16(src_a(s), a_off[c & 3], dst); else async_copy16(src_b(s, c & 3), b_off, dst);
        } else {
            const int kvalid = p.K - s * BK;
            uintx4 v = {0u, 0u, 0u, 0u};
            if (c < 4) { if (8 * a_chunk < kvalid) v = *reinterpret_cast<const uintx4*>((const char*)src_a(s) + a_off[c & 3]); }
            else if (b_krow + 16 * (c & 3) < kvalid) v = *reinterpret_cast<const uintx4*>((const char*)src_b(s, c & 3) + b_off);
            *(__attribute__((address_space(3))) uintx4*)(uintptr_t)(dst + 16 * lane) = v;
        }
    };

    // ---- fragment read addresses (as in gemm_w4a128.hip) ----------------------------------
    uint32_t a_rd[2], b_rd[4];
    {
        const uint32_t row_off = (uint32_t)(wm_base + (lane & 15)) * (BK * 2);
        const int sw = (lane & 15) >> 1;
#pragma unroll
        for (int s = 0; s < 2; s++) a_rd[s] = smem_base + row_off + (uint32_t)(((4 * s + (lane >> 4)) ^ sw) * 16);
        const int blk = lane >> 4, j = lane & 15;
        const uint32_t krow_off = (uint32_t)(8 * blk + (j >> 2)) * QB_ROW;
        const int swz = ((j >> 2) << 2) | ((blk & 1) << 1);
#pragma unroll
        for (int fn = 0; fn < 4; fn++) {
            const int chunk = 2 * ((wn_base >> 4) + fn) + ((j & 3) >> 1);
            b_rd[fn] = smem_base + QA_BUF + krow_off + (uint32_t)((chunk ^ swz) * 16 + 8 * (j & 1));
        }
    }

    // ---- steps 0 .. 3 on their way: like all later ones, by the group that does not read them
#pragma unroll
    for (int s = 0; s < 4; s++)
        if (s < KT && (s & 1) != grp) {
#pragma unroll
            for (int c = 0; c < 8; c++) copy_now(s, c);
        }

    floatx4 acc[4][4];
#pragma unroll
    for (int fm = 0; fm < 4; fm++)
#pragma unroll
        for (int fn = 0; fn < 4; fn++) acc[fm][fn] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    half8 fa[2][4], fb[2][4];
    auto read_fragments = [&](uint32_t stage) {
#pragma unroll
        for (int s = 0; s < 2; s++) {
            uint32_t a0 = a_rd[s] + stage;
            asm volatile("" : "+v"(a0));
#pragma unroll
            for (int fm = 0; fm < 4; fm++) fa[s][fm] = lds_read_b128(a0 + fm * 16 * (BK * 2));
        }
#pragma unroll
        for (int fn = 0; fn < 4; fn++) {
            uint32_t b0 = b_rd[fn] + stage;
            asm volatile("" : "+v"(b0));
#pragma unroll
            for (int s = 0; s < 2; s++) {
                const half4 lo = lds_read_tr16(b0 + s * 32 * QB_ROW), hi = lds_read_tr16(b0 + s * 32 * QB_ROW + 4 * QB_ROW);
                fb[s][fn] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            }
        }
    };
    // copies: 0 none, 1 of step s + 5, a whole one, between the MFMAs, 2 of step s + 5, the k tail
    auto multiply = [&](int s, uint32_t copy_stage, auto copies) {
        constexpr int L = decltype(copies)::value;
        const uint32_t dst = dst_wave + copy_stage;
#pragma unroll
        for (int i = 0; i < 32; i++) {
            // two rows of blocks at a time, down, right, up, right: one operand changes per MFMA (gemm_pingpong.hip)
            const int sl = i / 16, pr = (i % 16) / 8, q = i % 8, gm = 2 * pr + ((q % 4 == 1 || q % 4 == 2) ? 1 : 0), gn = (pr & 1) ? 3 - q / 2 : q / 2;
            acc[gm][gn] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fb[sl][gn], fa[sl][gm], acc[gm][gn], 0, 0, 0);
            const int c = i / 4;
            if constexpr (L == 1) {
                // M0 behind MFMA 4c, the load behind 4c + 1
                if (i % 4 == 0) { __builtin_amdgcn_sched_barrier(0); if (c < 4) set_m0(dst, 4096 * c); else set_m0(dst, QA_BUF + 4096 * (c - 4)); __builtin_amdgcn_sched_barrier(0); }
                if (i % 4 == 1) { __builtin_amdgcn_sched_barrier(0); if (c < 4) async_copy16_m0(src_a(s + 5), a_off[c & 3]); else async_copy16_m0(src_b(s + 5, c & 3), b_off); __builtin_amdgcn_sched_barrier(0); }
            } else if (L == 2 && i % 4 == 1) {
                __builtin_amdgcn_sched_barrier(0);
                copy_now(s + 5, c);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    auto lds_done = [&]() {
        __builtin_amdgcn_s_waitcnt(0xC07F);                           // lgkmcnt(0)
        asm volatile("" ::: "memory");
    };

    // ---- C: addresses -------------------------------------------------------------------------
    // A wavefront adds and stores 16 whole rows of the tile, two (512 bytes of f32) an instruction: rows of C a power of two apart are
    // written faster that way than four rows of 256 bytes at a time (a kernel that only stores such tiles of a 2048 x 2048 f32 C 5.3 -> 4.8 us, at a pitch of 64 more 4.6 both).
    typedef typename CVec4<CT>::type ctx4;
    constexpr int RPP = 2;                                            // rows an instruction
    const int c_col = n0 + 4 * (lane & 31), c_row = m0 + 16 * wave_all + (lane >> 5);
    const bool col_ok = !edge || c_col < p.N;                         // N is a multiple of 8: all 4 columns or none
    CT* const cptr = (CT*)p.C + (int64_t)c_row * p.ldc + c_col;
    ctx4 cin[8];
    auto fetch_c = [&](int p0, int p1) {
#pragma unroll
        for (int ps = p0; ps < p1; ps++) {
            const bool ok = col_ok && (!edge || c_row + RPP * ps < p.M);
            const CT* src = ok ? cptr + (int64_t)(RPP * ps) * p.ldc : (const CT*)p.C + (int64_t)m0 * p.ldc + n0;
            cin[ps] = *reinterpret_cast<const ctx4*>(src);
        }
    };

    // ---- phases ----------------------------------------------------------------------------------
    typedef std::integral_constant<int, 0> I0; typedef std::integral_constant<int, 1> I1; typedef std::integral_constant<int, 2> I2;
    if (2 < kt_full && grp == 1) asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)" ::: "memory");       // step 0 has landed, step 2 may be on its way
    else if (grp == 1)           asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    else                         lds_done();                          // (step 1, if it went through registers; else the wait of phase 0 is in time)
    phase_barrier();
    if (grp == 1) {                                                   // phase 0: X reads step 0
        if (4 < KT) {
#pragma unroll
            for (int c = 0; c < 8; c++) copy_now(4, c);
        }
        lds_done();
        phase_barrier();
    }
    int s = grp;
    uint32_t st = stage_at(s);                                        // of step s; the copies of step s + 5 go there too
    auto next = [&]() {
        s += 2;
        st += 2 * QSTAGE;
        if (st >= QSTAGES * QSTAGE) st -= QSTAGES * QSTAGE;
    };
    for (; s + 5 + 2 * C_STEPS < kt_full; next()) {
        read_fragments(st);
        lds_done();
        asm volatile("s_waitcnt vmcnt(8)" ::: "memory");              // step s + 1 has landed, step s + 3 may be on its way
        phase_barrier();
        multiply(s, st, I1{});
        phase_barrier();
    }
    // The last ones request C behind their copies, two loads each, and C is then there when the loop ends.  (All 8 behind the
    // last copies, as before: the loop was done before C had come.)  The loads come from memory and loads complete in order, but
    // a copy has the three steps of its own lead to wait for them.  One load a step over eight steps, or four over two, gain less.
#pragma unroll
    for (int c = 0; c < C_STEPS; c++) {
        if (s + 5 < kt_full) {
            read_fragments(st);
            lds_done();
            asm volatile("s_waitcnt vmcnt(%0)" :: "n"(8 + CQ * (c < 2 ? c : 2)) : "memory");      // as above; what was requested of C behind the copies of step s + 1 may be on its way too
            phase_barrier();
            multiply(s, st, I1{});
            fetch_c(CQ * c, CQ * c + CQ);
            __builtin_amdgcn_sched_barrier(0);
            phase_barrier();
            next();
        } else {
            fetch_c(CQ * c, CQ * c + CQ);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if constexpr (TAIL) {
        for (; s + 5 < KT; next()) {                                  // at most once: fetches the k tail
            read_fragments(st);
            lds_done();
            asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
            phase_barrier();
            multiply(s, st, I2{});
            lds_done();
            phase_barrier();
        }
    }
    for (; s < KT; next()) {
        read_fragments(st);
        lds_done();
        // (at least 8 + 2 CQ loads and copies were issued behind the copies of step s + 1, or CQ where those are the last ones)
        if (s + 3 < kt_full) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(8 + 2 * CQ) : "memory");     // step s + 1; step s + 3 and the last of C may be on their way
        else                 asm volatile("s_waitcnt vmcnt(%0)" :: "n"(CQ) : "memory");             // step s + 1; the last of C may be
        phase_barrier();
        multiply(s, st, I0{});
        if (s + 1 < KT) phase_barrier();
    }

    // ---- sums of both groups + C, + bias, ReLU, -> C ------------------------------------------
    float bias4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (p.bias && col_ok) {
#pragma unroll
        for (int e = 0; e < 4; e++) bias4[e] = (float)reinterpret_cast<const CT*>(p.bias)[c_col + e];
    }
    // No barrier in front of these writes: the group that multiplies the last step has read it into registers before the last barrier, the
    // other group, which read its last step earlier, writes its sums meanwhile.  Block ((group, half of the rows), wavefront) of 32 rows x 64 columns each.
    const uint32_t t_w = smem_base + (uint32_t)(lane & 15) * QT_PITCH + (uint32_t)(lane >> 4) * 16;
#pragma unroll
    for (int h = 0; h < 2; h++)
#pragma unroll
        for (int r = 0; r < 2; r++)
#pragma unroll
            for (int fn = 0; fn < 4; fn++)
                *(__attribute__((address_space(3))) floatx4*)(uintptr_t)(t_w + (uint32_t)((grp * 2 + h) * 4 + wave) * QT_HALF + r * 16 * QT_PITCH + fn * 64) = acc[2 * h + r][fn];
    lds_done();
    phase_barrier();
    const uint32_t t_r = smem_base + (uint32_t)(((wave_all >> 1) & 1) * 4 + (wave_all >> 2) * 2 + ((lane >> 4) & 1)) * QT_HALF
                                   + (uint32_t)(16 * (wave_all & 1) + (lane >> 5)) * QT_PITCH + (uint32_t)(lane & 15) * 16;
#pragma unroll
    for (int ps = 0; ps < 8; ps++) {
        floatx4 s4 = *(__attribute__((address_space(3))) const floatx4*)(uintptr_t)(t_r + RPP * ps * QT_PITCH);
        s4 += *(__attribute__((address_space(3))) const floatx4*)(uintptr_t)(t_r + 8 * QT_HALF + RPP * ps * QT_PITCH);
        ctx4 o;
#pragma unroll
        for (int e = 0; e < 4; e++) o[e] = (CT)epilogue_value(s4[e] + (float)cin[ps][e], bias4[e], p.relu);     // f16: one rounding, to nearest even
        if (col_ok && (!edge || c_row + RPP * ps < p.M)) *reinterpret_cast<ctx4*>(cptr + (int64_t)(RPP * ps) * p.ldc) = o;
    }
}

int64_t grid_pp128(int64_t M, int64_t N)
{
    const int64_t tm = (M + QB - 1) / QB, tn = (N + QB - 1) / QB;
    if (tm > 0 && tn > INT32_MAX / tm) return -1;
    return tm * tn;
}

int launch_pp128(const GemmArgs& a)
{
    const int64_t g = grid_pp128(a.M, a.N);
    if (g < 0) return GEMM_F16_ERR_SIZE;
    const TiledParams p = make_tiled_params(a, QB, QB, 8);
    const dim3 grid((unsigned)g), block(512);
    const bool tail = a.K % BK != 0;
#define PP128_LAUNCH(CT, TAIL) hipLaunchKernelGGL((gemm_pp128_kernel<CT, TAIL>), grid, block, 0, a.stream, p)
    if (a.c_is_f16) { if (tail) PP128_LAUNCH(half_t, true); else PP128_LAUNCH(half_t, false); }
    else            { if (tail) PP128_LAUNCH(float, true); else PP128_LAUNCH(float, false); }
#undef PP128_LAUNCH
    return hipGetLastError() == hipSuccess ? GEMM_F16_OK : GEMM_F16_ERR_LAUNCH;
}

const GemmConfigDesc kPp128 = {"pp128x128x64_w2x2_k2", QB, QB, BK, 4, 64, 64, QSTAGES * QSTAGE, true, launch_pp128, grid_pp128};

}  // namespace

const GemmConfigDesc* pp128_config() { return &kPp128; }
