// Large problems whose operands have no 16-byte alignment: the phase-alternating schedule of
// gemm_pingpong.hip (two groups of four wavefronts, one reads fragments while the other multiplies;
// 16x16x32 MFMAs, the same LDS image, epilogue through LDS) with the operands on their way through
// registers, as in gemm_unaligned.hip: a chunk of 8 elements is one 16-byte load at 2-byte alignment
// and one ds_write_b128, issued between the MFMAs of the multiplying phase.  Chunks that would
// reach past the end of a row are loaded as the row's last 8 elements; what is then there twice
// is zeroed in both operands (k) or not stored (columns).
//
// Against the 128 x 128 tiles of gemm_unaligned.hip a result costs half the loads, which bound those (a 16-byte load at an odd
// element takes the CU's memory pipeline a lane a clock): (4001,3999,4003) f32 198 -> 144 us, in rows that begin at
// 4-byte addresses 185 -> 130.  What bounds it: a k step of 1.6 to 1.8 us (the aligned kernel's, power-limited, 1.4) and some 25 us
// for the read and write of C by all compute units at once, which nothing hides.  128 x 256 tiles are for problems that
// leave 256 x 256 ones too few: (2001,3999,4003) f32 116 -> 80 us (256 x 256: 95).
// The writes to LDS stand late in the multiplying phase, when the other group's reads are through: (4096,4096,8192) 236 us with them
// spread over its first half, 231 late, 233 in the reading phase, 248 in a row at the start.
#include "gemm_device.h"
#include "../../include/gemm_f16.h"
#include <type_traits>

namespace {

using namespace gemm_dev;

constexpr int VBN = 256, VB_BUF = BK * VBN * 2, VB_ROW = VBN * 2;     // B: two stages of 32 KB
constexpr int VT_PITCH = 64 * 4 + 16;                                 // epilogue: bytes per row of 64 columns, 32 rows a wavefront
template <int BM> constexpr int unaligned_pp_lds() { return BM * BK * 2 + 2 * VB_BUF; }   // A: one stage

typedef uintx4 uintx4_any __attribute__((aligned(2)));

// Phases (k = k step, h = its halves of 32): group X reads the fragments of (k, h) in phase 4k + 2h and
// multiplies them in the next, group Y one phase later.  A wavefront holds one k step of its copies in
// registers: multiplying (k, 0) it writes its chunks of B(k + 1) to LDS and requests those of B(k + 2),
// multiplying (k, 1) the same of A.  A(k + 1) may overwrite A(k): only the group that copies a row of
// A reads it, and it has read (k, 1) one phase earlier.  B(k + 1) overwrites B(k - 1), last read by Y two
// phases before X writes.
template <typename CT, int BM>
__global__ __launch_bounds__(512) void gemm_unaligned_pp_kernel(const TiledParams p)
{
    __shared__ __attribute__((aligned(1024))) char smem[unaligned_pp_lds<BM>()];
    const uint32_t smem_base = (uint32_t)(uintptr_t)(lds_ptr_t)smem;
    constexpr int HM = BM / 2, FM = HM / 16, FN = 4, TA = HM / 32, TB = 4;
    constexpr uint32_t B_REGION = BM * BK * 2;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = wave >> 2, wn = wave & 3;

    int tile_m, tile_n;
    tile_of_block(p, blockIdx.x, tile_m, tile_n);
    const int m0 = tile_m * BM, n0 = tile_n * VBN;
    const bool edge = (m0 + BM > p.M) || (n0 + VBN > p.N);

    // ---- copy plan: load t takes rows 8 (wn + 4t) .. +7 of the group's half of A, 8 lanes a row, and k rows 2 (wn + 4t),
    // +1 of its half of B, 32 lanes a row
    const int a_chunk = lane & 7, b_chunk = lane & 31;
    uint32_t a_off[TA];
#pragma unroll
    for (int t = 0; t < TA; t++) {
        int row = grp * HM + 8 * (wn + 4 * t) + (lane >> 3);
        row = (m0 + row < p.M) ? row : p.M - 1 - m0;                  // loaded, never stored
        a_off[t] = ((uint32_t)row * (uint32_t)p.lda + 8 * a_chunk) * 2;
    }
    const int b_krow0 = 2 * wn + (lane >> 5);                         // k row of load t within the group's half: b_krow0 + 8t
    int b_col = n0 + 8 * b_chunk;
    if (b_col > p.N - 8) b_col = p.N - 8;
    uint32_t b_off = ((uint32_t)b_krow0 * (uint32_t)p.ldb + (uint32_t)b_col) * 2u;
    const char* const a_tile = (const char*)(p.A + (int64_t)m0 * p.lda);
    const char* const b_half = (const char*)(p.B + (int64_t)(32 * grp) * p.ldb);
    const uint32_t a_wr = smem_base + (uint32_t)(grp * HM + 8 * wn + (lane >> 3)) * (BK * 2) + 16u * (a_chunk ^ (4 * (wn & 1) + (lane >> 4)));
    const uint32_t b_wr = smem_base + B_REGION + (uint32_t)(32 * grp + b_krow0) * VB_ROW + 16u * (b_chunk ^ ((b_krow0 & 3) << 2));
    const uint32_t b_wr_odd = b_wr ^ 32u;                             // k rows 8 further on: bit 1 of the chunk flips

    // ---- fragment read addresses (as in gemm_pingpong.hip) -------------------------------------
    uint32_t a_rd[2], b_rd[FN];
    {
        const int lr = lane & 15, lk = lane >> 4;
        const uint32_t row_off = (uint32_t)(grp * HM + lr) * (BK * 2);
#pragma unroll
        for (int h = 0; h < 2; h++) a_rd[h] = smem_base + row_off + (uint32_t)(((4 * h + lk) ^ (lr >> 1)) * 16);
        const int blk = lane >> 4, j = lane & 15, krow = 8 * blk + (j >> 2);
#pragma unroll
        for (int fn = 0; fn < FN; fn++) {
            const int chunk = (wn * 64 + fn * 16 + 4 * (j & 3)) >> 3;
            b_rd[fn] = smem_base + B_REGION + (uint32_t)krow * VB_ROW + (uint32_t)((chunk ^ (((krow & 3) << 2) | ((blk & 1) << 1))) * 16 + 8 * (j & 1));
        }
    }

    const int k_full = p.K / BK, KT = (p.K + BK - 1) / BK;
    uintx4 ra[TA], rb[TB];                                            // a k step on its way

    // (offsets that the compiler cannot see through: it then forms addresses from a uniform base and 32 bits a lane
    // instead of keeping a pair of registers for every load)
    auto load_a = [&](int k, int t) {
        asm volatile("" : "+v"(a_off[t]));
        ra[t] = *reinterpret_cast<const uintx4_any*>(a_tile + (int64_t)k * (BK * 2) + a_off[t]);
    };
    auto load_b = [&](int k, int t) {
        asm volatile("" : "+v"(b_off));
        rb[t] = *reinterpret_cast<const uintx4_any*>(b_half + ((int64_t)k * BK + 8 * t) * p.ldb * 2 + b_off);
    };
    // The step with the k tail: chunk c covers k = k0 + 8c .. + 7; past K - 8 it is loaded as the last 8 and
    // what belongs to the chunk before it is zeroed; the k rows of B that sit in the same slots likewise.
    auto load_a_tail = [&](int k, int t) {
        const int k0 = k * BK, over = k0 + 8 * a_chunk - (p.K - 8), back = over > 0 ? over : 0;
        uintx4 v = *reinterpret_cast<const uintx4_any*>(a_tile + ((int64_t)k0 - back) * 2 + a_off[t]);
#pragma unroll
        for (int e = 0; e < 4; e++) v[e] = (2 * e + 1 < back) ? 0u : (2 * e < back) ? (v[e] & 0xffff0000u) : v[e];
        ra[t] = v;
    };
    auto load_b_tail = [&](int k, int t) {
        const int k0 = k * BK, slot = 32 * grp + b_krow0 + 8 * t, over = k0 + (slot & ~7) - (p.K - 8), back = over > 0 ? over : 0;
        const uintx4 v = *reinterpret_cast<const uintx4_any*>((const char*)p.B + (((int64_t)(k0 + slot) - back) * p.ldb + b_col) * 2);
        rb[t] = (slot & 7) < back ? uintx4{0u, 0u, 0u, 0u} : v;
    };
    auto put_a = [&](int t) { *(__attribute__((address_space(3))) uintx4*)(uintptr_t)(a_wr + 4096u * t) = ra[t]; };
    auto put_b = [&](int k, int t) {
        *(__attribute__((address_space(3))) uintx4*)(uintptr_t)(((t & 1) ? b_wr_odd : b_wr) + (uint32_t)(k & 1) * VB_BUF + 4096u * t) = rb[t];
    };
    auto load_step = [&](int k) {
        if (k >= KT) return;
        if (k < k_full) {
#pragma unroll
            for (int t = 0; t < TB; t++) load_b(k, t);
#pragma unroll
            for (int t = 0; t < TA; t++) load_a(k, t);
        } else {
#pragma unroll
            for (int t = 0; t < TB; t++) load_b_tail(k, t);
#pragma unroll
            for (int t = 0; t < TA; t++) load_a_tail(k, t);
        }
    };

    load_step(0);
#pragma unroll
    for (int t = 0; t < TB; t++) put_b(0, t);
#pragma unroll
    for (int t = 0; t < TA; t++) put_a(t);
    load_step(1);

    floatx4 acc[FM][FN];
#pragma unroll
    for (int fm = 0; fm < FM; fm++)
#pragma unroll
        for (int fn = 0; fn < FN; fn++) acc[fm][fn] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    half8 fa[FM], fb[FN];
    auto read_fragments = [&](int k, int h) {
        uint32_t a0 = a_rd[h];
        asm volatile("" : "+v"(a0));
#pragma unroll
        for (int fm = 0; fm < FM; fm++) fa[fm] = lds_read_b128(a0 + fm * 16 * (BK * 2));
#pragma unroll
        for (int fn = 0; fn < FN; fn++) {
            uint32_t b0 = b_rd[fn] + (uint32_t)(k & 1) * VB_BUF;
            asm volatile("" : "+v"(b0));
            const half4 lo = lds_read_tr16(b0 + h * 32 * VB_ROW), hi = lds_read_tr16(b0 + h * 32 * VB_ROW + 4 * VB_ROW);
            fb[fn] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        }
    };
    auto lds_done = [&]() {
        __builtin_amdgcn_s_waitcnt(0xC07F);                           // lgkmcnt(0)
        asm volatile("" ::: "memory");
    };
    // loads: 0 none, 1 step k + 2 is a whole one, 2 it has the tail; puts: there is a step k + 1
    auto multiply = [&](int k, int h, auto loads, auto puts) {
        constexpr int L = decltype(loads)::value;
        constexpr int N = FM * FN;
#pragma unroll
        for (int i = 0; i < N; i++) {
            // two rows of blocks at a time, down, right, up, right: one operand changes per MFMA (gemm_pingpong.hip)
            const int pr = i / (2 * FN), q = i % (2 * FN), gm = 2 * pr + ((q % 4 == 1 || q % 4 == 2) ? 1 : 0), gn = (pr & 1) ? FN - 1 - q / 2 : q / 2;
            acc[gm][gn] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fb[gn], fa[gm], acc[gm][gn], 0, 0, 0);
            // chunk t is written behind MFMA 12 + 4t and the next one requested behind 14 + 4t (of 32)
#pragma unroll
            for (int t = 0; t < 4; t++) {
                if (h == 1 && t >= TA) continue;
                if (decltype(puts)::value != 0 && i == (12 + 4 * t) * N / 32) {
                    __builtin_amdgcn_sched_barrier(0);
                    if (h == 0) put_b(k + 1, t); else put_a(t);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (L != 0 && i == (14 + 4 * t) * N / 32) {
                    __builtin_amdgcn_sched_barrier(0);
                    if (h == 0) { if constexpr (L == 1) load_b(k + 2, t); else load_b_tail(k + 2, t); }
                    else        { if constexpr (L == 1) load_a(k + 2, t); else load_a_tail(k + 2, t); }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        if constexpr (decltype(puts)::value != 0) lds_done();         // the barrier that follows publishes the writes
    };
    auto k_step = [&](int k, auto loads, auto puts) {
#pragma unroll
        for (int h = 0; h < 2; h++) {
            read_fragments(k, h);                                     // X: phase 4k + 2h, Y: 4k + 2h + 1
            lds_done();
            phase_barrier();
            multiply(k, h, loads, puts);                              // X: phase 4k + 2h + 1, Y: 4k + 2h + 2
            if (decltype(puts)::value != 0 || grp == 0 || h == 0) phase_barrier();
        }
    };
    typedef std::integral_constant<int, 0> I0; typedef std::integral_constant<int, 1> I1; typedef std::integral_constant<int, 2> I2;

    lds_done();
    phase_barrier();
    if (grp == 1) phase_barrier();                                    // phase 0: X reads, Y has nothing to do yet
    int k = 0;
    for (; k + 2 < k_full; k++) k_step(k, I1{}, I1{});
    if (k + 2 < KT) { k_step(k, I2{}, I1{}); k++; }                   // fetches the tail
    if (k + 1 < KT) { k_step(k, I0{}, I1{}); k++; }

    // ---- C: addresses, and the first rows on their way under the last k step --------------------
    typedef typename CVec4<CT>::type ctx4;
    constexpr int NPRE = sizeof(CT) == 2 ? 2 : 1;
    int lane_e = lane;
    asm volatile("" : "+v"(lane_e));                                  // (nothing of the epilogue is worth registers during the k loop)
    const uint32_t tbuf = smem_base + (uint32_t)wave * (32u * VT_PITCH);
    const uint32_t t_w = tbuf + (uint32_t)(lane_e & 15) * VT_PITCH + (uint32_t)(lane_e >> 4) * 16;
    const uint32_t t_r = tbuf + (uint32_t)(lane_e >> 4) * VT_PITCH + (uint32_t)(lane_e & 15) * 16;
    const int x = wn * 64 + 4 * (lane_e & 15), nominal = n0 + (x & ~7);  // this lane_e's 4 columns within the tile; first column of their chunk
    const int first = (nominal < p.N - 8 ? nominal : p.N - 8) + (x & 7);   // ... and where those results belong
    const int row0 = m0 + grp * HM + (lane_e >> 4);
    // (columns before `nominal` are read, maybe while another workgroup stores them, and never used; rows beyond M read the last one)
    // (the pointers of all slabs at once would not fit the registers: each slab's are formed from a copy
    // that the compiler cannot see through)
    CT* cptr = (CT*)p.C + (int64_t)row0 * p.ldc + first;
    ctx4 cin[2][8];
    auto fetch = [&](int s, ctx4 (&dst)[8], auto edge_tag) {
        asm volatile("" : "+v"(cptr));
#pragma unroll
        for (int ps = 0; ps < 8; ps++) {
            int down = 32 * s + 4 * ps;
            if (decltype(edge_tag)::value) down = (row0 + down < p.M) ? down : p.M - 1 - row0;    // (within C, not stored)
            dst[ps] = *reinterpret_cast<const ctx4*>(cptr + (int64_t)down * p.ldc);
        }
    };
    if (edge) {
#pragma unroll
        for (int s = 0; s < NPRE; s++) fetch(s, cin[s], I1{});
    } else {
#pragma unroll
        for (int s = 0; s < NPRE; s++) fetch(s, cin[s], I0{});
    }
    __builtin_amdgcn_sched_barrier(0);
    for (; k < KT; k++) k_step(k, I0{}, I0{});                        // (one trip; as a loop it keeps the accumulators in their registers)

    // ---- + C, + bias, ReLU, -> C: 32 rows x 64 columns of a wavefront at a time through LDS, 4 columns a lane ----
    float bias4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (p.bias) {
#pragma unroll
        for (int e = 0; e < 4; e++) bias4[e] = (float)reinterpret_cast<const CT*>(p.bias)[first + e];
    }
    auto finish = [&](auto edge_tag) {
#pragma unroll
        for (int s = 0; s < HM / 32; s++) {
            if (s + 1 < HM / 32 && s + 1 >= NPRE) fetch(s + 1, cin[(s + 1) & 1], edge_tag);
#pragma unroll
            for (int r = 0; r < 2; r++)
#pragma unroll
                for (int fn = 0; fn < FN; fn++)
                    *(__attribute__((address_space(3))) floatx4*)(uintptr_t)(t_w + r * 16 * VT_PITCH + fn * 64) = acc[2 * s + r][fn];
            asm volatile("" : "+v"(cptr));
#pragma unroll
            for (int ps = 0; ps < 8; ps++) {
                const floatx4 s4 = *(__attribute__((address_space(3))) const floatx4*)(uintptr_t)(t_r + 4 * ps * VT_PITCH);
                const ctx4 c4 = cin[s & 1][ps];
                ctx4 o;
#pragma unroll
                for (int e = 0; e < 4; e++) o[e] = (CT)epilogue_value(s4[e] + (float)c4[e], bias4[e], p.relu);      // f16: one rounding, to nearest even
                CT* const dst = cptr + (int64_t)(32 * s + 4 * ps) * p.ldc;
                const bool row_ok = !decltype(edge_tag)::value || row0 + 32 * s + 4 * ps < p.M;
                if (row_ok && (!decltype(edge_tag)::value || first >= nominal)) *reinterpret_cast<ctx4*>(dst) = o;
                else if (row_ok) {
#pragma unroll
                    for (int e = 0; e < 4; e++) if (first + e >= nominal) dst[e] = o[e];
                }
            }
        }
    };
    if (edge) finish(I1{});
    else      finish(I0{});
}

template <int BM>
int64_t grid_unaligned_pp(int64_t M, int64_t N)
{
    const int64_t tm = (M + BM - 1) / BM, tn = (N + VBN - 1) / VBN;
    if (tm > 0 && tn > INT32_MAX / tm) return -1;
    return tm * tn;
}

template <int BM>
int launch_unaligned_pp(const GemmArgs& a)
{
    const int64_t g = grid_unaligned_pp<BM>(a.M, a.N);
    if (g < 0 || a.N < 8 || a.K < 8) return GEMM_F16_ERR_SIZE;
    const TiledParams p = make_tiled_params(a, BM, VBN, 8);
    const dim3 grid((unsigned)g), block(512);
    if (a.c_is_f16) hipLaunchKernelGGL((gemm_unaligned_pp_kernel<half_t, BM>), grid, block, 0, a.stream, p);
    else            hipLaunchKernelGGL((gemm_unaligned_pp_kernel<float, BM>), grid, block, 0, a.stream, p);
    return hipGetLastError() == hipSuccess ? GEMM_F16_OK : GEMM_F16_ERR_LAUNCH;
}

const GemmConfigDesc kUnaligned256 = {"generic256x256x64", 256, VBN, BK, 8, 128, 64, unaligned_pp_lds<256>(), false, launch_unaligned_pp<256>, grid_unaligned_pp<256>};
const GemmConfigDesc kUnaligned128x256 = {"generic128x256x64", 128, VBN, BK, 8, 64, 64, unaligned_pp_lds<128>(), false, launch_unaligned_pp<128>, grid_unaligned_pp<128>};

}  // namespace

const GemmConfigDesc* unaligned_pp_config(int block_m) { return block_m == 128 ? &kUnaligned128x256 : &kUnaligned256; }
